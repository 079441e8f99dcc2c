// Exact-operator baseline (Sec. 1.2; the "Exact" columns of the experiments
// of Sec. 5): Alg. 1 on the wavelet coefficients with the gradient of
// 1/2 ||H Psi x - u0||^2 computed from the blur itself rather than from the
// thresholded Theta_K:
//
//   g = Psi^* H^* (H Psi y - u0)    (synthesis, blur, adjoint blur, analysis)
//
// For a spatially varying PSF there is no fast exact H (the paper's FFT
// applies to convolutions only), so both products evaluate the truncated
// PSFs on the fly, in float64 with the field's own cut-off decisions,
// accumulating in float64; images and coefficients are float32.  Because Psi
// is orthogonal, Psi^* H Psi is the untruncated Theta, so this solves the
// problem before thresholding.
//
// The products are bound by the float64 arithmetic of the weights.  So a
// weight costs as little as it can: per source the handle keeps the rotated
// axes divided by the sigmas (q is then two products and four fused sums
// instead of two divisions) and 1 / Z; per 16 x 16 tile of sources and row
// offset it keeps the interval of column offsets any of them reaches (at sigma 4
// and 1, 150 of the 625 offsets of the box); and a block stages its
// neighbourhood in LDS.  Where q is so near the cut-off that its rounding could
// decide, the decision is taken again with the field's own formula.
// 512 x 512, sigma 4 and 1: H 302 -> 60 us, H^* 203 -> 27 us (its H^* needs half of
// the weights); about 30 instructions per weight, 3 of 4 issue slots used.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <functional>
#include <type_traits>
#include <vector>

#include "common.hpp"
#include "prox.hpp"
#include "psf.hpp"

struct wdb_exact {
  int device = 0;
  int32_t n = 0, levels = 0, wavelet = 0;
  int64_t N = 0;
  wdb::PsfField F;
  wdb::DevBuf<double> coef;   // per source, in planes: (c / a, s / a, c / b, s / b) kScale, 1 / Z
  wdb::DevBuf<short2> reach;  // per 16 x 16 tile of sources and dy: the dx any of them reaches
  int ntile = 0;              // tiles per side
  double near = 0.0;          // q is within this of the formula's value
  bool has_L = false;
  double L = 0.0;
  // workspace
  wdb::DevBuf<float> u0, y, img, r, gimg, g, sa, sb;
  wdb::DevBuf<double> part, scal;
  double* host = nullptr;     // pinned, 4 doubles
};

namespace wdb {
namespace {

constexpr int kT = 16;        // side of the tiles whose reach is kept

// The coefficients hold q scaled by log2(e) / 2, so that the weight is 2^-q.
constexpr double kScale = 0.8493218002880191;   // sqrt(log2(e) / 2)

// Device view of the handle's precomputed field.
struct ExDev {
  PsfDev P;
  const double* coef;
  const short2* reach;   // [tile][2 R + 1], dy = -R .. R; lo > hi: nothing
  int ntile;
  double sure, never;    // q <= sure is inside, q > never outside
};

__global__ __launch_bounds__(256) void k_exact_coef(PsfDev P, double* __restrict__ coef) {
  const int64_t s = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t N = static_cast<int64_t>(P.n) * P.n;
  if (s >= N) return;
  const double a = P.sM[s], b = P.sm[s], c = P.c[s], sn = P.s[s];
  coef[s] = kScale * c / a;
  coef[N + s] = kScale * sn / a;
  coef[2 * N + s] = kScale * c / b;
  coef[3 * N + s] = kScale * sn / b;
  coef[4 * N + s] = 1.0 / P.Z[s];
  // a PSF without weights (the squares of its sigmas underflow, so that not even its
  // centre is inside): a NaN is never inside either
  if (!(P.Z[s] > 0.0)) {
    for (int k = 0; k < 4; ++k) coef[k * N + s] = __longlong_as_double(0x7ff8000000000000ll);
    coef[4 * N + s] = 0.0;
  }
}

// a b + c with c from scalar registers.  (The compiler would copy each constant
// into the accumulator of a two-address v_fmac: a third more instructions here.)
__device__ __forceinline__ double fma_const(double a, double b, double c) {
  double d;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
  return d;
}

// 2^-x for 0 <= x < 2^31: -x = n + r, |r| <= 1/2, and the Taylor polynomial of
// degree 13 of 2^r (its remainder is below 5e-18) times 2^n.  n comes from the
// low 32 bits of a sum with 1.5 * 2^52.
__device__ __forceinline__ double exp2_neg(double x) {
  constexpr double kShift = 6755399441055744.0, kLn2 = 0.6931471805599453;
  const double t = kShift - x;
  const double r = (kShift - t) - x;
  double c[14] = {1.0};
#pragma unroll
  for (int k = 1; k < 14; ++k) c[k] = c[k - 1] * kLn2 / k;
  double p = c[13];
#pragma unroll
  for (int k = 12; k > 0; --k) p = fma_const(p, r, c[k]);
  return ldexp(fma(p, r, 1.0), __double2loint(t));
}

// Scaled q of coefficients k at offset (dy, dx).
__device__ __forceinline__ double scaled_q(double k0, double k1, double k2, double k3, double fy, double fx) {
  const double u1 = fma(fx, k0, fy * k1), u2 = fma(-fx, k3, fy * k2);
  return fma(u1, u1, u2 * u2);
}

// acc + w v, with w the weight (before 1 / Z) of source s, coefficients k, at
// offset (dy, dx); acc past the cut-off.
__device__ __forceinline__ double weigh(const ExDev& E, int64_t s, double k0, double k1, double k2, double k3,
                                        int dy, int dx, double fy, double fx, double v, double acc) {
  const double q = scaled_q(k0, k1, k2, k3, fy, fx);
  const bool maybe = q <= E.never;
  if (!__any(maybe)) return acc;
  bool in = q <= E.sure;
  if (maybe && !in) in = psf_q(E.P, s, dy, dx) <= E.P.T2;
  const double sum = fma(exp2_neg(q), v, acc);
  return in ? sum : acc;
}

// Reach at dy = blockIdx.y and at -dy of a tile of sources (blockIdx.x), thread =
// source.  An interval's ends come from the roots of q in dx, one offset more on
// either side, and are then tried; what rounding could let in is let in (the
// products decide).  A block per dy: with all of a tile's in one block and every
// offset tried with the field's formula, creating the handle took 1.44 ms for 64 x
// 64 at radius 30 and 6.15 ms for 512 x 512 at radius 27; now 0.79 and 5.4 ms.
__global__ __launch_bounds__(kT * kT) void k_exact_reach(ExDev E, short2* __restrict__ reach) {
  __shared__ int lo, hi;
  const int n = E.P.n, R = E.P.R, dy = blockIdx.y;
  const int64_t N = static_cast<int64_t>(n) * n;
  const int r = static_cast<int>(blockIdx.x) / E.ntile * kT + static_cast<int>(threadIdx.x) / kT;
  const int col = static_cast<int>(blockIdx.x) % E.ntile * kT + static_cast<int>(threadIdx.x) % kT;
  if (threadIdx.x == 0) {
    lo = R + 1;
    hi = -R - 1;
  }
  __syncthreads();
  int first = R + 1, last = -R - 1;
  if (r < n && col < n) {
    const int64_t s = static_cast<int64_t>(r) * n + col;
    const double k0 = E.coef[s], k1 = E.coef[N + s], k2 = E.coef[2 * N + s], k3 = E.coef[3 * N + s];
    const double fy = static_cast<double>(dy), R1 = static_cast<double>(R);
    // q = a (dx - mid)^2 + (c dy^2 - a mid^2)
    const double a = fma(k0, k0, k3 * k3), c = fma(k1, k1, k2 * k2), mid = -fy * (k0 * k1 - k3 * k2) / a;
    const double half = sqrt(fmax((E.never - fy * fy * c) / a + mid * mid, 0.0)) + 1.0;
    // squares that overflow, PSFs without weights (NaN): every offset is tried
    const bool known = a < 1e300 && c < 1e300;
    int x0 = known ? static_cast<int>(fmin(fmax(floor(mid - half), -R1), R1 + 1.0)) : -R;
    int x1 = known ? static_cast<int>(fmax(fmin(ceil(mid + half), R1), -R1 - 1.0)) : R;
    while (x0 <= x1 && !(scaled_q(k0, k1, k2, k3, fy, static_cast<double>(x0)) <= E.never)) ++x0;
    while (x1 >= x0 && !(scaled_q(k0, k1, k2, k3, fy, static_cast<double>(x1)) <= E.never)) --x1;
    if (x0 <= x1) {
      first = x0;
      last = x1;
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    first = min(first, __shfl_xor(first, off));
    last = max(last, __shfl_xor(last, off));
  }
  if ((threadIdx.x & 63) == 0) {
    atomicMin(&lo, first);
    atomicMax(&hi, last);
  }
  __syncthreads();
  if (threadIdx.x) return;
  short2* at = reach + static_cast<int64_t>(blockIdx.x) * (2 * R + 1) + R;
  at[-dy] = make_short2(static_cast<short>(-hi), static_cast<short>(-lo));   // a PSF is even
  at[dy] = make_short2(static_cast<short>(lo), static_cast<short>(hi));
}

// Interval of dx that any source of the tiles covering rows [r0, r1] and columns
// [c0, c1] (any integers, periodic) reaches at dy.
__device__ __forceinline__ int2 reach_of(const ExDev& E, int r0, int r1, int c0, int c1, int dy) {
  const int rows = min((r1 >> 4) - (r0 >> 4) + 1, E.ntile), cols = min((c1 >> 4) - (c0 >> 4) + 1, E.ntile);
  int lo = E.P.R + 1, hi = -E.P.R - 1;
  for (int i = 0; i < rows; ++i)
    for (int j = 0; j < cols; ++j) {
      const int tr = ((r0 >> 4) + i) & (E.ntile - 1), tc = ((c0 >> 4) + j) & (E.ntile - 1);
      const short2 v = E.reach[static_cast<int64_t>(tr * E.ntile + tc) * (2 * E.P.R + 1) + dy + E.P.R];
      lo = min(lo, static_cast<int>(v.x));
      hi = max(hi, static_cast<int>(v.y));
    }
  return make_int2(lo, hi);
}

struct Source {
  double k[4], v;   // coefficients, in / Z
};

__device__ __forceinline__ Source source(const ExDev& E, int64_t N, int64_t s, double in) {
  return Source{{E.coef[s], E.coef[N + s], E.coef[2 * N + s], E.coef[3 * N + s]}, E.coef[4 * N + s] * in};
}

// A product's block: kTW x TH targets (sources for H^*), each summed by
// kThreads / (kTW TH) threads over the row offsets dealt to them in turn.
constexpr int kTW = 32, kThreads = 1024;

// The targets' sums from their threads' (red: kThreads float64 of LDS), thread < kTW TH.
template <int TH>
__device__ __forceinline__ double sum_groups(double* red, double acc) {
  if (TH == 32) return acc;
  __syncthreads();
  red[threadIdx.x] = acc;
  __syncthreads();
  if (threadIdx.x < kTW * TH)
    for (int k = threadIdx.x + kTW * TH; k < kThreads; k += kTW * TH) acc += red[k];
  return acc;
}

// H: out[i] = sum over sources s of k_s(i - s) in[s]  (- sub[i]).  `rows` row
// offsets at a time have their sources staged in LDS (40 bytes each: neighbouring
// sources are on different banks); rows = 0: straight from memory.
template <typename TI, typename TO, int TH>
__global__ __launch_bounds__(kThreads) void k_exact_fwd(ExDev E, int rows, const TI* __restrict__ in,
                                                        const float* __restrict__ sub, TO* __restrict__ out) {
  extern __shared__ __align__(16) double lds[];
  const int n = E.P.n, R = E.P.R, m = n - 1, span = 2 * R + 1;
  const int64_t N = static_cast<int64_t>(n) * n;
  const int y0 = blockIdx.y * TH, x0 = blockIdx.x * kTW, W = kTW + 2 * R;
  int2* rng = reinterpret_cast<int2*>(lds + kThreads);
  Source* src = reinterpret_cast<Source*>(rng + span);
  for (int k = threadIdx.x; k < span; k += kThreads) {
    const int dy = k - R;
    rng[k] = reach_of(E, y0 - dy, y0 + TH - 1 - dy, x0 - R, x0 + kTW - 1 + R, dy);
  }
  const int id = static_cast<int>(threadIdx.x) % (kTW * TH), group = static_cast<int>(threadIdx.x) / (kTW * TH);
  const int ty = id / kTW, tx = id % kTW;
  double acc = 0.0;
  for (int d0 = -R; d0 <= R; d0 += rows ? rows : span) {
    const int d1 = rows ? min(d0 + rows - 1, R) : R;   // offsets d0 .. d1: source rows y0 - d1 .. y0 + TH - 1 - d0
    __syncthreads();
    if (rows)
      for (int e = threadIdx.x; e < W * (TH + d1 - d0); e += kThreads) {
        const int r = e / W, c = e - r * W;
        const int64_t s = static_cast<int64_t>((y0 - d1 + r) & m) * n + ((x0 - R + c) & m);
        src[e] = source(E, N, s, static_cast<double>(in[s]));
      }
    __syncthreads();
    for (int dy = d0 + group; dy <= d1; dy += kThreads / (kTW * TH)) {
      const int2 d = rng[dy + R];
      const int lo = __builtin_amdgcn_readfirstlane(d.x), hi = __builtin_amdgcn_readfirstlane(d.y);
      const double fy = static_cast<double>(dy);
      const int64_t row = static_cast<int64_t>((y0 + ty - dy) & m) * n;
      double fx = static_cast<double>(lo);
      if (rows) {
        const Source* p = src + (ty + d1 - dy) * W + tx + R - lo;
        for (int dx = lo; dx <= hi; ++dx, --p, fx += 1.0)
          acc = weigh(E, row + ((x0 + tx - dx) & m), p->k[0], p->k[1], p->k[2], p->k[3], dy, dx, fy, fx, p->v, acc);
      } else {
        for (int dx = lo; dx <= hi; ++dx, fx += 1.0) {
          const int64_t s = row + ((x0 + tx - dx) & m);
          const Source q = source(E, N, s, static_cast<double>(in[s]));
          acc = weigh(E, s, q.k[0], q.k[1], q.k[2], q.k[3], dy, dx, fy, fx, q.v, acc);
        }
      }
    }
  }
  acc = sum_groups<TH>(lds, acc);
  if (group || y0 + ty >= n || x0 + tx >= n) return;
  const int64_t i = static_cast<int64_t>(y0 + ty) * n + x0 + tx;
  out[i] = static_cast<TO>(sub ? acc - static_cast<double>(sub[i]) : acc);
}

// H^*: out[s] = sum_d k_s(d) in[s + d].  With STAGE the image within the field's
// radius is staged in LDS.  A PSF is even in d, also in its roundings, so half of
// the offsets are enough (47 -> 27 us).
template <typename TI, typename TO, int TH, bool STAGE>
__global__ __launch_bounds__(kThreads) void k_exact_adj(ExDev E, const TI* __restrict__ in, TO* __restrict__ out) {
  extern __shared__ __align__(16) double lds[];
  const int n = E.P.n, R = E.P.R, m = n - 1;
  const int64_t N = static_cast<int64_t>(n) * n;
  const int y0 = blockIdx.y * TH, x0 = blockIdx.x * kTW, W = kTW + 2 * R;
  int2* rng = reinterpret_cast<int2*>(lds + kThreads);   // dy = 0 .. R
  double* img = reinterpret_cast<double*>(rng + R + 1);
  for (int k = threadIdx.x; k <= R; k += kThreads) rng[k] = reach_of(E, y0, y0 + TH - 1, x0, x0 + kTW - 1, k);
  if (STAGE)
    for (int e = threadIdx.x; e < W * (TH + 2 * R); e += kThreads) {
      const int r = e / W, c = e - r * W;
      img[e] = static_cast<double>(in[static_cast<int64_t>((y0 - R + r) & m) * n + ((x0 - R + c) & m)]);
    }
  __syncthreads();
  const int id = static_cast<int>(threadIdx.x) % (kTW * TH), group = static_cast<int>(threadIdx.x) / (kTW * TH);
  const int ty = id / kTW, tx = id % kTW;
  const int64_t s = static_cast<int64_t>((y0 + ty) & m) * n + ((x0 + tx) & m);
  const Source src = source(E, N, s, 1.0);
  const auto at = [&](int dy, int dx) {
    return static_cast<double>(in[static_cast<int64_t>((y0 + ty + dy) & m) * n + ((x0 + tx + dx) & m)]);
  };
  const double* mid = img + (ty + R) * W + tx + R;
  double acc = 0.0;
  if (group == 0)
    acc = weigh(E, s, src.k[0], src.k[1], src.k[2], src.k[3], 0, 0, 0.0, 0.0, STAGE ? *mid : at(0, 0), acc);
  for (int dy = group; dy <= R; dy += kThreads / (kTW * TH)) {
    const int2 d = rng[dy];
    const int lo = dy ? __builtin_amdgcn_readfirstlane(d.x) : 1, hi = __builtin_amdgcn_readfirstlane(d.y);
    const double fy = static_cast<double>(dy);
    const double *p = mid + dy * W + lo, *q = mid - dy * W - lo;
    double fx = static_cast<double>(lo);
    for (int dx = lo; dx <= hi; ++dx, ++p, --q, fx += 1.0) {
      const double v = STAGE ? *p + *q : at(dy, dx) + at(-dy, -dx);
      acc = weigh(E, s, src.k[0], src.k[1], src.k[2], src.k[3], dy, dx, fy, fx, v, acc);
    }
  }
  acc = sum_groups<TH>(lds, acc);
  if (group || y0 + ty >= n || x0 + tx >= n) return;
  out[s] = static_cast<TO>(acc * src.v);
}

// Proximal step and momentum of Alg. 1 (beta from the host: the iteration
// index is known there).
__global__ __launch_bounds__(256) void k_exact_prox(const float* __restrict__ g, float* __restrict__ x,
                                                    float* __restrict__ y, float tau, float thr, float beta,
                                                    int64_t N) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const float xn = prox_plain(y[i], tau * g[i], thr);
  const float xo = x[i];
  x[i] = xn;
  y[i] = xn + beta * (xn - xo);
}

// Per-block partials: sum r^2, sum r u0, sum |x|, max |g| (4 * nblocks).
__global__ __launch_bounds__(256) void k_exact_obj(const float* __restrict__ r, const float* __restrict__ u0,
                                                   const float* __restrict__ x, const float* __restrict__ g,
                                                   int64_t N, double* __restrict__ part, int64_t nblocks) {
  __shared__ double sh[4][256];
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  if (i < N) {
    const double rr = r[i];
    v[0] = rr * rr;
    v[1] = rr * static_cast<double>(u0[i]);
    v[2] = fabs(static_cast<double>(x[i]));
    v[3] = fabs(static_cast<double>(g[i]));
  }
  for (int k = 0; k < 4; ++k) sh[k][threadIdx.x] = v[k];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w)
      for (int k = 0; k < 4; ++k)
        sh[k][threadIdx.x] = k == 3 ? fmax(sh[k][threadIdx.x], sh[k][threadIdx.x + w])
                                    : sh[k][threadIdx.x] + sh[k][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x < 4) part[threadIdx.x * nblocks + blockIdx.x] = sh[threadIdx.x][0];
}

__global__ __launch_bounds__(256) void k_exact_fin(const double* __restrict__ part, int64_t nblocks,
                                                   double* __restrict__ out) {
  __shared__ double sh[4][256];
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  for (int64_t b = threadIdx.x; b < nblocks; b += 256)
    for (int k = 0; k < 4; ++k) v[k] = k == 3 ? fmax(v[k], part[k * nblocks + b]) : v[k] + part[k * nblocks + b];
  for (int k = 0; k < 4; ++k) sh[k][threadIdx.x] = v[k];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w)
      for (int k = 0; k < 4; ++k)
        sh[k][threadIdx.x] = k == 3 ? fmax(sh[k][threadIdx.x], sh[k][threadIdx.x + w])
                                    : sh[k][threadIdx.x] + sh[k][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x < 4) out[threadIdx.x] = sh[threadIdx.x][0];
}

__global__ void k_exact_init(const float* __restrict__ src, float* __restrict__ x, float* __restrict__ y, int64_t N) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const float v = src ? src[i] : 0.0f;
  x[i] = v;
  y[i] = v;
}

dim3 pix_grid(int64_t N) { return dim3(static_cast<unsigned>((N + 255) / 256)); }

// Largest scaled q whose weight 2^-q is not 0 in float64.
constexpr double kLeast = 1074.0;

// A cut-off beyond kLeast (any trunc above 38.6) is brought down to it: the same
// sums, and exp2_neg's argument stays in its range (q reaches trunc^2).
ExDev view(const wdb_exact* ex) {
  const double T2 = ex->F.trunc * ex->F.trunc;
  const double k2 = kScale * kScale;
  return ExDev{ex->F.dev(), ex->coef.p, ex->reach.p, ex->ntile, std::min(k2 * (T2 - ex->near), kLeast),
               std::min(k2 * (T2 + ex->near), kLeast)};
}

// f(TH): 32 x 32 targets per block where those fill the chip, else 32 x 8 with four
// threads per target, else 32 x 2 with sixteen.  Always 16 waves a block: one wave
// of 32 x 2 alone is a serial chain (side 256, sigma 4 and 1: H 41 -> 22 us with
// four threads per target; side 128: 54 -> 12 us with sixteen).
template <typename F>
void with_tile(int n, F&& f) {
  using std::integral_constant;
  if (n >= 512)
    f(integral_constant<int, 32>{});
  else if (n >= 256)
    f(integral_constant<int, 8>{});
  else
    f(integral_constant<int, 2>{});
}

dim3 grid_of(int n, int TH) { return dim3((n + kTW - 1) / kTW, (n + TH - 1) / TH); }

constexpr size_t kLds = 160 * 1024;

// More than 64 KiB of LDS needs the kernel's limit raised, once per device (`done`: a bit per device).
void raise_lds(const void* kernel, int device, std::atomic<uint64_t>& done) {
  const uint64_t bit = uint64_t{1} << (device & 63);
  if (done.load() & bit) return;
  WDB_HIP(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kLds));
  done.fetch_or(bit);
}

// Row offsets of H staged at a time: all where the LDS holds their sources, else
// as many as it holds (512 x 512, sigma 6 and 1, two parts: 112 us, straight from
// memory 243 us), unless each source row would then serve few offsets.
int staged_rows(int R, int TH) {
  const size_t row = sizeof(Source) * (kTW + 2 * R);
  const size_t room = kLds - kThreads * sizeof(double) - (2 * static_cast<size_t>(R) + 1) * sizeof(int2);
  const int fit = static_cast<int>(room / row) - TH + 1, groups = kThreads / (kTW * TH);
  if (fit >= 2 * R + 1) return 2 * R + 1;
  return fit >= 8 ? std::max(fit / groups, 1) * groups : 0;
}

template <typename TI, typename TO>
void apply_H(const wdb_exact* ex, const TI* in, const float* sub, TO* out, hipStream_t s) {
  with_tile(ex->n, [&](auto Hc) {
    constexpr int TH = decltype(Hc)::value;
    const int R = ex->F.R, rows = std::min(staged_rows(R, TH), 2 * R + 1);
    const size_t bytes = kThreads * sizeof(double) + (2 * static_cast<size_t>(R) + 1) * sizeof(int2) +
                         (rows ? sizeof(Source) * (kTW + 2 * R) * (TH + rows - 1) : 0);
    static std::atomic<uint64_t> done{0};
    raise_lds(reinterpret_cast<const void*>(k_exact_fwd<TI, TO, TH>), ex->device, done);
    hipLaunchKernelGGL((k_exact_fwd<TI, TO, TH>), grid_of(ex->n, TH), dim3(kThreads), bytes, s, view(ex), rows, in,
                       sub, out);
  });
}

template <typename TI, typename TO>
void apply_Ht(const wdb_exact* ex, const TI* in, TO* out, hipStream_t s) {
  with_tile(ex->n, [&](auto Hc) {
    constexpr int TH = decltype(Hc)::value;
    const size_t R = ex->F.R, fixed = kThreads * sizeof(double) + (R + 1) * sizeof(int2);
    const size_t all = fixed + sizeof(double) * (kTW + 2 * R) * (TH + 2 * R);
    const auto go = [&](auto Sc, size_t bytes) {
      constexpr bool ST = decltype(Sc)::value;
      static std::atomic<uint64_t> done{0};
      raise_lds(reinterpret_cast<const void*>(k_exact_adj<TI, TO, TH, ST>), ex->device, done);
      hipLaunchKernelGGL((k_exact_adj<TI, TO, TH, ST>), grid_of(ex->n, TH), dim3(kThreads), bytes, s, view(ex), in,
                         out);
    };
    if (all <= kLds)
      go(std::true_type{}, all);
    else
      go(std::false_type{}, fixed);
  });
}

// g = Psi^* H^* (H Psi v - u0); leaves H Psi v - u0 in ex->r.
void gradient(wdb_exact* ex, const Filter& f, const float* v, float* g, hipStream_t s) {
  dwt_inverse(ex->n, ex->levels, f, v, ex->img.p, s);
  apply_H(ex, ex->img.p, ex->u0.p, ex->r.p, s);
  apply_Ht(ex, ex->r.p, ex->gimg.p, s);
  dwt_forward(ex->n, ex->levels, f, ex->gimg.p, g, ex->sa.p, ex->sb.p, s);
}

struct ExCheck {
  double E, rel_gap;
};

// E(x) = 1/2 ||H Psi x - u0||^2 + lambda ||x||_1 and the relative gap with the
// dual point s r, s = min(1, lambda / ||Psi^* H^* r||_inf) (float32 products,
// float64 sums).
ExCheck check(wdb_exact* ex, const Filter& f, const float* x, double lambda, hipStream_t s) {
  gradient(ex, f, x, ex->g.p, s);
  const int64_t nb = pix_grid(ex->N).x;
  hipLaunchKernelGGL(k_exact_obj, pix_grid(ex->N), dim3(256), 0, s, ex->r.p, ex->u0.p, x, ex->g.p, ex->N, ex->part.p,
                     nb);
  hipLaunchKernelGGL(k_exact_fin, dim3(1), dim3(256), 0, s, ex->part.p, nb, ex->scal.p);
  WDB_HIP(hipGetLastError());
  WDB_HIP(hipMemcpyAsync(ex->host, ex->scal.p, 4 * sizeof(double), hipMemcpyDeviceToHost, s));
  WDB_HIP(hipStreamSynchronize(s));
  const double rr = ex->host[0], ru = ex->host[1], l1 = ex->host[2], gm = ex->host[3];
  const double E = 0.5 * rr + lambda * l1;
  const double sc = gm <= lambda ? 1.0 : lambda / gm;
  const double D = -0.5 * sc * sc * rr - sc * ru;
  return ExCheck{E, E > 0 ? (E - D) / E : 0.0};
}

LanczosResult exact_lanczos(wdb_exact* ex, const double* start, double tol, int max_steps, hipStream_t s) {
  DevBuf<double> t(ex->N);
  auto apply = [&](const double* v, double* u) {   // u = H^* H v (pixel domain; Psi is orthogonal)
    apply_H(ex, v, static_cast<const float*>(nullptr), t.p, s);
    apply_Ht(ex, static_cast<const double*>(t.p), u, s);
  };
  return lanczos_core(ex->N, apply, start, tol, max_steps, s);
}

}  // namespace
}  // namespace wdb

extern "C" {

wdb_status wdb_exact_create(const wdb_psf_field* field, int32_t wavelet, int32_t levels, void* stream,
                            wdb_exact** out) {
  WDB_API_BEGIN
  WDB_REQUIRE(field && out, WDB_ERR_ARG, "null argument");
  const wdb::Filter f = wdb::make_filter(wavelet);
  wdb::check_geometry(field->n, levels, static_cast<int>(f.h.size()));
  hipStream_t s = static_cast<hipStream_t>(stream);
  auto* ex = new wdb_exact;
  try {
    WDB_HIP(hipGetDevice(&ex->device));
    ex->n = field->n;
    ex->levels = levels;
    ex->wavelet = wavelet;
    ex->N = static_cast<int64_t>(field->n) * field->n;
    ex->F.upload(field, s);
    const int64_t N = ex->N;
    ex->ntile = (ex->n + wdb::kT - 1) / wdb::kT;
    WDB_REQUIRE(ex->F.R < 32767, WDB_ERR_SIZE, "PSF radius %d too large", ex->F.R);
    // error of q against the formula's: each axis' rotated offset is off by a few
    // roundings of its terms, at most R / sigma, and q <= trunc^2 or so there
    ex->near = 1e-14 * (1.0 + ex->F.trunc) * (1.0 + ex->F.trunc + ex->F.R / ex->F.smin);
    ex->coef.alloc(5 * static_cast<size_t>(N));
    const size_t tiles = static_cast<size_t>(ex->ntile) * ex->ntile;
    ex->reach.alloc(tiles * (2 * static_cast<size_t>(ex->F.R) + 1));
    hipLaunchKernelGGL(wdb::k_exact_coef, wdb::pix_grid(N), dim3(256), 0, s, ex->F.dev(), ex->coef.p);
    hipLaunchKernelGGL(wdb::k_exact_reach, dim3(static_cast<unsigned>(tiles), static_cast<unsigned>(ex->F.R + 1)),
                       dim3(wdb::kT * wdb::kT), 0, s, wdb::view(ex), ex->reach.p);
    for (auto* b : {&ex->u0, &ex->y, &ex->img, &ex->r, &ex->gimg, &ex->g}) b->alloc(N);
    const wdb::DwtScratch need = wdb::dwt_scratch(ex->n, levels);
    ex->sa.alloc(need.a);
    ex->sb.alloc(need.b);
    const int64_t nb = wdb::pix_grid(N).x;
    ex->part.alloc(4 * nb);
    ex->scal.alloc(4);
    WDB_HIP(hipHostMalloc(reinterpret_cast<void**>(&ex->host), 4 * sizeof(double), hipHostMallocDefault));
    WDB_HIP(hipGetLastError());
    WDB_HIP(hipStreamSynchronize(s));
  } catch (...) {
    if (ex->host) (void)hipHostFree(ex->host);
    delete ex;
    throw;
  }
  *out = ex;
  WDB_API_END
}

void wdb_exact_free(wdb_exact* ex) {
  if (!ex) return;
  (void)hipSetDevice(ex->device);
  (void)hipDeviceSynchronize();
  if (ex->host) (void)hipHostFree(ex->host);
  delete ex;
}

wdb_status wdb_exact_apply(wdb_exact* ex, int32_t adjoint, const float* in, float* out, void* stream) {
  WDB_API_BEGIN
  WDB_REQUIRE(ex && in && out, WDB_ERR_ARG, "null argument");
  WDB_REQUIRE(in != out, WDB_ERR_ARG, "in and out must not alias");
  WDB_HIP(hipSetDevice(ex->device));
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (adjoint)
    wdb::apply_Ht(ex, in, out, s);
  else
    wdb::apply_H(ex, in, static_cast<const float*>(nullptr), out, s);
  WDB_HIP(hipGetLastError());
  WDB_API_END
}

wdb_status wdb_exact_lipschitz(wdb_exact* ex, const double* start, double tol, int32_t max_steps, double* L_out,
                               int32_t* steps_out, double* resid_out) {
  WDB_API_BEGIN
  WDB_REQUIRE(ex, WDB_ERR_ARG, "null handle");
  WDB_HIP(hipSetDevice(ex->device));
  const wdb::LanczosResult r = wdb::exact_lanczos(ex, start, tol, max_steps, nullptr);
  ex->L = r.theta + r.resid;
  ex->has_L = true;
  if (L_out) *L_out = ex->L;
  if (steps_out) *steps_out = r.steps;
  if (resid_out) *resid_out = r.resid;
  if (!r.converged)
    wdb::fail(WDB_ERR_NOT_CONVERGED, "Lanczos reached max_steps = %d with residual %.3e > tol * theta", max_steps,
              r.resid);
  WDB_API_END
}

wdb_status wdb_exact_solve(wdb_exact* ex, const float* u, float lambda, const wdb_solve_opts* opts, float* x_out,
                           wdb_solve_info* info) {
  WDB_API_BEGIN
  WDB_REQUIRE(ex && u && opts && x_out, WDB_ERR_ARG, "null argument");
  WDB_REQUIRE(std::isfinite(lambda) && lambda >= 0.0f, WDB_ERR_NONFINITE, "lambda must be finite and >= 0");
  WDB_REQUIRE(opts->max_iters >= 0 && opts->check_every >= 0 && opts->k0 >= 0, WDB_ERR_ARG, "bad iteration counts");
  WDB_REQUIRE(!opts->use_precond, WDB_ERR_ARG, "the exact-operator solver has no preconditioner");
  WDB_HIP(hipSetDevice(ex->device));
  hipStream_t s = static_cast<hipStream_t>(opts->stream);
  if (!ex->has_L) {
    const wdb::LanczosResult r = wdb::exact_lanczos(ex, nullptr, 1e-12, 2000, s);
    ex->L = r.theta + r.resid;
    ex->has_L = true;
  }
  WDB_REQUIRE(ex->L > 0.0 && std::isfinite(ex->L), WDB_ERR_ARG, "operator has no positive Lipschitz constant");
  const double tau = 1.0 / ex->L;
  const float tau_f = static_cast<float>(tau), thr_f = static_cast<float>(tau * static_cast<double>(lambda));
  const wdb::Filter f = wdb::make_filter(ex->wavelet);
  const int64_t N = ex->N;
  WDB_HIP(hipMemcpyAsync(ex->u0.p, u, N * sizeof(float), hipMemcpyDeviceToDevice, s));
  hipLaunchKernelGGL(wdb::k_exact_init, wdb::pix_grid(N), dim3(256), 0, s, opts->x_init, x_out, ex->y.p, N);
  const int k0 = opts->k0 > 0 ? opts->k0 : 1;
  const int c = opts->check_every, total = opts->max_iters;
  int done = 0, checks = 0;
  bool converged = false;
  wdb::ExCheck last{0.0, 0.0};
  while (done < total || (total == 0 && checks == 0)) {
    if (done < total) {
      const int k = k0 + done;
      const float beta = opts->ista ? 0.0f : static_cast<float>((k - 1.0) / (k + 2.0));
      wdb::gradient(ex, f, ex->y.p, ex->g.p, s);
      hipLaunchKernelGGL(wdb::k_exact_prox, wdb::pix_grid(N), dim3(256), 0, s, ex->g.p, x_out, ex->y.p, tau_f, thr_f,
                         beta, N);
      WDB_HIP(hipGetLastError());
      ++done;
    }
    if ((c > 0 && done % c == 0) || done == total) {
      last = wdb::check(ex, f, x_out, lambda, s);
      ++checks;
      if (opts->trace && checks <= opts->trace_cap) {
        opts->trace[3 * (checks - 1) + 0] = static_cast<double>(k0 - 1 + done);
        opts->trace[3 * (checks - 1) + 1] = last.E;
        opts->trace[3 * (checks - 1) + 2] = last.rel_gap;
      }
      WDB_REQUIRE(std::isfinite(last.E), WDB_ERR_DIVERGED, "objective became non-finite at iteration %d", done);
      if ((opts->tol_rel_gap > 0 && last.rel_gap <= opts->tol_rel_gap) ||
          (opts->target_objective > 0 && last.E <= opts->target_objective)) {
        converged = true;
        break;
      }
      if (total == 0) break;
    }
  }
  WDB_HIP(hipStreamSynchronize(s));
  if (info) {
    info->iters = done;
    info->checks = checks;
    info->objective = last.E;
    info->rel_gap = last.rel_gap;
    info->lipschitz = ex->L;
    info->tau = tau;
  }
  if ((opts->tol_rel_gap > 0 || opts->target_objective > 0) && !converged)
    wdb::fail(WDB_ERR_NOT_CONVERGED, "stopping test not met after %d iterations (relative gap %.3e)", done,
              last.rel_gap);
  WDB_API_END
}

}  // extern "C"
