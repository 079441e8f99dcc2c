// Periodic separable 2D orthogonal wavelet transform on the GPU (Sec. 2:
// tensor-product wavelets at one scale, circular boundaries), float32.
//
// Both directions keep the levels between the image and the coefficients in
// LDS instead of passing each through memory in a launch of its own (a level's
// launch took 5 us however small the level, and its scratch had to be
// allocated): one forward transform at 512 x 512 with 8 taps and 5 levels takes
// 10.5 us in 2 launches (5 launches: 26 us; the whole call 27 against 44 us), the
// inverse of 21 images of 1024 x 1024 with 6 levels 111 us in one (18 launches:
// 349 us).
//
// Forward: c_e[i][j] = sum_{m, m'} f_erow[m] f_ecol[m'] A[(2i+m) mod M][(2j+m') mod M]
// with f_0 = h (low-pass) and f_1 = g (high-pass).  k_dwt_fwd takes up to three
// levels at once: a block owns 8 x 8 to 32 x 32 positions of its last level, loads the
// footprint these depend on (the positions 2i .. 2i + L - 1 of every level
// above), filters rows, then columns, level by level, and writes the details
// it owns.  The overlap of the footprints (2.7 times the pixels for 8 taps and
// three levels) costs less than a launch per level.  Once a level's side is at
// most 128, one block per image (k_dwt_fwd_tail) does all that is left: the
// level fits in its LDS, and since it has read all of it before it writes, it
// works in place on the coefficient vector.  Every output is the same chain of
// products and sums, in the order of the taps, whatever the split.
//
// Inverse (the transpose): a pixel depends on L / 2 positions per axis of the
// level below, so a block's footprint on a coarser level is half its own size
// plus L / 2 and all levels together cost little more than the finest.
// k_dwt_inv therefore does the whole transform in one launch: a block owns 64 x
// 64 or 32 x 32 pixels, loads the coefficients they depend on at once, and works from the
// coarsest level up, columns (vertical), then rows, two pixels of either
// parity per thread from the same coefficients.  Half of a block's time goes
// to the coarse levels, whose few positions leave most threads idle; more
// threads or loads in flight did not change that.
#include <algorithm>
#include <atomic>
#include <mutex>
#include <type_traits>
#include <vector>

#include "common.hpp"

namespace wdb {
namespace {

struct Taps {
  float h[kMaxTaps];
  float g[kMaxTaps];
  int L;
};

Taps to_taps(const Filter& f) {
  Taps t{};
  t.L = static_cast<int>(f.h.size());
  for (int i = 0; i < t.L; ++i) {
    t.h[i] = static_cast<float>(f.h[i]);
    t.g[i] = static_cast<float>(f.g[i]);
  }
  return t;
}

// Up to kBatch images per launch (blockIdx.z): per image the first level's
// input, the last level's approximation and the coefficient vector that holds
// the details.  The details (0,1), (1,0), (1,1) of a level with side s start
// at s^2, 2 s^2 and 3 s^2 of that vector.
constexpr int kBatch = 32;
struct FwdPtrs {
  const float* src[kBatch];
  float* ll[kBatch];
  float* out[kBatch];
};
struct InvPtrs {
  const float* in[kBatch];
  float* dst[kBatch];
};

// One float per lane from memory to LDS without passing through registers: lane
// i of the wavefront fills dst[i] (dst the same for the whole wavefront).  All
// loads of a block are in flight at once; loads_done waits for them.
__device__ __forceinline__ void load_lds(const float* src, float* dst) {
  __builtin_amdgcn_global_load_lds(
      (const __attribute__((address_space(1))) void*)reinterpret_cast<uintptr_t>(src),
      (__attribute__((address_space(3))) void*)static_cast<uint32_t>(reinterpret_cast<uintptr_t>(dst)), 4, 0, 0);
}
__device__ __forceinline__ void loads_done() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}
// First thread of this thread's wavefront.
__device__ __forceinline__ int wave_first() {
  return __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) & ~63);
}

// Low and high pass of one row at output j (x: the row from position 2 j on,
// 8-byte aligned).
template <int L>
__device__ __forceinline__ float2 row_taps(const float* __restrict__ x, const Taps& t) {
  float l = 0.f, h = 0.f;
#pragma unroll
  for (int m = 0; m < L; m += 2) {
    const float2 v = *reinterpret_cast<const float2*>(x + m);
    l = fmaf(t.h[m], v.x, l);
    h = fmaf(t.g[m], v.x, h);
    l = fmaf(t.h[m + 1], v.y, l);
    h = fmaf(t.g[m + 1], v.y, h);
  }
  return make_float2(l, h);
}

// The same for a column of row results (low pass and high pass interleaved,
// `stride` float2 per row): the four subbands {00, 01, 10, 11}.
template <int L>
__device__ __forceinline__ float4 col_taps(const float2* __restrict__ x, int stride, const Taps& t) {
  float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int m = 0; m < L; ++m) {
    const float2 v = x[m * stride];
    a.x = fmaf(t.h[m], v.x, a.x);
    a.y = fmaf(t.h[m], v.y, a.y);
    a.z = fmaf(t.g[m], v.x, a.z);
    a.w = fmaf(t.g[m], v.y, a.w);
  }
  return a;
}

// Footprint side on the input of `nl` levels whose last level has T positions.
constexpr int footprint(int L, int nl, int T) { return nl == 0 ? T : footprint(L, nl - 1, 2 * T + L - 2); }

constexpr int kFwdThreads = 1024;

template <int L, int NL, int T>
constexpr int fwd_lds_floats() {
  const int s0 = footprint(L, NL, T), s1 = (s0 - L + 2) / 2;
  return s0 * s0 + 2 * s0 * s1;
}

// Level `lev` (1-based within the launch) of a block whose footprint of side
// S is in X; recurses to the last level.
template <int L, int NL, int T, int LEV>
__device__ __forceinline__ void fwd_levels(float* X, float2* R, int M, int i0, int j0, float* __restrict__ ll,
                                           float* __restrict__ out, const Taps& t) {
  constexpr int S = footprint(L, NL - LEV + 1, T), SO = (S - L + 2) / 2;
  constexpr int OWN = T << (NL - LEV);
  for (int e = threadIdx.x; e < S * SO; e += kFwdThreads) {
    const int r = e / SO, j = e - r * SO;
    R[e] = row_taps<L>(X + r * S + 2 * j, t);
  }
  __syncthreads();
  const int Mh = M >> 1;
  const int64_t q = static_cast<int64_t>(Mh) * Mh;
  for (int e = threadIdx.x; e < SO * SO; e += kFwdThreads) {
    const int i = e / SO, j = e - i * SO;
    const float4 c = col_taps<L>(R + 2 * i * SO + j, SO, t);
    if (LEV < NL) X[e] = c.x;
    if (i < OWN && j < OWN && i0 * OWN + i < Mh && j0 * OWN + j < Mh) {
      const int64_t at = static_cast<int64_t>(i0 * OWN + i) * Mh + j0 * OWN + j;
      out[q + at] = c.y;
      out[2 * q + at] = c.z;
      out[3 * q + at] = c.w;
      if (LEV == NL) ll[at] = c.x;
    }
  }
  if constexpr (LEV < NL) {
    __syncthreads();
    fwd_levels<L, NL, T, LEV + 1>(X, R, Mh, i0, j0, ll, out, t);
  }
}

template <int L, int NL, int T>
__global__ __launch_bounds__(kFwdThreads) void k_dwt_fwd(FwdPtrs P, int M, Taps t) {
  extern __shared__ __align__(16) float lds[];
  constexpr int S = footprint(L, NL, T), OWN = T << NL;
  const float* __restrict__ A = P.src[blockIdx.z];
  const int i0 = blockIdx.y, j0 = blockIdx.x;
  constexpr int IT = (S * S + kFwdThreads - 1) / kFwdThreads;
  const int w0 = wave_first();
#pragma unroll
  for (int k = 0; k < IT; ++k) {   // the last wavefronts' lanes beyond the footprint fill the row buffer's start
    const int e = static_cast<int>(threadIdx.x) + k * kFwdThreads;
    if (w0 + k * kFwdThreads < S * S) {
      const int r = e / S, c = e - r * S;
      load_lds(A + static_cast<size_t>((i0 * OWN + r) & (M - 1)) * M + ((j0 * OWN + c) & (M - 1)), lds + w0 + k * kFwdThreads);
    }
  }
  loads_done();
  fwd_levels<L, NL, T, 1>(lds, reinterpret_cast<float2*>(lds + S * S), M, i0, j0, P.ll[blockIdx.z], P.out[blockIdx.z], t);
}

// All levels from side M <= kTailSide down, one block per image.
constexpr int kTailSide = 128, kTailThreads = 1024;

template <int L>
__global__ __launch_bounds__(kTailThreads) void k_dwt_fwd_tail(FwdPtrs P, int lm, int levels, Taps t) {
  extern __shared__ __align__(16) float lds[];
  int M = 1 << lm;
  const float* A = P.src[blockIdx.z];   // may be out: all of it is read before the first store
  float* out = P.out[blockIdx.z];
  float* X = lds;
  float2* R = reinterpret_cast<float2*>(lds + M * M);
  const int w0 = wave_first();
  if (M >= 8) {   // whole wavefronts
    for (int e = w0; e < M * M; e += kTailThreads) load_lds(A + e + (threadIdx.x & 63), X + e);
  } else if (threadIdx.x < M * M) {
    X[threadIdx.x] = A[threadIdx.x];
  }
  loads_done();
  for (int lev = 0; lev < levels; ++lev, M >>= 1, --lm) {
    const int Mh = M >> 1, q = Mh * Mh;
    for (int e = threadIdx.x; e < M * Mh; e += kTailThreads) {
      const int r = e >> (lm - 1), j = e & (Mh - 1);
      float l = 0.f, h = 0.f;
#pragma unroll
      for (int m = 0; m < L; m += 2) {
        const float2 v = *reinterpret_cast<const float2*>(X + r * M + ((2 * j + m) & (M - 1)));
        l = fmaf(t.h[m], v.x, l);
        h = fmaf(t.g[m], v.x, h);
        l = fmaf(t.h[m + 1], v.y, l);
        h = fmaf(t.g[m + 1], v.y, h);
      }
      R[e] = make_float2(l, h);
    }
    __syncthreads();
    const bool last = lev + 1 == levels;
    for (int e = threadIdx.x; e < q; e += kTailThreads) {
      const int i = e >> (lm - 1), j = e & (Mh - 1);
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int m = 0; m < L; ++m) {
        const float2 v = R[((2 * i + m) & (M - 1)) * Mh + j];
        a.x = fmaf(t.h[m], v.x, a.x);
        a.y = fmaf(t.h[m], v.y, a.y);
        a.z = fmaf(t.g[m], v.x, a.z);
        a.w = fmaf(t.g[m], v.y, a.w);
      }
      (last ? out : X)[e] = a.x;
      out[q + e] = a.y;
      out[2 * q + e] = a.z;
      out[3 * q + e] = a.w;
    }
    __syncthreads();
  }
}

// Inverse.  An interval of E positions needs the positions (first - L + 2) / 2
// .. last / 2 of the level below; the largest extent that can be:
constexpr int coarser(int L, int E) { return (E + L - 1) / 2 + 1; }
constexpr int kInvThreads = 512;
constexpr int kMaxLevels = 24;

struct InvPlan {
  int levels;
  int wide;                  // the outputs are 8-byte aligned
  int log_row[kMaxLevels + 1];   // levels from 2 on: log2 of the row stride in LDS
  int plane[kMaxLevels + 1];     // floats of one subband (whole wavefronts)
  int off[kMaxLevels + 1];       // LDS floats before level l's three details
  int ll, rows;              // LDS floats before the approximation and the row buffer
};

// First position and extent on the level below of [a0, a0 + e).
template <int L>
__device__ __forceinline__ void below(int a0, int e, int& a1, int& e1) {
  a1 = (a0 - L + 2) >> 1;
  e1 = ((a0 + e - 1) >> 1) - a1 + 1;
}

// Rows r0 .. r0 + re - 1 (one column) from the level below: rows 2 i and 2 i +
// 1 from positions i - L / 2 + 1 .. i of the column at `at` (row i there).
template <int L>
__device__ __forceinline__ void inv_column(const float* LLb, const float* d, int dstride, int at, int X, const Taps& t,
                                           float2& ev, float2& od) {
  ev = od = make_float2(0.f, 0.f);
#pragma unroll
  for (int k = 0; k < L / 2; ++k, at -= X) {
    const float x00 = LLb[at], x01 = d[at], x10 = d[dstride + at], x11 = d[2 * dstride + at];
    ev.x = fmaf(t.g[2 * k], x10, fmaf(t.h[2 * k], x00, ev.x));
    ev.y = fmaf(t.g[2 * k], x11, fmaf(t.h[2 * k], x01, ev.y));
    od.x = fmaf(t.g[2 * k + 1], x10, fmaf(t.h[2 * k + 1], x00, od.x));
    od.y = fmaf(t.g[2 * k + 1], x11, fmaf(t.h[2 * k + 1], x01, od.y));
  }
}

// The same along a row of column results {from the row low-pass, high-pass}.
template <int L>
__device__ __forceinline__ float2 inv_row(const float2* row, const Taps& t) {
  float2 o = make_float2(0.f, 0.f);
#pragma unroll
  for (int k = 0; k < L / 2; ++k) {
    const float2 v = row[-k];
    o.x = fmaf(t.g[2 * k], v.y, fmaf(t.h[2 * k], v.x, o.x));
    o.y = fmaf(t.g[2 * k + 1], v.y, fmaf(t.h[2 * k + 1], v.x, o.y));
  }
  return o;
}

// T x T pixels per block, T even and a divisor of n: on level 1 every extent is
// a constant, coarser ones depend on the parity of the block's place.
template <int L, int T>
__global__ __launch_bounds__(kInvThreads) void k_dwt_inv(InvPtrs P, InvPlan pl, int n, Taps t) {
  extern __shared__ __align__(16) float lds[];
  constexpr int H = T / 2, X1 = H + L / 2 - 1;   // level 1: new pairs and footprint
  constexpr int kPlane = (X1 * X1 + 63) & ~63;
  const float* __restrict__ in = P.in[blockIdx.z];
  float* __restrict__ dst = P.dst[blockIdx.z];
  const int p0 = blockIdx.y * T, q0 = blockIdx.x * T;
  const int r1 = p0 / 2 - L / 2 + 1, c1 = q0 / 2 - L / 2 + 1;
  float* LLb = lds + pl.ll;
  __shared__ int4 ivals[kMaxLevels + 1];   // first row, first column, rows, columns of each level
  const auto iv = [&](int l, int k) { return __builtin_amdgcn_readfirstlane(reinterpret_cast<const int*>(ivals + l)[k]); };
  if (threadIdx.x == 0) ivals[1] = make_int4(r1, c1, X1, X1);
  // every coefficient the block depends on
  {
    const int s = n >> 1, m = s - 1;
    const int64_t q = static_cast<int64_t>(s) * s;
    const int w0 = wave_first();
#pragma unroll
    for (int k = 0; k < (X1 * X1 + kInvThreads - 1) / kInvThreads; ++k) {
      const int e = static_cast<int>(threadIdx.x) + k * kInvThreads, we = w0 + k * kInvThreads;
      if (we < X1 * X1) {   // lanes beyond fill the padding of each plane
        const int r = e / X1, c = e - r * X1;
        const float* src = in + static_cast<int64_t>((r1 + r) & m) * s + ((c1 + c) & m);
        load_lds(src + q, lds + we);
        load_lds(src + 2 * q, lds + kPlane + we);
        load_lds(src + 3 * q, lds + 2 * kPlane + we);
        if (pl.levels == 1) load_lds(src, LLb + we);
      }
    }
    int ra = r1, ca = c1, re = X1, ce = X1;
    for (int l = 2; l <= pl.levels; ++l) {
      int rb, cb, rn, cn;
      below<L>(ra, re, rb, rn);
      below<L>(ca, ce, cb, cn);
      if (threadIdx.x == 0) ivals[l] = make_int4(rb, cb, rn, cn);
      const int sl = n >> l, ml = sl - 1, lw = pl.log_row[l];
      const int64_t ql = static_cast<int64_t>(sl) * sl;
      float* d = lds + pl.off[l];
      const int plane = pl.plane[l], cnt = rn << lw;
      for (int we = w0; we < cnt; we += kInvThreads) {
        const int e = we + (static_cast<int>(threadIdx.x) & 63), r = e >> lw, c = e & ((1 << lw) - 1);
        const float* src = in + static_cast<int64_t>((rb + r) & ml) * sl + ((cb + c) & ml);
        load_lds(src + ql, d + we);
        load_lds(src + 2 * ql, d + plane + we);
        load_lds(src + 3 * ql, d + 2 * plane + we);
        if (l == pl.levels) load_lds(src, LLb + we);
      }
      ra = rb;
      ca = cb;
      re = rn;
      ce = cn;
    }
  }
  loads_done();
  float2* R = reinterpret_cast<float2*>(lds + pl.rows);
  for (int l = pl.levels; l >= 2; --l) {
    // the intervals of level l - 1, which this makes, and of level l
    const int r0 = iv(l - 1, 0), c0 = iv(l - 1, 1), re = iv(l - 1, 2), ce = iv(l - 1, 3);
    const int ra = iv(l, 0), ca = iv(l, 1), cn = iv(l, 3);
    const int lw = pl.log_row[l], X = 1 << lw, Y = l == 2 ? X1 : 1 << pl.log_row[l - 1];
    const float* d = lds + pl.off[l];
    {
      const int i0 = r0 >> 1, ni = ((r0 + re - 1) >> 1) - i0 + 1, c = threadIdx.x & ((1 << lw) - 1);
      if (c < cn)
        for (int i = threadIdx.x >> lw; i < ni; i += kInvThreads >> lw) {
          float2 ev, od;
          inv_column<L>(LLb, d, pl.plane[l], (i0 + i - ra) * X + c, X, t, ev, od);
          const int o = 2 * (i0 + i) - r0;
          if (o >= 0) R[o * X + c] = ev;
          if (o + 1 < re) R[(o + 1) * X + c] = od;
        }
    }
    __syncthreads();
    {
      const int j0 = c0 >> 1, nj = ((c0 + ce - 1) >> 1) - j0 + 1, j = threadIdx.x & ((1 << lw) - 1);
      if (j < nj)
        for (int r = threadIdx.x >> lw; r < re; r += kInvThreads >> lw) {
          const float2 v = inv_row<L>(R + r * X + (j0 + j - ca), t);
          const int o = 2 * (j0 + j) - c0;
          if (o >= 0) LLb[r * Y + o] = v.x;
          if (o + 1 < ce) LLb[r * Y + o + 1] = v.y;
        }
    }
    __syncthreads();
  }
  for (int e = threadIdx.x; e < H * X1; e += kInvThreads) {
    const int i = e / X1, c = e - i * X1;
    float2 ev, od;
    inv_column<L>(LLb, lds, kPlane, (i + L / 2 - 1) * X1 + c, X1, t, ev, od);
    R[2 * i * X1 + c] = ev;
    R[(2 * i + 1) * X1 + c] = od;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < T * H; e += kInvThreads) {
    const int r = e / H, j = e - r * H;
    const float2 v = inv_row<L>(R + r * X1 + j + L / 2 - 1, t);
    float* o = dst + static_cast<int64_t>(p0 + r) * n + q0 + 2 * j;
    if (pl.wide) {
      *reinterpret_cast<float2*>(o) = v;
    } else {
      o[0] = v.x;
      o[1] = v.y;
    }
  }
}

// Calls f with the filter length as a compile-time constant.
template <typename F>
void with_taps(int L, F&& f) {
  switch (L) {
    case 2: f(std::integral_constant<int, 2>{}); return;
    case 8: f(std::integral_constant<int, 8>{}); return;
    case 12: f(std::integral_constant<int, 12>{}); return;
    default: fail(WDB_ERR_ARG, "no transform for a filter of %d taps", L);
  }
}

// Dynamic LDS that a block of any of these kernels may take: what is left beside
// k_dwt_inv's intervals (the runtime refuses a limit that does not fit with them).
constexpr size_t kDynLds = 160 * 1024 - sizeof(int4) * (kMaxLevels + 1);

// Launches with more than 64 KiB of LDS (on the inverse: 12 taps from 6 levels
// on, 8 taps from 10) need the kernel's limit raised, once per device (`done`: a
// bit per device).
void raise_lds(const void* kernel, size_t bytes, std::atomic<uint64_t>& done) {
  if (bytes <= 64 * 1024) return;
  int dev = 0;
  WDB_HIP(hipGetDevice(&dev));
  const uint64_t bit = uint64_t{1} << (dev & 63);
  if (done.load() & bit) return;
  WDB_HIP(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kDynLds));
  done.fetch_or(bit);
}

// Levels of a launch that starts at side M > kTailSide with `left` levels to
// go: down to a side of 64 for the tail (a block alone takes 6 us on 128 x 128,
// 2 us on 64 x 64), at most three.  Above a side of 1024 another launch of many
// blocks follows anyway, and two levels with their larger tile cost less.
int launch_levels(int M, int left) {
  const int most = M > 1024 ? 2 : 3;
  int nl = 1;
  while (nl < most && nl < left && (M >> nl) > 64) ++nl;
  return nl;
}

}  // namespace

DwtScratch dwt_scratch(int n, int levels) {
  DwtScratch need;
  int M = n, left = levels, turn = 0;
  while (M > kTailSide && left > 0) {
    const int nl = launch_levels(M, left);
    M >>= nl;
    left -= nl;
    if (left > 0 && M > kTailSide) {   // the approximation another launch of many blocks reads
      size_t& part = turn ? need.b : need.a;
      part = std::max(part, static_cast<size_t>(M) * M);
      turn ^= 1;
    }
  }
  return need;
}

void dwt_forward_many(int n, int levels, const Filter& f, int count, const float* const* in, float* const* out,
                      float* const* scratch_a, float* const* scratch_b, hipStream_t s) {
  const Taps t = to_taps(f);
  with_taps(t.L, [&](auto Lc) {
    constexpr int L = decltype(Lc)::value;
    for (int b0 = 0; b0 < count; b0 += kBatch) {
      const int nb = std::min(kBatch, count - b0);
      FwdPtrs P{};
      for (int z = 0; z < nb; ++z) {
        P.src[z] = in[b0 + z];
        P.out[z] = out[b0 + z];
      }
      int M = n, left = levels, turn = 0;
      while (left > 0) {
        // one level of an image of side 128 alone: 16 blocks an image instead of one
        // (8 taps: a call 23.3 -> 19.1 us for one image, 29.5 -> 21.9 us for 60; two
        // levels from one block take 24.5 us, a launch per level 27.8 us)
        const bool alone = M == kTailSide && M == n && left == 1;
        if (M <= kTailSide && !alone) {
          const size_t bytes = (static_cast<size_t>(M) * M * 2) * sizeof(float);
          static std::atomic<uint64_t> done{0};
          raise_lds(reinterpret_cast<const void*>(k_dwt_fwd_tail<L>), bytes, done);
          hipLaunchKernelGGL(k_dwt_fwd_tail<L>, dim3(1, 1, nb), dim3(kTailThreads), bytes, s, P,
                             __builtin_ctz(static_cast<unsigned>(M)), left, t);
          break;
        }
        const int nl = launch_levels(M, left);
        const bool on = left > nl && (M >> nl) > kTailSide;   // another launch of many blocks follows
        for (int z = 0; z < nb; ++z)
          P.ll[z] = on ? (turn ? scratch_b : scratch_a)[b0 + z] : out[b0 + z];
        turn ^= 1;
        // the larger tile (less overlap) where it gives every compute unit a block
        const int big = nl == 1 ? 32 : nl == 2 ? 16 : 8;
        const int64_t blocks = static_cast<int64_t>((M >> nl) / big) * ((M >> nl) / big) * nb;
        const auto go = [&](auto Nc, auto Tc) {
          constexpr int NL = decltype(Nc)::value, T = decltype(Tc)::value;
          constexpr size_t bytes = fwd_lds_floats<L, NL, T>() * sizeof(float);
          static std::atomic<uint64_t> done{0};
          raise_lds(reinterpret_cast<const void*>(k_dwt_fwd<L, NL, T>), bytes, done);
          const int side = ((M >> nl) + T - 1) / T;
          hipLaunchKernelGGL((k_dwt_fwd<L, NL, T>), dim3(side, side, nb), dim3(kFwdThreads), bytes, s, P, M, t);
        };
        using std::integral_constant;
        if (nl == 1 && blocks >= 256) go(integral_constant<int, 1>{}, integral_constant<int, 32>{});
        else if (nl == 1) go(integral_constant<int, 1>{}, integral_constant<int, 16>{});
        else if (nl == 2 && blocks >= 256) go(integral_constant<int, 2>{}, integral_constant<int, 16>{});
        else if (nl == 2) go(integral_constant<int, 2>{}, integral_constant<int, 8>{});
        else go(integral_constant<int, 3>{}, integral_constant<int, 8>{});
        for (int z = 0; z < nb; ++z) P.src[z] = P.ll[z];
        M >>= nl;
        left -= nl;
      }
      WDB_HIP(hipGetLastError());
    }
  });
}

void dwt_inverse_many(int n, int levels, const Filter& f, int count, const float* const* in, float* const* out,
                      hipStream_t s) {
  const Taps t = to_taps(f);
  WDB_REQUIRE(levels <= kMaxLevels, WDB_ERR_LEVELS, "at most %d levels", kMaxLevels);
  // 64 x 64 pixels per block where that gives every compute unit one, smaller below
  const int64_t tiles64 = static_cast<int64_t>(n / 64) * (n / 64) * count;
  const int T = n < 32 ? n : tiles64 >= 256 ? 64 : 32;
  with_taps(t.L, [&](auto Lc) {
    constexpr int L = decltype(Lc)::value;
    InvPlan pl{};
    pl.levels = levels;
    int ext = T / 2 + L / 2 - 1, plane = (ext * ext + 63) & ~63;   // of level 1
    int at = 3 * plane, big = plane, most = T * ext;
    for (int l = 2; l <= levels; ++l) {
      const int above = ext;
      ext = coarser(L, ext);
      const int lw = ext <= 16 ? 4 : ext <= 32 ? 5 : 6;
      pl.log_row[l] = lw;
      pl.plane[l] = ((ext << lw) + 63) & ~63;
      pl.off[l] = at;
      at += 3 * pl.plane[l];
      big = std::max(big, pl.plane[l]);
      most = std::max(most, above << lw);   // the row buffer: rows of a level by the row stride below
    }
    pl.ll = at;
    pl.rows = at + big;
    const size_t bytes = (pl.rows + 2 * static_cast<size_t>(most)) * sizeof(float);
    WDB_REQUIRE(bytes <= kDynLds, WDB_ERR_LEVELS, "the inverse transform's levels do not fit on chip");
    for (int b0 = 0; b0 < count; b0 += kBatch) {
      const int nb = std::min(kBatch, count - b0);
      InvPtrs P{};
      pl.wide = 1;
      for (int z = 0; z < nb; ++z) {
        P.in[z] = in[b0 + z];
        P.dst[z] = out[b0 + z];
        if (reinterpret_cast<uintptr_t>(P.dst[z]) & 7) pl.wide = 0;
      }
      const auto go = [&](auto Tc) {
        constexpr int TT = decltype(Tc)::value;
        static std::atomic<uint64_t> done{0};
        raise_lds(reinterpret_cast<const void*>(k_dwt_inv<L, TT>), bytes, done);
        hipLaunchKernelGGL((k_dwt_inv<L, TT>), dim3(n / TT, n / TT, nb), dim3(kInvThreads), bytes, s, P, pl, n, t);
      };
      switch (T) {
        case 2: go(std::integral_constant<int, 2>{}); break;
        case 4: go(std::integral_constant<int, 4>{}); break;
        case 8: go(std::integral_constant<int, 8>{}); break;
        case 16: go(std::integral_constant<int, 16>{}); break;
        case 32: go(std::integral_constant<int, 32>{}); break;
        default: go(std::integral_constant<int, 64>{}); break;
      }
      WDB_HIP(hipGetLastError());
    }
  });
}

void dwt_forward(int n, int levels, const Filter& f, const float* in, float* out, float* scratch_a,
                 float* scratch_b, hipStream_t s) {
  dwt_forward_many(n, levels, f, 1, &in, &out, &scratch_a, &scratch_b, s);
}

void dwt_inverse(int n, int levels, const Filter& f, const float* in, float* out, hipStream_t s) {
  dwt_inverse_many(n, levels, f, 1, &in, &out, s);
}

}  // namespace wdb

extern "C" wdb_status wdb_dwt(int32_t n, int32_t wavelet, int32_t levels, const float* in, float* out,
                              int32_t inverse, void* stream) {
  WDB_API_BEGIN
  WDB_REQUIRE(in && out, WDB_ERR_ARG, "null buffer");
  WDB_REQUIRE(in != out, WDB_ERR_ARG, "in and out must not alias");
  wdb::Filter f = wdb::make_filter(wavelet);
  wdb::check_geometry(n, levels, static_cast<int>(f.h.size()));
  hipStream_t s = static_cast<hipStream_t>(stream);
  const wdb::DwtScratch need = inverse ? wdb::DwtScratch{} : wdb::dwt_scratch(n, levels);
  wdb::DevBuf<float> scratch(need.a + need.b);
  if (inverse)
    wdb::dwt_inverse(n, levels, f, in, out, s);
  else
    wdb::dwt_forward(n, levels, f, in, out, scratch.p, scratch.p + need.a, s);
  WDB_HIP(hipStreamSynchronize(s));
  WDB_API_END
}

extern "C" wdb_status wdb_dwt_batched(int32_t n, int32_t wavelet, int32_t levels, int32_t count, const float* in,
                                      float* out, int32_t inverse, void* stream) {
  WDB_API_BEGIN
  WDB_REQUIRE(in && out, WDB_ERR_ARG, "null buffer");
  WDB_REQUIRE(count >= 1, WDB_ERR_ARG, "count %d must be >= 1", count);
  wdb::Filter f = wdb::make_filter(wavelet);
  wdb::check_geometry(n, levels, static_cast<int>(f.h.size()));
  const int64_t N = static_cast<int64_t>(n) * n;
  const char* ib = reinterpret_cast<const char*>(in);
  const char* ie = reinterpret_cast<const char*>(in + N * count);
  const char* ob = reinterpret_cast<const char*>(out);
  const char* oe = reinterpret_cast<const char*>(out + N * count);
  WDB_REQUIRE(ie <= ob || oe <= ib, WDB_ERR_ARG, "in and out must not overlap");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const wdb::DwtScratch need = inverse ? wdb::DwtScratch{} : wdb::dwt_scratch(n, levels);
  const int nsc = std::min(count, wdb::kBatch);
  wdb::DevBuf<float> scratch((need.a + need.b) * nsc);
  std::vector<const float*> ip(count);
  std::vector<float*> op(count), sa(count), sb(count);
  for (int i = 0; i < count; ++i) {
    ip[i] = in + N * i;
    op[i] = out + N * i;
    sa[i] = scratch.p + (need.a + need.b) * (i % nsc);   // images of one launch use distinct scratch; launches are in order
    sb[i] = sa[i] + need.a;
  }
  if (inverse)
    wdb::dwt_inverse_many(n, levels, f, count, ip.data(), op.data(), s);
  else
    wdb::dwt_forward_many(n, levels, f, count, ip.data(), op.data(), sa.data(), sb.data(), s);
  WDB_HIP(hipStreamSynchronize(s));
  WDB_API_END
}

extern "C" wdb_status wdb_synthesize(const wdb_theta* th, const float* x, float* u_hat, void* stream) {
  WDB_API_BEGIN
  WDB_REQUIRE(th && x && u_hat, WDB_ERR_ARG, "null argument");
  WDB_REQUIRE(static_cast<const void*>(x) != static_cast<const void*>(u_hat), WDB_ERR_ARG,
              "x and u_hat must not alias");
  WDB_HIP(hipSetDevice(th->device));
  wdb::Filter f = wdb::make_filter(th->wavelet);
  wdb::dwt_inverse(th->n, th->levels, f, x, u_hat, static_cast<hipStream_t>(stream));
  WDB_API_END
}

// ---------------------------------------------------------------------------
// Transform without allocation.  The level-to-level intermediates live in a
// fixed device array instead of a per-call allocation: each GPU the library
// runs on holds its own copy (kNoAllocScratch floats, 8 MiB, enough for
// n <= 2048) until the process ends.  Host code never passes the array's name
// to a kernel: its device address is looked up once per device with
// hipGetSymbolAddress and only that address is used.  Every level writes the
// intermediate it later reads, so the array needs no clearing; calls that
// overlap on one GPU (different streams or threads) share it and race.
// ---------------------------------------------------------------------------
namespace {
constexpr int kNoAllocMaxN = 2048;
constexpr size_t kNoAllocScratch = 2 * static_cast<size_t>(kNoAllocMaxN / 2) * (kNoAllocMaxN / 2);
constexpr int kMaxDevices = 64;
static __device__ __align__(256) float scratch[kNoAllocScratch];

std::mutex g_scratch_mu;
float* g_scratch_ptr[kMaxDevices] = {};

// Device address of this device's scratch array (looked up on first use).
float* scratch_address() {
  int dev = 0;
  WDB_HIP(hipGetDevice(&dev));
  WDB_REQUIRE(dev >= 0 && dev < kMaxDevices, WDB_ERR_ARG, "device index %d beyond %d", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    WDB_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    WDB_REQUIRE(ptr != nullptr, WDB_ERR_HIP, "no device address for the transform scratch array");
    g_scratch_ptr[dev] = static_cast<float*>(ptr);
  }
  return g_scratch_ptr[dev];
}
}  // namespace

extern "C" wdb_status wdb_dwt_noalloc(int32_t n, int32_t wavelet, int32_t levels, const float* in, float* out,
                                      int32_t inverse, void* stream) {
  WDB_API_BEGIN
  WDB_REQUIRE(in && out, WDB_ERR_ARG, "null buffer");
  WDB_REQUIRE(in != out, WDB_ERR_ARG, "in and out must not alias");
  wdb::Filter f = wdb::make_filter(wavelet);
  wdb::check_geometry(n, levels, static_cast<int>(f.h.size()));
  WDB_REQUIRE(n <= kNoAllocMaxN, WDB_ERR_SIZE,
              "wdb_dwt_noalloc: image side %d exceeds the fixed scratch limit of %d (use wdb_dwt)", n, kNoAllocMaxN);
  float* sc = scratch_address();
  const size_t q = static_cast<size_t>(n / 2) * (n / 2);
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (inverse)
    wdb::dwt_inverse(n, levels, f, in, out, s);
  else
    wdb::dwt_forward(n, levels, f, in, out, sc, sc + q, s);
  WDB_API_END
}
