// Theta_K = K largest-magnitude entries of Theta = Psi^* H Psi (Sec. 3.4,
// Sec. 3.7 naive rule), computed on the GPU in float64.
//
// Column b of Theta is Psi^*(H psi_b).  The paper notes that applying H to
// all N atoms and transforming them is O(N^3) for a spatially varying blur
// (Sec. 3.4).  Here each column is computed on its support only:
//
//  * psi_b is separable: f_erow,l(r - 2^l p) * f_ecol,l(c - 2^l q), with the
//    level-l equivalent filters f_0,l / f_1,l (the cascade of h and g that
//    maps pixels to level-l coefficients, periodised to n).
//  * H psi_b is non-zero only on the atom's window dilated by the PSF radius
//    R; it is gathered pixel by pixel in float64 from the source PSFs.
//  * Psi^* of that window is a local pyramid: at each level only the
//    coefficients whose footprint meets the current window are formed, with
//    periodic index arithmetic, so every non-zero <psi_a, H psi_b> of the
//    column is produced exactly once.
//
// One workgroup owns one column at a time (float64 window buffers in LDS, or in
// a per-workgroup slab of global memory where they do not fit).  The K largest
// magnitudes are found by a radix select on the IEEE bit pattern of |theta|: each
// histogram pass recomputes every column and counts 12-bit digits of the keys
// that match the prefix fixed so far; once the boundary digit holds few enough
// entries, an emit pass writes the entries above the boundary and collects the
// boundary digit, of which the same select on the collected list then keeps the
// entries by (|theta| descending, a*N + b ascending).  The kept triples are
// then sorted into CSR.
//
// A column is bound by its weights: every one of them is met by hundreds of
// columns.  So they are computed once into a table (all offsets of all sources),
// and a column reads only the offsets that lie in its atom and that any source
// nearby reaches.  The sums keep their terms and their order.  256 x 256,
// sigma 3 and 1, db4, 4 levels: a pass over all columns 48 -> 16 ms, the kept
// part of the boundary (a sort on the host before) 110 -> 0.5 ms.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <numeric>

#include "common.hpp"
#include "psf.hpp"

namespace wdb {

namespace {

constexpr int kMaxSub = 48;
constexpr int kMaxLev = 16;
constexpr int kDigits = 4096;
constexpr unsigned long long kBoundaryCap = 1ull << 22;

struct Geom {
  int n, J, L, R, nsub;
  int sub_level[kMaxSub], sub_er[kMaxSub], sub_ec[kMaxSub], sub_side[kMaxSub];
  int64_t sub_off[kMaxSub + 1];
  int flen[kMaxLev];
  int64_t foff[kMaxLev];
  double h[kMaxTaps], g[kMaxTaps];
};

struct Select {
  int mode;   // 0: histogram, 1: emit above prefix + collect prefix, 2: emit every non-zero
  int scaled; // 1: rank by sigma_b |theta| with sigma_b = 2^-k = 1 / (side of b's subband) (Sec. 3.7)
  int pbits;  // bits of the key already fixed
  int shift;  // histogram digit position
  unsigned long long prefix;
  unsigned long long dmask;
};

struct Emit {
  int32_t* row;
  int32_t* col;
  double* val;
  unsigned long long* count;
  unsigned long long cap;
};

struct Win {
  int s, len, M;  // positions (s + t) mod M for t < len
};

__host__ __device__ inline int floordiv2(int a) { return a >= 0 ? a / 2 : -((-a + 1) / 2); }

// Window of level-(l+1) positions whose footprint [2i, 2i + L - 1] meets w.
__host__ __device__ inline Win next_win(Win w, int L) {
  const int Mh = w.M >> 1;
  if (w.len >= w.M) return Win{0, Mh, Mh};
  const int lo = floordiv2(w.s - L + 2);
  const int hi = floordiv2(w.s + w.len - 1);
  const int len = hi - lo + 1;
  if (len >= Mh) return Win{0, Mh, Mh};
  return Win{lo & (Mh - 1), len, Mh};
}

__device__ inline void emit_one(bool want, int a, int b, double v, const Emit& E, int* err) {
  const unsigned long long mask = __ballot(want);
  if (mask == 0ull) return;
  const int lane = __lane_id();
  const int leader = __ffsll(static_cast<long long>(mask)) - 1;
  unsigned long long base = 0;
  if (lane == leader) base = atomicAdd(E.count, static_cast<unsigned long long>(__popcll(mask)));
  const unsigned lo = __shfl(static_cast<unsigned>(base & 0xffffffffull), leader);
  const unsigned hi = __shfl(static_cast<unsigned>(base >> 32), leader);
  base = (static_cast<unsigned long long>(hi) << 32) | lo;
  if (want) {
    const unsigned long long idx = base + __popcll(mask & ((1ull << lane) - 1ull));
    if (idx < E.cap) {
      E.row[idx] = a;
      E.col[idx] = b;
      E.val[idx] = v;
    } else {
      atomicOr(err, 2);
    }
  }
}

// sb: the column's ranking weight (1, or sigma_b; a power of two, so the
// scaled magnitude is exact).
__device__ inline void handle(const Select& S, double v, double sb, int a, int b, unsigned* lhist, const Emit& out,
                              const Emit& bnd, int* err) {
  const bool nz = v != 0.0;
  const unsigned long long key = static_cast<unsigned long long>(__double_as_longlong(fabs(v) * sb));
  if (S.mode == 0) {
    if (nz && (S.pbits == 0 || (key >> (64 - S.pbits)) == S.prefix))
      atomicAdd(&lhist[(key >> S.shift) & S.dmask], 1u);
  } else if (S.mode == 2) {
    emit_one(nz, a, b, v, out, err);
  } else {
    const unsigned long long top = key >> (64 - S.pbits);
    emit_one(nz && top > S.prefix, a, b, v, out, err);
    emit_one(nz && top == S.prefix, a, b, v, bnd, err);
  }
}

// Normalised weights of all sources: wt[(dy (2R + 1) + dx + R) N + s], dy = 0 .. R.
__global__ __launch_bounds__(256) void k_weights(PsfDev P, double* __restrict__ wt) {
  const int64_t N = static_cast<int64_t>(P.n) * P.n;
  const int64_t s = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (s >= N) return;
  const int dy = static_cast<int>(blockIdx.y);
  for (int dx = -P.R; dx <= P.R; ++dx) {
    const double w = psf_unnormalised(P, s, dy, dx);
    wt[(static_cast<int64_t>(blockIdx.y) * (2 * P.R + 1) + dx + P.R) * N + s] = w != 0.0 ? w / P.Z[s] : 0.0;
  }
}

constexpr int kReach = 16;   // side of the tiles whose reach is kept

// Table of the field's weights and, per row offset and kReach x kReach tile
// (source rows, target columns), the column offsets with a weight other than 0.
// Row offsets below 0 read the weights and offsets of -dy, -dx.
struct Weights {
  const double* wt = nullptr;   // nullptr: weights are evaluated where they are used
  short2* reach = nullptr;      // [dy][row tile][column tile], dy = 0 .. R
  int tiles = 0;
};

// Reach of the sources of rows 16 blockIdx.y .. and of all columns that a target of
// columns 16 blockIdx.x .. meets, at dy = blockIdx.z.
__global__ __launch_bounds__(256) void k_weight_reach(int n, int R, Weights T) {
  __shared__ int lo, hi;
  if (threadIdx.x == 0) {
    lo = R + 1;
    hi = -R - 1;
  }
  __syncthreads();
  const int64_t N = static_cast<int64_t>(n) * n;
  const int rows = min(kReach, n), cols = min(kReach + 2 * R, n);
  for (int e = threadIdx.x; e < rows * cols; e += blockDim.x) {
    const int r = static_cast<int>(blockIdx.y) * kReach + e / cols;
    const int c = (static_cast<int>(blockIdx.x) * kReach - R + e % cols) & (n - 1);
    const double* w = T.wt + static_cast<int64_t>(blockIdx.z) * (2 * R + 1) * N + static_cast<int64_t>(r) * n + c;
    int first = -R, last = R;
    while (first <= R && w[(first + R) * N] == 0.0) ++first;
    while (last >= first && w[(last + R) * N] == 0.0) --last;
    if (first <= last) {
      atomicMin(&lo, first);
      atomicMax(&hi, last);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0)
    T.reach[(static_cast<int64_t>(blockIdx.z) * T.tiles + blockIdx.y) * T.tiles + blockIdx.x] =
        make_short2(static_cast<short>(lo), static_cast<short>(hi));
}

// H psi_b at pixel (orow, ocol) of its window: the terms in ascending (dy, dx).
struct Atom {
  const double *fr, *fc;   // row and column filter of length wl
  int wl, r0, c0, hr0, hc0;
};

// From the table, where the window does not wrap onto itself.
__device__ __forceinline__ double blurred_atom_table(const Weights& T, int n, int R, const Atom& A, int orow, int ocol) {
  const int64_t N = static_cast<int64_t>(n) * n;
  const int ic = (A.hc0 + ocol) & (n - 1);
  // atom row (column) tr = orow - R - dy, tc = ocol - R - dx
  const int dy0 = max(-R, orow - R - A.wl + 1), dy1 = min(R, orow - R);
  const int dx0 = max(-R, ocol - R - A.wl + 1), dx1 = min(R, ocol - R);
  double acc = 0.0;
  for (int dy = dy0; dy <= dy1; ++dy) {
    const int tr = orow - R - dy, sr = (A.r0 + tr) & (n - 1);
    const int up = dy < 0 ? -dy : dy;
    const short2 d = T.reach[(static_cast<int64_t>(up) * T.tiles + sr / kReach) * T.tiles + ic / kReach];
    const int lo = max(dx0, dy < 0 ? -static_cast<int>(d.y) : static_cast<int>(d.x));
    const int hi = min(dx1, dy < 0 ? -static_cast<int>(d.x) : static_cast<int>(d.y));
    const int64_t step = dy < 0 ? -N : N;
    const double vr = A.fr[tr];
    const double* w = T.wt + (static_cast<int64_t>(up) * (2 * R + 1) + R) * N + static_cast<int64_t>(sr) * n;
    // a weight of 0 leaves acc as it is (acc is never -0, the filters are finite)
#pragma unroll 8
    for (int dx = lo; dx <= hi; ++dx) acc += (vr * A.fc[ocol - R - dx]) * w[dx * step + ((ic - dx) & (n - 1))];
  }
  return acc;
}

__device__ double blurred_atom(const PsfDev& P, int n, int R, const Atom& A, int orow, int ocol) {
  const int ir = (A.hr0 + orow) & (n - 1), ic = (A.hc0 + ocol) & (n - 1);
  double acc = 0.0;
  for (int dy = -R; dy <= R; ++dy) {
    const int tr = (ir - dy - A.r0) & (n - 1);
    if (tr >= A.wl) continue;
    const double vr = A.fr[tr];
    const int sr = (A.r0 + tr) & (n - 1);
    for (int dx = -R; dx <= R; ++dx) {
      const int tc = (ic - dx - A.c0) & (n - 1);
      if (tc >= A.wl) continue;
      const int64_t s = static_cast<int64_t>(sr) * n + ((A.c0 + tc) & (n - 1));
      const double w = psf_unnormalised(P, s, dy, dx);
      if (w != 0.0) acc += (vr * A.fc[tc]) * (w / P.Z[s]);
    }
  }
  return acc;
}

// Doubles of a column's buffers: the window, the next level's window (which also
// takes the third, the first the second after it), the row-transformed window.
struct Caps {
  int64_t in = 0, out = 0, mid = 0;
  size_t bytes() const { return static_cast<size_t>(in + out + mid) * sizeof(double); }
};

// Columns b_begin .. b_end - 1, with their buffers in LDS or in scratch.
template <bool LDS>
__global__ __launch_bounds__(256) void k_theta_columns(Geom G, PsfDev P, Weights T, const double* __restrict__ ftab,
                                                       double* __restrict__ scratch, Caps cap,
                                                       int64_t b_begin, int64_t b_end, Select S,
                                                       unsigned long long* __restrict__ ghist, Emit out,
                                                       Emit bnd, int* err) {
  extern __shared__ double win[];
  __shared__ unsigned lhist[kDigits];
  const int tid = threadIdx.x, nt = blockDim.x;
  if (S.mode == 0)
    for (int i = tid; i < kDigits; i += nt) lhist[i] = 0u;
  __syncthreads();
  double* bufA = LDS ? win : scratch + static_cast<size_t>(blockIdx.x) * (cap.in + cap.out + cap.mid);
  double* bufB = bufA + cap.in;
  double* mid = bufB + cap.out;
  const int n = G.n, R = G.R, L = G.L;
  for (int64_t b = b_begin + blockIdx.x; b < b_end; b += gridDim.x) {
    int k = 0;
    while (k + 1 < G.nsub && b >= G.sub_off[k + 1]) ++k;
    const int lev = G.sub_level[k], side = G.sub_side[k];
    const double sb = S.scaled ? 1.0 / static_cast<double>(side) : 1.0;
    const int64_t pos = b - G.sub_off[k];
    const int p = static_cast<int>(pos / side), q = static_cast<int>(pos % side);
    const int wl = G.flen[lev];
    const int r0 = (p << lev) & (n - 1), c0 = (q << lev) & (n - 1);
    // H psi_b on the atom window dilated by R (whole torus if that is wider).
    const int hl = min(wl + 2 * R, n);
    const int hr0 = (r0 - R) & (n - 1), hc0 = (c0 - R) & (n - 1);
    const Atom A{ftab + G.foff[lev] + (G.sub_er[k] ? wl : 0), ftab + G.foff[lev] + (G.sub_ec[k] ? wl : 0),
                 wl, r0, c0, hr0, hc0};
    const bool table = T.wt && wl + 2 * R <= n;
    for (int o = tid; o < hl * hl; o += nt) {
      const int orow = o / hl, ocol = o - orow * hl;
      bufA[o] = table ? blurred_atom_table(T, n, R, A, orow, ocol) : blurred_atom(P, n, R, A, orow, ocol);
    }
    __syncthreads();
    // Local analysis pyramid of the window: rows, then columns.
    Win inr{hr0, hl, n}, inc{hc0, hl, n};
    double* in = bufA;
    double* ob = bufB;
    for (int lv = 1; lv <= G.J; ++lv) {
      const int M = n >> (lv - 1), Mh = M >> 1;
      const Win onr = next_win(inr, L), onc = next_win(inc, L);
      const int cnt = onr.len * onc.len, rows = inr.len * onc.len;
      if (cnt > (lv % 2 ? cap.out : cap.in) || 2 * rows > cap.mid) {
        if (tid == 0) atomicOr(err, 1);
        break;
      }
      for (int o = tid; o < rows; o += nt) {
        const int rr = o / onc.len, oj = o - rr * onc.len;
        const int Jc = (onc.s + oj) & (Mh - 1);
        const double* rowp = in + static_cast<size_t>(rr) * inc.len;
        double lo = 0.0, hi = 0.0;
        for (int m2 = 0; m2 < L; ++m2) {
          const int cc = (2 * Jc + m2 - inc.s) & (M - 1);
          if (cc >= inc.len) continue;
          const double v = rowp[cc];
          lo += G.h[m2] * v;
          hi += G.g[m2] * v;
        }
        mid[2 * o] = lo;
        mid[2 * o + 1] = hi;
      }
      __syncthreads();
      const int ks = 1 + (G.J - lv) * 3;
      for (int o = tid; o < cnt; o += nt) {
        const int oi = o / onc.len, oj = o - oi * onc.len;
        const int I = (onr.s + oi) & (Mh - 1), Jc = (onc.s + oj) & (Mh - 1);
        double a00 = 0.0, a01 = 0.0, a10 = 0.0, a11 = 0.0;
        for (int m = 0; m < L; ++m) {
          const int rr = (2 * I + m - inr.s) & (M - 1);
          if (rr >= inr.len) continue;
          const double lo = mid[2 * (rr * onc.len + oj)], hi = mid[2 * (rr * onc.len + oj) + 1];
          a00 += G.h[m] * lo;
          a01 += G.h[m] * hi;
          a10 += G.g[m] * lo;
          a11 += G.g[m] * hi;
        }
        ob[o] = a00;
        const int64_t loc = static_cast<int64_t>(I) * Mh + Jc;
        handle(S, a01, sb, static_cast<int>(G.sub_off[ks] + loc), static_cast<int>(b), lhist, out, bnd, err);
        handle(S, a10, sb, static_cast<int>(G.sub_off[ks + 1] + loc), static_cast<int>(b), lhist, out, bnd, err);
        handle(S, a11, sb, static_cast<int>(G.sub_off[ks + 2] + loc), static_cast<int>(b), lhist, out, bnd, err);
        if (lv == G.J) handle(S, a00, sb, static_cast<int>(G.sub_off[0] + loc), static_cast<int>(b), lhist, out, bnd, err);
      }
      __syncthreads();
      double* t = in;
      in = ob;
      ob = t;
      inr = onr;
      inc = onc;
    }
  }
  if (S.mode == 0) {
    __syncthreads();
    for (int i = tid; i < kDigits; i += nt)
      if (lhist[i]) atomicAdd(&ghist[i], static_cast<unsigned long long>(lhist[i]));
  }
}

// The collected boundary entries (COO, col < N): their ranked magnitude, or with
// `index` their linear index a * N + b.
struct Boundary {
  Emit e;
  int64_t N, count;
  const double* sigma;   // sigma_b of column b, nullptr: 1
};

__device__ __forceinline__ unsigned long long boundary_key(const Boundary& B, int64_t i) {
  const double v = fabs(B.e.val[i]);
  return static_cast<unsigned long long>(__double_as_longlong(B.sigma ? v * B.sigma[B.e.col[i]] : v));
}

__device__ __forceinline__ unsigned long long boundary_index(const Boundary& B, int64_t i) {
  return static_cast<unsigned long long>(static_cast<int64_t>(B.e.row[i]) * B.N + B.e.col[i]);
}

// Counts a digit: of the magnitudes whose bits above it equal `prefix`; with INDEX
// of the linear indices whose bits above it equal `prefix`, among the entries of
// magnitude `key`.
template <bool INDEX>
__global__ __launch_bounds__(256) void k_boundary_digits(Boundary B, unsigned long long key, unsigned long long prefix,
                                                         int shift, int width, unsigned long long* __restrict__ ghist) {
  __shared__ unsigned lhist[kDigits];
  for (int i = threadIdx.x; i < kDigits; i += blockDim.x) lhist[i] = 0u;
  __syncthreads();
  const int64_t step = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < B.count; i += step) {
    if (INDEX && boundary_key(B, i) != key) continue;
    const unsigned long long x = (INDEX ? boundary_index(B, i) : boundary_key(B, i)) >> shift;
    if ((x >> width) == prefix) atomicAdd(&lhist[x & ((1ull << width) - 1ull)], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kDigits; i += blockDim.x)
    if (lhist[i]) atomicAdd(&ghist[i], static_cast<unsigned long long>(lhist[i]));
}

// Appends the entries above `key`, and those of `key` up to the linear index `last`.
__global__ __launch_bounds__(256) void k_boundary_keep(Boundary B, unsigned long long key, unsigned long long last,
                                                       Emit out, int* err) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  bool want = false;
  int a = 0, b = 0;
  double v = 0.0;
  if (i < B.count) {
    a = B.e.row[i];
    b = B.e.col[i];
    v = B.e.val[i];
    const unsigned long long k = boundary_key(B, i);
    want = k > key || (k == key && boundary_index(B, i) <= last);
  }
  emit_one(want, a, b, v, out, err);
}

// Level-l equivalent filters (index l = 1..J): phi_l = cascade of h,
// psi_l = g applied after l-1 low-pass steps, periodised to length <= n.
void level_filters(const Filter& f, int n, int J, std::vector<double>& tab, Geom& G) {
  const int L = static_cast<int>(f.h.size());
  std::vector<double> phi{1.0};
  tab.clear();
  for (int l = 1; l <= J; ++l) {
    const int up = 1 << (l - 1);
    const int len = static_cast<int>(phi.size()) + up * (L - 1);
    std::vector<double> nphi(len, 0.0), npsi(len, 0.0);
    for (size_t t = 0; t < phi.size(); ++t)
      for (int m = 0; m < L; ++m) {
        nphi[t + up * m] += f.h[m] * phi[t];
        npsi[t + up * m] += f.g[m] * phi[t];
      }
    const int plen = std::min(len, n);
    std::vector<double> pphi(plen, 0.0), ppsi(plen, 0.0);
    for (int t = 0; t < len; ++t) {
      pphi[t % n] += nphi[t];
      ppsi[t % n] += npsi[t];
    }
    G.flen[l] = plen;
    G.foff[l] = static_cast<int64_t>(tab.size());
    tab.insert(tab.end(), pphi.begin(), pphi.end());
    tab.insert(tab.end(), ppsi.begin(), ppsi.end());
    phi.swap(nphi);
  }
}

// For a level-l column.
Caps window_caps(const Geom& G, int l) {
  int len = std::min(G.flen[l] + 2 * G.R, G.n), M = G.n;
  Caps c;
  c.in = static_cast<int64_t>(len) * len;
  for (int lv = 1; lv <= G.J; ++lv) {
    int next = 0;
    for (int s = 0; s < 2; ++s) next = std::max(next, next_win(Win{s, len, M}, G.L).len);
    c.mid = std::max(c.mid, 2 * static_cast<int64_t>(len) * next);
    int64_t& to = lv % 2 ? c.out : c.in;
    to = std::max(to, static_cast<int64_t>(next) * next);
    len = next;
    M >>= 1;
  }
  return c;
}

Caps larger(const Caps& a, const Caps& b) {
  return Caps{std::max(a.in, b.in), std::max(a.out, b.out), std::max(a.mid, b.mid)};
}

// LDS for the window buffers of a block: three blocks per CU beside their digit counts.
constexpr size_t kWindowLds = 36 * 1024;

struct Builder {
  Geom G{};
  PsfField psf;
  DevBuf<double> ftab, scratch, wt;
  DevBuf<short2> reach;
  DevBuf<unsigned long long> hist, counters;
  DevBuf<int> err;
  Weights T;
  Caps cap;               // of the columns in scratch
  int64_t lds_begin = 0;  // first of the columns in LDS (the finer levels)
  int nwg = 0;
  hipStream_t s = nullptr;
  bool log = false;

  // The weights' table, where there is room for it beside the kept entries
  // (WDB_BUILD_TABLE=0: never; the same sums).
  void tabulate(int64_t nnz_budget) {
    const int64_t N = static_cast<int64_t>(G.n) * G.n, rows = G.R + 1;
    const char* off = std::getenv("WDB_BUILD_TABLE");
    size_t free = 0, all = 0;
    WDB_HIP(hipMemGetInfo(&free, &all));
    const size_t entry = 2 * sizeof(int32_t) + sizeof(double);
    const size_t kept = (static_cast<size_t>(nnz_budget) + kBoundaryCap) * entry;
    const size_t bytes = weight_table_bytes(G.n, G.R);
    T.tiles = (G.n + kReach - 1) / kReach;
    const bool fits = !(off && *off == '0') && bytes <= weight_table_room(free, kept) && try_alloc([&] {
      wt.alloc(bytes / sizeof(double));   // fails if the memory was taken meanwhile (another thread)
      reach.alloc(static_cast<size_t>(rows) * T.tiles * T.tiles);
    });
    if (log) std::fprintf(stderr, "[wdb] build: weights' table of %zu bytes %s\n", bytes, fits ? "kept" : "left out");
    if (!fits) {
      wt.reset();
      reach.reset();
      return;
    }
    T.wt = wt.p;
    T.reach = reach.p;
    hipLaunchKernelGGL(k_weights, dim3(static_cast<unsigned>((N + 255) / 256), static_cast<unsigned>(rows)), dim3(256),
                       0, s, psf.dev(), wt.p);
    hipLaunchKernelGGL(k_weight_reach, dim3(T.tiles, T.tiles, static_cast<unsigned>(rows)), dim3(256), 0, s, G.n, G.R,
                       T);
    WDB_HIP(hipGetLastError());
  }

  void columns(int64_t b0, int64_t b1, int blocks, const Select& S, Emit out, Emit bnd) {
    if (b0 < std::min(b1, lds_begin))
      hipLaunchKernelGGL(k_theta_columns<false>, dim3(blocks), dim3(256), 0, s, G, psf.dev(), T, ftab.p, scratch.p,
                         cap, b0, std::min(b1, lds_begin), S, hist.p, out, bnd, err.p);
    for (int l = G.J; l >= 1; --l) {   // a level's own buffers: the finer, the more blocks per CU
      const int k = 1 + (G.J - l) * 3;
      const int64_t from = std::max({b0, lds_begin, G.sub_off[l == G.J ? 0 : k]}), to = std::min(b1, G.sub_off[k + 3]);
      const Caps c = window_caps(G, l);
      if (from < to)
        hipLaunchKernelGGL(k_theta_columns<true>, dim3(blocks), dim3(256), c.bytes(), s, G, psf.dev(), T, ftab.p,
                           scratch.p, c, from, to, S, hist.p, out, bnd, err.p);
    }
    WDB_HIP(hipGetLastError());
  }

  void run(const Select& S, Emit out, Emit bnd) {
    const int64_t N = static_cast<int64_t>(G.n) * G.n;
    const int64_t chunk = 32768;
    for (int64_t b0 = 0; b0 < N; b0 += chunk) columns(b0, std::min(N, b0 + chunk), nwg, S, out, bnd);
    WDB_HIP(hipStreamSynchronize(s));
    int e = 0;
    WDB_HIP(hipMemcpy(&e, err.p, sizeof(int), hipMemcpyDeviceToHost));
    WDB_REQUIRE(e == 0, WDB_ERR_HIP, "theta build consistency check failed (code %d)", e);
  }

  // Counts of one digit, as `launch` adds them to the cleared hist.
  template <typename F>
  void digits(std::vector<unsigned long long>& h, F&& launch) {
    WDB_HIP(hipMemsetAsync(hist.p, 0, kDigits * sizeof(unsigned long long), s));
    launch();
    WDB_HIP(hipGetLastError());
    WDB_HIP(hipMemcpyAsync(h.data(), hist.p, kDigits * sizeof(unsigned long long), hipMemcpyDeviceToHost, s));
    WDB_HIP(hipStreamSynchronize(s));
  }

  // Appends the `need` first entries of `B`, by magnitude descending, then linear
  // index ascending, to out; all agree with `prefix` in the upper pbits of the
  // magnitude.  Returns the last one's magnitude.
  double keep_boundary(const Boundary& B, unsigned long long prefix, int pbits, unsigned long long need, Emit out) {
    std::vector<unsigned long long> h(kDigits);
    const dim3 grid(static_cast<unsigned>(std::min<int64_t>((B.count + 255) / 256, 1024)));
    unsigned long long same = static_cast<unsigned long long>(B.count);   // entries with the prefix
    while (pbits < 64) {
      const int w = std::min(12, 64 - pbits), shift = 64 - pbits - w;
      digits(h, [&] { hipLaunchKernelGGL(k_boundary_digits<false>, grid, dim3(256), 0, s, B, 0ull, prefix, shift, w, hist.p); });
      int d = (1 << w) - 1;
      while (d > 0 && h[d] < need) need -= h[d--];
      same = h[d];
      prefix = (prefix << w) | static_cast<unsigned long long>(d);
      pbits += w;
    }
    unsigned long long last = ~0ull;
    if (need < same) {   // equal magnitudes straddle the cut
      last = 0;
      for (int shift = 60; shift >= 0; shift -= 12) {
        digits(h, [&] { hipLaunchKernelGGL(k_boundary_digits<true>, grid, dim3(256), 0, s, B, prefix, last, shift, 12, hist.p); });
        int d = 0;
        while (d < kDigits - 1 && h[d] < need) need -= h[d++];
        last = (last << 12) | static_cast<unsigned long long>(d);
      }
    }
    hipLaunchKernelGGL(k_boundary_keep, dim3(static_cast<unsigned>((B.count + 255) / 256)), dim3(256), 0, s, B, prefix,
                       last, out, err.p);
    WDB_HIP(hipGetLastError());
    double threshold;
    std::memcpy(&threshold, &prefix, sizeof(threshold));
    return threshold;
  }
};

// ---------------------------------------------------------------------------
// Convolution fast path (Alg. 3; circulant subband blocks, Sec. 3.6).
//
// With the same PSF at every pixel, H is a circular convolution with a kernel
// symmetric under x -> -x (the Gaussian of psf.hip), so H = H^* and Theta is
// symmetric.  Every block (R, C) of Theta is then a rectangular circulant
// matrix generated by the column gamma_k = Psi^*(H psi_k0) of one atom per
// subband k:
//   * C coarser than R:  Theta[(R, p + r q), (C, q)] = gamma_C[(R, p)],
//   * C as fine as R or finer: Theta[(R, m), (C, p + r m)] = gamma_R[(C, p)]
// (r the ratio of the two sides, positions taken modulo the finer side).  So
// the 3J + 1 representative columns are computed exactly as the general
// build computes any column, each non-zero becomes a generator with a known
// number of copies, the K largest magnitudes are selected on the generators
// (equal magnitudes at the cut ordered by a * N + b like the general build)
// and the kept copies are written out in parallel.
// ---------------------------------------------------------------------------
bool field_is_stationary(const wdb_psf_field* f) {
  const int64_t N = static_cast<int64_t>(f->n) * f->n;
  for (int64_t i = 1; i < N; ++i)
    if (f->sig_major[i] != f->sig_major[0] || f->sig_minor[i] != f->sig_minor[0] || f->angle[i] != f->angle[0])
      return false;
  return true;
}

struct GenDev {
  int64_t off_k, off_b;  // subband offsets: k enumerates the copies, b holds the moving position
  int side_k, side_b;
  int p1, p2, r, form;   // form 0: row in k, column in b; 1: row in b, column in k
  double v;
};

__device__ __host__ inline void gen_entry(const GenDev& g, int64_t idx, int32_t* row, int32_t* col) {
  const int i1 = static_cast<int>(idx / g.side_k), i2 = static_cast<int>(idx % g.side_k);
  const int q1 = (g.p1 + g.r * i1) & (g.side_b - 1), q2 = (g.p2 + g.r * i2) & (g.side_b - 1);
  const int64_t ak = g.off_k + static_cast<int64_t>(i1) * g.side_k + i2;
  const int64_t ab = g.off_b + static_cast<int64_t>(q1) * g.side_b + q2;
  *row = static_cast<int32_t>(g.form == 0 ? ak : ab);
  *col = static_cast<int32_t>(g.form == 0 ? ab : ak);
}

__global__ void k_expand(const GenDev* __restrict__ gens, const int64_t* __restrict__ first, int ngen,
                         int64_t total, int32_t* __restrict__ row, int32_t* __restrict__ col,
                         double* __restrict__ val) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= total) return;
  int lo = 0, hi = ngen - 1;  // last generator with first[g] <= t
  while (lo < hi) {
    const int mid = (lo + hi + 1) / 2;
    if (first[mid] <= t) lo = mid;
    else hi = mid - 1;
  }
  gen_entry(gens[lo], t - first[lo], row + t, col + t);
  val[t] = gens[lo].v;
}

// Builds Theta_K of a stationary field; returns the handle's CSR pieces.
void build_stationary(Builder& B, int64_t nnz_budget, int scaled, unsigned long long* K_out, double* thr_out,
                      DevBuf<int32_t>& orow, DevBuf<int32_t>& ocol, DevBuf<double>& oval,
                      std::vector<CircGen>& kept, std::vector<int32_t>& tie_r, std::vector<int32_t>& tie_c,
                      std::vector<double>& tie_v) {
  const Geom& G = B.G;
  const int64_t N = static_cast<int64_t>(G.n) * G.n;
  hipStream_t s = B.s;
  // 1. representative columns gamma_k (every non-zero, float64)
  DevBuf<int32_t> er(N), ec(N);
  DevBuf<double> ev(N);
  std::vector<GenDev> gens;
  std::vector<int32_t> hr;
  std::vector<double> hv;
  auto band_of = [&](int64_t a) {
    int k = 0;
    while (k + 1 < G.nsub && a >= G.sub_off[k + 1]) ++k;
    return k;
  };
  for (int k = 0; k < G.nsub; ++k) {
    WDB_HIP(hipMemsetAsync(B.counters.p, 0, sizeof(unsigned long long), s));
    Emit out{er.p, ec.p, ev.p, B.counters.p, static_cast<unsigned long long>(N)};
    Emit none{nullptr, nullptr, nullptr, B.counters.p + 1, 0};
    Select S{2, 0, 0, 0, 0, 0};
    B.columns(G.sub_off[k], G.sub_off[k] + 1, 1, S, out, none);
    unsigned long long cnt = 0;
    WDB_HIP(hipMemcpyAsync(&cnt, B.counters.p, sizeof(cnt), hipMemcpyDeviceToHost, s));
    WDB_HIP(hipStreamSynchronize(s));
    int e = 0;
    WDB_HIP(hipMemcpy(&e, B.err.p, sizeof(int), hipMemcpyDeviceToHost));
    WDB_REQUIRE(e == 0 && cnt <= static_cast<unsigned long long>(N), WDB_ERR_HIP,
                "representative column %d failed (code %d)", k, e);
    hr.resize(cnt);
    hv.resize(cnt);
    WDB_HIP(hipMemcpy(hr.data(), er.p, cnt * sizeof(int32_t), hipMemcpyDeviceToHost));
    WDB_HIP(hipMemcpy(hv.data(), ev.p, cnt * sizeof(double), hipMemcpyDeviceToHost));
    const int sk = G.sub_side[k];
    for (unsigned long long i = 0; i < cnt; ++i) {
      const int b = band_of(hr[i]);
      const int sb = G.sub_side[b];
      const int64_t pos = hr[i] - G.sub_off[b];
      GenDev g{G.sub_off[k], G.sub_off[b], sk, sb, static_cast<int>(pos / sb), static_cast<int>(pos % sb),
               sb / sk, 0, hv[i]};
      if (sb > sk) {  // block (R = b, C = k), C coarser: copies over the columns of k
        g.form = 1;
        gens.push_back(g);
      }
      if (sb >= sk) {  // block (R = k, C = b), C as fine or finer: copies over the rows of k
        g.form = 0;
        gens.push_back(g);
      }
    }
  }
  // 2. the K largest (weighted) magnitudes over the generators and their copies
  auto mag = [scaled](const GenDev& g) {
    const int side_col = g.form == 0 ? g.side_b : g.side_k;
    return scaled ? std::fabs(g.v) / side_col : std::fabs(g.v);
  };
  std::sort(gens.begin(), gens.end(), [&](const GenDev& x, const GenDev& y) { return mag(x) > mag(y); });
  const unsigned long long budget = static_cast<unsigned long long>(nnz_budget);
  unsigned long long cum = 0;
  size_t full = 0;
  std::vector<std::pair<int64_t, std::pair<int32_t, int32_t>>> tie;  // (a*N + b, (a, b))
  double threshold = 0.0;
  std::vector<double> tie_val;
  while (full < gens.size()) {
    size_t e = full;
    unsigned long long grp = 0;
    while (e < gens.size() && mag(gens[e]) == mag(gens[full])) {
      grp += static_cast<unsigned long long>(gens[e].side_k) * gens[e].side_k;
      ++e;
    }
    if (cum + grp <= budget) {
      cum += grp;
      threshold = mag(gens[full]);
      full = e;
      continue;
    }
    // equal magnitudes straddle the cut: keep the smallest linear indices
    const unsigned long long need = budget - cum;
    if (need == 0) break;
    std::vector<std::pair<int64_t, size_t>> cand;  // (a*N + b, generator * 2^32 + copy)
    cand.reserve(grp);
    for (size_t g = full; g < e; ++g) {
      const int64_t m = static_cast<int64_t>(gens[g].side_k) * gens[g].side_k;
      for (int64_t i = 0; i < m; ++i) {
        int32_t a, b;
        gen_entry(gens[g], i, &a, &b);
        cand.push_back({static_cast<int64_t>(a) * N + b, ((g - full) << 32) | static_cast<size_t>(i)});
      }
    }
    std::nth_element(cand.begin(), cand.begin() + (need - 1), cand.end());
    for (unsigned long long i = 0; i < need; ++i) {
      const size_t g = full + (cand[i].second >> 32);
      tie.push_back({cand[i].first, {static_cast<int32_t>(cand[i].first / N), static_cast<int32_t>(cand[i].first % N)}});
      tie_val.push_back(gens[g].v);
    }
    threshold = mag(gens[full]);
    cum += need;
    break;
  }
  // 3. write the kept copies
  const unsigned long long K = cum;
  const int ngen = static_cast<int>(full);
  std::vector<int64_t> first(ngen + 1, 0);
  for (int g = 0; g < ngen; ++g) first[g + 1] = first[g] + static_cast<int64_t>(gens[g].side_k) * gens[g].side_k;
  orow.alloc(std::max<unsigned long long>(K, 1));
  ocol.alloc(std::max<unsigned long long>(K, 1));
  oval.alloc(std::max<unsigned long long>(K, 1));
  if (ngen > 0) {
    DevBuf<GenDev> dg(ngen);
    DevBuf<int64_t> df(ngen + 1);
    WDB_HIP(hipMemcpy(dg.p, gens.data(), ngen * sizeof(GenDev), hipMemcpyHostToDevice));
    WDB_HIP(hipMemcpy(df.p, first.data(), (ngen + 1) * sizeof(int64_t), hipMemcpyHostToDevice));
    const int64_t tot = first[ngen];
    hipLaunchKernelGGL(k_expand, dim3(static_cast<unsigned>((tot + 255) / 256)), dim3(256), 0, s, dg.p, df.p, ngen,
                       tot, orow.p, ocol.p, oval.p);
    WDB_HIP(hipGetLastError());
    WDB_HIP(hipStreamSynchronize(s));
  }
  if (!tie.empty()) {
    std::vector<int32_t> tr(tie.size()), tc(tie.size());
    for (size_t i = 0; i < tie.size(); ++i) {
      tr[i] = tie[i].second.first;
      tc[i] = tie[i].second.second;
    }
    const int64_t at = first[ngen];
    WDB_HIP(hipMemcpy(orow.p + at, tr.data(), tie.size() * sizeof(int32_t), hipMemcpyHostToDevice));
    WDB_HIP(hipMemcpy(ocol.p + at, tc.data(), tie.size() * sizeof(int32_t), hipMemcpyHostToDevice));
    WDB_HIP(hipMemcpy(oval.p + at, tie_val.data(), tie.size() * sizeof(double), hipMemcpyHostToDevice));
  }
  kept.clear();
  for (int g = 0; g < ngen; ++g) {
    const GenDev& d = gens[g];
    kept.push_back(CircGen{d.off_k, d.off_b, d.side_k, d.side_b, d.p1, d.p2, d.r, d.form, d.v});
  }
  tie_r.clear();
  tie_c.clear();
  tie_v.clear();
  for (size_t i = 0; i < tie.size(); ++i) {
    tie_r.push_back(tie[i].second.first);
    tie_c.push_back(tie[i].second.second);
    tie_v.push_back(tie_val[i]);
  }
  *K_out = K;
  *thr_out = threshold;
}

}  // namespace

}  // namespace wdb

extern "C" wdb_status wdb_build_theta(const wdb_psf_field* field, int32_t wavelet, int32_t levels,
                                      int64_t nnz_budget, void* stream, wdb_theta** out) {
  return wdb_build_theta_rule(field, wavelet, levels, nnz_budget, WDB_THRESH_NAIVE, stream, out);
}

extern "C" wdb_status wdb_build_theta_rule(const wdb_psf_field* field, int32_t wavelet, int32_t levels,
                                           int64_t nnz_budget, int32_t rule, void* stream, wdb_theta** out) {
  using namespace wdb;
  WDB_API_BEGIN
  WDB_REQUIRE(field && out, WDB_ERR_ARG, "null argument");
  WDB_REQUIRE(rule == WDB_THRESH_NAIVE || rule == WDB_THRESH_SCALE, WDB_ERR_ARG, "unknown thresholding rule %d", rule);
  const int scaled = rule == WDB_THRESH_SCALE ? 1 : 0;
  const Filter f = make_filter(wavelet);
  const int n = field->n;
  check_geometry(n, levels, static_cast<int>(f.h.size()));
  WDB_REQUIRE(levels < kMaxLev && 3 * levels + 1 <= kMaxSub, WDB_ERR_LEVELS, "too many levels");
  const int64_t N = static_cast<int64_t>(n) * n;
  WDB_REQUIRE(nnz_budget >= 1 && nnz_budget <= N * N, WDB_ERR_ARG, "nnz_budget %lld outside [1, N^2]",
              static_cast<long long>(nnz_budget));
  hipStream_t s = static_cast<hipStream_t>(stream);
  Builder B;
  B.s = s;
  B.log = std::getenv("WDB_LOG") != nullptr;
  B.psf.upload(field, s);  // validates the field before any device call
  int dev = 0;
  WDB_HIP(hipGetDevice(&dev));
  Geom& G = B.G;
  G.n = n;
  G.J = levels;
  G.L = static_cast<int>(f.h.size());
  G.R = B.psf.R;
  const std::vector<Subband> lay = layout(n, levels);
  G.nsub = static_cast<int>(lay.size());
  for (int k = 0; k < G.nsub; ++k) {
    G.sub_level[k] = lay[k].level;
    G.sub_er[k] = lay[k].erow;
    G.sub_ec[k] = lay[k].ecol;
    G.sub_side[k] = lay[k].side;
    G.sub_off[k] = lay[k].offset;
  }
  G.sub_off[G.nsub] = N;
  for (int m = 0; m < G.L; ++m) {
    G.h[m] = f.h[m];
    G.g[m] = f.g[m];
  }
  std::vector<double> tab;
  level_filters(f, n, levels, tab, G);
  B.ftab.alloc(tab.size());
  WDB_HIP(hipMemcpy(B.ftab.p, tab.data(), tab.size() * sizeof(double), hipMemcpyHostToDevice));
  B.nwg = static_cast<int>(std::min<int64_t>(1024, N));
  // columns of the levels whose windows fit go through LDS (the finer levels come last)
  B.lds_begin = N;
  for (int k = G.nsub - 1; k >= 0; --k) {
    if (window_caps(G, G.sub_level[k]).bytes() > kWindowLds) break;
    B.lds_begin = G.sub_off[k];
  }
  if (B.lds_begin > 0) {
    for (int l = 1; l <= G.J; ++l) B.cap = larger(B.cap, window_caps(G, l));
    // as many workgroups as two windows each would leave room for
    const size_t windows = 2 * static_cast<size_t>(B.cap.in) * sizeof(double);
    if (B.nwg * windows > (size_t{1} << 30))
      B.nwg = std::max(1, static_cast<int>(B.nwg * windows / std::max(windows, B.cap.bytes())));
    B.scratch.alloc(B.nwg * B.cap.bytes() / sizeof(double));
  }
  B.hist.alloc(kDigits);
  B.counters.alloc(2);
  B.err.alloc(1);
  WDB_HIP(hipMemset(B.err.p, 0, sizeof(int)));

  const char* force_general = std::getenv("WDB_BUILD_GENERAL");
  if (field_is_stationary(field) && !(force_general && *force_general == '1')) {
    unsigned long long K = 0;
    double threshold = 0.0;
    DevBuf<int32_t> orow, ocol;
    DevBuf<double> oval;
    std::vector<CircGen> kept;
    std::vector<int32_t> tie_r, tie_c;
    std::vector<double> tie_v;
    build_stationary(B, nnz_budget, scaled, &K, &threshold, orow, ocol, oval, kept, tie_r, tie_c, tie_v);
    B.scratch.reset();
    wdb_theta* th = new wdb_theta();
    try {
      th->device = dev;
      th->n = n;
      th->levels = levels;
      th->wavelet = wavelet;
      th->N = N;
      th->nnz = static_cast<int64_t>(K);
      th->threshold = threshold;
      th->conv_build = 1;
      th->rule = rule;
      coo_to_csr(N, th->nnz, orow.p, ocol.p, oval.p, &th->csr, s);
      finish_theta(th, s);
      build_stencils(th, kept, tie_r, tie_c, tie_v);
    } catch (...) {
      wdb_theta_free(th);
      throw;
    }
    *out = th;
    return WDB_OK;
  }

  B.tabulate(nnz_budget);
  Emit none{nullptr, nullptr, nullptr, B.counters.p, 0};
  // Radix select of the nnz_budget-th largest |theta|.
  unsigned long long need = static_cast<unsigned long long>(nnz_budget);
  unsigned long long prefix = 0, bcount = 0, total = 0;
  int pbits = 0;
  bool keep_all = false;
  std::vector<unsigned long long> h(kDigits);
  while (true) {
    const int w = std::min(12, 64 - pbits);
    Select S{0, scaled, pbits, 64 - pbits - w, prefix, (1ull << w) - 1ull};
    WDB_HIP(hipMemsetAsync(B.hist.p, 0, kDigits * sizeof(unsigned long long), s));
    B.run(S, none, none);
    WDB_HIP(hipMemcpy(h.data(), B.hist.p, kDigits * sizeof(unsigned long long), hipMemcpyDeviceToHost));
    if (pbits == 0) {
      total = std::accumulate(h.begin(), h.end(), 0ull);
      if (total <= need) {
        keep_all = true;
        break;
      }
    }
    unsigned long long cum = 0;
    int digit = -1;
    for (int d = (1 << w) - 1; d >= 0; --d) {
      if (cum + h[d] >= need) {
        digit = d;
        break;
      }
      cum += h[d];
    }
    WDB_REQUIRE(digit >= 0, WDB_ERR_HIP, "radix select lost entries");
    need -= cum;
    prefix = (prefix << w) | static_cast<unsigned long long>(digit);
    pbits += w;
    bcount = h[digit];
    if (B.log)
      std::fprintf(stderr, "[wdb] build: digit pass %d bits, boundary %llu, need %llu\n", pbits, bcount, need);
    if (bcount <= kBoundaryCap || pbits >= 64) break;
  }
  const unsigned long long K = keep_all ? total : static_cast<unsigned long long>(nnz_budget);
  const unsigned long long above = keep_all ? total : K - need;
  DevBuf<int32_t> orow(K), ocol(K);
  DevBuf<double> oval(K);
  DevBuf<int32_t> brow(keep_all ? 0 : bcount), bcol(keep_all ? 0 : bcount);
  DevBuf<double> bval(keep_all ? 0 : bcount);
  WDB_HIP(hipMemsetAsync(B.counters.p, 0, 2 * sizeof(unsigned long long), s));
  Emit eo{orow.p, ocol.p, oval.p, B.counters.p, above};
  Emit eb{brow.p, bcol.p, bval.p, B.counters.p + 1, keep_all ? 0 : bcount};
  Select S{keep_all ? 2 : 1, scaled, pbits, 0, prefix, 0};
  B.run(S, eo, eb);
  unsigned long long cnt[2];
  WDB_HIP(hipMemcpy(cnt, B.counters.p, sizeof(cnt), hipMemcpyDeviceToHost));
  WDB_REQUIRE(cnt[0] == above && (keep_all || cnt[1] == bcount), WDB_ERR_HIP,
              "theta emit pass produced %llu/%llu entries, expected %llu/%llu", cnt[0], cnt[1], above, bcount);
  double threshold = 0.0;
  if (!keep_all) {
    DevBuf<double> sigma;
    if (scaled) {   // the ranked magnitude is times sigma_b of the column
      std::vector<double> sg(N);
      for (int k = 0; k < G.nsub; ++k)
        for (int64_t b = G.sub_off[k]; b < G.sub_off[k + 1]; ++b) sg[b] = 1.0 / static_cast<double>(G.sub_side[k]);
      sigma.alloc(N);
      WDB_HIP(hipMemcpy(sigma.p, sg.data(), N * sizeof(double), hipMemcpyHostToDevice));
    }
    Emit rest{orow.p + above, ocol.p + above, oval.p + above, B.counters.p, need};
    WDB_HIP(hipMemsetAsync(B.counters.p, 0, sizeof(unsigned long long), s));
    threshold = B.keep_boundary(Boundary{eb, N, static_cast<int64_t>(bcount), sigma.p}, prefix, pbits, need, rest);
    unsigned long long kept = 0;
    int e = 0;
    WDB_HIP(hipMemcpyAsync(&kept, B.counters.p, sizeof(kept), hipMemcpyDeviceToHost, s));
    WDB_HIP(hipMemcpyAsync(&e, B.err.p, sizeof(e), hipMemcpyDeviceToHost, s));
    WDB_HIP(hipStreamSynchronize(s));
    WDB_REQUIRE(e == 0 && kept == need, WDB_ERR_HIP, "boundary select kept %llu entries, expected %llu (code %d)", kept,
                need, e);
  }
  B.scratch.reset();
  B.wt.reset();

  wdb_theta* th = new wdb_theta();
  try {
    th->device = dev;
    th->n = n;
    th->levels = levels;
    th->wavelet = wavelet;
    th->N = N;
    th->nnz = static_cast<int64_t>(K);
    th->threshold = threshold;
    th->rule = rule;
    coo_to_csr(N, th->nnz, orow.p, ocol.p, oval.p, &th->csr, s);
    finish_theta(th, s);
  } catch (...) {
    wdb_theta_free(th);
    throw;
  }
  *out = th;
  WDB_API_END
}
