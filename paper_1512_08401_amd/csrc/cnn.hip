// Warm-start network on wavelet coefficients (not in the paper): one stack of
// three circular 3x3 convolutions per wavelet level (A_J with 1 channel, the
// detail levels with their 3 subbands as channels), ReLU after the first two,
// a residual connection, MSE loss and Adam with float32 master weights.
// Compute uses bfloat16 copies of the parameters and float32 accumulation.
//
//   h1 = relu(conv(z; W1, b1)), h2 = relu(conv(h1; W2, b2)), out = z + conv(h2; W3, b3),
//   conv(z; W, b)[o, i, j] = b[o] + sum_{c, di, dj} W[o, c, di, dj] z[c, (i+di-1) mod s, (j+dj-1) mod s].
//
// Two kernels do all of it, for every stack of the network in one launch each:
//   k_net_fwd   the three convolutions of a tile of positions, the hidden
//               activations in LDS; for training also the loss, its gradient
//               and the pre-activations a1, a2 for the backward pass;
//   k_net_bwd   both data gradients and the three weight gradients of a tile.
//
// The products run on the bfloat16 matrix cores without rounding the float32
// operands: a float32 x is the exact sum of three bfloat16 numbers (8 + 8 + 8
// bits of its significand, split3), a weight is one bfloat16 number, and the
// products of two bfloat16 numbers are exact in float32.  So three bfloat16
// products with float32 accumulation replace one float32 product, at 3/16 of
// the float32 matrix time; the weight gradients, whose operands are both
// float32, take six of the nine partial products (what is left out is below
// 2^-24 of the product).  Measured against float64 the convolutions' part of a
// prediction is off by 0.8 to 1.2e-7 (float32 matrix products: 1.3 to 2.5e-7)
// and the gradient by 0.56 to 0.74e-7 (0.66 to 0.81e-7).
//
// A tile is 256 positions of one image, 8 x 32 for sides of 32 and more and 16
// x 16 below (sides under 16 cover the tile several times over and count each
// position once).  Blocks are dealt to the stacks in proportion to their tiles
// and walk their stack's tiles with the stack's weights in registers.  Weight
// gradients are reduced in two deterministic stages (per-block partial sums
// over the block's tiles, then a fixed-order sum).
// Parameters are flattened stack by stack: W1, b1, W2, b2, W3, b3.
#include <cmath>
#include <cstring>
#include <algorithm>
#include <type_traits>

#include "common.hpp"

namespace {
constexpr int kF = 32;       // hidden channels
constexpr int kBlk = 256;
constexpr int kTileP = 256;  // positions of a tile
constexpr int kMaxStacks = 24;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float(static_cast<uint32_t>(h) << 16); }

__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t b = __float_as_uint(f);
  b += 0x7FFFu + ((b >> 16) & 1u);
  return static_cast<uint16_t>(b >> 16);
}

// D += A B on the matrix cores, 32 x 32 x 16: lane l holds A[l mod 32][8 (l /
// 32) + i] and B[8 (l / 32) + i][l mod 32], i < 8, and in accumulator j
// D[drow(j, l)][l mod 32].
__device__ __forceinline__ f32x16 mma(const u32x4& a, const u32x4& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                 0);
}
__device__ __forceinline__ int drow(int j, int hi) { return 8 * (j >> 2) + 4 * hi + (j & 3); }

// The upper halves of x and y as one dword (x in the low half).
__device__ __forceinline__ uint32_t pack_hi(float x, float y) {
  return __builtin_amdgcn_perm(__float_as_uint(y), __float_as_uint(x), 0x07060302u);
}

// What the bfloat16 prefix of x leaves of it (exact; 0 for infinities, so that
// their parts are {inf, 0, 0}).  POS: x >= 0 and not NaN.
template <bool POS>
__device__ __forceinline__ float rest(float x) {
  const float r = x - __uint_as_float(__float_as_uint(x) & 0xFFFF0000u);
  if constexpr (POS) return fmaxf(r, 0.0f);
  else return (__float_as_uint(x) & 0x7FFFFFFFu) == 0x7F800000u ? 0.0f : r;
}

// x and y as three bfloat16 parts each, x = p[0] + p[1] + p[2] (low halves),
// by truncation: the remainders have x's sign.
template <bool POS>
__device__ __forceinline__ void split3(float x, float y, uint32_t (&p)[3]) {
  p[0] = pack_hi(x, y);
  x = rest<POS>(x);
  y = rest<POS>(y);
  p[1] = pack_hi(x, y);
  p[2] = pack_hi(x - __uint_as_float(__float_as_uint(x) & 0xFFFF0000u),
                 y - __uint_as_float(__float_as_uint(y) & 0xFFFF0000u));
}

// The same rounding to nearest, for products of two split operands: there the
// small products that are left out then have either sign and cancel in a sum
// instead of shortening it.  (The parts of an infinity hold a NaN: a gradient
// that meets one is not finite either way.)
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void split3r(float x, float y, uint32_t (&p)[3]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    p[k] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{x, y}), bf16x2));
    x -= __uint_as_float(p[k] << 16);
    y -= __uint_as_float(p[k] & 0xFFFF0000u);
  }
}

// Scheduling of a run of N products that read one LDS operand each: the reads
// stay AHEAD products ahead of their use.
template <int N, int AHEAD>
__device__ __forceinline__ void pipeline_reads() {
  __builtin_amdgcn_sched_group_barrier(0x100, AHEAD, 0);   // LDS reads
#pragma unroll
  for (int i = 0; i < N - AHEAD; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);     // a product
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x008, AHEAD, 0);
}

// Packed weights of one stack, per matrix a list of operands [step][lane][8]:
// the conv1, conv2 and conv3 weights as A operands, W3^T and W2^T (data
// gradients) as B operands.
constexpr int kPk1 = 0, kPk2 = 3, kPk3 = 21, kPk3T = 23, kPk2T = 26, kPkSteps = 44;
constexpr int64_t kPkStack = int64_t{kPkSteps} * 64 * 8;   // bfloat16 values per stack

struct StackArg {
  int64_t off;              // of the stack's coefficients
  int C, s;                 // channels, side
  int blk0, nblk;           // blocks of the launch
  int tiles_x, tiles_img, ntiles;
  const uint16_t* pk;       // packed weights
  const uint16_t* b[3];     // biases
  int64_t prow;             // first parameter
  float* a1;                // pre-activations of the batch, [b][32][s][s]
  float* a2;
};
struct NetArg {
  int nstacks;
  StackArg st[kMaxStacks];
};

__device__ __forceinline__ int stack_of(const NetArg& n) {
  int k = 0;
  while (k + 1 < n.nstacks && static_cast<int>(blockIdx.x) >= n.st[k + 1].blk0) ++k;
  return k;
}

// Image and origin of tile t of a stack.
template <int TX>
__device__ __forceinline__ void tile_at(const StackArg& S, int t, int& b, int& y0, int& x0) {
  b = t / S.tiles_img;
  const int i = t - b * S.tiles_img, ty = i / S.tiles_x;
  y0 = ty * (kTileP / TX);
  x0 = (i - ty * S.tiles_x) * TX;
}

__device__ __forceinline__ u32x4 pk_at(const uint16_t* __restrict__ pk, int step, int lane) {
  return reinterpret_cast<const u32x4*>(pk)[step * 64 + lane];
}

// ---------------------------------------------------------------------------
// Forward
// ---------------------------------------------------------------------------
// LDS of a tile: z on the tile and 3 positions around it as [part][pos][4]
// (channels, zero beyond C), h1 on 2 around as [part][pos][32] with 80 bytes
// per position (the 16-byte reads of 8 consecutive positions then fall on
// different banks), the per-tap products T[q][9 o + d] on 1 around.
template <int TX>
struct FwdG {
  static constexpr int TY = kTileP / TX;
  static constexpr int ZW = TX + 6, NZ = ZW * (TY + 6);
  static constexpr int W1 = TX + 4, N1 = W1 * (TY + 4), G1 = (N1 + 31) / 32;
  static constexpr int W2 = TX + 2, N2 = W2 * (TY + 2), G2 = (N2 + 31) / 32;
};
constexpr int kFwdWaves = 8, kFwdThreads = 64 * kFwdWaves;
constexpr int kZPlane = 532 * 8;          // bytes; the larger of the two tiles (14 x 38)
constexpr int kHPos = 80, kHPlane = 432 * kHPos;
constexpr int kTM = 27;                   // floats of T per position (odd: no bank conflicts)
constexpr int kFwdH = 3 * kZPlane, kFwdT = kFwdH + 3 * kHPlane, kFwdLds = kFwdT + 340 * kTM * 4;
static_assert(FwdG<32>::NZ == 532 && FwdG<16>::NZ <= 532 && FwdG<32>::N1 == 432 && FwdG<16>::N1 <= 432 &&
                  FwdG<32>::N2 == 340 && FwdG<16>::N2 <= 340,
              "LDS regions");
static_assert(kFwdH % 16 == 0 && kFwdT % 16 == 0 && kFwdLds <= 160 * 1024, "LDS layout");

struct TrainArg {        // null tgt: inference
  const float* tgt;
  float* gout;           // gradient of the loss with respect to the output
  double* loss;          // per-block sums of squared errors
  float scale;
};

template <int TX, bool TRAIN>
__device__ __forceinline__ void fwd_stack(const StackArg& S, const float* __restrict__ x0, int64_t N,
                                          float* __restrict__ out, const TrainArg& tr, char* lds) {
  using G = FwdG<TX>;
  const int lane = threadIdx.x & 63, l32 = lane & 31, hi = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int s = S.s, m = s - 1, C = S.C;
  const int64_t per = static_cast<int64_t>(s) * s;
  float* T = reinterpret_cast<float*>(lds + kFwdT);
  u32x4 w1[3], w2[18], w3[2];
#pragma unroll
  for (int k = 0; k < 3; ++k) w1[k] = pk_at(S.pk, kPk1 + k, lane);
#pragma unroll
  for (int k = 0; k < 18; ++k) w2[k] = pk_at(S.pk, kPk2 + k, lane);
#pragma unroll
  for (int k = 0; k < 2; ++k) w3[k] = pk_at(S.pk, kPk3 + k, lane);
  f32x16 b1, b2;   // biases of the lane's 16 outputs
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    b1[j] = bf2f(S.b[0][drow(j, hi)]);
    b2[j] = bf2f(S.b[1][drow(j, hi)]);
  }
  // byte offsets of this lane half's two taps of each conv1 step (taps above 8:
  // zero weights and, for an infinite input's sake, zero operands)
  int zo[3][2];
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int t = min(4 * k + 2 * hi + i, 8);
      zo[k][i] = ((t / 3) * G::ZW + t % 3) * 8;
    }
  constexpr int ZIT = (G::NZ + kFwdThreads - 1) / kFwdThreads;
  float zv[ZIT][3];
  const auto load_z = [&](int t) {
    int b, y0, xt;
    tile_at<TX>(S, t, b, y0, xt);
    const float* zb = x0 + b * N + S.off;
#pragma unroll
    for (int i = 0; i < ZIT; ++i) {
      const int q = static_cast<int>(threadIdx.x) + i * kFwdThreads;
      zv[i][1] = zv[i][2] = 0.0f;
      if (q < G::NZ) {
        const int y = q / G::ZW, x = q - y * G::ZW;
        const float* p = zb + static_cast<int64_t>((y0 + y - 3) & m) * s + ((xt + x - 3) & m);
        zv[i][0] = p[0];
        if (C == 3) {
          zv[i][1] = p[per];
          zv[i][2] = p[2 * per];
        }
      }
    }
  };
  double lsum = 0.0;
  int t = static_cast<int>(blockIdx.x) - S.blk0;
  if (t < S.ntiles) load_z(t);
  for (; t < S.ntiles; t += S.nblk) {
    int b, y0, xt;
    tile_at<TX>(S, t, b, y0, xt);
#pragma unroll
    for (int i = 0; i < ZIT; ++i) {
      const int q = static_cast<int>(threadIdx.x) + i * kFwdThreads;
      if (q < G::NZ) {
        uint32_t p[3], r[3];
        split3<false>(zv[i][0], zv[i][1], p);
        split3<false>(zv[i][2], 0.0f, r);
#pragma unroll
        for (int k = 0; k < 3; ++k) *reinterpret_cast<u32x2*>(lds + k * kZPlane + q * 8) = u32x2{p[k], r[k]};
      }
    }
    __syncthreads();
    if (t + S.nblk < S.ntiles) load_z(t + S.nblk);   // in flight during this tile's products
    // first convolution on the tile and 2 around
    for (int g = wv; g < G::G1; g += kFwdWaves) {
      const int q = g * 32 + l32, qc = min(q, G::N1 - 1);
      const int y = qc / G::W1, x = qc - y * G::W1;
      const char* zp = lds + (y * G::ZW + x) * 8;
      // the small parts first; the sum starts from the bias
      f32x16 acc = b1;
#pragma unroll
      for (int p = 2; p >= 0; --p)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          u32x2 a = *reinterpret_cast<const u32x2*>(zp + p * kZPlane + zo[k][0]);
          u32x2 c = {0, 0};
          if (k < 2) c = *reinterpret_cast<const u32x2*>(zp + p * kZPlane + zo[k][1]);
          else if (hi) a = u32x2{0, 0};
          acc = mma(w1[k], u32x4{a.x, a.y, c.x, c.y}, acc);
        }
      if (q < G::N1) {
        const int gy = y0 + y - 2, gx = xt + x - 2;
        const bool keep = TRAIN && y >= 2 && y < G::TY + 2 && x >= 2 && x < TX + 2 && gy < s && gx < s;
        const uint32_t at = static_cast<uint32_t>(gy * s + gx) + 4 * hi * static_cast<uint32_t>(per);
        float* ap = TRAIN ? S.a1 + b * kF * per : nullptr;
#pragma unroll
        for (int jq = 0; jq < 4; ++jq) {
          float v[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            v[j] = acc[4 * jq + j];
            if (TRAIN && keep) (ap + (8 * jq + j) * per)[at] = v[j];
            v[j] = fmaxf(v[j], 0.0f);
          }
          uint32_t p[3], r[3];
          split3<true>(v[0], v[1], p);
          split3<true>(v[2], v[3], r);
#pragma unroll
          for (int k = 0; k < 3; ++k)
            *reinterpret_cast<u32x2*>(lds + kFwdH + k * kHPlane + q * kHPos + 16 * jq + 8 * hi) = u32x2{p[k], r[k]};
        }
      }
    }
    __syncthreads();
    // what the last part reads from memory, in flight during the products
    constexpr int OIT = (kTileP * 3 + kFwdThreads - 1) / kFwdThreads;
    float res[OIT], want[OIT];
#pragma unroll
    for (int i = 0; i < OIT; ++i) {
      const int e = static_cast<int>(threadIdx.x) + i * kFwdThreads;
      const int p = e & (kTileP - 1), o = e / kTileP, y = p / TX, x = p % TX;
      if (o < C && y0 + y < s && xt + x < s) {
        const int64_t at = b * N + S.off + o * per + static_cast<int64_t>(y0 + y) * s + xt + x;
        res[i] = x0[at];
        if (TRAIN) want[i] = tr.tgt[at];
      }
    }
    // second convolution on the tile and 1 around, and from its registers the
    // per-tap products of the third
    for (int g = wv; g < G::G2; g += kFwdWaves) {
      const int q = g * 32 + l32, qc = min(q, G::N2 - 1);
      const int y = qc / G::W2, x = qc - y * G::W2;
      const char* hp = lds + kFwdH + (y * G::W1 + x) * kHPos + 16 * hi;
      f32x16 acc = b2;
#pragma unroll
      for (int p = 2; p >= 0; --p)
#pragma unroll
        for (int k = 0; k < 18; ++k) {
          const int d = k >> 1;
          acc = mma(w2[k],
                    *reinterpret_cast<const u32x4*>(hp + p * kHPlane + ((d / 3) * G::W1 + d % 3) * kHPos + 32 * (k & 1)),
                    acc);
        }
      pipeline_reads<54, 6>();
      const int gy = y0 + y - 1, gx = xt + x - 1;
      const bool keep = TRAIN && q < G::N2 && y >= 1 && y <= G::TY && x >= 1 && x <= TX && gy < s && gx < s;
      const uint32_t at = static_cast<uint32_t>(gy * s + gx) + 4 * hi * static_cast<uint32_t>(per);
      float* ap = TRAIN ? S.a2 + b * kF * per : nullptr;
      f32x16 tap = {}, tlo = {};
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        uint32_t v[3][4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          float f[2];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const int j = 8 * h + 2 * u + e;
            f[e] = acc[j];
            if (TRAIN && keep) (ap + drow(j, 0) * per)[at] = f[e];
            f[e] = fmaxf(f[e], 0.0f);
          }
          uint32_t p[3];
          split3<true>(f[0], f[1], p);
#pragma unroll
          for (int k = 0; k < 3; ++k) v[k][u] = p[k];
        }
        tap = mma(w3[h], u32x4{v[0][0], v[0][1], v[0][2], v[0][3]}, tap);
        tlo = mma(w3[h], u32x4{v[2][0], v[2][1], v[2][2], v[2][3]}, tlo);
        tlo = mma(w3[h], u32x4{v[1][0], v[1][1], v[1][2], v[1][3]}, tlo);
      }
      if (q < G::N2) {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int r = drow(j, hi);
          if (r < kTM) T[q * kTM + r] = tap[j] + tlo[j];
        }
      }
    }
    __syncthreads();
    // third convolution: the nine shifted taps, bias and the input
#pragma unroll
    for (int i = 0; i < OIT; ++i) {
      const int e = static_cast<int>(threadIdx.x) + i * kFwdThreads;
      const int p = e & (kTileP - 1), o = e / kTileP, y = p / TX, x = p % TX;
      if (o >= C || y0 + y >= s || xt + x >= s) continue;
      const float* tp = T + (y * G::W2 + x) * kTM + 9 * o;
      float v = 0.0f;
#pragma unroll
      for (int d = 0; d < 9; ++d) v += tp[((d / 3) * G::W2 + d % 3) * kTM + d];
      v += bf2f(S.b[2][o]);
      v += res[i];
      const int64_t at = b * N + S.off + o * per + static_cast<int64_t>(y0 + y) * s + xt + x;
      if (TRAIN) {
        const float d = v - want[i];
        tr.gout[at] = tr.scale * d;
        lsum += static_cast<double>(d) * d;
      } else {
        out[at] = v;
      }
    }
  }
  if (TRAIN) {
    double* red = reinterpret_cast<double*>(lds);   // z: read by no wavefront any more
    __syncthreads();
    red[threadIdx.x] = lsum;
    __syncthreads();
    for (int w = kFwdThreads / 2; w > 0; w >>= 1) {
      if (static_cast<int>(threadIdx.x) < w) red[threadIdx.x] += red[threadIdx.x + w];
      __syncthreads();
    }
    if (threadIdx.x == 0) tr.loss[blockIdx.x] = red[0];
  }
}

// Bound by the matrix cores and by the vector work between their runs (the
// splits): per 8 x 32 tile 14 thousand cycles, 6.2 of them products.  77
// images of 256 x 256 in 164 us, 226 TFLOP/s; three float32 kernels per stack,
// with the activations in memory, took 613 us.  The taps' operands are read
// ahead of the products (pipeline_reads; without it 10% slower), and what the
// tile's first and last part read from memory is requested a part earlier.
template <bool TRAIN>
__global__ __launch_bounds__(kFwdThreads, 2) void k_net_fwd(NetArg net, const float* __restrict__ x0, int64_t N,
                                                            float* __restrict__ out, TrainArg tr) {
  extern __shared__ __align__(16) char lds[];
  const StackArg& S = net.st[stack_of(net)];
  if (S.s >= 32) fwd_stack<32, TRAIN>(S, x0, N, out, tr, lds);
  else fwd_stack<16, TRAIN>(S, x0, N, out, tr, lds);
}

// ---------------------------------------------------------------------------
// Backward
// ---------------------------------------------------------------------------
// With off(d) the displacement of tap d and everything periodic,
//   g2[p][c] = [a2 > 0] sum_{o,d} W3[o][c][d] gout[p - off(d)][o],
//   g1[p][c] = [a1 > 0] sum_{o,d} W2[o][c][d] g2[p - off(d)][o],
//   dW3[o][c][d] = sum_q h2[q][c] gout[q - off(d)][o],
//   dW2[o][c][d] = sum_p g2[p][o] h1[p + off(d)][c],
//   dW1[o][c][d] = sum_p g1[p][o] z[p + off(d)][c].
// A wavefront computes g2 (then g1) of 32 positions as D[p][c], lane = channel:
// its accumulators, split into bfloat16 parts, are the A operand of the weight
// gradient (rows = channel, k = position: step h takes the positions drow(8 h +
// i, lane half)), whose B operands are runs of four positions of h1, z or gout
// from planes [part][channel][y][x].  One window of a row serves its three
// taps (the odd shift is a funnel shift of the packed pairs).
//
// LDS of a tile: g2 on the tile and 1 around as [part][pos][32] (64 bytes per
// position, 16-byte pieces exchanged by position against bank conflicts), the
// planes of h1, gout and z with 1 around, and gout on 2 around as
// [part][pos][4].
template <int TX>
struct BwdG {
  static constexpr int TY = kTileP / TX;
  static constexpr int W2 = TX + 2, H2 = TY + 2, N2 = W2 * H2;   // halo 1
  static constexpr int GW = TX + 4, NG = GW * (TY + 4);          // halo 2
  static constexpr int RowB = TX == 32 ? 72 : 40;                // bytes of a plane's row (W2 values, 8-byte steps)
  static constexpr int ChB = 728;                                // bytes of a channel's plane
  static constexpr int GR = 3;                                  // groups of 32 positions around the tile
};
constexpr int kBwdWaves = 8, kBwdThreads = 64 * kBwdWaves;
constexpr int kG2Plane = 340 * 64, kH1Plane = kF * 728, kGoPlane = 432 * 8, kThinPlane = 3 * 728;
constexpr int kBwdH1 = 3 * kG2Plane, kBwdGo = kBwdH1 + 3 * kH1Plane, kBwdGp = kBwdGo + 3 * kGoPlane,
              kBwdZp = kBwdGp + 3 * kThinPlane, kBwdLds = kBwdZp + 3 * kThinPlane + 16;
constexpr int kStackParams = 32 * 27 + 32 + 32 * 288 + 32 + 3 * 288 + 3;   // most parameters of a stack
constexpr int kRowFloats = (kStackParams + 15) / 16 * 16;                  // a block's row of partial gradients
static_assert(BwdG<32>::H2 * BwdG<32>::RowB <= 728 && BwdG<16>::H2 * BwdG<16>::RowB <= 728, "channel plane");
static_assert(kBwdH1 % 16 == 0 && kBwdGo % 8 == 0 && kBwdGp % 8 == 0 && kBwdZp % 8 == 0 && kBwdLds <= 160 * 1024,
              "LDS layout");
static_assert(BwdG<32>::NG <= kBwdThreads && BwdG<16>::NG <= kBwdThreads, "one thread per position");
static_assert(2 * BwdG<32>::H2 <= 32 && BwdG<16>::H2 <= 32, "the columns beside a tile");
static_assert(kRowFloats * 4 <= kBwdLds, "the block's gradient row is assembled in LDS");

__device__ __forceinline__ uint32_t funnel(uint32_t hi, uint32_t lo, int shift) {
  return __builtin_amdgcn_alignbit(hi, lo, shift);
}

// D += A b for part k of a second operand of three parts (small parts first):
// the products below 2^-24 of the whole are left out.
template <int K>
__device__ __forceinline__ void mma_part(const u32x4 (&a)[3], const u32x4& b, f32x16& d) {
#pragma unroll
  for (int i = 2 - K; i >= 0; --i) d = mma(a[i], b, d);
}

// B operand of a thin weight gradient (lane = (channel, tap)): two runs of four
// values at `p` (this lane's row and first value, dx <= 2 beyond an 8-byte
// step) and 8 values on.
__device__ __forceinline__ u32x4 thin_run(const char* p, int shift) {
  const uint32_t* a = reinterpret_cast<const uint32_t*>(p);
  return u32x4{funnel(a[1], a[0], shift), funnel(a[2], a[1], shift), funnel(a[5], a[4], shift),
               funnel(a[6], a[5], shift)};
}

// WHOLE: every position of a tile counts (sides of at least 16).
template <int TX, bool WHOLE>
__device__ __forceinline__ void bwd_stack(const StackArg& S, const float* __restrict__ x0,
                                          const float* __restrict__ gout, int64_t N, float* __restrict__ partial,
                                          char* lds) {
  using G = BwdG<TX>;
  const int lane = threadIdx.x & 63, l32 = lane & 31, hi = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int pw = wv & 3, half = wv >> 2;
  const int s = S.s, m = s - 1, C = S.C;
  const int64_t per = static_cast<int64_t>(s) * s;
  u32x4 w3t[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) w3t[k] = pk_at(S.pk, kPk3T + k, lane);
  int go[3][2];   // byte offsets of this lane half's taps in the [pos][4] gradient
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int t = min(4 * k + 2 * hi + i, 8);
      go[k][i] = ((t / 3) * G::GW + t % 3) * 8;
    }
  // this lane's column n = (channel, tap) of the thin weight gradients
  const int nc = min(l32 / 9, C - 1), nd = l32 % 9;
  const int zofs = kBwdZp + nc * G::ChB + (nd / 3) * G::RowB + (nd % 3 >> 1) * 4, zsh = (nd % 3 & 1) * 16;
  const int gofs = kBwdGp + nc * G::ChB + ((8 - nd) / 3) * G::RowB + ((8 - nd) % 3 >> 1) * 4;
  const int gsh = ((8 - nd) % 3 & 1) * 16;
  // dw: taps 0..3 of W2 and W3 (half 0), taps 4..8 of W2 (half 1)
  f32x16 dw[5] = {}, dw1 = {};
  float db2 = 0.0f, db1 = 0.0f, db3[3] = {0.0f, 0.0f, 0.0f};
  for (int t = static_cast<int>(blockIdx.x) - S.blk0; t < S.ntiles; t += S.nblk) {
    int b, y0, xt;
    tile_at<TX>(S, t, b, y0, xt);
    // the index arithmetic of the tile is done in the tile: hoisted out of the
    // loop it would take more registers than there are
    int tid = threadIdx.x, ln = lane;
    asm volatile("" : "+v"(tid), "+v"(ln));
    const int l32 = ln & 31, hi = ln >> 5;
    const float* zb = x0 + b * N + S.off;
    const float* gb = gout + b * N + S.off;
    const float* a2c = S.a2 + (b * kF + l32) * per;
    // --- staging: the planes of h1 (16 threads per channel), gout and z in
    // pairs along x, gout as [pos][4]
    {
      // pair px of row y: px < TX / 2 in rows of 16 (two of 8) threads, the last
      // pair of each row by one thread a row
      constexpr int PX = G::W2 / 2, NP = G::H2 * PX, AIT = TX == 32 ? G::H2 : G::H2 / 2, AEX = TX == 32 ? 1 : 2;
      constexpr int TIT = (2 * 3 * NP + kBwdThreads - 1) / kBwdThreads;
      const int gy = tid / G::GW, gx = tid - gy * G::GW;
      float vg[3] = {0.0f, 0.0f, 0.0f}, vt[TIT][2];
      if (tid < G::NG) {
        const float* p = gb + static_cast<int64_t>((y0 + gy - 2) & m) * s + ((xt + gx - 2) & m);
        vg[0] = p[0];
        if (C == 3) {
          vg[1] = p[per];
          vg[2] = p[2 * per];
        }
      }
#pragma unroll
      for (int i = 0; i < TIT; ++i) {
        const int e = min(tid + i * kBwdThreads, 2 * C * NP - 1), cc = e / NP, r = e - cc * NP, y = r / PX, px = r - y * PX;
        const float* row = (cc < C ? zb + cc * per : gb + (cc - C) * per) + static_cast<int64_t>((y0 + y - 1) & m) * s;
        vt[i][0] = row[(xt + 2 * px - 1) & m];
        vt[i][1] = row[(xt + 2 * px) & m];
      }
      const int ac = tid >> 4, ai = tid & 15, apx = TX == 32 ? ai : ai & 7;
      const float* a1c = S.a1 + b * kF * per;
      const auto row_of = [&](int i) { return TX == 32 ? i : 2 * i + (ai >> 3); };
      const size_t c0 = ac * per + ((xt + 2 * apx - 1) & m), c1 = ac * per + ((xt + 2 * apx) & m);
      const size_t e0 = ac * per + ((xt + TX - 1) & m), e1 = ac * per + ((xt + TX) & m);
      float v[AIT + AEX][2];
#pragma unroll
      for (int i = 0; i < AIT; ++i) {
        const float* row = a1c + static_cast<int64_t>((y0 + row_of(i) - 1) & m) * s;
        v[i][0] = row[c0];
        v[i][1] = row[c1];
      }
#pragma unroll
      for (int i = 0; i < AEX; ++i) {
        const float* row = a1c + static_cast<int64_t>((y0 + min(16 * i + ai, G::H2 - 1) - 1) & m) * s;
        v[AIT + i][0] = row[e0];
        v[AIT + i][1] = row[e1];
      }
      if (tid < G::NG) {
        const int yi = gy - 2, xi = gx - 2;
        if (yi >= 0 && yi < G::TY && xi >= 0 && xi < TX && y0 + yi < s && xt + xi < s) {
#pragma unroll
          for (int c = 0; c < 3; ++c) db3[c] += vg[c];
        }
        uint32_t a[3], c[3];
        split3r(vg[0], vg[1], a);
        split3r(vg[2], 0.0f, c);
#pragma unroll
        for (int k = 0; k < 3; ++k)
          *reinterpret_cast<u32x2*>(lds + kBwdGo + k * kGoPlane + tid * 8) = u32x2{a[k], c[k]};
      }
#pragma unroll
      for (int i = 0; i < TIT; ++i) {
        const int e = tid + i * kBwdThreads, cc = e / NP, r = e - cc * NP, y = r / PX, px = r - y * PX;
        if (cc < 2 * C) {
          uint32_t p[3];
          split3r(vt[i][0], vt[i][1], p);
          const int o = (cc < C ? kBwdZp + cc * G::ChB : kBwdGp + (cc - C) * G::ChB) + y * G::RowB + 4 * px;
#pragma unroll
          for (int k = 0; k < 3; ++k) *reinterpret_cast<uint32_t*>(lds + o + k * kThinPlane) = p[k];
        }
      }
      const auto put_h1 = [&](int i, int y, int px) {
        uint32_t p[3];
        split3r(fmaxf(v[i][0], 0.0f), fmaxf(v[i][1], 0.0f), p);
#pragma unroll
        for (int k = 0; k < 3; ++k)
          *reinterpret_cast<uint32_t*>(lds + kBwdH1 + k * kH1Plane + ac * G::ChB + y * G::RowB + 4 * px) = p[k];
      };
#pragma unroll
      for (int i = 0; i < AIT; ++i) put_h1(i, row_of(i), apx);
#pragma unroll
      for (int i = 0; i < AEX; ++i)
        if (16 * i + ai < G::H2) put_h1(AIT + i, 16 * i + ai, TX / 2);
    }
    __syncthreads();
    // D[p][c] of g2 before its mask: rows at `gp` (the lane's position in the
    // [pos][4] gradient, tap (0, 0))
    const auto conv3t = [&](const char* gp, f32x16& acc) {
      acc = f32x16{};
#pragma unroll
      for (int p = 2; p >= 0; --p)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const u32x2 a = *reinterpret_cast<const u32x2*>(gp + p * kGoPlane + go[k][0]);
          const u32x2 c = *reinterpret_cast<const u32x2*>(gp + p * kGoPlane + go[k][1]);
          acc = mma(u32x4{a.x, a.y, c.x, c.y}, w3t[k], acc);
        }
    };
    // part k of g2 of this lane's channel at halo position (yy, xx)
    const auto put_g2 = [&](int yy, int xx, int k, uint32_t bits) {
      *reinterpret_cast<uint16_t*>(lds + k * kG2Plane + (yy * G::W2 + xx) * 64 + (((l32 >> 3) ^ (xx >> 1 & 3)) << 4) +
                                   (l32 & 7) * 2) = static_cast<uint16_t>(bits);
    };
    // --- g2 around the tile
    if (wv >= 4 && wv < 4 + G::GR) {
      // rows above and below the tile, then the columns beside it (repeated
      // entries write the same value again)
      const int g = wv - 4;
      const auto ring = [&](int i, int& yy, int& xx) {
        if (TX == 32 ? g < 2 : g == 0) {
          yy = (TX == 32 ? g : i >> 4) ? G::H2 - 1 : 0;
          xx = 1 + (TX == 32 ? i : i & 15);
        } else if (TX == 32) {
          const int k = min(i, 2 * G::H2 - 1);
          yy = k >= G::H2 ? k - G::H2 : k;
          xx = k >= G::H2 ? G::W2 - 1 : 0;
        } else {
          yy = min(i, G::H2 - 1);
          xx = g == 1 ? 0 : G::W2 - 1;
        }
      };
      float a[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        int yy, xx;
        ring(drow(j, hi), yy, xx);
        a[j] = a2c[static_cast<int64_t>((y0 + yy - 1) & m) * s + ((xt + xx - 1) & m)];
      }
      int yl, xl;
      ring(l32, yl, xl);
      f32x16 acc;
      conv3t(lds + kBwdGo + (yl * G::GW + xl) * 8, acc);
#pragma unroll
      for (int j = 0; j < 16; j += 2) {
        uint32_t p[3];
        split3r(a[j] > 0.0f ? acc[j] : 0.0f, a[j + 1] > 0.0f ? acc[j + 1] : 0.0f, p);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          int yy, xx;
          ring(drow(j + e, hi), yy, xx);
#pragma unroll
          for (int k = 0; k < 3; ++k) put_g2(yy, xx, k, p[k] >> (16 * e));
        }
      }
    }
    // --- g2, dW3 and dW2 on the tile: 8 groups of 32 positions (a row of 32
    // or two of 16), each by two wavefronts, one for either half of the
    // accumulators (both compute g2)
    const auto grads = [&](auto Hc) {
    constexpr int HALF = decltype(Hc)::value;
#pragma unroll 1
    for (int gi = pw; gi < kTileP / 32; gi += 4) {
      const auto at = [&](int i, int& y, int& x) {
        y = TX == 32 ? gi : 2 * gi + (i >> 4);
        x = TX == 32 ? i : i & 15;
      };
      float a[16];
      uint32_t ok = 0xFFFFu;   // positions that count (bit j)
      if constexpr (WHOLE) {
#pragma unroll
        for (int jq = 0; jq < 4; ++jq) {
          int y, x;
          at(8 * jq + 4 * hi, y, x);
          const float4 q = *reinterpret_cast<const float4*>(a2c + static_cast<int64_t>(y0 + y) * s + xt + x);
          a[4 * jq] = q.x;
          a[4 * jq + 1] = q.y;
          a[4 * jq + 2] = q.z;
          a[4 * jq + 3] = q.w;
        }
      } else {
        ok = 0;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          int y, x;
          at(drow(j, hi), y, x);
          a[j] = a2c[static_cast<int64_t>(y & m) * s + (x & m)];
          ok |= (y < s && x < s ? 1u : 0u) << j;
        }
      }
      int yl, xl;
      at(l32, yl, xl);
      f32x16 acc;
      conv3t(lds + kBwdGo + ((yl + 1) * G::GW + xl + 1) * 8, acc);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        u32x4 gp[3], hp[3];   // parts of g2 and h2 of this step's positions
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int j = 8 * h + 2 * u;
          const float g0 = a[j] > 0.0f ? acc[j] : 0.0f, g1 = a[j + 1] > 0.0f ? acc[j + 1] : 0.0f;
          uint32_t p[3], q[3] = {0, 0, 0};
          split3r(g0, g1, p);
          const uint32_t keep = WHOLE ? 0xFFFFFFFFu
                                      : ((ok >> j & 1) ? 0xFFFFu : 0u) | ((ok >> j & 2) ? 0xFFFF0000u : 0u);
          if constexpr (HALF == 0) {
            split3r(fmaxf(a[j], 0.0f), fmaxf(a[j + 1], 0.0f), q);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              int y, x;
              at(drow(j + e, hi), y, x);
#pragma unroll
              for (int k = 0; k < 3; ++k) put_g2(y + 1, x + 1, k, p[k] >> (16 * e));
            }
            db2 += (keep & 0xFFFFu) ? g0 : 0.0f;
            db2 += (keep >> 16) ? g1 : 0.0f;
          }
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            gp[k][u] = p[k] & keep;
            hp[k][u] = q[k] & keep;
          }
        }
        const int y = TX == 32 ? gi : 2 * gi + h, x = (TX == 32 ? 16 * h : 0) + 4 * hi;
        const char* hb = lds + kBwdH1 + l32 * G::ChB + y * G::RowB + 2 * x;
        // part k of h1 at the step's positions moved by the three taps of row dy
        const auto window = [&](int dy, int k, u32x4 (&r)[3]) {
          const char* q = hb + k * kH1Plane + dy * G::RowB;
          const u32x2 w = *reinterpret_cast<const u32x2*>(q), u = *reinterpret_cast<const u32x2*>(q + 16);
          const uint32_t w2 = *reinterpret_cast<const uint32_t*>(q + 8);
          const uint32_t u2 = *reinterpret_cast<const uint32_t*>(q + 24);
          r[0] = u32x4{w.x, w.y, u.x, u.y};
          r[1] = u32x4{funnel(w.y, w.x, 16), funnel(w2, w.y, 16), funnel(u.y, u.x, 16), funnel(u2, u.y, 16)};
          r[2] = u32x4{w.y, w2, u.y, u2};
        };
        const auto part = [&](auto Kc) {
          constexpr int K = decltype(Kc)::value;
          u32x4 r[3];
          if constexpr (HALF == 0) {
            mma_part<K>(hp, thin_run(lds + gofs + K * kThinPlane + y * G::RowB + 2 * x, gsh), dw[4]);
            window(0, K, r);
#pragma unroll
            for (int d = 0; d < 3; ++d) mma_part<K>(gp, r[d], dw[d]);
            window(1, K, r);
            mma_part<K>(gp, r[0], dw[3]);
          } else {
            window(1, K, r);
            mma_part<K>(gp, r[1], dw[0]);
            mma_part<K>(gp, r[2], dw[1]);
            window(2, K, r);
#pragma unroll
            for (int d = 0; d < 3; ++d) mma_part<K>(gp, r[d], dw[2 + d]);
          }
        };
        part(std::integral_constant<int, 2>{});
        part(std::integral_constant<int, 1>{});
        part(std::integral_constant<int, 0>{});
      }
    }
    };
    if (half == 0) grads(std::integral_constant<int, 0>{});
    else grads(std::integral_constant<int, 1>{});
    // W2^T in registers for the next part only: the accumulators of the weight
    // gradients and all weights together do not fit
    const uint16_t* pk = S.pk;
    asm volatile("" : "+s"(pk));   // not hoisted out of the tile loop
    u32x4 w2t[18];
#pragma unroll
    for (int k = 0; k < 18; ++k) w2t[k] = pk_at(pk, kPk2T + k, lane);
    __syncthreads();
    // --- g1 and dW1, a group per wavefront
    {
      const int gi = wv;
      const int yl = TX == 32 ? gi : 2 * gi + (l32 >> 4), xl = TX == 32 ? l32 : l32 & 15;
      f32x16 acc = {};
      int at0[3];   // of the taps (0, dx)
#pragma unroll
      for (int d = 0; d < 3; ++d) at0[d] = (yl * G::W2 + xl + d) * 64 + ((hi ^ (xl + d >> 1 & 3)) << 4);
#pragma unroll
      for (int p = 2; p >= 0; --p)
#pragma unroll
        for (int k = 0; k < 18; ++k)
          acc = mma(*reinterpret_cast<const u32x4*>(lds + p * kG2Plane + (k / 6) * (G::W2 * 64) +
                                                    (at0[(k >> 1) % 3] ^ (32 * (k & 1)))),
                    w2t[k], acc);
      pipeline_reads<54, 6>();
      u32x4 gp[2][3];
#pragma unroll
      for (int jq = 0; jq < 4; ++jq) {
        const int r = 8 * jq + 4 * hi, y = TX == 32 ? gi : 2 * gi + (r >> 4), x = TX == 32 ? r : r & 15;
        const char* q = lds + kBwdH1 + l32 * G::ChB + (y + 1) * G::RowB + 2 * x;
        const u32x2 w = *reinterpret_cast<const u32x2*>(q);
        const uint32_t w2 = *reinterpret_cast<const uint32_t*>(q + 8);
        // h1 > 0 at the four positions: its leading part is not zero
        const uint32_t on[4] = {w.x >> 16, w.y & 0xFFFFu, w.y >> 16, w2 & 0xFFFFu};
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool keep = on[e] != 0 && (WHOLE || (y < s && x + e < s));
          v[e] = keep ? acc[4 * jq + e] : 0.0f;
          db1 += v[e];
        }
        uint32_t p[3], u[3];
        split3r(v[0], v[1], p);
        split3r(v[2], v[3], u);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          gp[jq >> 1][k][2 * (jq & 1)] = p[k];
          gp[jq >> 1][k][2 * (jq & 1) + 1] = u[k];
        }
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int y = TX == 32 ? gi : 2 * gi + h, x = (TX == 32 ? 16 * h : 0) + 4 * hi;
        mma_part<2>(gp[h], thin_run(lds + zofs + 2 * kThinPlane + y * G::RowB + 2 * x, zsh), dw1);
        mma_part<1>(gp[h], thin_run(lds + zofs + kThinPlane + y * G::RowB + 2 * x, zsh), dw1);
        mma_part<0>(gp[h], thin_run(lds + zofs + y * G::RowB + 2 * x, zsh), dw1);
      }
    }
    __syncthreads();
  }
  // --- the block's row of partial gradients: wavefront pair pw writes (pw < 2)
  // or adds (pw >= 2) its sums to row pw mod 2, then the two rows and the second
  // half's dW1 are added
  constexpr int kRow = kRowFloats + 28 * kF;
  static_assert(2 * kRow * 4 <= kBwdLds, "two rows of gradients");
  float* red = reinterpret_cast<float*>(lds) + (pw & 1) * kRow;
  const int oB1 = 9 * kF * C, oW2 = oB1 + kF, oB2 = oW2 + 9 * kF * kF, oW3 = oB2 + kF, oB3 = oW3 + 9 * kF * C;
  const int oD1 = half == 0 ? 0 : kRowFloats;   // dW1 and db1 of this half
  db1 += __shfl_xor(db1, 32);
  db2 += __shfl_xor(db2, 32);
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) db3[c] += __shfl_xor(db3[c], o);
  float* sum3 = reinterpret_cast<float*>(lds) + 2 * kRow;   // db3 of the wavefronts
  static_assert((2 * kRow + 4 * kBwdWaves) * 4 <= kBwdLds, "and the last bias");
  if (lane == 0) {
#pragma unroll
    for (int c = 0; c < 3; ++c) sum3[4 * wv + c] = db3[c];
  }
  for (int round = 0; round < 2; ++round) {
    if (pw >> 1 == round) {
      const auto put = [&](const f32x16& v, int first, int step) {   // entry j at first + step drow(j)
        float o[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) o[j] = round == 0 ? 0.0f : red[first + step * drow(j, hi)];
#pragma unroll
        for (int j = 0; j < 16; ++j) red[first + step * drow(j, hi)] = o[j] + v[j];
      };
#pragma unroll
      for (int d = 0; d < 5; ++d) {
        if (half == 1 || d < 4) put(dw[d], oW2 + l32 * 9 + 4 * half + d, 9 * kF);
        else if (l32 < 9 * C) put(dw[d], oW3 + (l32 / 9) * (9 * kF) + l32 % 9, 9);
      }
      if (l32 < 9 * C) put(dw1, oD1 + l32, 9 * C);
      if (hi == 0) {
        red[oD1 + oB1 + l32] = (round == 0 ? 0.0f : red[oD1 + oB1 + l32]) + db1;
        if (half == 0) red[oB2 + l32] = (round == 0 ? 0.0f : red[oB2 + l32]) + db2;
      }
    }
    __syncthreads();
  }
  const float* r0 = reinterpret_cast<const float*>(lds);
  for (int e = threadIdx.x; e < oB3; e += kBwdThreads) {
    float v = r0[e] + r0[kRow + e];
    if (e < oW2) v += r0[kRowFloats + e] + r0[kRow + kRowFloats + e];
    partial[static_cast<int64_t>(blockIdx.x) * kRowFloats + e] = v;
  }
  if (static_cast<int>(threadIdx.x) < C) {
    float v = 0.0f;
    for (int w = 0; w < kBwdWaves; ++w) v += sum3[4 * w + threadIdx.x];
    partial[static_cast<int64_t>(blockIdx.x) * kRowFloats + oB3 + threadIdx.x] = v;
  }
}

// Bound by the vector work of the splits and the staging beside the products
// (per 8 x 32 tile 40 thousand cycles, 13 of them products, two thirds of these
// dW2).  The nine taps' accumulators are split over two wavefronts, so that two
// fit on a SIMD and one's loads and splits run beside the other's products
// (with one wavefront per SIMD holding them all: 316 us, this one 290 us).  They
// fit with 256 registers each because the compiler keeps 324 values in scratch
// (700 bytes a lane, over the three forms of bwd_stack together); what these cost
// is not known apart from the rest.  A
// training step of 32 images of 256 x 256 takes 0.42 ms (forward 0.12 ms, this
// kernel 0.29 ms); with float32 matrix products, a kernel per layer and the
// forward pass twice it took 1.29 ms.
__global__ __launch_bounds__(kBwdThreads, 2) void k_net_bwd(NetArg net, const float* __restrict__ x0,
                                                            const float* __restrict__ gout, int64_t N,
                                                            float* __restrict__ partial) {
  extern __shared__ __align__(16) char lds[];
  const StackArg& S = net.st[stack_of(net)];
  if (S.s >= 32) bwd_stack<32, true>(S, x0, gout, N, partial, lds);
  else if (S.s >= 16) bwd_stack<16, true>(S, x0, gout, N, partial, lds);
  else bwd_stack<16, false>(S, x0, gout, N, partial, lds);
}

// grad[i] = sum over the stack's blocks of their partial rows (blockIdx.y: the
// stack): a block of 16 wavefronts takes 64 consecutive i, wavefront w the rows
// w, w + 16, ..., and the 16 sums are added in a fixed order.
constexpr int kSumWaves = 16;
__global__ __launch_bounds__(64 * kSumWaves) void k_sum_partials(NetArg net, const float* __restrict__ partial,
                                                                 float* __restrict__ grad,
                                                                 const double* __restrict__ loss, int nblocks,
                                                                 double count, double* __restrict__ dloss,
                                                                 double* __restrict__ hloss) {
  __shared__ float red[kSumWaves][64];
  if (blockIdx.x == gridDim.x - 1) {   // the mean squared error, on the device and for the host
    if (blockIdx.y == 0 && threadIdx.x < 64) {
      double a = 0.0;
      for (int b = threadIdx.x; b < nblocks; b += 64) a += loss[b];
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o);
      if (threadIdx.x == 0) *dloss = *hloss = a / count;
    }
    return;
  }
  const StackArg& S = net.st[blockIdx.y];
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + l;
  const int np = 18 * kF * S.C + 9 * kF * kF + 2 * kF + S.C;
  float a = 0.0f;
  if (i < np) {
    const float* p = partial + static_cast<int64_t>(S.blk0) * kRowFloats + i;
    int b = w;
    for (; b + 3 * kSumWaves < S.nblk; b += 4 * kSumWaves) {
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = p[static_cast<int64_t>(b + u * kSumWaves) * kRowFloats];
#pragma unroll
      for (int u = 0; u < 4; ++u) a += v[u];
    }
    for (; b < S.nblk; b += kSumWaves) a += p[static_cast<int64_t>(b) * kRowFloats];
  }
  red[w][l] = a;
  __syncthreads();
  if (w == 0 && i < np) {
    float t = 0.0f;
    for (int k = 0; k < kSumWaves; ++k) t += red[k][l];
    grad[S.prow + i] = t;
  }
}

// One packed weight: operand `step` of its stack, lane, element i (the layout
// of mma's operands; k of conv1 and of W3^T = 4 tap + channel, of conv2 and W2^T
// = 32 tap + channel, of conv3 the channel order of conv2's accumulators).
__device__ __forceinline__ uint16_t pk_value(const uint16_t* __restrict__ w1, const uint16_t* __restrict__ w2,
                                             const uint16_t* __restrict__ w3, int C, int step, int lane, int i) {
  const int r = lane & 31, hi = lane >> 5, slot = 8 * hi + i;
  if (step < kPk2) {
    const int k = 16 * step + slot, t = k >> 2, c = k & 3;
    return t < 9 && c < C ? w1[(r * C + c) * 9 + t] : 0;
  }
  if (step < kPk3) {
    const int k = step - kPk2;
    return w2[(r * kF + 16 * (k & 1) + slot) * 9 + (k >> 1)];
  }
  if (step < kPk3T) {
    const int c = drow(8 * (step - kPk3) + i, hi);
    return r < 9 * C ? w3[((r / 9) * kF + c) * 9 + r % 9] : 0;
  }
  if (step < kPk2T) {
    const int k = 16 * (step - kPk3T) + slot, t = k >> 2, o = k & 3;
    return t < 9 && o < C ? w3[(o * kF + r) * 9 + 8 - t] : 0;
  }
  const int k = step - kPk2T;
  return w2[((16 * (k & 1) + slot) * kF + r) * 9 + 8 - (k >> 1)];
}

__global__ void k_pack(NetArg net, const uint16_t* __restrict__ wbf, uint16_t* __restrict__ wpk) {
  const StackArg& S = net.st[blockIdx.y];
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= kPkStack) return;
  const uint16_t* w1 = wbf + S.prow;
  const uint16_t* w2 = w1 + 9 * kF * S.C + kF;
  const uint16_t* w3 = w2 + 9 * kF * kF + kF;
  wpk[blockIdx.y * kPkStack + e] = pk_value(w1, w2, w3, S.C, e >> 9, (e >> 3) & 63, e & 7);
}

__global__ void k_adam(float* __restrict__ master, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ g, int64_t n, float lr, float b1, float b2, float c1, float c2,
                       float eps, uint16_t* __restrict__ wbf, const double* __restrict__ loss) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n || !isfinite(*loss)) return;   // a step that diverged changes nothing
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float w = master[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  master[i] = w;
  wbf[i] = f2bf(w);
}

__global__ void k_round_bf16(const float* __restrict__ master, uint16_t* __restrict__ wbf, int64_t n) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) wbf[i] = f2bf(master[i]);
}

inline dim3 grid_for(int64_t n) { return dim3(static_cast<unsigned>((n + kBlk - 1) / kBlk)); }

}  // namespace

struct wdb_cnn {
  int device = 0;
  int n = 0, levels = 0, F = kF;
  int cus = 0;               // compute units: a block of either kernel fills one
  int64_t N = 0;
  struct Stack {
    int64_t off;
    int C, s;
    int64_t p[6];  // offsets of W1, b1, W2, b2, W3, b3
  };
  std::vector<Stack> stacks;
  int64_t nparam = 0;
  float* master = nullptr;
  uint16_t* wbf = nullptr;
  uint16_t* wpk = nullptr;   // the kernels' packed weights, kPkStack per stack
  float* m = nullptr;
  float* v = nullptr;
  float* grad = nullptr;
  int64_t t = 0;
  // training workspace
  int bcap = 0;
  float* a1 = nullptr;      // pre-activations of all stacks, 32 per position
  float* a2 = nullptr;
  float* gout = nullptr;    // B*N
  float* partial = nullptr; // a row of partial gradients per block
  double* dpart = nullptr;  // the loss, then a sum per block
  double* hloss = nullptr;  // pinned
};

namespace {

void cnn_free_ws(wdb_cnn* c) {
  float* fs[] = {c->a1, c->a2, c->gout, c->partial};
  for (float* p : fs)
    if (p) (void)hipFree(p);
  if (c->dpart) (void)hipFree(c->dpart);
  if (c->hloss) (void)hipHostFree(c->hloss);
  c->a1 = c->a2 = c->gout = c->partial = nullptr;
  c->dpart = nullptr;
  c->hloss = nullptr;
  c->bcap = 0;
}

// Positions of all stacks of one image.
int64_t cnn_positions(const wdb_cnn* c) {
  int64_t p = 0;
  for (const auto& S : c->stacks) p += static_cast<int64_t>(S.s) * S.s;
  return p;
}

int cnn_most_blocks(const wdb_cnn* c) { return std::max(c->cus, static_cast<int>(c->stacks.size())); }

void cnn_ensure(wdb_cnn* c, int B) {
  if (B <= c->bcap) return;
  cnn_free_ws(c);
  const int64_t act = static_cast<int64_t>(B) * kF * cnn_positions(c);
  const size_t nb = static_cast<size_t>(cnn_most_blocks(c));
  WDB_HIP(hipMalloc(reinterpret_cast<void**>(&c->a1), act * sizeof(float)));
  WDB_HIP(hipMalloc(reinterpret_cast<void**>(&c->a2), act * sizeof(float)));
  WDB_HIP(hipMalloc(reinterpret_cast<void**>(&c->gout), static_cast<int64_t>(B) * c->N * sizeof(float)));
  WDB_HIP(hipMalloc(reinterpret_cast<void**>(&c->partial), nb * kRowFloats * sizeof(float)));
  WDB_HIP(hipMalloc(reinterpret_cast<void**>(&c->dpart), (nb + 1) * sizeof(double)));
  WDB_HIP(hipHostMalloc(reinterpret_cast<void**>(&c->hloss), sizeof(double), hipHostMallocDefault));
  c->bcap = B;
}

// The stacks' shares of a launch over B images: the least work per block that
// fits all blocks on the compute units at once (a block per unit; each stack
// has at least one).  A 16 x 16 tile of the backward pass takes 1.2 times an 8 x
// 32 one (48 against 40 thousand cycles): work in fifths.  Returns the number
// of blocks.
int net_arg(const wdb_cnn* c, int B, bool train, NetArg* net) {
  int64_t most = 1;
  net->nstacks = static_cast<int>(c->stacks.size());
  int64_t at = 0;
  for (int k = 0; k < net->nstacks; ++k) {
    const auto& S = c->stacks[k];
    StackArg& a = net->st[k];
    const int tx = S.s >= 32 ? 32 : 16, ty = kTileP / tx;
    a.off = S.off;
    a.C = S.C;
    a.s = S.s;
    a.tiles_x = std::max(S.s / tx, 1);
    a.tiles_img = a.tiles_x * std::max(S.s / ty, 1);
    WDB_REQUIRE(static_cast<int64_t>(B) * a.tiles_img < (int64_t{1} << 30), WDB_ERR_ARG, "batch too large");
    a.ntiles = B * a.tiles_img;
    a.prow = S.p[0];
    a.pk = c->wpk + k * kPkStack;
    for (int l = 0; l < 3; ++l) a.b[l] = c->wbf + S.p[2 * l + 1];
    a.a1 = c->a1 ? c->a1 + at : nullptr;
    a.a2 = c->a2 ? c->a2 + at : nullptr;
    at += static_cast<int64_t>(c->bcap) * kF * S.s * S.s;
    most = std::max<int64_t>(most, a.ntiles * int64_t{6});
  }
  const auto share = [&](int k, int64_t work) {   // blocks of stack k with that much work each
    const int64_t tiles = std::max<int64_t>(1, work / (train && net->st[k].s < 32 ? 6 : 5));
    return (net->st[k].ntiles + tiles - 1) / tiles;
  };
  const auto blocks = [&](int64_t work) {
    int64_t n = 0;
    for (int k = 0; k < net->nstacks; ++k) n += share(k, work);
    return n;
  };
  int64_t lo = 1, hi = most;   // the least work whose blocks fit
  while (lo < hi) {
    const int64_t mid = (lo + hi) / 2;
    if (blocks(mid) <= cnn_most_blocks(c)) hi = mid;
    else lo = mid + 1;
  }
  int first = 0;
  for (int k = 0; k < net->nstacks; ++k) {
    net->st[k].blk0 = first;
    net->st[k].nblk = static_cast<int>(share(k, lo));
    first += net->st[k].nblk;
  }
  return first;
}

// Refresh the packed weights from the bfloat16 parameters (after every change of wbf).
void pack_weights(wdb_cnn* c, hipStream_t st) {
  NetArg net{};
  (void)net_arg(c, 1, false, &net);
  hipLaunchKernelGGL(k_pack, dim3(static_cast<unsigned>((kPkStack + kBlk - 1) / kBlk), net.nstacks), dim3(kBlk), 0, st,
                     net, c->wbf, c->wpk);
  WDB_HIP(hipGetLastError());
}

void forward(wdb_cnn* c, const float* x0, int B, float* out, hipStream_t st) {
  NetArg net{};
  const int nb = net_arg(c, B, false, &net);
  hipLaunchKernelGGL(k_net_fwd<false>, dim3(nb), dim3(kFwdThreads), kFwdLds, st, net, x0, c->N, out, TrainArg{});
  WDB_HIP(hipGetLastError());
}

// Enqueue the loss (c->dpart[0] and, once the stream has passed it, *c->hloss)
// and the gradient (c->grad, float32).
void loss_grad(wdb_cnn* c, const float* x0, const float* tgt, int B, hipStream_t st) {
  const int64_t tot = static_cast<int64_t>(B) * c->N;
  NetArg net{};
  const int nb = net_arg(c, B, true, &net);
  const TrainArg tr{tgt, c->gout, c->dpart + 1, static_cast<float>(2.0 / static_cast<double>(tot))};
  hipLaunchKernelGGL(k_net_fwd<true>, dim3(nb), dim3(kFwdThreads), kFwdLds, st, net, x0, c->N,
                     static_cast<float*>(nullptr), tr);
  hipLaunchKernelGGL(k_net_bwd, dim3(nb), dim3(kBwdThreads), kBwdLds, st, net, x0, c->gout, c->N, c->partial);
  hipLaunchKernelGGL(k_sum_partials, dim3((kStackParams + 63) / 64 + 1, net.nstacks), dim3(64 * kSumWaves), 0, st, net,
                     c->partial, c->grad, c->dpart + 1, nb, static_cast<double>(tot), c->dpart, c->hloss);
  WDB_HIP(hipGetLastError());
}

uint64_t splitmix(uint64_t& s) {
  uint64_t z = (s += 0x9e3779b97f4a7c15ull);
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

}  // namespace

extern "C" {

wdb_status wdb_cnn_create(int32_t n, int32_t levels, int32_t features, uint64_t seed, wdb_cnn** out) {
  using namespace wdb;
  WDB_API_BEGIN
  WDB_REQUIRE(out, WDB_ERR_ARG, "null output");
  WDB_REQUIRE(features == kF, WDB_ERR_ARG, "only %d hidden channels are built", kF);
  check_geometry(n, levels, 2);
  WDB_REQUIRE((n >> levels) >= 2, WDB_ERR_LEVELS, "coarsest level too small for 3x3 convolutions");
  wdb_cnn* c = new wdb_cnn();
  try {
    WDB_HIP(hipGetDevice(&c->device));
    WDB_HIP(hipDeviceGetAttribute(&c->cus, hipDeviceAttributeMultiprocessorCount, c->device));
    for (const void* k : {reinterpret_cast<const void*>(k_net_fwd<false>), reinterpret_cast<const void*>(k_net_fwd<true>)})
      WDB_HIP(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kFwdLds));
    WDB_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_net_bwd), hipFuncAttributeMaxDynamicSharedMemorySize,
                                kBwdLds));
    c->n = n;
    c->levels = levels;
    c->N = static_cast<int64_t>(n) * n;
    const std::vector<Subband> lay = layout(n, levels);
    int64_t pos = 0;
    auto add = [&](int64_t off, int C, int s) {
      wdb_cnn::Stack S{off, C, s, {0, 0, 0, 0, 0, 0}};
      const int64_t sizes[6] = {int64_t(kF) * C * 9, kF, int64_t(kF) * kF * 9, kF, int64_t(C) * kF * 9, C};
      for (int k = 0; k < 6; ++k) {
        S.p[k] = pos;
        pos += sizes[k];
      }
      c->stacks.push_back(S);
    };
    WDB_REQUIRE(levels < kMaxStacks, WDB_ERR_LEVELS, "at most %d levels", kMaxStacks - 1);
    add(lay[0].offset, 1, lay[0].side);
    for (size_t k = 1; k < lay.size(); k += 3) add(lay[k].offset, 3, lay[k].side);
    c->nparam = pos;
    // He-normal convolution weights (SplitMix64 + Box-Muller), zero biases; the
    // last convolution of each stack starts 10x smaller so the network starts
    // close to the identity map.
    std::vector<float> h(pos, 0.0f);
    uint64_t st = seed;
    auto normal = [&]() {
      const double u1 = (static_cast<double>(splitmix(st) >> 11) + 0.5) * 0x1.0p-53;
      const double u2 = static_cast<double>(splitmix(st) >> 11) * 0x1.0p-53;
      return std::sqrt(-2.0 * std::log(u1)) * std::cos(2.0 * M_PI * u2);
    };
    for (auto& S : c->stacks) {
      const int fan[3] = {S.C * 9, kF * 9, kF * 9};
      const int64_t len[3] = {int64_t(kF) * S.C * 9, int64_t(kF) * kF * 9, int64_t(S.C) * kF * 9};
      for (int l = 0; l < 3; ++l) {
        const double sd = std::sqrt(2.0 / fan[l]) * (l == 2 ? 0.1 : 1.0);
        for (int64_t i = 0; i < len[l]; ++i) h[S.p[2 * l] + i] = static_cast<float>(sd * normal());
      }
    }
    WDB_HIP(hipMalloc(reinterpret_cast<void**>(&c->master), pos * sizeof(float)));
    WDB_HIP(hipMalloc(reinterpret_cast<void**>(&c->wbf), pos * sizeof(uint16_t)));
    WDB_HIP(hipMalloc(reinterpret_cast<void**>(&c->wpk), c->stacks.size() * kPkStack * sizeof(uint16_t)));
    WDB_HIP(hipMalloc(reinterpret_cast<void**>(&c->m), pos * sizeof(float)));
    WDB_HIP(hipMalloc(reinterpret_cast<void**>(&c->v), pos * sizeof(float)));
    WDB_HIP(hipMalloc(reinterpret_cast<void**>(&c->grad), pos * sizeof(float)));
    WDB_HIP(hipMemcpy(c->master, h.data(), pos * sizeof(float), hipMemcpyHostToDevice));
    WDB_HIP(hipMemset(c->m, 0, pos * sizeof(float)));
    WDB_HIP(hipMemset(c->v, 0, pos * sizeof(float)));
    hipLaunchKernelGGL(k_round_bf16, grid_for(pos), dim3(kBlk), 0, nullptr, c->master, c->wbf, pos);
    pack_weights(c, nullptr);
    WDB_HIP(hipGetLastError());
    WDB_HIP(hipDeviceSynchronize());
  } catch (...) {
    wdb_cnn_free(c);
    throw;
  }
  *out = c;
  WDB_API_END
}

wdb_status wdb_cnn_param_count(const wdb_cnn* c, int64_t* count) {
  WDB_API_BEGIN
  WDB_REQUIRE(c && count, WDB_ERR_ARG, "null argument");
  *count = c->nparam;
  WDB_API_END
}

wdb_status wdb_cnn_set_params(wdb_cnn* c, const float* host, int64_t count) {
  WDB_API_BEGIN
  WDB_REQUIRE(c && host, WDB_ERR_ARG, "null argument");
  WDB_REQUIRE(count == c->nparam, WDB_ERR_ARG, "expected %lld parameters", static_cast<long long>(c->nparam));
  for (int64_t i = 0; i < count; ++i)
    WDB_REQUIRE(std::isfinite(host[i]), WDB_ERR_NONFINITE, "non-finite parameter %lld", static_cast<long long>(i));
  WDB_HIP(hipSetDevice(c->device));
  WDB_HIP(hipMemcpy(c->master, host, count * sizeof(float), hipMemcpyHostToDevice));
  WDB_HIP(hipMemset(c->m, 0, count * sizeof(float)));
  WDB_HIP(hipMemset(c->v, 0, count * sizeof(float)));
  c->t = 0;
  hipLaunchKernelGGL(k_round_bf16, grid_for(count), dim3(kBlk), 0, nullptr, c->master, c->wbf, count);
  pack_weights(c, nullptr);
  WDB_HIP(hipGetLastError());
  WDB_HIP(hipDeviceSynchronize());
  WDB_API_END
}

wdb_status wdb_cnn_get_params(const wdb_cnn* c, float* host, int32_t rounded) {
  WDB_API_BEGIN
  WDB_REQUIRE(c && host, WDB_ERR_ARG, "null argument");
  WDB_HIP(hipSetDevice(c->device));
  if (!rounded) {
    WDB_HIP(hipMemcpy(host, c->master, c->nparam * sizeof(float), hipMemcpyDeviceToHost));
  } else {
    std::vector<uint16_t> b(c->nparam);
    WDB_HIP(hipMemcpy(b.data(), c->wbf, c->nparam * sizeof(uint16_t), hipMemcpyDeviceToHost));
    for (int64_t i = 0; i < c->nparam; ++i) {
      const uint32_t u = static_cast<uint32_t>(b[i]) << 16;
      std::memcpy(&host[i], &u, 4);
    }
  }
  WDB_API_END
}

wdb_status wdb_cnn_predict(wdb_cnn* c, const float* x0, int32_t batch, float* out, void* stream) {
  WDB_API_BEGIN
  WDB_REQUIRE(c && x0 && out, WDB_ERR_ARG, "null argument");
  WDB_REQUIRE(batch >= 1, WDB_ERR_ARG, "batch must be >= 1");
  WDB_REQUIRE(x0 != out, WDB_ERR_ARG, "x0 and out must not alias");
  WDB_HIP(hipSetDevice(c->device));
  forward(c, x0, batch, out, static_cast<hipStream_t>(stream));
  WDB_API_END
}

wdb_status wdb_cnn_loss_grad(wdb_cnn* c, const float* x0, const float* target, int32_t batch, double* loss,
                             float* grad_host, void* stream) {
  WDB_API_BEGIN
  WDB_REQUIRE(c && x0 && target, WDB_ERR_ARG, "null argument");
  WDB_REQUIRE(batch >= 1, WDB_ERR_ARG, "batch must be >= 1");
  WDB_HIP(hipSetDevice(c->device));
  cnn_ensure(c, batch);
  loss_grad(c, x0, target, batch, static_cast<hipStream_t>(stream));
  WDB_HIP(hipStreamSynchronize(static_cast<hipStream_t>(stream)));
  if (loss) *loss = *c->hloss;
  if (grad_host) WDB_HIP(hipMemcpy(grad_host, c->grad, c->nparam * sizeof(float), hipMemcpyDeviceToHost));
  WDB_API_END
}

wdb_status wdb_cnn_train_step(wdb_cnn* c, const float* x0, const float* target, int32_t batch, float lr,
                              double* loss, void* stream) {
  WDB_API_BEGIN
  WDB_REQUIRE(c && x0 && target, WDB_ERR_ARG, "null argument");
  WDB_REQUIRE(batch >= 1 && std::isfinite(lr) && lr > 0, WDB_ERR_ARG, "bad batch or learning rate");
  WDB_HIP(hipSetDevice(c->device));
  cnn_ensure(c, batch);
  hipStream_t st = static_cast<hipStream_t>(stream);
  loss_grad(c, x0, target, batch, st);
  // the step follows without waiting for the loss: the kernel looks at it
  const double b1 = 0.9, b2 = 0.999;
  const double t = static_cast<double>(c->t + 1);
  const float c1 = static_cast<float>(1.0 - std::pow(b1, t));
  const float c2 = static_cast<float>(1.0 - std::pow(b2, t));
  hipLaunchKernelGGL(k_adam, grid_for(c->nparam), dim3(kBlk), 0, st, c->master, c->m, c->v, c->grad, c->nparam, lr,
                     static_cast<float>(b1), static_cast<float>(b2), c1, c2, 1e-8f, c->wbf, c->dpart);
  pack_weights(c, st);
  WDB_HIP(hipGetLastError());
  WDB_HIP(hipStreamSynchronize(st));
  const double L = *c->hloss;
  WDB_REQUIRE(std::isfinite(L), WDB_ERR_DIVERGED, "training loss became non-finite");
  c->t += 1;
  if (loss) *loss = L;
  WDB_API_END
}

void wdb_cnn_free(wdb_cnn* c) {
  if (!c) return;
  (void)hipSetDevice(c->device);
  (void)hipDeviceSynchronize();
  cnn_free_ws(c);
  float* fs[] = {c->master, c->m, c->v, c->grad};
  for (float* p : fs)
    if (p) (void)hipFree(p);
  if (c->wbf) (void)hipFree(c->wbf);
  if (c->wpk) (void)hipFree(c->wpk);
  delete c;
}

}  // extern "C"
