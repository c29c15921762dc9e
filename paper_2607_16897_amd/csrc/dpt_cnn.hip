// Learned initialiser: a small CNN that proposes the reference-to-current
// twist from the coarsest pyramid pair (60 x 94, two channels), replacing the
// constant-velocity start of the coarse-to-fine Gauss-Newton track.
//
// Network: four 3x3 stride-2 padding-1 convolutions with ReLU (2-16-32-64-64
// channels), global average pool, FC 64-64 ReLU, FC 64-6.  Activations and
// convolution weights are BF16 in NHWC / [co][ky][kx][ci] layouts; the
// forward convolutions are implicit GEMMs on the matrix cores
// (v_mfma_f32_16x16x16bf16_1k, FP32 accumulation) with bias and ReLU fused in
// the epilogue.  The backward convolutions are implicit GEMMs too: the data
// gradient per stride-parity class of the input pixels (only the taps that reach a
// class) on the same instruction, the weight gradient as dZ^T Xcol
// (v_mfma_f32_16x16x32_bf16) split over samples, with the bias gradient as a column
// of ones; gradients flowing between layers are stored in BF16, split reductions are
// summed in a fixed order.  Pooling, the FC layers, the loss and Adam run on the vector
// units; master weights and Adam moments are FP32.
#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "../../include/dptrack.h"
#include "dpt_device.h"
#include "dpt_internal.h"

struct dpt_cnn;

namespace dpt {
namespace cnn {

constexpr int kH0 = 60, kW0 = 94;
constexpr int kC[5] = {2, 16, 32, 64, 64};
constexpr int kHs[5] = {60, 30, 15, 8, 4};
constexpr int kWs[5] = {94, 47, 24, 12, 6};
constexpr int kHidden = 64, kOut = 6;

typedef short short4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);  // round to nearest even
  return (uint16_t)(u >> 16);
}
// The same of two floats (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t f2bf_pair(float lo, float hi) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{lo, hi}, b2));
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ short4_t bf16x4(uint2 v) {
  typedef uint32_t words __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(short4_t, words{v.x, v.y});
}

// ---------------------------------------------------------------- layout
// Flat FP32 parameter vector, tensor order w1 b1 w2 b2 w3 b3 w4 b4 fw1 fb1 fw2 fb2.
// Conv weights are stored [co][ky][kx][ci] internally; the ABI uses [co][ci][ky][kx].
struct Offsets {
  int w[4], b[4], fw1, fb1, fw2, fb2, total;
};

__host__ __device__ inline Offsets offsets() {
  Offsets o{};
  int s = 0;
  for (int l = 0; l < 4; ++l) {
    o.w[l] = s;
    s += kC[l + 1] * kC[l] * 9;
    o.b[l] = s;
    s += kC[l + 1];
  }
  o.fw1 = s;
  s += kHidden * 64;
  o.fb1 = s;
  s += kHidden;
  o.fw2 = s;
  s += kOut * kHidden;
  o.fb2 = s;
  s += kOut;
  o.total = s;
  return o;
}

// The BF16 convolution weights, in the layouts the kernels stage in LDS: layer l
// forward as [co][tap][ci], rows of kWRow[l] elements, and (l >= 1) for the data
// gradient as [tap][ci][co], rows of kTRow[l].  Sixteen lanes read 8 bytes each
// from sixteen consecutive rows, four lane groups 8 bytes apart; rows an odd
// multiple of 16 bytes apart spread a half wave over all banks (rows of 576 or
// 1152 bytes put eight or sixteen lanes on the same ones), so rows are padded to
// that.  The same holds for the activations' pixels, two apart in the forward
// convolutions (kXRow, layers' inputs: an odd multiple of 8) and adjacent in the
// data gradient (kDRow).
constexpr int kWRow[4] = {18, 152, 296, 584};
constexpr int kTRow[4] = {0, 40, 72, 72};
constexpr int kXRow[4] = {2, 20, 36, 68};
constexpr int kDRow[5] = {0, 0, 40, 72, 72};
// Activations and gradients lie in LDS with the zero pixels the convolutions pad
// with, so that every tap is at a fixed distance: inputs of layer l + 1 from row
// and column -1 to 2 Ho - 1 and 2 Wo - 1, gradients with a row and column past the
// last.
constexpr int xrows(int l) { return 2 * kHs[l + 1] + 1; }
constexpr int xcols(int l) { return 2 * kWs[l + 1] + 1; }
constexpr int xbytes(int l) { return (2 * xrows(l) * xcols(l) * kXRow[l] + 15) / 16 * 16; }
constexpr int drows(int l) { return kHs[l] + 1; }
constexpr int dcols(int l) { return kWs[l] + 1; }
constexpr int dbytes(int l) { return (2 * drows(l) * dcols(l) * kDRow[l] + 15) / 16 * 16; }
__host__ __device__ constexpr int wrow_off(int l) { return l == 0 ? 0 : wrow_off(l - 1) + kC[l] * kWRow[l - 1]; }
__host__ __device__ constexpr int trow_off(int l) { return l <= 1 ? 0 : trow_off(l - 1) + 9 * kC[l - 1] * kTRow[l - 1]; }
constexpr int kPbTotal = wrow_off(4), kPbTTotal = trow_off(4);

// ---------------------------------------------------------------- head forward and proposal (device parts)

// The network's outputs are twists scaled to unit range: 5 degrees (in
// radians) for the rotation part, 0.1 m for the translation part.
__constant__ double kTwistScaleDev[6] = {0.08726646259971647, 0.08726646259971647, 0.08726646259971647,
                                         0.1, 0.1, 0.1};

// rel = exp(xi) as 3x4 FP64, xi = the six scaled outputs o6 (rotation first).
__device__ __forceinline__ void propose_twist(const float* o6, double* rel) {
  double xi[6];
  for (int j = 0; j < 6; ++j) xi[j] = (double)o6[j] * kTwistScaleDev[j];
  const double th2 = fma(xi[0], xi[0], fma(xi[1], xi[1], xi[2] * xi[2]));
  double A, Bc, C;
  if (th2 < 1e-8) {  // |w| < 1e-4: series, truncation below 1e-17
    A = 1.0 - th2 * (1.0 / 6.0);
    Bc = 0.5 - th2 * (1.0 / 24.0);
    C = (1.0 / 6.0) - th2 * (1.0 / 120.0);
  } else {
    const double th = sqrt(th2), sn = sin(th), sh = sin(0.5 * th);
    A = sn / th;
    Bc = 2.0 * sh * sh / th2;
    C = (th - sn) / (th2 * th);
  }
  double T[12] = {1.0, 0.0, 0.0, 0.0, 0.0, 1.0, 0.0, 0.0, 0.0, 0.0, 1.0, 0.0};
  compose_exp(T, xi[0], xi[1], xi[2], xi[3], xi[4], xi[5], th2, A, Bc, C);
  for (int j = 0; j < 12; ++j) rel[j] = T[j];
}

// ---------------------------------------------------------------- forward convolutions (fused, MFMA)

constexpr int kFuseThreads = 1024;

// Zero the border pixels of a layer's input (rows and columns outside the image)
// or of a gradient (past the last row and column).
template <int ROWS, int COLS, int S, int R0, int R1, int C0, int C1>
__device__ __forceinline__ void zero_border(uint16_t* __restrict__ x) {  // inside: rows R0 .. R1 - 1, columns C0 .. C1 - 1
  constexpr int TOP = R0 * COLS, BOT = (ROWS - R1) * COLS, SIDE = C0 + COLS - C1, N = TOP + BOT + ROWS * SIDE;
#pragma unroll
  for (int k = (int)threadIdx.x; k < N; k += kFuseThreads) {
    int p = k < TOP ? k : R1 * COLS + k - TOP;
    if (k >= TOP + BOT) {
      const int r = (k - TOP - BOT) / SIDE, c = (k - TOP - BOT) % SIDE;
      p = r * COLS + (c < C0 ? c : C1 + c - C0);
    }
#pragma unroll
    for (int c = 0; c < S; c += 2) *reinterpret_cast<uint32_t*>(x + p * S + c) = 0u;
  }
}
template <int L>
__device__ __forceinline__ void zero_input_border(uint16_t* x) {
  zero_border<xrows(L), xcols(L), kXRow[L], 1, kHs[L] + 1, 1, kWs[L] + 1>(x);
}
template <int L>
__device__ __forceinline__ void zero_grad_border(uint16_t* d) {
  zero_border<drows(L), dcols(L), kDRow[L], 0, kHs[L], 0, kWs[L]>(d);
}

// Layer L + 1 of one sample inside a workgroup, as an implicit GEMM: rows n =
// output channels, columns m = output pixels (i, j), k = (ky, kx, ci), stride 2
// and one pixel of zero padding; BF16 operands, FP32 accumulation, then bias and
// ReLU, BF16 out: into the padded input of the layer after (L < 3) or dense.  The
// sample's activations and the layer's weights are in LDS; the waves take the
// (16-channel tile, 16-pixel tile) pairs in turn, a wave always the same channels,
// whose weights it keeps where they fit.  Lane l supplies A[n0 + l%16][k0 +
// 4(l/16) .. +3] and B[k0 + 4(l/16) .. +3][m0 + l%16] and receives D[4(l/16) +
// j][l%16]: four channels of one pixel, stored as one word pair; columns past the
// last repeat pixel 0 and are not stored.
//
// Vector instructions take four cycles each and four waves share a SIMD, so what
// surrounds a product is a layer's time: taps lie at fixed distances (no bounds
// checks or selects, nineteen instructions a step before), and a lane's results
// share one address (eleven instructions a value with pixels as rows).  The reads
// of nine steps are in flight together.
template <int L>
__device__ __forceinline__ void conv_sample(const uint16_t* __restrict__ x, const uint16_t* __restrict__ w,
                                            const float* __restrict__ bias, uint16_t* __restrict__ y) {
  constexpr int CI = kC[L], CO = kC[L + 1], Ho = kHs[L + 1], Wo = kWs[L + 1];
  constexpr int XS = kXRow[L], WS = kWRow[L], K = 9 * CI, NT = CO / 16, M = Ho * Wo, ITEMS = (M + 15) / 16 * NT;
  constexpr int NW = kFuseThreads / 64;
  static_assert(NW % NT == 0, "a wave keeps its channels");
  const int lane = threadIdx.x & 63, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int n = wave % NT * 16 + (lane & 15), no = wave % NT * 16 + 4 * kq;  // of the operand, of the results
  const float4 bn = *reinterpret_cast<const float4*>(bias + no);
  constexpr int STEPS = (K + 15) / 16;
  constexpr bool KEEP = STEPS <= 18;  // the wave's weights in registers
  uint2 u[KEEP ? STEPS : 1];
  int tap2[CI == 2 ? 2 * STEPS : 1];  // two channels: a lane's four k are two taps, a word of both channels each
  if constexpr (CI == 2) {
#pragma unroll
    for (int k = 0; k < STEPS; ++k) {
      uint32_t h[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int tap = 8 * k + 2 * kq + e;
        h[e] = *reinterpret_cast<const uint32_t*>(w + n * WS + (tap < 9 ? 2 * tap : 0));
        h[e] = tap < 9 ? h[e] : 0u;
        tap2[2 * k + e] = tap < 9 ? (tap / 3 * xcols(L) + tap % 3) * XS : 0;
      }
      u[k] = make_uint2(h[0], h[1]);
    }
  } else if constexpr (KEEP) {
#pragma unroll
    for (int k = 0; k < STEPS; ++k) u[k] = *reinterpret_cast<const uint2*>(w + n * WS + 16 * k + 4 * kq);
  }
  for (int it = wave; it < ITEMS; it += NW) {
    const int m = it / NT * 16 + (lane & 15), mi = m < M ? m : 0, i = mi / Wo, j = mi - i * Wo;
    const uint16_t* xp = x + (2 * i * xcols(L) + 2 * j) * XS + (CI == 2 ? 0 : 4 * kq);
    float4_t acc = float4_t{0.f, 0.f, 0.f, 0.f};
    constexpr int G = STEPS < 9 ? STEPS : 9;
    static_assert(STEPS % G == 0, "whole batches");
#pragma unroll
    for (int k0 = 0; k0 < STEPS; k0 += G) {
      uint2 v[G], uk[G];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int k = k0 + g;
        if constexpr (CI == 2) {
          v[g] = make_uint2(*reinterpret_cast<const uint32_t*>(xp + tap2[2 * k]),
                            *reinterpret_cast<const uint32_t*>(xp + tap2[2 * k + 1]));
        } else {
          static_assert(CI == 2 || CI % 16 == 0, "one tap per step");
          const int tap = 16 * k / CI;
          v[g] = *reinterpret_cast<const uint2*>(xp + (tap / 3 * xcols(L) + tap % 3) * XS + 16 * k % CI);
        }
        if constexpr (!KEEP) uk[g] = *reinterpret_cast<const uint2*>(w + n * WS + 16 * k + 4 * kq);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if constexpr (KEEP) uk[g] = u[k0 + g];
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(bf16x4(uk[g]), bf16x4(v[g]), acc, 0, 0, 0);
      }
    }
    int at = mi * CO;
    if constexpr (L < 3) at = ((i + 1) * xcols(L < 3 ? L + 1 : 0) + j + 1) * kXRow[L < 3 ? L + 1 : 0];
    if (m < M)
      *reinterpret_cast<uint2*>(y + at + no) = make_uint2(f2bf_pair(fmaxf(acc[0] + bn.x, 0.0f), fmaxf(acc[1] + bn.y, 0.0f)),
                                                          f2bf_pair(fmaxf(acc[2] + bn.z, 0.0f), fmaxf(acc[3] + bn.w, 0.0f)));
  }
}

// Data gradient of layer L + 1 of one sample inside a workgroup, fused with the
// ReLU mask of its input: dZprev[y][x][c] = (aprev > 0) * sum over taps (ky, kx)
// and channels o of W[o][ky][kx][c] dZ[i][j][o], where 2i + ky - 1 = y and 2j +
// kx - 1 = x.  Stride 2 makes the reaching taps depend only on the parities of
// (y, x): an even row is reached by ky = 1 alone, an odd one by ky = 0 and 2
// (columns likewise), so the pixels of the implicit GEMM are those of one
// parity class and k = (reaching tap, o); columns are pixels as in conv_sample.
// dZ and the weights ([tap][ci][co]) are in LDS; the waves take (class, 16 pixels, 16 channels) in turn, the classes
// of most taps first.  out: dZprev in LDS for the next layer, or null; gout: dense.
template <int L>
__device__ __forceinline__ void conv_bwd_sample(const uint16_t* __restrict__ dz, const uint16_t* __restrict__ wT,
                                                const uint16_t* __restrict__ aprev, uint16_t* __restrict__ out,
                                                uint16_t* __restrict__ gout) {
  constexpr int CI = kC[L], CO = kC[L + 1], H = kHs[L], W = kWs[L];
  constexpr int NT = CI / 16, DS = kDRow[L + 1], WS = kTRow[L], OS = kDRow[L];
  static_assert(CI % 16 == 0 && CO % 16 == 0, "16-channel tiles");
  const int lane = threadIdx.x & 63, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const auto tiles = [](int cls) {
    return (((H - (cls >> 1) + 1) / 2) * ((W - (cls & 1) + 1) / 2) + 15) / 16 * NT;
  };
  const int items = tiles(0) + tiles(1) + tiles(2) + tiles(3);
  for (int it = wave; it < items; it += kFuseThreads / 64) {
    int cls = 3, r0 = it;
    while (r0 >= tiles(cls)) r0 -= tiles(cls--);
    const int py = cls >> 1, px = cls & 1, Hc = (H - py + 1) / 2, Wc = (W - px + 1) / 2, M = Hc * Wc;
    const int m = r0 / NT * 16 + (lane & 15), n = r0 % NT * 16 + (lane & 15), no = r0 % NT * 16 + 4 * q;
    const int r = m < M ? m : 0, i = r / Wc, j = r - i * Wc, y = 2 * i + py, x = 2 * j + px;
    const uint2 mask = *reinterpret_cast<const uint2*>(aprev + (y * W + x) * CI + no);  // at the lane's four results
    float4_t acc = float4_t{0.f, 0.f, 0.f, 0.f};
    // tap (ky, kx) is reached from pixel ((y + 1 - ky) / 2, (x + 1 - kx) / 2), at
    // most a row or column past the last
    constexpr int S = CO / 16;
    const uint16_t* drow = dz + (i * dcols(L + 1) + j) * DS + 4 * q;
    const uint16_t* wcol = wT + n * WS + 4 * q;
    for (int ta = 0; ta < (py ? 2 : 1); ++ta)
      for (int tb = 0; tb < (px ? 2 : 1); ++tb) {
        const int ky = py ? 2 * ta : 1, kx = px ? 2 * tb : 1;
        const uint16_t* d = drow + ((py & (ta == 0)) * dcols(L + 1) + (px & (tb == 0))) * DS;
        const uint16_t* w = wcol + (ky * 3 + kx) * CI * WS;
#pragma unroll
        for (int o = 0; o < S; ++o)
          acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(bf16x4(*reinterpret_cast<const uint2*>(w + 16 * o)),
                                                           bf16x4(*reinterpret_cast<const uint2*>(d + 16 * o)), acc, 0, 0, 0);
      }
    // ReLU outputs are >= 0: kept where any bit but the sign is set
    const auto keep = [](uint32_t v, uint32_t a) {
      return (a & 0x7fffu ? v & 0xffffu : 0u) | (a & 0x7fff0000u ? v & 0xffff0000u : 0u);
    };
    const uint2 v = make_uint2(keep(f2bf_pair(acc[0], acc[1]), mask.x), keep(f2bf_pair(acc[2], acc[3]), mask.y));
    if (m < M) {
      if (out) *reinterpret_cast<uint2*>(out + (y * dcols(L) + x) * OS + no) = v;
      *reinterpret_cast<uint2*>(gout + (size_t)(y * W + x) * CI + no) = v;
    }
  }
}

// A layer's BF16 weights ([co][tap][ci], BYTES a multiple of 16 from a
// 16-byte aligned source) copied into LDS by the workgroup, global memory
// straight into LDS; the caller waits (s_waitcnt 0, then a barrier).
template <int BYTES>
__device__ __forceinline__ void stage_weights(const uint16_t* __restrict__ src, uint16_t* lds) {
  constexpr int NG = BYTES / 16;
  static_assert(BYTES % 16 == 0, "whole granules");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
#pragma unroll
  for (int q = 0; q < NG; q += kFuseThreads) {
    const int q0 = q + 64 * wave;
    if (q0 + lane < NG)
      __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint32_t*>(src) + 4 * (q0 + lane),
                                       (__attribute__((address_space(3))) void*)(lds + 8 * q0), 16, 0, 0);
  }
}

// Where the fused pass reads and writes: the input pairs as per-sample level
// pointers (refs, curs) or planar [B][2][60][94] bytes (pairs); act[l]
// (non-null) receives layer l's activations for the weight gradient (act[0] the
// BF16 input), act[4] always; out the head's outputs, rel (non-null) their
// exponentials.  Training: targets [B][6], and the squared errors, FC gradients
// ([B][fc parameters]) and layers' gradients dz[1..4] out.
struct FusedIO {
  const uint8_t* const* refs;
  const uint8_t* const* curs;
  const uint8_t* pairs;
  uint16_t* act[5];
  float* out;
  double* rel;
  const float* targets;
  float *sqerr, *fcg;
  uint16_t* dz[5];
  int B;
};

// The N BF16 activations of layer L (a padded input) or 4 (dense) from LDS to
// global memory, 16 bytes a thread.
template <int L, int N>
__device__ __forceinline__ void store_act(const uint16_t* __restrict__ src, uint16_t* __restrict__ dst) {
  constexpr int C = kC[L];
  static_assert(N % 8 == 0, "16-byte copies");
#pragma unroll
  for (int e = 8 * (int)threadIdx.x; e < N; e += 8 * kFuseThreads) {
    uint2 v[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = e + 4 * h, p = k / C, y = p / kWs[L], x = p % kWs[L];
      if constexpr (C == 2) {  // two pixels
        const int x2 = (p + 1) % kWs[L], y2 = (p + 1) / kWs[L];
        v[h] = make_uint2(*reinterpret_cast<const uint32_t*>(src + ((y + 1) * xcols(0) + x + 1) * 2),
                          *reinterpret_cast<const uint32_t*>(src + ((y2 + 1) * xcols(0) + x2 + 1) * 2));
      } else if constexpr (L < 4) {
        v[h] = *reinterpret_cast<const uint2*>(src + ((y + 1) * xcols(L < 4 ? L : 0) + x + 1) * kXRow[L < 4 ? L : 0] + k % C);
      } else {
        v[h] = *reinterpret_cast<const uint2*>(src + k);
      }
    }
    *reinterpret_cast<uint4*>(dst + e) = make_uint4(v[0].x, v[0].y, v[1].x, v[1].y);
  }
}

// LDS of the fused pass in bytes.  What a step reads and what is being staged for
// the steps after it are apart; a region is reused once its last reader is done.
//   forward:  A   input, then layer 2's activations, then layer 4's
//             W3  staged from the start; the head's weights once layer 3 is done
//             B   layer 1's activations; from layer 3 on its activations (C3) and W4
//             W2, W1 staged from the start
//   backward: D4, D3 (gradients) and T2 from the start, T3 over C3 and W4;
//             D2 and T1 over T3
struct FuseLds {
  static constexpr int kA = 0, kW3 = xbytes(2) > xbytes(0) ? xbytes(2) : xbytes(0), kB = kW3 + 2 * kC[3] * kWRow[2],
                       kW2 = kB + xbytes(1), kW1 = kW2 + 2 * kC[2] * kWRow[1], kFwdEnd = kW1 + 2 * kC[1] * kWRow[0];
  static constexpr int kC3 = kB, kW4 = kC3 + xbytes(3), kEnd4 = kW4 + 2 * kC[4] * kWRow[3];
  static constexpr int kHead = kW3, kHeadEnd = kHead + 4 * (64 * 65 + kOut * kHidden);
  static constexpr int kD4 = 2 * kHs[4] * kWs[4] * kC[4], kD3 = kD4 + dbytes(4), kT2 = kD3 + dbytes(3),
                       kT3 = kT2 + 2 * 9 * kC[2] * kTRow[2], kEndT3 = kT3 + 2 * 9 * kC[3] * kTRow[3];
  static constexpr int kD2 = kT3, kT1 = kD2 + dbytes(2), kEndT1 = kT1 + 2 * 9 * kC[1] * kTRow[1];
  static constexpr int kFwd = kFwdEnd > kEnd4 ? kFwdEnd : kEnd4, kBwd = kEndT3 > kEndT1 ? kEndT3 : kEndT1;
  static constexpr int kBytes = kFwd > kBwd ? kFwd : kBwd;
};
static_assert(FuseLds::kHeadEnd <= FuseLds::kB && FuseLds::kT2 <= FuseLds::kHead && FuseLds::kT3 >= FuseLds::kHeadEnd &&
                  FuseLds::kBytes <= 160 * 1024 - 3072 && FuseLds::kW3 % 16 == 0 && FuseLds::kB % 16 == 0 &&
                  FuseLds::kW2 % 16 == 0 && FuseLds::kW1 % 16 == 0 && FuseLds::kW4 % 16 == 0 && FuseLds::kD4 % 16 == 0 &&
                  FuseLds::kD3 % 16 == 0 && FuseLds::kT2 % 16 == 0 && FuseLds::kT3 % 16 == 0 && FuseLds::kT1 % 16 == 0,
              "the regions follow the layer shapes");

// Sample blockIdx.x in one workgroup: the input, the four convolutions and the
// head, the activations never leaving LDS (save the copies io asks for); then the
// proposal's exponential or, training, the loss, the head's backward and the
// gradients of the layers' outputs down to layer 1 (mean(a4) = g, h1 = relu(fw1 g
// + fb1), out = fw2 h1 + fb2).  The steps are short and depend on each other, so
// latency bounds them: each layer's weights are on their way while the layer
// before is computed, and 1024 threads share a layer's tiles.  64 pairs with the
// proposal: 27 us with unpadded rows and each layer's weights waited for, now 16.2;
// the training pass of 256 pairs: 97 us as five launches, 51.5 in one, now 35.
template <bool TRAIN>
__global__ __launch_bounds__(kFuseThreads) void conv_net_fused(FusedIO io, const uint16_t* __restrict__ Pb,
                                                               const uint16_t* __restrict__ PbT,
                                                               const float* __restrict__ P) {
  using R = FuseLds;
  __shared__ __align__(16) uint8_t lds[R::kBytes];
  __shared__ __align__(16) float sh_bias[kC[1] + kC[2] + kC[3] + kC[4]];
  __shared__ float sh_g[64], sh_h1[64], sh_out[kOut], sh_dout[kOut], sh_dz1[64];
  __shared__ uint16_t sh_dg[64];
  const auto at = [&](int o) { return reinterpret_cast<uint16_t*>(lds + o); };
  constexpr int N0 = kH0 * kW0 * 2, N1 = kHs[1] * kWs[1] * kC[1], N2 = kHs[2] * kWs[2] * kC[2],
                N3 = kHs[3] * kWs[3] * kC[3], N4 = kHs[4] * kWs[4] * kC[4], HW = kHs[4] * kWs[4];
  const int b = blockIdx.x, t = threadIdx.x;
  const Offsets o = offsets();
  const uint8_t* ref = io.pairs ? io.pairs + (size_t)(2 * b) * kH0 * kW0 : io.refs[b];
  const uint8_t* cur = io.pairs ? io.pairs + (size_t)(2 * b + 1) * kH0 * kW0 : io.curs[b];
  constexpr int PX = (kH0 * kW0 + kFuseThreads - 1) / kFuseThreads;
  uint8_t pr[PX], pc[PX];
#pragma unroll
  for (int k = 0; k < PX; ++k) {
    const int r = min(t + k * kFuseThreads, kH0 * kW0 - 1);
    pr[k] = gload(ref + r), pc[k] = gload(cur + r);
  }
  // the biases too: a read of global memory inside a layer would wait for the
  // weights being staged
  constexpr int B1 = kC[1], B2 = B1 + kC[2], B3 = B2 + kC[3], B4 = B3 + kC[4];
  const float bias = t < B4 ? gload(P + (t < B1 ? o.b[0] + t : t < B2 ? o.b[1] + t - B1 : t < B3 ? o.b[2] + t - B2
                                                                                              : o.b[3] + t - B3))
                            : 0.f;
  stage_weights<kC[1] * kWRow[0] * 2>(Pb + wrow_off(0), at(R::kW1));
  stage_weights<kC[2] * kWRow[1] * 2>(Pb + wrow_off(1), at(R::kW2));
  stage_weights<kC[3] * kWRow[2] * 2>(Pb + wrow_off(2), at(R::kW3));
#pragma unroll
  for (int k = 0; k < PX; ++k) {  // (I - 128) / 64, exact in BF16
    const int r = t + k * kFuseThreads;
    if (r < kH0 * kW0)
      *reinterpret_cast<uint32_t*>(at(R::kA) + 2 * ((r / kW0 + 1) * xcols(0) + r % kW0 + 1)) =
          f2bf_pair(((float)pr[k] - 128.0f) * (1.0f / 64.0f), ((float)pc[k] - 128.0f) * (1.0f / 64.0f));
  }
  zero_input_border<0>(at(R::kA));
  zero_input_border<1>(at(R::kB));
  if (t < B4) sh_bias[t] = bias;
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (io.act[0]) store_act<0, N0>(at(R::kA), io.act[0] + (size_t)b * N0);
  conv_sample<0>(at(R::kA), at(R::kW1), sh_bias, at(R::kB));
  __syncthreads();
  if (io.act[1]) store_act<1, N1>(at(R::kB), io.act[1] + (size_t)b * N1);
  zero_input_border<2>(at(R::kA));
  conv_sample<1>(at(R::kB), at(R::kW2), sh_bias + B1, at(R::kA));
  __syncthreads();
  stage_weights<kC[4] * kWRow[3] * 2>(Pb + wrow_off(3), at(R::kW4));
  if (io.act[2]) store_act<2, N2>(at(R::kA), io.act[2] + (size_t)b * N2);
  zero_input_border<3>(at(R::kC3));
  conv_sample<2>(at(R::kA), at(R::kW3), sh_bias + B2, at(R::kC3));
  // the head's weights, to LDS once W3 is done with: fw1 transposed in rows of 65,
  // so that both fw1 g and fw1^T dz1 read it without conflicts
  static_assert(kFuseThreads * 4 == kHidden * 64, "four elements of fw1 per thread");
  const float4 f1 = gload(reinterpret_cast<const float4*>(P + o.fw1) + t);
  const float f2 = t < kOut * kHidden ? P[o.fw2 + t] : 0.f, fb1 = t < kHidden ? P[o.fb1 + t] : 0.f,
              fb2 = t < kOut ? P[o.fb2 + t] : 0.f;
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (io.act[3]) store_act<3, N3>(at(R::kC3), io.act[3] + (size_t)b * N3);
  float* fw1 = reinterpret_cast<float*>(lds + R::kHead);  // [q][t]
  float* fw2 = fw1 + 64 * 65;
  {
    float* d = fw1 + 4 * (t & 15) * 65 + (t >> 4);
    d[0] = f1.x, d[65] = f1.y, d[130] = f1.z, d[195] = f1.w;
    if (t < kOut * kHidden) fw2[t] = f2;
  }
  uint16_t* a4 = at(R::kA);
  conv_sample<3>(at(R::kC3), at(R::kW4), sh_bias + B3, a4);
  __syncthreads();
  if constexpr (TRAIN) stage_weights<9 * kC[3] * kTRow[3] * 2>(PbT + trow_off(3), at(R::kT3));
  store_act<4, N4>(a4, io.act[4] + (size_t)b * N4);
  if (t < 64) {
    float v = 0.f;
#pragma unroll
    for (int p = 0; p < HW; ++p) v += bf2f(a4[p * 64 + t]);
    sh_g[t] = v * (1.0f / HW);
  }
  __syncthreads();
  if (t < 64) {
    float z = fb1;
#pragma unroll 16
    for (int q = 0; q < 64; ++q) z = fmaf(fw1[q * 65 + t], sh_g[q], z);
    sh_h1[t] = fmaxf(z, 0.f);
  }
  __syncthreads();
  if (t < kOut) {
    float v = fb2;
#pragma unroll 16
    for (int q = 0; q < kHidden; ++q) v = fmaf(fw2[t * kHidden + q], sh_h1[q], v);
    io.out[b * kOut + t] = v;
    sh_out[t] = v;
    if constexpr (TRAIN) {
      const float d = v - io.targets[b * kOut + t];
      sh_dout[t] = 2.0f * d / (float)(io.B * kOut);
      io.sqerr[b * kOut + t] = d * d;
    }
  }
  __syncthreads();
  if constexpr (!TRAIN) {
    if (io.rel && t == 0) propose_twist(sh_out, io.rel + 12 * b);
    return;
  }
  // FC gradients of this sample (fixed layout: fw1, fb1, fw2, fb2 relative to o.fw1)
  float* G = io.fcg + (size_t)b * (o.total - o.fw1);
  if (t < kOut * kHidden) G[o.fw2 - o.fw1 + t] = sh_dout[t / kHidden] * sh_h1[t % kHidden];
  if (t < kOut) G[o.fb2 - o.fw1 + t] = sh_dout[t];
  if (t < 64) {
    float dh = 0.f;
#pragma unroll
    for (int q = 0; q < kOut; ++q) dh = fmaf(fw2[q * kHidden + t], sh_dout[q], dh);
    const float dz1 = sh_h1[t] > 0.f ? dh : 0.f;
    sh_dz1[t] = dz1;
    G[o.fb1 - o.fw1 + t] = dz1;
  }
  __syncthreads();
  for (int e = t; e < kHidden * 64; e += kFuseThreads) G[e] = sh_dz1[e >> 6] * sh_g[e & 63];
  if (t < 64) {
    float dg = 0.f;
#pragma unroll 16
    for (int q = 0; q < kHidden; ++q) dg = fmaf(fw1[t * 65 + q], sh_dz1[q], dg);
    sh_dg[t] = f2bf(dg * (1.0f / HW));
  }
  __syncthreads();
  uint16_t* d4 = at(R::kD4);
  zero_grad_border<4>(d4);
  zero_grad_border<3>(at(R::kD3));
  for (int e = t; e < N4; e += kFuseThreads) {
    const uint16_t v = bf2f(a4[e]) > 0.f ? sh_dg[e & 63] : (uint16_t)0;
    d4[((e >> 6) / kWs[4] * dcols(4) + (e >> 6) % kWs[4]) * kDRow[4] + (e & 63)] = v;
    io.dz[4][(size_t)b * N4 + e] = v;
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  stage_weights<9 * kC[2] * kTRow[2] * 2>(PbT + trow_off(2), at(R::kT2));
  conv_bwd_sample<3>(d4, at(R::kT3), io.act[3] + (size_t)b * N3, at(R::kD3), io.dz[3] + (size_t)b * N3);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  stage_weights<9 * kC[1] * kTRow[1] * 2>(PbT + trow_off(1), at(R::kT1));
  zero_grad_border<2>(at(R::kD2));
  conv_bwd_sample<2>(at(R::kD3), at(R::kT2), io.act[2] + (size_t)b * N2, at(R::kD2), io.dz[2] + (size_t)b * N2);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  conv_bwd_sample<1>(at(R::kD2), at(R::kT1), io.act[1] + (size_t)b * N1, nullptr, io.dz[1] + (size_t)b * N1);
}

// The fused pass over B samples on stream s.
hipError_t launch_fused(const FusedIO& io, int B, const uint16_t* Pb, const uint16_t* PbT, const float* P,
                        hipStream_t s) {
  if (io.targets)
    hipLaunchKernelGGL(conv_net_fused<true>, dim3(B), dim3(kFuseThreads), 0, s, io, Pb, PbT, P);
  else
    hipLaunchKernelGGL(conv_net_fused<false>, dim3(B), dim3(kFuseThreads), 0, s, io, Pb, PbT, P);
  return hipGetLastError();
}

// ---------------------------------------------------------------- weight gradient

// Weight and bias gradient of layer L + 1 over the samples b0 .. b1 - 1, in one
// workgroup of sixteen waves: dW[o][n] = sum over pixels p of dZ[p][o] Xcol[p][n],
// where Xcol[p][tap * CI + c] = X[2i + ky - 1][2j + kx - 1][c] (zero outside the
// image) and column n = 9 CI is all ones (the bias); columns up to the next
// multiple of 16 are zero.  v_mfma_f32_16x16x32_bf16 over four groups of eight
// pixels of a row.
//
// A lane's operand is eight pixels of one channel, so a sample is transposed into
// LDS: dZ as [o][i][j] and X by the parities of its pixels, [c][row][kx][j], where
// row i of the first Ho is y = 2i (ky = 1), row i of the rest y = 2i - 1 (ky = 0;
// ky = 2 one on), and column j of variant kx is x = 2j + kx - 1: each tap of eight
// output pixels is eight consecutive elements, whatever the stride.  Rows are
// padded to groups of eight, channels so that sixteen lanes' 16-byte reads fall on
// different banks.  The products are few (a 16x16 tile takes 1 to 45 steps a
// sample): the transposition and its latency bound it, so the next sample is read
// while one is multiplied and each element is read once per layer, where a wave
// per output tile that gathers from global memory reads it 37 to 148 times.
template <int L>
struct Wgrad {
  static constexpr int CI = kC[L], CO = kC[L + 1], H = kHs[L], W = kWs[L], Ho = kHs[L + 1], Wo = kWs[L + 1];
  static constexpr int Wp = (Wo + 7) / 8 * 8, GR = Wp / 8, NG = Ho * GR, STEPS = (NG + 3) / 4;
  static constexpr int MT = CO / 16, NT = (9 * CI + 1 + 15) / 16, NPAD = 16 * NT;
  // waves: MT x NGRP groups of NTW column tiles x KG shares of the steps
  static constexpr int NTW = L == 3 ? 10 : L == 0 ? 2 : 5, NGRP = (NT + NTW - 1) / NTW, KG = 16 / (MT * NGRP);
  static_assert(MT * NGRP * KG == 16, "sixteen waves");
  static constexpr int XROW = 3 * Wp, XP = (2 * Ho + 1) * XROW + (L == 2 ? 8 : 0), DP = STEPS * 32 + 8;
  static constexpr int XN = CI * XP, DN = CO * DP, BYTES = 2 * (XN + DN);
  static_assert(XP % 8 == 0 && BYTES >= (KG > 1 ? KG * MT * NT * 1024 : 0), "16-byte rows; room for the shares' sums");
  // what a thread moves of a sample: pixels of eight channels (X of layer 1: of two)
  static constexpr int XG = CI == 2 ? 1 : CI / 8, DG = CO / 8;
  static constexpr int XI = (H * W * XG + kFuseThreads - 1) / kFuseThreads, DI = (Ho * Wo * DG + kFuseThreads - 1) / kFuseThreads;
};

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

template <int L>
__device__ __forceinline__ void wgrad_layer(const uint16_t* __restrict__ x, const uint16_t* __restrict__ dz, int b0,
                                            int b1, uint16_t* lds, float* __restrict__ out) {
  using C = Wgrad<L>;
  using XV = typename std::conditional<C::CI == 2, uint32_t, uint4>::type;
  constexpr int XC = C::CI == 2 ? 2 : 8;  // channels of an X item
  const int t = threadIdx.x, lane = t & 63, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  uint16_t* xt = lds;
  uint16_t* dt = lds + C::XN;
  XV xr[C::XI];
  uint4 dr[C::DI];
  const auto load = [&](int b) {
    const uint16_t* xs = x + (size_t)b * C::H * C::W * C::CI;
    const uint16_t* ds = dz + (size_t)b * C::Ho * C::Wo * C::CO;
#pragma unroll
    for (int k = 0; k < C::XI; ++k) {  // consecutive threads: consecutive pixels of a channel group
      const int e = min(t + k * kFuseThreads, C::H * C::W * C::XG - 1), px = e % (C::H * C::W), g = e / (C::H * C::W);
      xr[k] = gload(reinterpret_cast<const XV*>(xs + px * C::CI + XC * g));
    }
#pragma unroll
    for (int k = 0; k < C::DI; ++k) {
      const int e = min(t + k * kFuseThreads, C::Ho * C::Wo * C::DG - 1), px = e % (C::Ho * C::Wo), g = e / (C::Ho * C::Wo);
      dr[k] = gload(reinterpret_cast<const uint4*>(ds + px * C::CO + 8 * g));
    }
  };
  load(b0);
  for (int e = t; e < C::BYTES / 16; e += kFuseThreads) reinterpret_cast<uint4*>(lds)[e] = make_uint4(0u, 0u, 0u, 0u);
  // this wave's tiles: row tile mt, column tiles nt0 .. nt0 + NTW - 1, steps kg, kg + KG, ...
  const int mt = wave % C::MT, nt0 = wave / C::MT % C::NGRP * C::NTW, kg = wave / (C::MT * C::NGRP);
  int col[C::NTW];  // where column n's taps start in xt
  bool real[C::NTW], ones[C::NTW];
#pragma unroll
  for (int k = 0; k < C::NTW; ++k) {
    const int n = (nt0 + k) * 16 + (lane & 15);
    real[k] = n < 9 * C::CI, ones[k] = n == 9 * C::CI;
    const int tap = real[k] ? n / C::CI : 0, c = real[k] ? n % C::CI : 0, ky = tap / 3, kx = tap % 3;
    col[k] = c * C::XP + ((ky == 1 ? 0 : C::Ho) + (ky == 2)) * C::XROW + kx * C::Wp;
  }
  float4_t acc[C::NTW];
#pragma unroll
  for (int k = 0; k < C::NTW; ++k) acc[k] = float4_t{0.f, 0.f, 0.f, 0.f};
  for (int b = b0; b < b1; ++b) {
    __syncthreads();  // the previous sample's products (first: the zeros) are done
#pragma unroll
    for (int k = 0; k < C::XI; ++k) {
      const int e = t + k * kFuseThreads, px = e % (C::H * C::W), g = e / (C::H * C::W);
      if (e >= C::H * C::W * C::XG) continue;
      const int y = px / C::W, xx = px % C::W;
      uint16_t* r = xt + XC * g * C::XP + ((y & 1) ? C::Ho + (y + 1) / 2 : y / 2) * C::XROW;
      const uint32_t* v = reinterpret_cast<const uint32_t*>(&xr[k]);
      if (xx & 1) {
        uint16_t *r2 = r + 2 * C::Wp + (xx - 1) / 2, *r0 = r + (xx + 1) / 2;
#pragma unroll
        for (int c = 0; c < XC; ++c) {
          const uint16_t h = (uint16_t)(v[c / 2] >> (16 * (c & 1)));
          r2[c * C::XP] = h, r0[c * C::XP] = h;
        }
      } else {
        uint16_t* r1 = r + C::Wp + xx / 2;
#pragma unroll
        for (int c = 0; c < XC; ++c) r1[c * C::XP] = (uint16_t)(v[c / 2] >> (16 * (c & 1)));
      }
    }
#pragma unroll
    for (int k = 0; k < C::DI; ++k) {
      const int e = t + k * kFuseThreads, px = e % (C::Ho * C::Wo), g = e / (C::Ho * C::Wo);
      if (e >= C::Ho * C::Wo * C::DG) continue;
      uint16_t* r = dt + 8 * g * C::DP + px / C::Wo * C::Wp + px % C::Wo;
      const uint32_t* v = reinterpret_cast<const uint32_t*>(&dr[k]);
#pragma unroll
      for (int c = 0; c < 8; ++c) r[c * C::DP] = (uint16_t)(v[c / 2] >> (16 * (c & 1)));
    }
    if (b + 1 < b1) load(b + 1);
    __syncthreads();
    for (int s = kg; s < C::STEPS; s += C::KG) {
      const int grp = 4 * s + q, gx = grp < C::NG ? grp : 0;  // past the last group: zeros in dt
      const int xo = gx / C::GR * C::XROW + gx % C::GR * 8;
      const bf16x8_t av = *reinterpret_cast<const bf16x8_t*>(dt + (mt * 16 + (lane & 15)) * C::DP + 8 * grp);
#pragma unroll
      for (int k = 0; k < C::NTW; ++k) {
        uint4 u = *reinterpret_cast<const uint4*>(xt + col[k] + xo);
        const uint32_t fill = ones[k] ? 0x3f803f80u : 0u;  // 1.0 twice
        u = make_uint4(real[k] ? u.x : fill, real[k] ? u.y : fill, real[k] ? u.z : fill, real[k] ? u.w : fill);
        acc[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8_t, u), acc[k], 0, 0, 0);
      }
    }
  }
  if constexpr (C::KG > 1) {  // the shares of the steps, summed in pairs
    float* sh = reinterpret_cast<float*>(lds);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < C::NTW; ++k)
      *reinterpret_cast<float4_t*>(sh + (((kg * C::MT + mt) * C::NT + nt0 + k) * 64 + lane) * 4) = acc[k];
    __syncthreads();
    for (int e = t; e < C::MT * C::NT * 256; e += kFuseThreads) {
      float v[C::KG];
#pragma unroll
      for (int g = 0; g < C::KG; ++g) v[g] = sh[g * C::MT * C::NT * 256 + e];
#pragma unroll
      for (int w = C::KG / 2; w > 0; w >>= 1)
#pragma unroll
        for (int g = 0; g < w; ++g) v[g] += v[g + w];
      const int tile = e >> 8, l = e >> 2 & 63;
      out[(tile / C::NT * 16 + 4 * (l >> 4) + (e & 3)) * C::NPAD + tile % C::NT * 16 + (l & 15)] = v[0];
    }
  } else {
#pragma unroll
    for (int k = 0; k < C::NTW; ++k)
      if (nt0 + k < C::NT)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          out[(mt * 16 + 4 * q + j) * C::NPAD + (nt0 + k) * 16 + (lane & 15)] = acc[k][j];
  }
}

// Samples per workgroup of layer l for B samples, in 1/256 of B: the workgroups of
// all layers together are at most 246, one turn of the chip.  Above 512 samples a
// workgroup's stay at what they are there (6 to 16) and the workgroups take turns:
// the products of a workgroup's samples meet in one accumulator, whose rounding
// grows with their number.  One turn at any size lost 1.3e-6 of a gradient at 4096
// equal samples, so 1.5e-7, for 4 % of the step's time (4096 samples 819 to 869 us,
// and 919 with turns from 256 samples on).
constexpr int kWgradShare[4] = {4, 3, 4, 8}, kWgradMost = 2;
constexpr int wgrad_samples(int l, int B) {
  return B <= 256 * kWgradMost ? (int)(((int64_t)B * kWgradShare[l] + 255) / 256) : kWgradMost * kWgradShare[l];
}
constexpr int wgrad_slots(int l, int B) { return (B + wgrad_samples(l, B) - 1) / wgrad_samples(l, B); }
constexpr int npad(int l) { return (9 * kC[l] + 1 + 15) / 16 * 16; }

struct WgradIO {
  const uint16_t* act[4];  // layer inputs
  const uint16_t* dz[4];   // layer output gradients
  float* partial[4];       // [slot][CO][NPAD]
  int B;
};

// The weight gradients of all layers' slots, a workgroup each.  256 pairs: four
// launches of 99 us together with a wave per output tile, now 18.
__global__ __launch_bounds__(kFuseThreads) void conv_bwd_weight(WgradIO io) {
  __shared__ __align__(16) uint16_t lds[Wgrad<1>::BYTES / 2];
  static_assert(Wgrad<0>::BYTES <= Wgrad<1>::BYTES && Wgrad<2>::BYTES <= Wgrad<1>::BYTES &&
                    Wgrad<3>::BYTES <= Wgrad<1>::BYTES && Wgrad<1>::BYTES <= 160 * 1024,
                "the largest layer's LDS");
  int slot = blockIdx.x;
  const auto run = [&](auto layer) {
    constexpr int L = decltype(layer)::value;
    const int n = wgrad_slots(L, io.B), S = wgrad_samples(L, io.B);
    if (slot >= 0 && slot < n)
      wgrad_layer<L>(io.act[L], io.dz[L], slot * S, min(io.B, (slot + 1) * S), lds,
                     io.partial[L] + (size_t)slot * kC[L + 1] * Wgrad<L>::NPAD);
    slot -= n;
  };
  run(std::integral_constant<int, 1>{});
  run(std::integral_constant<int, 0>{});
  run(std::integral_constant<int, 2>{});
  run(std::integral_constant<int, 3>{});
}

// ---------------------------------------------------------------- sums over slots, Adam

// The BF16 copies of convolution weight e ([co][ky][kx][ci] in P).
__device__ __forceinline__ void store_bf16_param(int e, float p, uint16_t* __restrict__ Pb,
                                                 uint16_t* __restrict__ PbT) {
  const uint16_t h = f2bf(p);
  const Offsets o = offsets();
#pragma unroll
  for (int l = 0; l < 4; ++l) {
    const int CI = kC[l], CO = kC[l + 1], r = e - o.w[l];
    if (r >= 0 && r < CO * 9 * CI) {
      const int co = r / (9 * CI), k = r % (9 * CI);
      Pb[wrow_off(l) + co * kWRow[l] + k] = h;
      if (l > 0) PbT[trow_off(l) + k * kTRow[l] + co] = h;
    }
  }
}

// Where the gradient's sums come from and what they update.
struct UpdateIO {
  const float* partial[4];  // weight gradients per slot
  int slots[4];
  const float *fcg, *sqerr;  // per sample: FC gradients, squared errors
  int B;
  float *G, *loss;  // the gradient; the squared errors' sums (pinned host memory)
  float *P, *M, *V;
  uint16_t *Pb, *PbT;
  float lr, c1, c2;  // lr = 0: the gradient only
};

// Every element of the gradient (weights at [co][ky][kx][ci]) and the six squared
// errors: the sum of its slots or samples in a fixed order, sixteen threads to an
// element (each sums every sixteenth, then a pairwise tree), and Adam
// (Kingma & Ba 2015) on the FP32 master weights, beta 0.9 / 0.999, eps 1e-8, with
// bias correction c1 = 1 - b1^t, c2 = 1 - b2^t, refreshing the BF16 weights.  A
// thread's sum (4096 samples at the largest batch) is of pairwise sums of eight,
// eight of those in a chain, and so many such: in a single chain it rounded off 8e-6
// of a gradient at 16,384 equal samples, now 2e-7.  One
// launch for all of them: each of seven took its launch and little more (50 us
// for 256 pairs), now 8.8.
__global__ __launch_bounds__(256) void update_kernel(UpdateIO io) {
  constexpr int PARTS = 16, EPB = 256 / PARTS;
  __shared__ float sh[256];
  const Offsets o = offsets();
  const int el = (int)threadIdx.x % EPB, part = (int)threadIdx.x / EPB;
  const int e = (int)blockIdx.x * EPB + el;
  const float* v = io.sqerr + (e - o.total);
  int stride = kOut, K = e < o.total + kOut ? io.B : 0;
  if (e < o.fw1) {
#pragma unroll
    for (int l = 0; l < 4; ++l) {
      const int CI = kC[l], CO = kC[l + 1], r = e - o.w[l], rb = e - o.b[l];
      if (r < 0 || rb >= CO) continue;
      const int co = rb < 0 ? r / (9 * CI) : rb, n = rb < 0 ? r % (9 * CI) : 9 * CI;
      v = io.partial[l] + co * npad(l) + n, stride = CO * npad(l), K = io.slots[l];
    }
  } else if (e < o.total) {
    v = io.fcg + (e - o.fw1), stride = o.total - o.fw1;
  }
  float s = 0.f;
  for (int k0 = part; k0 < K;) {
    float chain = 0.f;
    for (int q = 0; q < 8 && k0 < K; ++q, k0 += 8 * PARTS) {
      float x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int k = k0 + j * PARTS;
        x[j] = 0.f;
        if (k < K) x[j] = gload(v + (size_t)k * stride);
      }
      chain += ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
    }
    s += chain;
  }
  sh[threadIdx.x] = s;
  __syncthreads();
#pragma unroll
  for (int w = PARTS / 2; w > 0; w >>= 1) {
    if (part < w) sh[threadIdx.x] += sh[threadIdx.x + w * EPB];
    __syncthreads();
  }
  if (part != 0 || e >= o.total + kOut) return;
  const float g = sh[el];
  if (e >= o.total) {
    io.loss[e - o.total] = g;
    return;
  }
  io.G[e] = g;
  if (!(io.lr > 0.f)) return;
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float m = b1 * io.M[e] + (1.0f - b1) * g;
  const float w = b2 * io.V[e] + (1.0f - b2) * g * g;
  io.M[e] = m;
  io.V[e] = w;
  const float p = io.P[e] - io.lr * (m / io.c1) / (sqrtf(w / io.c2) + eps);
  io.P[e] = p;
  if (e < o.fw1) store_bf16_param(e, p, io.Pb, io.PbT);
}

__global__ void to_bf16(const float* __restrict__ P, int n, uint16_t* __restrict__ Pb, uint16_t* __restrict__ PbT) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n) store_bf16_param(e, P[e], Pb, PbT);
}

__global__ void bf16_to_f32(const uint16_t* __restrict__ a, size_t n, float* __restrict__ out) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n) out[e] = bf2f(a[e]);
}

}  // namespace cnn
}  // namespace dpt

// ---------------------------------------------------------------- host

using namespace dpt;
using namespace dpt::cnn;

struct dpt_cnn {
  int32_t max_batch = 0;
  hipStream_t stream = nullptr;
  Offsets o;
  float *P = nullptr, *G = nullptr, *M = nullptr, *V = nullptr;  // FP32 master, gradient, Adam moments
  uint16_t* Pb = nullptr;                                          // BF16 conv weights, kWRow layout
  uint16_t* PbT = nullptr;                                         // BF16 conv weights as [tap][ci][co], kTRow layout
  uint16_t* act[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};
  // dz[l]: gradient at layer l's output (pre-ReLU), BF16 NHWC; sized for FP32
  // so that the activation test hook can stage an FP32 copy there
  uint16_t* dz[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};
  float *out = nullptr, *tgt = nullptr, *sqerr = nullptr, *fcg = nullptr, *partial = nullptr;
  uint8_t* pairs = nullptr;
  const uint8_t** d_lv = nullptr;  // [2][max_batch] level pointers
  int step = 0;
  float* h_buf = nullptr;  // pinned
  float* h_buf_dev = nullptr;  // its address on the device
  ~dpt_cnn() {
    for (void* p : {(void*)P, (void*)G, (void*)M, (void*)V, (void*)Pb, (void*)PbT, (void*)out, (void*)tgt, (void*)sqerr,
                    (void*)fcg, (void*)partial, (void*)pairs, (void*)d_lv})
      if (p) (void)hipFree(p);
    for (int l = 0; l < 5; ++l) {
      if (act[l]) (void)hipFree(act[l]);
      if (dz[l]) (void)hipFree(dz[l]);
    }
    if (h_buf) (void)hipHostFree(h_buf);
  }
};

namespace {

int cfail(int code, const char* msg) { return set_error(code, msg); }

#define CNN_TRY(expr)                                          \
  do {                                                         \
    hipError_t e_ = (expr);                                    \
    if (e_ != hipSuccess) return cfail(DPT_E_HIP, #expr);      \
  } while (0)

// Room for the weight gradients' slots at any B up to max_batch: at most 256 / share
// a layer up to 512 samples, and above as many as at max_batch.
size_t max_partial(int max_batch) {
  size_t n = 0;
  for (int l = 0; l < 4; ++l) {
    const size_t few = (256 + kWgradShare[l] - 1) / kWgradShare[l], all = wgrad_slots(l, max_batch);
    n += std::max(few, all) * kC[l + 1] * npad(l);
  }
  return n;
}

// Weight gradients, their sums with the FC gradients' and the loss's, and (lr > 0) Adam.
hipError_t update(dpt_cnn* c, int B, float lr, float c1, float c2) {
  WgradIO w{};
  UpdateIO u{};
  int blocks = 0;
  float* partial = c->partial;  // one layer's slots after the other
  for (int l = 0; l < 4; ++l) {
    w.act[l] = c->act[l], w.dz[l] = c->dz[l + 1];
    u.partial[l] = w.partial[l] = partial, u.slots[l] = wgrad_slots(l, B);
    partial += (size_t)u.slots[l] * kC[l + 1] * npad(l);
    blocks += u.slots[l];
  }
  w.B = B;
  hipLaunchKernelGGL(conv_bwd_weight, dim3(blocks), dim3(kFuseThreads), 0, c->stream, w);
  u.fcg = c->fcg, u.sqerr = c->sqerr, u.B = B, u.G = c->G, u.loss = c->h_buf_dev;
  u.P = c->P, u.M = c->M, u.V = c->V, u.Pb = c->Pb, u.PbT = c->PbT;
  u.lr = lr, u.c1 = c1, u.c2 = c2;
  hipLaunchKernelGGL(update_kernel, dim3((c->o.total + kOut + 15) / 16), dim3(256), 0, c->stream, u);
  return hipGetLastError();
}

// The fused pass over B planar pairs (host or device), every layer's activations
// kept and the head's outputs in c->out; with targets (device), the backward pass
// down to the layers' gradients too.
int forward_pairs(dpt_cnn* c, const uint8_t* pairs, int B, int on_device, const float* targets) {
  const uint8_t* src = pairs;
  if (!on_device) {
    CNN_TRY(hipMemcpyAsync(c->pairs, pairs, (size_t)B * 2 * kH0 * kW0, hipMemcpyHostToDevice, c->stream));
    src = c->pairs;
  }
  FusedIO io{};
  io.pairs = src;
  for (int l = 0; l < 5; ++l) io.act[l] = c->act[l];
  io.out = c->out;
  io.targets = targets;
  io.sqerr = c->sqerr, io.fcg = c->fcg, io.B = B;
  for (int l = 0; l < 5; ++l) io.dz[l] = c->dz[l];
  CNN_TRY(launch_fused(io, B, c->Pb, c->PbT, c->P, c->stream));
  return DPT_OK;
}

}  // namespace

extern "C" {

int dpt_cnn_create(int32_t max_batch, void* hip_stream, dpt_cnn** out) {
  if (!out) return cfail(DPT_E_ARG, "out is NULL");
  *out = nullptr;
  if (max_batch < 1 || max_batch > 65536) return cfail(DPT_E_ARG, "max_batch outside [1, 65536]");
  dpt_cnn* c = new (std::nothrow) dpt_cnn();
  if (!c) return cfail(DPT_E_OOM, "host allocation failed");
  c->max_batch = max_batch;
  c->stream = (hipStream_t)hip_stream;
  c->o = offsets();
  const size_t n = (size_t)c->o.total, B = (size_t)max_batch;
  bool ok = hipMalloc(&c->P, n * 4) == hipSuccess && hipMalloc(&c->G, n * 4) == hipSuccess &&
            hipMalloc(&c->M, n * 4) == hipSuccess && hipMalloc(&c->V, n * 4) == hipSuccess &&
            hipMalloc(&c->Pb, kPbTotal * 2) == hipSuccess && hipMalloc(&c->PbT, kPbTTotal * 2) == hipSuccess;
  for (int l = 0; l < 5 && ok; ++l) {
    const size_t e = B * kHs[l] * kWs[l] * kC[l];
    ok = hipMalloc(&c->act[l], e * 2) == hipSuccess && hipMalloc(&c->dz[l], e * 4) == hipSuccess;
  }
  ok = ok && hipMalloc(&c->out, B * kOut * 4) == hipSuccess && hipMalloc(&c->tgt, B * kOut * 4) == hipSuccess &&
       hipMalloc(&c->sqerr, B * kOut * 4) == hipSuccess &&
       hipMalloc(&c->fcg, B * (size_t)(c->o.total - c->o.fw1) * 4) == hipSuccess &&
       hipMalloc(&c->partial, max_partial(max_batch) * 4) == hipSuccess &&
       hipMalloc(&c->pairs, B * 2 * kH0 * kW0) == hipSuccess && hipMalloc(&c->d_lv, 2 * B * sizeof(void*)) == hipSuccess &&
       hipHostMalloc(&c->h_buf, std::max(n, B * kOut) * 4 + 64) == hipSuccess &&
       hipHostGetDevicePointer((void**)&c->h_buf_dev, c->h_buf, 0) == hipSuccess;
  if (!ok) {
    (void)hipGetLastError();
    delete c;
    return cfail(DPT_E_OOM, "device allocation failed");
  }
  (void)hipMemsetAsync(c->M, 0, n * 4, c->stream);
  (void)hipMemsetAsync(c->V, 0, n * 4, c->stream);
  (void)hipMemsetAsync(c->P, 0, n * 4, c->stream);
  (void)hipMemsetAsync(c->Pb, 0, kPbTotal * 2, c->stream);
  (void)hipMemsetAsync(c->PbT, 0, kPbTTotal * 2, c->stream);
  if (hipStreamSynchronize(c->stream) != hipSuccess) {
    delete c;
    return cfail(DPT_E_HIP, "stream synchronize");
  }
  *out = c;
  return DPT_OK;
}

void dpt_cnn_destroy(dpt_cnn* c) {
  if (!c) return;
  (void)hipStreamSynchronize(c->stream);
  delete c;
}

int32_t dpt_cnn_num_params(void) { return offsets().total; }

// params: host FP32, tensor order w1 b1 .. fb2, conv weights [co][ci][ky][kx]
int dpt_cnn_set_params(dpt_cnn* c, const float* params) {
  if (!c || !params) return cfail(DPT_E_ARG, "NULL argument");
  const Offsets& o = c->o;
  float* h = c->h_buf;
  std::memcpy(h, params, sizeof(float) * o.total);
  for (int l = 0; l < 4; ++l) {  // [co][ci][ky][kx] -> [co][ky][kx][ci]
    const int CI = kC[l], CO = kC[l + 1];
    for (int co = 0; co < CO; ++co)
      for (int ci = 0; ci < CI; ++ci)
        for (int t = 0; t < 9; ++t) h[o.w[l] + (co * 9 + t) * CI + ci] = params[o.w[l] + (co * CI + ci) * 9 + t];
  }
  CNN_TRY(hipMemcpyAsync(c->P, h, sizeof(float) * o.total, hipMemcpyHostToDevice, c->stream));
  hipLaunchKernelGGL(to_bf16, dim3((o.total + 255) / 256), dim3(256), 0, c->stream, c->P, o.total, c->Pb, c->PbT);
  CNN_TRY(hipGetLastError());
  CNN_TRY(hipMemsetAsync(c->M, 0, sizeof(float) * o.total, c->stream));
  CNN_TRY(hipMemsetAsync(c->V, 0, sizeof(float) * o.total, c->stream));
  CNN_TRY(hipStreamSynchronize(c->stream));
  c->step = 0;
  return DPT_OK;
}

static void to_abi_layout(const Offsets& o, const float* in, float* out) {
  std::memcpy(out, in, sizeof(float) * o.total);
  for (int l = 0; l < 4; ++l) {
    const int CI = kC[l], CO = kC[l + 1];
    for (int co = 0; co < CO; ++co)
      for (int ci = 0; ci < CI; ++ci)
        for (int t = 0; t < 9; ++t) out[o.w[l] + (co * CI + ci) * 9 + t] = in[o.w[l] + (co * 9 + t) * CI + ci];
  }
}

int dpt_cnn_get_params(dpt_cnn* c, float* params) {
  if (!c || !params) return cfail(DPT_E_ARG, "NULL argument");
  CNN_TRY(hipMemcpyAsync(c->h_buf, c->P, sizeof(float) * c->o.total, hipMemcpyDeviceToHost, c->stream));
  CNN_TRY(hipStreamSynchronize(c->stream));
  to_abi_layout(c->o, c->h_buf, params);
  return DPT_OK;
}

int dpt_cnn_get_grads(dpt_cnn* c, float* grads) {
  if (!c || !grads) return cfail(DPT_E_ARG, "NULL argument");
  CNN_TRY(hipMemcpyAsync(c->h_buf, c->G, sizeof(float) * c->o.total, hipMemcpyDeviceToHost, c->stream));
  CNN_TRY(hipStreamSynchronize(c->stream));
  to_abi_layout(c->o, c->h_buf, grads);
  return DPT_OK;
}

int dpt_cnn_forward(dpt_cnn* c, const uint8_t* pairs, int32_t B, int32_t on_device, float* out_host) {
  if (!c || !pairs || !out_host) return cfail(DPT_E_ARG, "NULL argument");
  if (B < 1 || B > c->max_batch) return cfail(DPT_E_ARG, "batch size");
  int e = forward_pairs(c, pairs, B, on_device, nullptr);
  if (e != DPT_OK) return e;
  CNN_TRY(hipMemcpyAsync(out_host, c->out, sizeof(float) * B * kOut, hipMemcpyDeviceToHost, c->stream));
  CNN_TRY(hipStreamSynchronize(c->stream));
  return DPT_OK;
}

// One training step on B pairs: forward, MSE loss against targets (normalised
// twists, B x 6), backward, Adam (lr, beta 0.9 / 0.999, eps 1e-8).  With
// lr == 0 only the gradients are computed (no update).  *loss_out: the loss
// before the update.
int dpt_cnn_train_step(dpt_cnn* c, const uint8_t* pairs, const float* targets, int32_t B, float lr,
                       int32_t on_device, float* loss_out) {
  if (!c || !pairs || !targets || !loss_out) return cfail(DPT_E_ARG, "NULL argument");
  if (B < 1 || B > c->max_batch) return cfail(DPT_E_ARG, "batch size");
  const float* tg = targets;
  if (!on_device) {
    CNN_TRY(hipMemcpyAsync(c->tgt, targets, sizeof(float) * B * kOut, hipMemcpyHostToDevice, c->stream));
    tg = c->tgt;
  }
  int e = forward_pairs(c, pairs, B, on_device, tg);
  if (e != DPT_OK) return e;
  float c1 = 1.f, c2 = 1.f;
  if (lr > 0.f) {
    c->step += 1;
    c1 = 1.0f - std::pow(0.9f, (float)c->step), c2 = 1.0f - std::pow(0.999f, (float)c->step);
  }
  CNN_TRY(update(c, B, lr, c1, c2));
  CNN_TRY(hipStreamSynchronize(c->stream));
  float s = 0.f;
  for (int q = 0; q < kOut; ++q) s += c->h_buf[q];
  *loss_out = s / (float)(B * kOut);
  return DPT_OK;
}

// Test hook: layer activation l (1..4) of the last forward as FP32 NHWC, or
// (l = 5) the network outputs [B][6].
int dpt_cnn_get_activation(dpt_cnn* c, int32_t l, int32_t B, float* host_out) {
  if (!c || !host_out || l < 1 || l > 5 || B < 1 || B > c->max_batch) return cfail(DPT_E_ARG, "argument");
  if (l == 5) {
    CNN_TRY(hipMemcpyAsync(host_out, c->out, sizeof(float) * B * kOut, hipMemcpyDeviceToHost, c->stream));
  } else {
    const size_t n = (size_t)B * kHs[l] * kWs[l] * kC[l];  // dz[l] has exactly this size
    float* tmp = reinterpret_cast<float*>(c->dz[l]);
    hipLaunchKernelGGL(bf16_to_f32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, c->act[l], n, tmp);
    CNN_TRY(hipGetLastError());
    CNN_TRY(hipMemcpyAsync(host_out, tmp, sizeof(float) * n, hipMemcpyDeviceToHost, c->stream));
  }
  CNN_TRY(hipStreamSynchronize(c->stream));
  return DPT_OK;
}

}  // extern "C"

namespace dpt {

// Forward pass on B pairs given as device pointers to coarsest pyramid levels
// (94 x 60, packed rows); writes B x 6 normalised twists to out_host.
int cnn_forward_levels(dpt_cnn* c, const uint8_t* const* refs, const uint8_t* const* curs, int B, float* out_host) {
  if (B < 1 || B > c->max_batch) return cfail(DPT_E_ARG, "batch size");
  std::vector<const uint8_t*> h(2 * (size_t)B);
  for (int b = 0; b < B; ++b) h[b] = refs[b], h[B + b] = curs[b];
  CNN_TRY(hipMemcpyAsync(c->d_lv, h.data(), sizeof(void*) * 2 * B, hipMemcpyHostToDevice, c->stream));
  FusedIO io{};
  io.refs = c->d_lv, io.curs = c->d_lv + B, io.act[4] = c->act[4], io.out = c->out;
  CNN_TRY(launch_fused(io, B, c->Pb, c->PbT, c->P, c->stream));
  CNN_TRY(hipMemcpyAsync(out_host, c->out, sizeof(float) * B * kOut, hipMemcpyDeviceToHost, c->stream));
  CNN_TRY(hipStreamSynchronize(c->stream));
  return DPT_OK;
}

int cnn_propose(dpt_cnn* c, const uint8_t* const* d_lv, int B, hipStream_t s, double* rel) {
  if (B < 1 || B > c->max_batch) return cfail(DPT_E_ARG, "batch size");
  FusedIO io{};
  io.refs = d_lv, io.curs = d_lv + B, io.act[4] = c->act[4], io.out = c->out, io.rel = rel;
  CNN_TRY(launch_fused(io, B, c->Pb, c->PbT, c->P, s));
  return DPT_OK;
}

}  // namespace dpt
