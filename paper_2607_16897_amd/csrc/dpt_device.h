// Device helpers shared by the tracker kernels: projection, sampling,
// workgroup reductions and the 6x6 solve with the SE(3) update.
#pragma once

#include <type_traits>

#include "dpt_internal.h"

namespace dpt {

// ---------------------------------------------------------------- helpers

__device__ __forceinline__ void transform(const float* T, float X, float Y, float Z, float& x, float& y,
                                          float& z) {
  x = fmaf(T[0], X, fmaf(T[1], Y, fmaf(T[2], Z, T[3])));
  y = fmaf(T[4], X, fmaf(T[5], Y, fmaf(T[6], Z, T[7])));
  z = fmaf(T[8], X, fmaf(T[9], Y, fmaf(T[10], Z, T[11])));
}

// Eq.(1): pinhole projection at one pyramid level, through one reciprocal of
// z (v_rcp_f32, 1 ulp).  Every sampling site (the precompute and every track
// path) projects with this same arithmetic, so a pose equal to the reference's
// reproduces the template's sample positions bit for bit.
__device__ __forceinline__ void project(const LevelGeom& g, float x, float y, float z, float& u, float& v) {
  const float iz = __builtin_amdgcn_rcpf(z);
  u = fmaf(g.fx * x, iz, g.cx);
  v = fmaf(g.fy * y, iz, g.cy);
}

// A point is usable when it is in front of the camera and every pattern
// position p satisfies 1 <= p.x < W-2 and 1 <= p.y < H-2 (the bilinear taps and
// their central differences stay inside the level).
__device__ __forceinline__ bool inside(const LevelGeom& g, const Pattern& p, float u, float v) {
  return (u + (float)p.dx_min >= 1.0f) && (u + (float)p.dx_max < (float)(g.W - 2)) &&
         (v + (float)p.dy_min >= 1.0f) && (v + (float)p.dy_max < (float)(g.H - 2));
}

// The K = 8 pattern held in registers for the whole track: offsets and their
// bounding box as floats (the same values inside() converts on the fly).
struct PatRegs {
  float dx[8], dy[8];
  float dx_min, dx_max, dy_min, dy_max;
};

__device__ __forceinline__ PatRegs pattern_regs(const Pattern& p) {
  PatRegs r;
#pragma unroll
  for (int k = 0; k < 8; ++k) r.dx[k] = (float)p.dx[k], r.dy[k] = (float)p.dy[k];
  r.dx_min = (float)p.dx_min, r.dx_max = (float)p.dx_max;
  r.dy_min = (float)p.dy_min, r.dy_max = (float)p.dy_max;
  return r;
}

// inside() on the register pattern, without branches.
__device__ __forceinline__ bool inside(const LevelGeom& g, const PatRegs& p, float u, float v) {
  return (u + p.dx_min >= 1.0f) & (u + p.dx_max < (float)(g.W - 2)) & (v + p.dy_min >= 1.0f) &
         (v + p.dy_max < (float)(g.H - 2));
}

// Bilinear sampling, pixel centres at integer coordinates.  A point projected
// to (u, v) lies in the cell with corner (iu, iv) = floor(u, v) at fractions
// (a, c); the pattern's offsets are whole pixels, so every sample of the point
// is the cell at (iu + dx_k, iv + dy_k) with the same fractions and weights.
// The weights are formed once per point, the same way at every sampling site.
struct Bilin {
  float w00, w10, w01, w11;
};

struct Cell {
  int iu, iv;
  Bilin w;
};

__device__ __forceinline__ Cell cell_of(float u, float v) {
  Cell q;
  const float fu = floorf(u), fv = floorf(v);
  const float a = u - fu, c = v - fv;  // exact: u and floor(u) are close
  q.iu = (int)fu, q.iv = (int)fv;
  q.w.w11 = a * c;
  q.w.w10 = a - q.w.w11;
  q.w.w01 = c - q.w.w11;
  q.w.w00 = (1.0f - a) - q.w.w01;
  return q;
}

// (1-a)(1-c) t00 + a(1-c) t10 + (1-a)c t01 + ac t11.
__device__ __forceinline__ float bilin_mix(const Bilin& w, float t00, float t10, float t01, float t11) {
  return fmaf(w.w11, t11, fmaf(w.w01, t01, fmaf(w.w10, t10, w.w00 * t00)));
}

// Intensity of a level (uint8 or float pixels) in the cell with corner (x, y).
template <class PIX>
__device__ __forceinline__ float sample_cell(const PIX* img, int W, int x, int y, const Bilin& w) {
  const PIX* p = img + y * W + x;
  return bilin_mix(w, (float)p[0], (float)p[1], (float)p[W], (float)p[W + 1]);
}

// Intensity in the cell with corner (x, y) as sample_cell, and the reference-side
// gradient: central differences / 2 at its four corners, blended with the same
// weights.  The 4 x 4 pixels around the cell, all inside the level, are read a
// row at a time from any address.
template <class PIX>
__device__ __forceinline__ void reference_cell(const PIX* img, int W, int x, int y, const Bilin& w, float& I0, float& gx,
                                               float& gy) {
  float r[4][4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const PIX* p = img + (y - 1 + j) * W + x - 1;
    if constexpr (std::is_same<PIX, uint8_t>::value) {
      struct __attribute__((packed)) Word {
        uint32_t w;
      };
      const uint32_t v = ((const __attribute__((address_space(1))) Word*)p)->w;
#pragma unroll
      for (int i = 0; i < 4; ++i) r[j][i] = (float)(v >> (8 * i) & 0xffu);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) r[j][i] = ((const __attribute__((address_space(1))) PIX*)p)[i];
    }
  }
  I0 = bilin_mix(w, r[1][1], r[1][2], r[2][1], r[2][2]);
  gx = bilin_mix(w, 0.5f * (r[1][2] - r[1][0]), 0.5f * (r[1][3] - r[1][1]), 0.5f * (r[2][2] - r[2][0]),
                 0.5f * (r[2][3] - r[2][1]));
  gy = bilin_mix(w, 0.5f * (r[2][1] - r[0][1]), 0.5f * (r[2][2] - r[0][2]), 0.5f * (r[3][1] - r[1][1]),
                 0.5f * (r[3][2] - r[1][2]));
}

// ---------------------------------------------------------------- pyramid

// One launch builds every level.  A workgroup owns a TILE x TILE block of
// level 0 (TILE >= 2^(levels-1)), so each level's 2x2 parents stay inside the
// tile; levels alternate between two LDS buffers.
// The tile at level-0 origin (ox, oy); write_l0 = false leaves level 0 of dst
// unwritten (a caller that reads level 0 from the source frame itself).
template <int TILE>
__device__ __forceinline__ void pyramid_tile_at(const uint8_t* __restrict__ src, int64_t pitch,
                                                uint8_t* __restrict__ dst, const PyrGeom& g, int vec4, int ox, int oy,
                                                bool write_l0) {
  __shared__ uint8_t buf0[TILE * TILE];
  __shared__ uint8_t buf1[TILE * TILE / 4];
  const int W0 = g.W[0], H0 = g.H[0];
  if (vec4) {
    // 4-byte loads: width, pitch and base are multiples of 4
    for (int q = threadIdx.x; q < TILE * TILE / 4; q += blockDim.x) {
      int ly = q / (TILE / 4), lx = (q % (TILE / 4)) * 4;
      int gx = ox + lx, gy = oy + ly;
      uint32_t v = 0;
      if (gy < H0 && gx < W0) {
        v = *reinterpret_cast<const uint32_t*>(src + gy * pitch + gx);
        if (write_l0) *reinterpret_cast<uint32_t*>(dst + g.off[0] + (int64_t)gy * W0 + gx) = v;
      }
      *reinterpret_cast<uint32_t*>(buf0 + ly * TILE + lx) = v;
    }
  } else {
    for (int q = threadIdx.x; q < TILE * TILE; q += blockDim.x) {
      int ly = q / TILE, lx = q % TILE;
      int gx = ox + lx, gy = oy + ly;
      uint8_t v = 0;
      if (gy < H0 && gx < W0) {
        v = src[gy * pitch + gx];
        if (write_l0) dst[g.off[0] + (int64_t)gy * W0 + gx] = v;
      }
      buf0[q] = v;
    }
  }
  __syncthreads();
  uint8_t* prev = buf0;
  uint8_t* next = buf1;
  for (int l = 1; l < g.levels; ++l) {
    const int T = TILE >> l, Tp = TILE >> (l - 1);
    const int Wl = g.W[l], Hl = g.H[l];
    const int oxl = ox >> l, oyl = oy >> l;
    for (int q = threadIdx.x; q < T * T; q += blockDim.x) {
      int ly = q / T, lx = q % T;
      int gx = oxl + lx, gy = oyl + ly;
      uint8_t v = 0;
      if (gx < Wl && gy < Hl) {
        const uint8_t* p = prev + (2 * ly) * Tp + 2 * lx;
        int s = (int)p[0] + (int)p[1] + (int)p[Tp] + (int)p[Tp + 1];
        v = (uint8_t)((s + 2) >> 2);
        dst[g.off[l] + (int64_t)gy * Wl + gx] = v;
      }
      next[q] = v;
    }
    __syncthreads();
    uint8_t* t = prev;
    prev = next;
    next = t;
  }
}

template <int TILE>
__device__ __forceinline__ void pyramid_tile(const uint8_t* __restrict__ src, int64_t pitch,
                                             uint8_t* __restrict__ dst, const PyrGeom& g, int vec4) {
  pyramid_tile_at<TILE>(src, pitch, dst, g, vec4, blockIdx.x * TILE, blockIdx.y * TILE, true);
}

// N words from or to any address.
template <int N>
struct __attribute__((packed)) Words {
  uint32_t w[N];
};
template <int N>
__device__ __forceinline__ void load_words(const uint8_t* p, uint32_t (&v)[N]) {
  const auto* q = (const __attribute__((address_space(1))) Words<N>*)p;
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = q->w[k];
}
template <int N>
__device__ __forceinline__ void store_words(uint8_t* p, const uint32_t (&v)[N]) {
  auto* q = (__attribute__((address_space(1))) Words<N>*)p;
#pragma unroll
  for (int k = 0; k < N; ++k) q->w[k] = v[k];
}

// pyramid_tile for 64x64 tiles and up to 7 levels: one 16-byte load and store per
// thread for level 0 (256 threads), four level-1 pixels per thread from two 8-byte
// LDS reads with one 4-byte store, then the coarser levels as pyramid_tile.  At
// any width, pitch and address: rows of odd frames start anywhere, and only the
// end of a row goes byte by byte (whole rows so, and four tiles in turn for each
// workgroup: a window of 9 641x479 frames took 21 us, now 5.6).
__device__ __forceinline__ void pyramid_tile64v_at(const uint8_t* __restrict__ src, int64_t pitch,
                                                   uint8_t* __restrict__ dst, const PyrGeom& g, int ox, int oy,
                                                   bool write_l0) {
  __shared__ __align__(16) uint8_t buf0[64 * 64];
  __shared__ __align__(16) uint8_t buf1[32 * 32];
  const int W0 = g.W[0], H0 = g.H[0];
  {
    const int r = threadIdx.x >> 2, c = (threadIdx.x & 3) * 16;
    const int gx = ox + c, gy = oy + r;
    uint32_t v[4] = {0u, 0u, 0u, 0u};
    if (gy < H0 && gx < W0) {
      const uint8_t* sp = src + gy * pitch + gx;
      uint8_t* dp = dst + g.off[0] + (int64_t)gy * W0 + gx;
      if (gx + 16 <= W0) {
        load_words<4>(sp, v);
        if (write_l0) store_words<4>(dp, v);
      } else {
#pragma unroll
        for (int k = 0; k < 16; ++k)
          if (gx + k < W0) v[k / 4] |= (uint32_t)((const __attribute__((address_space(1))) uint8_t*)sp)[k] << (8 * (k & 3));
        if (write_l0) {
#pragma unroll
          for (int k = 0; k < 16; ++k)
            if (gx + k < W0) dp[k] = (uint8_t)(v[k / 4] >> (8 * (k & 3)));
        }
      }
    }
    *reinterpret_cast<uint4*>(buf0 + r * 64 + c) = make_uint4(v[0], v[1], v[2], v[3]);
  }
  __syncthreads();
  if (g.levels < 2) return;
  {
    const int r = threadIdx.x >> 3, c = (threadIdx.x & 7) * 4;
    const uint2 a = *reinterpret_cast<const uint2*>(buf0 + (2 * r) * 64 + 2 * c);
    const uint2 b = *reinterpret_cast<const uint2*>(buf0 + (2 * r + 1) * 64 + 2 * c);
    const uint32_t top[2] = {a.x, a.y}, bot[2] = {b.x, b.y};
    uint32_t out = 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t t = top[j >> 1] >> (16 * (j & 1)), u = bot[j >> 1] >> (16 * (j & 1));
      const uint32_t s4 = (t & 0xffu) + ((t >> 8) & 0xffu) + (u & 0xffu) + ((u >> 8) & 0xffu);
      out |= ((s4 + 2u) >> 2) << (8 * j);
    }
    *reinterpret_cast<uint32_t*>(buf1 + r * 32 + c) = out;
    const int W1 = g.W[1], H1 = g.H[1];
    const int gx = (ox >> 1) + c, gy = (oy >> 1) + r;
    uint8_t* dp = dst + g.off[1] + (int64_t)gy * W1 + gx;
    if (gy < H1 && gx + 4 <= W1) {
      store_words<1>(dp, {out});
    } else if (gy < H1) {
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (gx + k < W1) dp[k] = (uint8_t)(out >> (8 * k));
    }
  }
  __syncthreads();
  uint8_t* prev = buf1;
  uint8_t* next = buf0;
  for (int l = 2; l < g.levels; ++l) {
    const int T = 64 >> l, Tp = 64 >> (l - 1);
    const int Wl = g.W[l], Hl = g.H[l];
    const int oxl = ox >> l, oyl = oy >> l;
    for (int q = threadIdx.x; q < T * T; q += blockDim.x) {
      const int ly = q >> (6 - l), lx = q & (T - 1);
      const int gx = oxl + lx, gy = oyl + ly;
      uint8_t v = 0;
      if (gx < Wl && gy < Hl) {
        const uint8_t* p = prev + (2 * ly) * Tp + 2 * lx;
        const int s4 = (int)p[0] + (int)p[1] + (int)p[Tp] + (int)p[Tp + 1];
        v = (uint8_t)((s4 + 2) >> 2);
        dst[g.off[l] + (int64_t)gy * Wl + gx] = v;
      }
      next[q] = v;
    }
    __syncthreads();
    uint8_t* t = prev;
    prev = next;
    next = t;
  }
}

// Rounded 2x2 box means of two rows of four bytes: bytes 0 and 1 of the
// result hold (t0 + t1 + b0 + b1 + 2) >> 2 and (t2 + t3 + b2 + b3 + 2) >> 2.
// The pair sums travel in two 16-bit lanes (at most 1022 each).
__device__ __forceinline__ uint32_t box_pairs(uint32_t top, uint32_t bot) {
  const uint32_t s = (top & 0x00ff00ffu) + ((top >> 8) & 0x00ff00ffu) + (bot & 0x00ff00ffu) + ((bot >> 8) & 0x00ff00ffu);
  const uint32_t r = ((s + 0x00020002u) >> 2) & 0x00ff00ffu;
  return (r & 0xffu) | ((r >> 8) & 0xff00u);
}

// The pyramid of one B x B block of level 0 (B = 2^(LV-1), LV = 3 or 4
// levels) in one thread's registers: block (bx, by) of a level 0 whose sizes
// are multiples of B, so every level's share of the block is whole and
// (levels' sizes halving exactly) each level is written with one aligned
// store per row.  Needs 8-byte aligned rows of src and dst.
template <int LV>
__device__ __forceinline__ void pyramid_block(const uint8_t* __restrict__ src, int64_t pitch,
                                              uint8_t* __restrict__ dst, const PyrGeom& g, int bx, int by,
                                              bool write_l0) {
  static_assert(LV == 3 || LV == 4, "three or four levels");
  constexpr int B = 1 << (LV - 1);
  const int W0 = g.W[0];
  if constexpr (LV == 4) {
    uint2 r0[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) r0[r] = *reinterpret_cast<const uint2*>(src + (int64_t)(8 * by + r) * pitch + 8 * bx);
    if (write_l0)
#pragma unroll
      for (int r = 0; r < 8; ++r) *reinterpret_cast<uint2*>(dst + g.off[0] + (int64_t)(8 * by + r) * W0 + 8 * bx) = r0[r];
    uint32_t r1[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      r1[i] = box_pairs(r0[2 * i].x, r0[2 * i + 1].x) | (box_pairs(r0[2 * i].y, r0[2 * i + 1].y) << 16);
      *reinterpret_cast<uint32_t*>(dst + g.off[1] + (int64_t)(4 * by + i) * g.W[1] + 4 * bx) = r1[i];
    }
    uint32_t r2[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      r2[i] = box_pairs(r1[2 * i], r1[2 * i + 1]);
      *reinterpret_cast<uint16_t*>(dst + g.off[2] + (int64_t)(2 * by + i) * g.W[2] + 2 * bx) = (uint16_t)r2[i];
    }
    dst[g.off[3] + (int64_t)by * g.W[3] + bx] = (uint8_t)box_pairs(r2[0], r2[1]);
  } else {
    uint32_t r0[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) r0[r] = *reinterpret_cast<const uint32_t*>(src + (int64_t)(4 * by + r) * pitch + 4 * bx);
    if (write_l0)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        *reinterpret_cast<uint32_t*>(dst + g.off[0] + (int64_t)(4 * by + r) * W0 + 4 * bx) = r0[r];
    uint32_t r1[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      r1[i] = box_pairs(r0[2 * i], r0[2 * i + 1]);
      *reinterpret_cast<uint16_t*>(dst + g.off[1] + (int64_t)(2 * by + i) * g.W[1] + 2 * bx) = (uint16_t)r1[i];
    }
    dst[g.off[2] + (int64_t)by * g.W[2] + bx] = (uint8_t)box_pairs(r1[0], r1[1]);
  }
  (void)B;
}

__device__ __forceinline__ void pyramid_tile64v(const uint8_t* __restrict__ src, int64_t pitch,
                                                uint8_t* __restrict__ dst, const PyrGeom& g) {
  pyramid_tile64v_at(src, pitch, dst, g, blockIdx.x * 64, blockIdx.y * 64, true);
}

// ---------------------------------------------------------------- reductions

// Row rotation within 16 lanes (DPP row_ror:K), a VALU operand modifier.
template <int K>
__device__ __forceinline__ float dpp_ror(float v) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x120 + K, 0xf, 0xf, false));
}

// Sum 32 per-lane values over a wave64.  Two halving steps exchange whole
// half-waves with the gfx950 lane-swap instructions: v_permlane32_swap pairs
// lane L with L ^ 32 and v_permlane16_swap pairs L with L ^ 16, each lane keeping
// half of its values, so 16 + 8 swaps leave 8 values per lane summed over 4
// lanes.  DPP row rotations then sum each over the 16 lanes of a row.  On return
// a[j] of every lane in row r = lane / 16 holds the wave total of value 8 r + j.
// No shuffle through LDS and no data-dependent indexing; fixed addition order.
__device__ __forceinline__ void wave_reduce32(float (&a)[32]) {
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[j]), __float_as_uint(a[j + 16]), false, false);
    a[j] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[j]), __float_as_uint(a[j + 8]), false, false);
    a[j] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    float v = a[j];
    v += dpp_ror<8>(v);
    v += dpp_ror<4>(v);
    v += dpp_ror<2>(v);
    v += dpp_ror<1>(v);
    a[j] = v;
  }
}

// wave_reduce32 for 16 values: one lane-swap step less.  On return a[j] of
// every lane in row r = lane / 16 holds the wave total of value 4 r + j, j < 4.
__device__ __forceinline__ void wave_reduce16(float (&a)[16]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[j]), __float_as_uint(a[j + 8]), false, false);
    a[j] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[j]), __float_as_uint(a[j + 4]), false, false);
    a[j] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float v = a[j];
    v += dpp_ror<8>(v);
    v += dpp_ror<4>(v);
    v += dpp_ror<2>(v);
    v += dpp_ror<1>(v);
    a[j] = v;
  }
}

// Workgroup total of 32 per-lane values into out[32] (LDS), fixed order.
// `scratch` is 16 x 32 floats of LDS.
__device__ __forceinline__ void block_reduce32(float (&a)[32], float* scratch, float* out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  wave_reduce32(a);
  if ((lane & 15) == 0) {
#pragma unroll
    for (int j = 0; j < 8; ++j) scratch[wave * 32 + 8 * (lane >> 4) + j] = a[j];
  }
  __syncthreads();
  if (threadIdx.x < 32) {
    float s = 0.0f;
    for (int w = 0; w < nw; ++w) s += scratch[w * 32 + threadIdx.x];
    out[threadIdx.x] = s;
  }
  __syncthreads();
}

// Index of H(i, j), i <= j, in the row-major upper-triangle order of the sums.
__host__ __device__ constexpr int tri(int i, int j) { return i * 6 - (i * (i - 1)) / 2 + (j - i); }

// T <- T exp(xi) for the twist xi = (w, v) (rotation part first) of squared
// angle th2 = |w|^2, given the coefficients A = sin(th) / th,
// B = (1 - cos th) / th^2 and C = (th - sin th) / th^3 of the SE(3) exponential:
// R = I + A [w]x + B [w]x^2 and t = (I + B [w]x + C [w]x^2) v.  With
// [w]x^2 = w w^T - th2 I and [w]x v = w x v these are written out entry by
// entry: R = (1 - B th2) I + A [w]x + B w w^T, t = (1 - C th2) v + B (w x v)
// + C (w.v) w.  F = float or double; every product is an explicit FMA.
template <class F>
__device__ __forceinline__ void compose_exp(F* T, F w0, F w1, F w2, F v0, F v1, F v2, F th2, F A, F B, F C) {
  const F Bw0 = B * w0, Bw1 = B * w1, Bw2 = B * w2, Aw0 = A * w0, Aw1 = A * w1, Aw2 = A * w2;
  const F dg = fma(-B, th2, F(1));
  const F E[3][4] = {
      {fma(Bw0, w0, dg), fma(Bw0, w1, -Aw2), fma(Bw0, w2, Aw1), F(0)},
      {fma(Bw0, w1, Aw2), fma(Bw1, w1, dg), fma(Bw1, w2, -Aw0), F(0)},
      {fma(Bw0, w2, -Aw1), fma(Bw1, w2, Aw0), fma(Bw2, w2, dg), F(0)}};
  const F c0 = fma(w1, v2, -(w2 * v1)), c1 = fma(w2, v0, -(w0 * v2)), c2 = fma(w0, v1, -(w1 * v0));
  const F Cwv = C * fma(w0, v0, fma(w1, v1, w2 * v2)), Cv = fma(-C, th2, F(1));
  const F t[3] = {fma(B, c0, fma(Cwv, w0, Cv * v0)), fma(B, c1, fma(Cwv, w1, Cv * v1)),
                  fma(B, c2, fma(Cwv, w2, Cv * v2))};
  F N[12];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
#pragma unroll
    for (int c = 0; c < 3; ++c) N[4 * r + c] = fma(T[4 * r], E[0][c], fma(T[4 * r + 1], E[1][c], T[4 * r + 2] * E[2][c]));
    N[4 * r + 3] = fma(T[4 * r], t[0], fma(T[4 * r + 1], t[1], fma(T[4 * r + 2], t[2], T[4 * r + 3])));
  }
#pragma unroll
  for (int j = 0; j < 12; ++j) T[j] = N[j];
}

// With H = L L^T given by its factor (L(i, j), i >= j, at tri(j, i), and
// invd = 1 / diag(L)), solve H delta = b by forward and back substitution and
// apply T <- T exp(-delta) in FP32; *max_step = max_j |delta_j|.
__device__ __forceinline__ void substitute_update(const float (&L)[21], const float (&invd)[6], const float (&b)[6],
                                                  float* T, float* max_step);

// Solve H delta = b (6x6 SPD from the 21 upper-triangle sums) by Cholesky in
// FP32 and apply T <- T exp(-delta).  Returns 0, or 1 if a pivot is <= 1e-6 of
// the largest diagonal entry (not positive definite).  Every loop is unrolled
// so the factor lives in registers.
__device__ __forceinline__ int solve_update(const float* tot_lds, float* T, float* max_step) {
  float tot[27];  // one batch of LDS reads, then registers only
#pragma unroll
  for (int q = 0; q < 27; ++q) tot[q] = tot_lds[q];
  float L[21];  // L(i, j), i >= j, stored at tri(j, i)
  float invd[6];
  float dmax = 0.f;
#pragma unroll
  for (int j = 0; j < 6; ++j) dmax = fmaxf(dmax, tot[tri(j, j)]);
  int bad = 0;
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    float s = tot[tri(j, j)];
#pragma unroll
    for (int k = 0; k < j; ++k) s = fmaf(-L[tri(k, j)], L[tri(k, j)], s);
    bad |= !(s > 1e-6f * dmax);
    // only 1/L(j, j) is used by the elimination and the substitutions
    const float inv = __builtin_amdgcn_rsqf(fmaxf(s, 1e-30f));
    invd[j] = inv;
#pragma unroll
    for (int i = j + 1; i < 6; ++i) {
      float t = tot[tri(j, i)];
#pragma unroll
      for (int k = 0; k < j; ++k) t = fmaf(-L[tri(k, i)], L[tri(k, j)], t);
      L[tri(j, i)] = t * inv;
    }
  }
  if (bad) return 1;
  float b[6];
#pragma unroll
  for (int i = 0; i < 6; ++i) b[i] = tot[kSlotB + i];
  substitute_update(L, invd, b, T, max_step);
  return 0;
}

// Fixed-H mode: the factor of the level's constant H comes precomputed
// (Lp[21], invdp[6], as in substitute_update); only the substitutions and the
// update remain.  b: the 6 reduced right-hand-side sums.
__device__ __forceinline__ void solve_fixed(const float* Lp, const float* invdp, const float* bp, float* T,
                                            float* max_step) {
  float L[21], invd[6], b[6];
#pragma unroll
  for (int q = 0; q < 21; ++q) L[q] = Lp[q];
#pragma unroll
  for (int q = 0; q < 6; ++q) invd[q] = invdp[q], b[q] = bp[q];
  substitute_update(L, invd, b, T, max_step);
}

__device__ __forceinline__ void substitute_update(const float (&L)[21], const float (&invd)[6], const float (&b)[6],
                                                  float* T, float* max_step) {
  float y[6], d[6];
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    float s = b[i];
#pragma unroll
    for (int k = 0; k < i; ++k) s = fmaf(-L[tri(k, i)], y[k], s);
    y[i] = s * invd[i];
  }
#pragma unroll
  for (int i = 5; i >= 0; --i) {
    float s = y[i];
#pragma unroll
    for (int k = i + 1; k < 6; ++k) s = fmaf(-L[tri(i, k)], d[k], s);
    d[i] = s * invd[i];
  }
  float m = 0.f;
#pragma unroll
  for (int j = 0; j < 6; ++j) m = fmaxf(m, fabsf(d[j]));
  *max_step = m;
  const float w0 = -d[0], w1 = -d[1], w2 = -d[2];
  const float th2 = fmaf(w0, w0, fmaf(w1, w1, w2 * w2));
  float A, B, C;
  if (th2 < 0.0025f) {  // |w| < 0.05
    A = 1.0f - th2 * (1.0f / 6.0f) * (1.0f - th2 * (1.0f / 20.0f));
    B = 0.5f - th2 * (1.0f / 24.0f) * (1.0f - th2 * (1.0f / 30.0f));
    C = (1.0f / 6.0f) - th2 * (1.0f / 120.0f) * (1.0f - th2 * (1.0f / 42.0f));
  } else {
    const float th = sqrtf(th2);
    const float sn = sinf(th), sh = sinf(0.5f * th);
    A = sn / th;
    B = 2.0f * sh * sh / th2;
    C = (th - sn) / (th2 * th);
  }
  compose_exp(T, w0, w1, w2, -d[3], -d[4], -d[5], th2, A, B, C);
}

// ---------------------------------------------------------------- solve and update across the lanes

// Lane K of each 16-lane row, in every lane of the row (DPP row_newbcast).
template <int K>
__device__ __forceinline__ float row_bcast(float v) {
  return __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0x150 + K, 0xf, 0xf, true));
}
template <int K>
__device__ __forceinline__ double row_bcast(double v) {
  const uint64_t u = __double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_mov_dpp((uint32_t)u, 0x150 + K, 0xf, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_mov_dpp((uint32_t)(u >> 32), 0x150 + K, 0xf, 0xf, true);
  return __longlong_as_double(((uint64_t)hi << 32) | lo);
}
// Lane K of each quad, in every lane of the quad (DPP quad_perm).
template <int K>
__device__ __forceinline__ float quad_bcast(float v) {
  return __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), K * 0x55, 0xf, 0xf, true));
}
template <int K>
__device__ __forceinline__ double quad_bcast(double v) {
  const uint64_t u = __double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_mov_dpp((uint32_t)u, K * 0x55, 0xf, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_mov_dpp((uint32_t)(u >> 32), K * 0x55, 0xf, 0xf, true);
  return __longlong_as_double(((uint64_t)hi << 32) | lo);
}

// The stream totals of an iteration as the solve reads them (floats, LDS): row
// i of the symmetric H at 8 i .. 8 i + 5 and b_i at 8 i + 6, then the cost and
// the counts.
constexpr int kTotB = 6, kTotE = 48, kTotN = 49, kTotPts = 50, kTotOk = 51, kTotals = 52;

// Where the total of reduction slot v goes: two places for an off-diagonal
// entry of H (else twice the same).  Slots without a use go to a spare word of
// the rows.
template <int NV>
__device__ __forceinline__ int2 total_place(int v) {
  if constexpr (NV == kFixSlots) {
    const int d = v < 6 ? 8 * v + kTotB : v == kFixE ? kTotE : v == kFixN ? kTotN : v == kFixPts ? kTotPts : 7;
    return make_int2(d, d);
  } else {
    const int r = (v >= 6) + (v >= 11) + (v >= 15) + (v >= 18) + (v >= 20);
    const int c = v - (6 * r - r * (r - 1) / 2) + r;
    if (v < kSlotB) return make_int2(8 * r + c, 8 * c + r);
    const int d = v < kSlotE ? 8 * (v - kSlotB) + kTotB
                             : v == kSlotE ? kTotE : v == kSlotN ? kTotN : v == kSlotPts ? kTotPts : 7;
    return make_int2(d, d);
  }
}

// 1 / p: the hardware estimate, in FP64 refined by two Newton steps.
__device__ __forceinline__ float recip(float p) { return __builtin_amdgcn_rcpf(p); }
__device__ __forceinline__ double recip(double p) {
  double r = __builtin_amdgcn_rcp(p);
  r = r * fma(-p, r, 2.0);
  return r * fma(-p, r, 2.0);
}

// One elimination step of solve_rows (K = 0..5), then the next.
template <int K, class F>
__device__ __forceinline__ void eliminate(F (&a)[7], int i, F& piv, F& inv_own) {
  const F p = row_bcast<K>(a[K]);
  const F inv = recip(p);
  const F f = (i == K ? F(0) : -a[K]) * inv;
  piv = i == K ? p : piv;
  inv_own = i == K ? inv : inv_own;
#pragma unroll
  for (int j = K + 1; j < 7; ++j) a[j] = fma(row_bcast<K>(a[j]), f, a[j]);
  if constexpr (K < 5) eliminate<K + 1>(a, i, piv, inv_own);
}

// Solve H delta = b (6x6 SPD) across the lanes of each 16-lane row: lane i < 6
// holds row i of (H | b) in a, Gauss-Jordan elimination without pivoting (the
// pivots are those of the Cholesky factorisation squared), every step one
// instruction per remaining column for all rows at once.  Lane i returns
// delta_i; *bad (every lane) is set if a pivot is not above eps times the
// largest diagonal entry (diag: the lane's own), NaN included.  A thread that
// solves the system and updates the pose by itself issues about 330
// instructions, these lanes 200 (the phase is bound by their issue, 4 cycles
// each, and by their chains).  With the exchange's poll offsets formed once
// and the iteration loop's branches scalar, a nine-frame window track of 2000
// points takes 434 instead of 475 us (two threads per point; one thread per
// point 479 instead of 535, fixed H 355 instead of 408, mixed precision 493
// instead of 534).
template <class F>
__device__ __forceinline__ F solve_rows(F (&a)[7], F diag, F eps, int i, bool* bad) {
  const F thr = eps * fmax(fmax(fmax(row_bcast<0>(diag), row_bcast<1>(diag)), fmax(row_bcast<2>(diag), row_bcast<3>(diag))),
                           fmax(row_bcast<4>(diag), row_bcast<5>(diag)));
  F piv = F(0), inv_own = F(0);
  eliminate<0>(a, i, piv, inv_own);
  *bad = __any((i < 6) & !(piv > thr));
  return a[6] * inv_own;
}

// The pose held across the lanes: element (r, c) of the 3x4 [R | t] in lane
// 4 r + c of each 16-lane row (lanes 12 to 15 hold a fourth row that nothing
// reads).  T <- T exp(-delta), lane i < 6 giving delta_i (rotation first);
// *max_step (every lane) = max |delta_i|.  Column c of the exponential is
// alpha q + beta (w x q) + gamma (w.q) w with q the unit vector c and
// (1 - B th2, A, B), or, for the translation, q = v and (1 - C th2, B, C): each
// lane forms its own column, so the update costs a third of the instructions
// of the entries one by one.
template <class F>
__device__ __forceinline__ F update_lanes(F T, F delta, F* max_step) {
  const F w0 = -row_bcast<0>(delta), w1 = -row_bcast<1>(delta), w2 = -row_bcast<2>(delta);
  const F v0 = -row_bcast<3>(delta), v1 = -row_bcast<4>(delta), v2 = -row_bcast<5>(delta);
  *max_step = fmax(fmax(fmax(fabs(w0), fabs(w1)), fmax(fabs(w2), fabs(v0))), fmax(fabs(v1), fabs(v2)));
  const int c = threadIdx.x & 3;
  const bool tr = c == 3;
  const F q0 = tr ? v0 : c == 0 ? F(1) : F(0), q1 = tr ? v1 : c == 1 ? F(1) : F(0),
          q2 = tr ? v2 : c == 2 ? F(1) : F(0);
  const F th2 = fma(w0, w0, fma(w1, w1, w2 * w2));
  F be, ga;  // A and B, or B and C in the translation's lanes
  if (__builtin_expect(th2 < F(0.0025), 1)) {  // |w| < 0.05
    const F k1 = tr ? F(0.5) : F(1), g1 = tr ? F(1.0 / 6.0) : F(0.5);
    const F k2 = tr ? F(1.0 / 24.0) : F(1.0 / 6.0), g2 = tr ? F(1.0 / 120.0) : F(1.0 / 24.0);
    const F k3 = tr ? F(1.0 / 30.0) : F(1.0 / 20.0), g3 = tr ? F(1.0 / 42.0) : F(1.0 / 30.0);
    if constexpr (sizeof(F) == 4) {
      be = fma(-th2 * k2, fma(-th2, k3, F(1)), k1);
      ga = fma(-th2 * g2, fma(-th2, g3, F(1)), g1);
    } else {  // through th^8: truncation below 1e-20
      const F k4 = tr ? F(1.0 / 56.0) : F(1.0 / 42.0), g4 = tr ? F(1.0 / 72.0) : F(1.0 / 56.0);
      const F k5 = tr ? F(1.0 / 90.0) : F(1.0 / 72.0), g5 = tr ? F(1.0 / 110.0) : F(1.0 / 90.0);
      be = fma(-th2 * k2, fma(-th2 * k3, fma(-th2 * k4, fma(-th2, k5, F(1)), F(1)), F(1)), k1);
      ga = fma(-th2 * g2, fma(-th2 * g3, fma(-th2 * g4, fma(-th2, g5, F(1)), F(1)), F(1)), g1);
    }
  } else {
    const F th = sqrt(th2);
    const F sn = sin(th), sh = sin(F(0.5) * th);
    const F A = sn / th, B = F(2) * sh * sh / th2, C = (th - sn) / (th2 * th);
    be = tr ? B : A, ga = tr ? C : B;
  }
  const F al = fma(-ga, th2, F(1)), gd = ga * fma(w0, q0, fma(w1, q1, w2 * q2));
  const F e0 = fma(al, q0, fma(be, fma(w1, q2, -(w2 * q1)), gd * w0));
  const F e1 = fma(al, q1, fma(be, fma(w2, q0, -(w0 * q2)), gd * w1));
  const F e2 = fma(al, q2, fma(be, fma(w0, q1, -(w1 * q0)), gd * w2));
  return fma(quad_bcast<0>(T), e0, fma(quad_bcast<1>(T), e1, fma(quad_bcast<2>(T), e2, tr ? T : F(0))));
}

// Every element of a pose held across the lanes, in every lane.
__device__ __forceinline__ void spread_pose(float Tl, float (&T)[12]) {
  T[0] = row_bcast<0>(Tl), T[1] = row_bcast<1>(Tl), T[2] = row_bcast<2>(Tl), T[3] = row_bcast<3>(Tl);
  T[4] = row_bcast<4>(Tl), T[5] = row_bcast<5>(Tl), T[6] = row_bcast<6>(Tl), T[7] = row_bcast<7>(Tl);
  T[8] = row_bcast<8>(Tl), T[9] = row_bcast<9>(Tl), T[10] = row_bcast<10>(Tl), T[11] = row_bcast<11>(Tl);
}

// One map point's IC cache (K = 8) held in registers across the iterations of
// a level: the reference-camera point x0, template intensities and gradients.
struct PointRegs {
  float X0, Y0, Z0;
  float iz, xp, yp;  // 1/Z0, X0/Z0, Y0/Z0 for the warp Jacobian
  float i0_[8], gx_[8], gy_[8];
  bool ok;
  __device__ __forceinline__ float i0(int k) const { return i0_[k]; }
  __device__ __forceinline__ float gx(int k) const { return gx_[k]; }
  __device__ __forceinline__ float gy(int k) const { return gy_[k]; }
};

// Mixed-precision variant: template intensity (minus 128) and gradients in FP16,
// 12 registers per point instead of 24.
struct PointRegsH {
  float X0, Y0, Z0;
  __half i0_[8];
  __half2 g_[8];
  bool ok;
  __device__ __forceinline__ float i0(int k) const { return __half2float(i0_[k]) + 128.0f; }
  __device__ __forceinline__ float gx(int k) const { return __low2float(g_[k]); }
  __device__ __forceinline__ float gy(int k) const { return __high2float(g_[k]); }
};

// Half of a point's 8-sample cache, for kernels that give each point two
// threads: samples 4 sub .. 4 sub + 3 of thread `sub` of the pair.
struct PointRegs4 {
  float X0, Y0, Z0;
  float i0_[4], gx_[4], gy_[4];
  bool ok;
  __device__ __forceinline__ float i0(int k) const { return i0_[k]; }
  __device__ __forceinline__ float gx(int k) const { return gx_[k]; }
  __device__ __forceinline__ float gy(int k) const { return gy_[k]; }
};

struct PointRegsH4 {
  float X0, Y0, Z0;
  __half i0_[4];
  __half2 g_[4];
  bool ok;
  __device__ __forceinline__ float i0(int k) const { return __half2float(i0_[k]) + 128.0f; }
  __device__ __forceinline__ float gx(int k) const { return __low2float(g_[k]); }
  __device__ __forceinline__ float gy(int k) const { return __high2float(g_[k]); }
};

// A load through a generic pointer into device memory, issued as a global
// (not flat) load: a flat load also counts on the LDS counter, so the next
// wait for LDS data would wait for it as well.
// The value moves as a plain word or word vector: HIP's vector structs copy
// through a generic reference, which would turn the load back into a flat one.
template <class T>
__device__ __forceinline__ T gload(const T* p) {
  static_assert(sizeof(T) == 1 || sizeof(T) == 4 || sizeof(T) == 8 || sizeof(T) == 16, "word or word vector");
  using W = typename std::conditional<
      sizeof(T) == 1, uint8_t,
      typename std::conditional<sizeof(T) == 4, uint32_t,
                                typename std::conditional<sizeof(T) == 8, uint32_t __attribute__((ext_vector_type(2))),
                                                          uint32_t __attribute__((ext_vector_type(4)))>::type>::type>::type;
  const W w = *(const __attribute__((address_space(1))) W*)p;
  T t;
  __builtin_memcpy(&t, &w, sizeof(T));
  return t;
}

// Load point i's registers for level l.  Branch-free: a point past the map
// (i >= n) reads entry 0 instead, and the geometry of an unusable point is
// selected to finite values (its warp Jacobian multiplies masked zeros); the
// template registers of such a point reach only sums that are selected away.
// The cache arrays hold at least one entry per level, so every read is inside.
__device__ __forceinline__ bool load_geometry(const TrackArgs& a, int l, int i, float4& p, int64_t& e) {
  const int64_t lo = (int64_t)l * a.ref.cap;
  const bool in = i < a.ref.n;
  const int j = in ? i : 0;
  e = lo + j;
  p = gload(a.ref.x0 + j);
  return in & (gload(a.ref.valid + e) != 0);
}

__device__ __forceinline__ void set_geometry(PointRegs& pr, bool ok, const float4& p) {
  pr.ok = ok;
  const float iz = 1.0f / p.z;
  pr.X0 = ok ? p.x : 0.0f;
  pr.Y0 = ok ? p.y : 0.0f;
  pr.Z0 = ok ? p.z : 1.0f;
  pr.iz = ok ? iz : 0.0f;
  pr.xp = ok ? p.x * iz : 0.0f;
  pr.yp = ok ? p.y * iz : 0.0f;
}

// The template registers of cache entry e: all 8 samples, or (PR4 variants)
// the four of thread `sub` of the point's pair.
__device__ __forceinline__ void load_template(const TrackArgs& a, int64_t e, int, PointRegs& pr) {
  const float4* q0 = reinterpret_cast<const float4*>(a.ref.I0 + e * 8);
  const float4* qx = reinterpret_cast<const float4*>(a.ref.gx + e * 8);
  const float4* qy = reinterpret_cast<const float4*>(a.ref.gy + e * 8);
  const float4 a0 = gload(q0), a1 = gload(q0 + 1), b0 = gload(qx), b1 = gload(qx + 1), c0 = gload(qy),
               c1 = gload(qy + 1);
  const float t0[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
  const float t1[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
  const float t2[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
#pragma unroll
  for (int k = 0; k < 8; ++k) pr.i0_[k] = t0[k], pr.gx_[k] = t1[k], pr.gy_[k] = t2[k];
}

__device__ __forceinline__ void load_template(const TrackArgs& a, int64_t e, int sub, PointRegs4& pr) {
  const float4 a0 = gload(reinterpret_cast<const float4*>(a.ref.I0 + e * 8) + sub);
  const float4 b0 = gload(reinterpret_cast<const float4*>(a.ref.gx + e * 8) + sub);
  const float4 c0 = gload(reinterpret_cast<const float4*>(a.ref.gy + e * 8) + sub);
  pr.i0_[0] = a0.x, pr.i0_[1] = a0.y, pr.i0_[2] = a0.z, pr.i0_[3] = a0.w;
  pr.gx_[0] = b0.x, pr.gx_[1] = b0.y, pr.gx_[2] = b0.z, pr.gx_[3] = b0.w;
  pr.gy_[0] = c0.x, pr.gy_[1] = c0.y, pr.gy_[2] = c0.z, pr.gy_[3] = c0.w;
}

__device__ __forceinline__ void load_template(const TrackArgs& a, int64_t e, int sub, PointRegsH4& pr) {
  const uint2 h = gload(reinterpret_cast<const uint2*>(a.ref.I0h + e * 8) + sub);
  const uint4 g = gload(reinterpret_cast<const uint4*>(a.ref.gh + e * 8) + sub);
  const uint32_t hw[2] = {h.x, h.y};
  const uint32_t gw[4] = {g.x, g.y, g.z, g.w};
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    pr.i0_[2 * k] = __ushort_as_half((unsigned short)(hw[k] & 0xffffu));
    pr.i0_[2 * k + 1] = __ushort_as_half((unsigned short)(hw[k] >> 16));
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    __half2 v;
    __builtin_memcpy(&v, &gw[k], 4);
    pr.g_[k] = v;
  }
}

__device__ __forceinline__ void load_template(const TrackArgs& a, int64_t e, int, PointRegsH& pr) {
  const uint4 h = gload(reinterpret_cast<const uint4*>(a.ref.I0h + e * 8));
  const uint4* q = reinterpret_cast<const uint4*>(a.ref.gh + e * 8);
  const uint4 g0 = gload(q), g1 = gload(q + 1);
  const uint32_t hw[4] = {h.x, h.y, h.z, h.w};
  const uint32_t gw[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    pr.i0_[2 * k] = __ushort_as_half((unsigned short)(hw[k] & 0xffffu));
    pr.i0_[2 * k + 1] = __ushort_as_half((unsigned short)(hw[k] >> 16));
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    __half2 v;
    __builtin_memcpy(&v, &gw[k], 4);
    pr.g_[k] = v;
  }
}

// Point i's registers for level l, one thread per point.
__device__ __forceinline__ void load_point(const TrackArgs& a, int l, int i, PointRegs& pr) {
  float4 p;
  int64_t e;
  const bool ok = load_geometry(a, l, i, p, e);
  set_geometry(pr, ok, p);
  load_template(a, e, 0, pr);
}

// The cooperative kernel's geometry of map point i, the same for every level
// and frame of a launch: X0, Y0, Z0 of pr.  A point past the map, behind the
// camera, not finite or with a Jacobian row that is not (|x / z| from 1.8e19 on,
// or 1 / z past FP32) becomes (0, 0, 1): no level holds it as valid, but the matrix
// products multiply every point's rows, by zero for an unusable one, and zero
// times infinity would reach the whole stream.  Returns whether the point can be
// valid; *j is its entry in a level's cache.
template <class PR>
__device__ __forceinline__ bool load_geometry_once(const TrackArgs& a, int i, PR& pr, int* j) {
  const bool in = i < a.ref.n;
  *j = in ? i : 0;
  const float4 p = gload(a.ref.x0 + *j);
  const float iz = 1.0f / p.z, xp = p.x * iz, yp = p.y * iz;
  // every entry of the rows (warp_rows) is at most one of these terms; NaN compares false
  const float rows = fmaf(xp, xp, 1.0f) + fmaf(yp, yp, 1.0f) + fabsf(xp * iz) + fabsf(yp * iz) + iz;
  const bool can = in && p.z > a.z_min && p.z < __builtin_inff() && fabsf(p.x) < __builtin_inff() &&
                   fabsf(p.y) < __builtin_inff() && rows < __builtin_inff();
  pr.X0 = can ? p.x : 0.0f;
  pr.Y0 = can ? p.y : 0.0f;
  pr.Z0 = can ? p.z : 1.0f;
  return can;
}

// Add one point's normal-equation terms (Eq.(2), Eq.(5)) at relative pose T.
// The K samples share the point's 2x6 warp Jacobian Jw with rows au, av, so with
// J_k = gx_k au + gy_k av:
//   H_i = m00 au^T au + m01 (au^T av + av^T au) + m11 av^T av,   b_i = -(v0 au + v1 av),
// m = sum_k w_k g_k^T g_k, v = sum_k w_k g_k r_k (five FMAs per sample, the
// 21-term product once per point).  Huber weight w = min(1, k/|r|).
// Branch-free: a point that is not usable (reference-invalid, behind the
// camera or a pattern position outside the level) runs the same instructions
// with its taps at the level's first pixels and its sums and counts masked to
// zero, so no exit path has to materialise a zeroed accumulator.
// `img` is the level in global memory or its copy in LDS.
__device__ __forceinline__ void accumulate_point(const TrackArgs& a, const PatRegs& pat, const LevelGeom& g,
                                                 const uint8_t* __restrict__ img, const float* T,
                                                 const PointRegs& pr, float (&acc)[32]) {
  const float kH = a.huber_k;
  float X, Y, Z;
  transform(T, pr.X0, pr.Y0, pr.Z0, X, Y, Z);
  float u, v;
  project(g, X, Y, Z, u, v);
  const bool ok = pr.ok & (Z > a.z_min) & inside(g, pat, u, v);
  // An unusable point continues from (0, 0): finite, integer sample positions
  // (zero bilinear fractions) and a tap offset forced to 0.
  u = ok ? u : 0.0f;
  v = ok ? v : 0.0f;
  // Phase 1: all 32 bilinear taps of the point are issued before any is used
  // (one memory round trip per point instead of one per sample).
  const Cell q0 = cell_of(u, v);
  float t00[8], t10[8], t01[8], t11[8];
  const int W = g.W;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int off = ((q0.iv + (int)pat.dy[k]) * W + q0.iu + (int)pat.dx[k]) & -(int)ok;  // masked, not branched
    const uint8_t* p = img + off;
    t00[k] = p[0], t10[k] = p[1], t01[k] = p[W], t11[k] = p[W + 1];
  }
  // Phase 2: residuals, Huber weights and the point's sums.  The interpolation
  // repeats the precompute's arithmetic exactly.
  float m00 = 0.f, m01 = 0.f, m11 = 0.f, v0 = 0.f, v1 = 0.f, E = 0.f;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const float Ic = bilin_mix(q0.w, t00[k], t10[k], t01[k], t11[k]);
    const float r = pr.i0(k) - Ic;
    const float ar = fabsf(r);
    const bool hub = (kH > 0.f) & (ar > kH);
    const float w = hub ? kH * __builtin_amdgcn_rcpf(ar) : 1.0f;  // v_rcp_f32, 1 ulp
    const float rho = hub ? kH * (ar - 0.5f * kH) : 0.5f * r * r;
    E += rho;
    const float gx = pr.gx(k), gy = pr.gy(k);
    const float wgx = w * gx, wgy = w * gy;
    m00 = fmaf(wgx, gx, m00);
    m01 = fmaf(wgx, gy, m01);
    m11 = fmaf(wgy, gy, m11);
    v0 = fmaf(wgx, r, v0);
    v1 = fmaf(wgy, r, v1);
  }
  acc[kSlotE] += ok ? E : 0.0f;
  acc[kSlotN] += ok ? 8.0f : 0.0f;
  acc[kSlotPts] += ok ? 1.0f : 0.0f;
  v0 = ok ? v0 : 0.0f, v1 = ok ? v1 : 0.0f;
  const float iz = pr.iz, xp = pr.xp, yp = pr.yp;
  const float au[6] = {-g.fx * xp * yp, g.fx * fmaf(xp, xp, 1.0f), -g.fx * yp, g.fx * iz, 0.0f, -g.fx * xp * iz};
  const float av[6] = {-g.fy * fmaf(yp, yp, 1.0f), g.fy * xp * yp, g.fy * xp, 0.0f, g.fy * iz, -g.fy * yp * iz};
  m00 = ok ? m00 : 0.0f, m01 = ok ? m01 : 0.0f, m11 = ok ? m11 : 0.0f;
  int q = 0;
#pragma unroll
  for (int r = 0; r < 6; ++r) {
    const float ma = fmaf(m00, au[r], m01 * av[r]);
    const float mc = fmaf(m01, au[r], m11 * av[r]);
#pragma unroll
    for (int c = r; c < 6; ++c) {
      acc[q] = fmaf(ma, au[c], fmaf(mc, av[c], acc[q]));
      ++q;
    }
    acc[kSlotB + r] -= fmaf(au[r], v0, av[r] * v1);
  }
}

// ---------------------------------------------------------------- LDS-staged accumulation (K = 8)

// Two neighbouring pixels, read in one go from any address.
template <class PIX>
struct __attribute__((packed)) PixPair {
  uint16_t w;
  __device__ __forceinline__ void load(const __attribute__((address_space(1))) PIX* p) {
    w = ((const __attribute__((address_space(1))) PixPair*)p)->w;
  }
  __device__ __forceinline__ float left() const { return (float)(w & 0xffu); }
  __device__ __forceinline__ float right() const { return (float)(w >> 8); }
};
template <>
struct __attribute__((packed)) PixPair<float> {
  float a, b;
  __device__ __forceinline__ void load(const __attribute__((address_space(1))) float* p) { a = p[0], b = p[1]; }
  __device__ __forceinline__ float left() const { return a; }
  __device__ __forceinline__ float right() const { return b; }
};

// The bytes of the current level a workgroup holds in LDS: rows lo..hi
// (inclusive), each W bytes, byte (r, x) of the level at offset
// delta + (r - lo) * W + x.  spans: the allocation is long enough for a pattern of
// the level whose first row is the tile's.
struct Tile8 {
  const __attribute__((address_space(3))) uint8_t* lds;
  int lo, hi, delta;
  bool spans;
};

// Byte offset in the level of the pattern's sample k relative to its base
// pixel: dy_k * W + dx_k, the same for every point of the level.
__device__ __forceinline__ void pattern_offsets(const PatRegs& pat, int W, int (&off)[8]) {
#pragma unroll
  for (int k = 0; k < 8; ++k) off[k] = (int)pat.dy[k] * W + (int)pat.dx[k];
}

// The scalar track parameters an iteration reads, copied to registers once
// per launch: the cooperative kernel keeps its TrackArgs in LDS, where a field
// read after a workgroup barrier is an LDS round trip on the iteration's path.
struct IterParams {
  float huber_k, z_min, step_eps;
  int max_iters, min_points;
  __device__ explicit IterParams(const TrackArgs& a)
      : huber_k(a.huber_k), z_min(a.z_min), step_eps(a.step_eps), max_iters(a.max_iters), min_points(a.min_points) {}
};

// What a thread's samples of its point sum to at a pose: m = sum w g^T g, v =
// sum w g r and the cost, and whether the point is usable there (else the sums
// are zero).
struct PointSums {
  float m00, m01, m11, v0, v1, E;
  bool ok;
};

// The sums of a point's samples with their templates in registers (Eq.(2),
// Eq.(5)), with the taps read from the workgroup's LDS copy of the level where
// every point of the wave lies inside it (else from global memory, as
// accumulate_point).  The pattern offsets are whole pixels, so all samples share
// the point's bilinear fractions: the weights are formed once per point.  Branch-free: an unusable
// point (reference-invalid, behind the camera or a pattern position outside the
// level) runs the same instructions and its sums are selected to zero.  Taps
// from global memory are read two pixels at a time, all of a batch in flight
// (one at a time: 397 against 386 us for a window of 9 frames).
// COST_ONLY: only the cost (the final pass).  Otherwise m and v, no cost (it is
// read only after the final pass).  FIXED: no weights, v only.
//
// The point has one thread (all 8 samples), two (NS = 4, each taking four of the
// samples with their offsets `off`) or, for other patterns, four (NS = 13 or 7
// slots, of which the lane fills `filled`); the point's sums are its threads'
// added.  A slot past `filled` has a zero gradient and repeats a sample of the
// pattern, so only the cost has to leave it out.  PIX: uint8 levels or the
// floating-point Gaussian pyramid.
template <bool COST_ONLY, bool FIXED, class PIX, int NS, class PR>
__device__ __forceinline__ PointSums sample_point(const IterParams& a, const PatRegs& pat, const int* off,
                                                  const LevelGeom& g, const PIX* __restrict__ img, const Tile8& tile,
                                                  const float* T, const PR& pr, int filled = NS) {
  constexpr bool BYTES = std::is_same<PIX, uint8_t>::value;
  constexpr bool QUAD = NS != 8 && NS != 4;
  const float kH = FIXED ? 0.0f : a.huber_k;
  // Huber weight min(1, k / |r|); without a threshold every weight is 1
  const float kHw = kH > 0.0f ? kH : __builtin_inff();
  float X, Y, Z;
  transform(T, pr.X0, pr.Y0, pr.Z0, X, Y, Z);
  float u, v;
  project(g, X, Y, Z, u, v);
  const bool ok = pr.ok & (Z > a.z_min) & inside(g, pat, u, v);
  u = ok ? u : 0.0f;
  v = ok ? v : 0.0f;
  const Cell q0 = cell_of(u, v);
  const int iu = q0.iu, iv = q0.iv, W = g.W;
  // Every usable point of the wave inside the tile?  An unusable one reads from
  // the tile position of a pattern whose top-left sample sits at the tile's first
  // byte, masked below; where the small tile is too short for that (8 samples 32
  // rows apart at a width of 2000, never the default pattern), and so holds no usable
  // point either, every point reads global memory.  Other patterns' unusable points
  // read the tile's first bytes.
  const bool in_tile = !ok | ((iv + (int)pat.dy_min >= tile.lo) & (iv + (int)pat.dy_max + 1 <= tile.hi));
  const bool use_tile = (QUAD || tile.spans) && __all(in_tile);
  PointSums s = {};
  s.ok = ok;
  // Up to eight samples at a time: all their taps are requested before any is
  // used (one LDS round trip); 13 at once would not fit the registers.
  constexpr int B = NS > 8 ? 7 : NS;
#pragma unroll
  for (int k0 = 0; k0 < NS; k0 += B) {
    float t00[B], t10[B], t01[B], t11[B];
    if (use_tile) {
      const int lb = (int)(uint32_t)(uintptr_t)tile.lds;
      const int lbase = lb + tile.delta +
                        (int)sizeof(PIX) * (ok ? (iv - tile.lo) * W + iu : -((int)pat.dy_min * W + (int)pat.dx_min));
      const int Wt = QUAD && !ok ? 0 : W;
      if constexpr (BYTES) {
        uint32_t w[B][4];
        int bt[B];
#pragma unroll
        for (int k = 0; k < B; ++k) {
          if (k0 + k >= NS) continue;
          bt[k] = QUAD && !ok ? lb : lbase + off[k0 + k];
          const __attribute__((address_space(3))) uint32_t* p =
              (const __attribute__((address_space(3))) uint32_t*)(uintptr_t)(uint32_t)(bt[k] & ~3);
          const __attribute__((address_space(3))) uint32_t* q =
              (const __attribute__((address_space(3))) uint32_t*)(uintptr_t)(uint32_t)((bt[k] + Wt) & ~3);
          w[k][0] = p[0], w[k][1] = p[1], w[k][2] = q[0], w[k][3] = q[1];
        }
#pragma unroll
        for (int k = 0; k < B; ++k) {
          if (k0 + k >= NS) continue;
          const uint32_t top = __builtin_amdgcn_alignbyte(w[k][1], w[k][0], (uint32_t)bt[k]);
          const uint32_t bot = __builtin_amdgcn_alignbyte(w[k][3], w[k][2], (uint32_t)(bt[k] + Wt));
          t00[k] = (float)(top & 0xffu), t10[k] = (float)((top >> 8) & 0xffu);
          t01[k] = (float)(bot & 0xffu), t11[k] = (float)((bot >> 8) & 0xffu);
        }
      } else {
#pragma unroll
        for (int k = 0; k < B; ++k) {
          if (k0 + k >= NS) continue;
          const __attribute__((address_space(3))) float* p =
              (const __attribute__((address_space(3))) float*)(uintptr_t)(uint32_t)(ok ? lbase + 4 * off[k0 + k] : lb);
          t00[k] = p[0], t10[k] = p[1], t01[k] = p[Wt], t11[k] = p[Wt + 1];
        }
      }
    } else {
      const __attribute__((address_space(1))) PIX* gimg = (const __attribute__((address_space(1))) PIX*)img;
      const int gbase = iv * W + iu;
      PixPair<PIX> r[B][2];
#pragma unroll
      for (int k = 0; k < B; ++k) {
        if (k0 + k >= NS) continue;
        const uint32_t o = ok ? gbase + off[k0 + k] : 0, q = o + W;  // an unusable point: the level's first pixels
        r[k][0].load(gimg + o), r[k][1].load(gimg + q);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < B; ++k) {
        if (k0 + k >= NS) continue;
        t00[k] = r[k][0].left(), t10[k] = r[k][0].right(), t01[k] = r[k][1].left(), t11[k] = r[k][1].right();
      }
    }
#pragma unroll
    for (int kk = 0; kk < B; ++kk) {
      const int k = k0 + kk;
      if (k >= NS) continue;
      const float Ic = bilin_mix(q0.w, t00[kk], t10[kk], t01[kk], t11[kk]);
      const float r = pr.i0(k) - Ic;
      if constexpr (COST_ONLY) {
        const float ar = fabsf(r);
        const bool hub = (kH > 0.f) & (ar > kH);
        const float rho = hub ? kH * (ar - 0.5f * kH) : 0.5f * r * r;
        s.E += k < filled ? rho : 0.0f;
      } else {
        const float gx = pr.gx(k), gy = pr.gy(k);
        if constexpr (FIXED) {
          s.v0 = fmaf(gx, r, s.v0);
          s.v1 = fmaf(gy, r, s.v1);
        } else {
          const float w = fminf(1.0f, kHw * __builtin_amdgcn_rcpf(fabsf(r)));
          const float wgx = w * gx, wgy = w * gy;
          s.m00 = fmaf(wgx, gx, s.m00);
          s.m01 = fmaf(wgx, gy, s.m01);
          s.m11 = fmaf(wgy, gy, s.m11);
          s.v0 = fmaf(wgx, r, s.v0);
          s.v1 = fmaf(wgy, r, s.v1);
        }
      }
    }
  }
  if constexpr (COST_ONLY) {
    s.E = ok ? s.E : 0.0f;
  } else {
    s.v0 = ok ? s.v0 : 0.0f, s.v1 = ok ? s.v1 : 0.0f;
    if constexpr (!FIXED) s.m00 = ok ? s.m00 : 0.0f, s.m01 = ok ? s.m01 : 0.0f, s.m11 = ok ? s.m11 : 0.0f;
  }
  return s;
}

// ---------------------------------------------------------------- generic-K cooperative accumulation

// Patterns other than the 8-pixel one (p x p patches) and the floating-point
// pyramid: four lanes share a point, lane `sub` of the quad taking samples
// sub, sub + 4, ... < K, so a 49-sample patch costs each lane 13 samples.
struct PointGeo {
  float X0, Y0, Z0;
  int64_t s0;  // cache index of the point's sample 0 at the level
  bool ok;
};

// Patterns of up to 4 x kQuadSlots samples keep their templates in registers
// like the 8-pixel one: slot j of lane `sub` is sample sub + 4 j, a slot past
// the pattern has zero gradients.  Reading them again in every iteration put 91
// loads per lane of a 7x7 patch on the address units, the path's bound; with
// templates in registers and taps in LDS the track of 2000 7x7 points at 752x480
// went from 191 to 153 us, of a 5x5-patch window of 9 frames from 771 to 594 us.
// 13 slots (K <= 52) are what fits beside the loop's own state without spills
// inside it.
constexpr int kQuadSlots = 13;
struct PointRegsQ {
  float X0, Y0, Z0;
  float i0_[kQuadSlots], gx_[kQuadSlots], gy_[kQuadSlots];
  bool ok;
  __device__ __forceinline__ float i0(int k) const { return i0_[k]; }
  __device__ __forceinline__ float gx(int k) const { return gx_[k]; }
  __device__ __forceinline__ float gy(int k) const { return gy_[k]; }
};

__device__ __forceinline__ void load_template(const TrackArgs& a, int64_t e, int sub, PointRegsQ& pr) {
  const int K = a.pat.K;
#pragma unroll
  for (int j = 0; j < kQuadSlots; ++j) {
    const int k = sub + kLanesPerPoint * j;
    const int64_t o = e * K + (k < K ? k : 0);
    pr.i0_[j] = gload(a.ref.I0 + o), pr.gx_[j] = gload(a.ref.gx + o), pr.gy_[j] = gload(a.ref.gy + o);
  }
#pragma unroll
  for (int j = 0; j < kQuadSlots; ++j) {
    const bool has = sub + kLanesPerPoint * j < K;
    pr.gx_[j] = has ? pr.gx_[j] : 0.0f, pr.gy_[j] = has ? pr.gy_[j] : 0.0f;
  }
}

// Their pixel offsets at a level of width W (a slot past the pattern: sample 0).
__device__ __forceinline__ void quad_offsets(const Pattern& pat, int W, int sub, int (&off)[kQuadSlots]) {
#pragma unroll
  for (int j = 0; j < kQuadSlots; ++j) {
    const int k = sub + kLanesPerPoint * j, kk = k < pat.K ? k : 0;
    off[j] = (int)pat.dy[kk] * W + (int)pat.dx[kk];
  }
}

// DPP quad permutation (quad_perm selector), a VALU operand modifier.
template <int SEL>
__device__ __forceinline__ float dpp_quad(float v) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), SEL, 0xf, 0xf, false));
}

// Sum over the four lanes of a quad, the same in every lane of it.
__device__ __forceinline__ float quad_sum(float v) {
  v += dpp_quad<0xB1>(v);  // lanes [1, 0, 3, 2]
  v += dpp_quad<0x4E>(v);  // lanes [2, 3, 0, 1]
  return v;
}

// Sums over the quad's lanes, the same in each.
template <bool COST_ONLY, bool FIXED>
__device__ __forceinline__ void quad_sums(PointSums& s) {
  if constexpr (COST_ONLY) {
    s.E = quad_sum(s.E);
  } else {
    s.v0 = quad_sum(s.v0), s.v1 = quad_sum(s.v1);
    if constexpr (!FIXED) s.m00 = quad_sum(s.m00), s.m01 = quad_sum(s.m01), s.m11 = quad_sum(s.m11);
  }
}

// sample_point for patterns past the register slots, this lane's share of the
// quad's point: taps and templates from global memory.
template <bool COST_ONLY, bool FIXED, class PIX>
__device__ __forceinline__ PointSums sample_point_generic(const TrackArgs& a, const Pattern& pat, const LevelGeom& g,
                                                          const PIX* __restrict__ img, const float* T,
                                                          const PointGeo& pg, int sub) {
  const float kH = FIXED ? 0.0f : a.huber_k;
  float X, Y, Z;
  transform(T, pg.X0, pg.Y0, pg.Z0, X, Y, Z);
  float u, v;
  project(g, X, Y, Z, u, v);
  const bool ok = pg.ok & (Z > a.z_min) & inside(g, pat, u, v);
  u = ok ? u : 0.0f;
  v = ok ? v : 0.0f;
  const Cell q0 = cell_of(u, v);
  const int K = pat.K, W = g.W;
  const __attribute__((address_space(1))) PIX* gimg = (const __attribute__((address_space(1))) PIX*)img;
  PointSums s = {};
  s.ok = ok;
  // Batches of four samples per lane: all their taps and cache entries are
  // issued before any is used (the barriers keep it so: left to itself the compiler
  // waits for each sample's taps, 262 instead of 192 us for five iterations of 1500
  // 11x11 patches over four levels).  A slot past the pattern reads sample 0 (always
  // in range) and is weighted by zero.
  constexpr int B = 4;
  for (int k0 = sub; k0 < K; k0 += B * kLanesPerPoint) {
    float t00[B], t10[B], t01[B], t11[B], i0[B], gxs[B], gys[B], msk[B];
    uint32_t off[B];
    PixPair<PIX> top[B], bot[B];
#pragma unroll
    for (int j = 0; j < B; ++j) {
      const int k = k0 + j * kLanesPerPoint;
      const bool has = k < K;
      const int kk = has ? k : 0;
      msk[j] = has ? 1.0f : 0.0f;
      // an unusable point reads the level's first taps
      off[j] = (uint32_t)(((q0.iv + (int)pat.dy[kk]) * W + q0.iu + (int)pat.dx[kk]) & -(int)ok);
      i0[j] = gload(a.ref.I0 + pg.s0 + kk);
      if (!COST_ONLY) gxs[j] = gload(a.ref.gx + pg.s0 + kk), gys[j] = gload(a.ref.gy + pg.s0 + kk);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < B; ++j) top[j].load(gimg + off[j]), bot[j].load(gimg + (off[j] + W));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < B; ++j)
      t00[j] = top[j].left(), t10[j] = top[j].right(), t01[j] = bot[j].left(), t11[j] = bot[j].right();
#pragma unroll
    for (int j = 0; j < B; ++j) {
      const float Ic = bilin_mix(q0.w, t00[j], t10[j], t01[j], t11[j]);
      const float r = i0[j] - Ic;
      const float ar = fabsf(r);
      const bool hub = (kH > 0.f) & (ar > kH);
      const float w = (hub ? kH * __builtin_amdgcn_rcpf(ar) : 1.0f) * msk[j];
      const float rho = hub ? kH * (ar - 0.5f * kH) : 0.5f * r * r;
      s.E = fmaf(msk[j], rho, s.E);
      if (!COST_ONLY) {
        const float wgx = w * gxs[j], wgy = w * gys[j];
        if (!FIXED) {
          s.m00 = fmaf(wgx, gxs[j], s.m00);
          s.m01 = fmaf(wgx, gys[j], s.m01);
          s.m11 = fmaf(wgy, gys[j], s.m11);
        }
        s.v0 = fmaf(wgx, r, s.v0);
        s.v1 = fmaf(wgy, r, s.v1);
      }
    }
  }
  if constexpr (COST_ONLY) {
    s.E = ok ? s.E : 0.0f;
  } else {
    s.v0 = ok ? s.v0 : 0.0f, s.v1 = ok ? s.v1 : 0.0f;
    if constexpr (!FIXED) s.m00 = ok ? s.m00 : 0.0f, s.m01 = ok ? s.m01 : 0.0f, s.m11 = ok ? s.m11 : 0.0f;
  }
  return s;
}

// ---------------------------------------------------------------- normal equations on the matrix cores

// The warp Jacobian of a point at x0 for unit focal lengths: rows ju, jv over
// the twist (omega, v), Eq.(6).  They depend on the map alone, not on level or
// pose: a level's focal lengths scale m and v instead.
__device__ __forceinline__ void warp_rows(float X, float Y, float Z, float (&ju)[6], float (&jv)[6]) {
  const float iz = 1.0f / Z, xp = X * iz, yp = Y * iz;
  ju[0] = -xp * yp, ju[1] = fmaf(xp, xp, 1.0f), ju[2] = -yp, ju[3] = iz, ju[4] = 0.0f, ju[5] = -xp * iz;
  jv[0] = -fmaf(yp, yp, 1.0f), jv[1] = xp * yp, jv[2] = xp, jv[3] = 0.0f, jv[4] = iz, jv[5] = -yp * iz;
}

// A quad's P points (4, 2 or 1 threads' worth: 1, 2 or 4 threads per point) with
// their Jacobian rows laid out for the 4x4x1 matrix product: lane q of the quad
// holds components q (low) and 4 + q (high) of every point's two rows.  The
// high components past 5 are the row that counts points: 1 in u, 0 in v, and 0.
template <int P>
struct QuadRows {
  float ul[P], uh[P], vl[P], vh[P];
};

template <int P, int I>
__device__ __forceinline__ void quad_rows_of(const float (&ju)[6], const float (&jv)[6], QuadRows<P>& r) {
  constexpr int S = I * (4 / P);  // the quad lane that holds point I
  const int q = threadIdx.x & 3;
  const auto pick = [&](float a, float b, float c, float d) { return q == 0 ? a : q == 1 ? b : q == 2 ? c : d; };
  r.ul[I] = pick(quad_bcast<S>(ju[0]), quad_bcast<S>(ju[1]), quad_bcast<S>(ju[2]), quad_bcast<S>(ju[3]));
  r.uh[I] = pick(quad_bcast<S>(ju[4]), quad_bcast<S>(ju[5]), 1.0f, 0.0f);
  r.vl[I] = pick(quad_bcast<S>(jv[0]), quad_bcast<S>(jv[1]), quad_bcast<S>(jv[2]), quad_bcast<S>(jv[3]));
  r.vh[I] = pick(quad_bcast<S>(jv[4]), quad_bcast<S>(jv[5]), 0.0f, 0.0f);
  if constexpr (I + 1 < P) quad_rows_of<P, I + 1>(ju, jv, r);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Add point I of the quad: D += A B with A = J (rows u and v, one product each)
// and B = (M J | -v | count), in three 4x4 blocks: low x low, low x high, high x
// high of the 8 x 8 product (H is symmetric).
template <int P, int I>
__device__ __forceinline__ void quad_products(const QuadRows<P>& r, float m00, float m01, float m11, float v0, float v1,
                                              float cnt, f32x4 (&D)[3]) {
  constexpr int S = I * (4 / P);
  const int q = threadIdx.x & 3;
  const auto at = [](float v) {
    if constexpr (P == 1) return v;
    return quad_bcast<S>(v);
  };
  const float a00 = at(m00), a01 = at(m01), a11 = at(m11), b0 = at(v0), b1 = at(v1), n = at(cnt);
  const float lu = fmaf(a01, r.vl[I], a00 * r.ul[I]), lv = fmaf(a11, r.vl[I], a01 * r.ul[I]);
  float hu = fmaf(a01, r.vh[I], a00 * r.uh[I]), hv = fmaf(a11, r.vh[I], a01 * r.uh[I]);
  hu = q == 2 ? -b0 : q == 3 ? n : hu;
  hv = q == 2 ? -b1 : hv;
  D[0] = __builtin_amdgcn_mfma_f32_4x4x1f32(r.ul[I], lu, D[0], 0, 0, 0);
  D[1] = __builtin_amdgcn_mfma_f32_4x4x1f32(r.ul[I], hu, D[1], 0, 0, 0);
  D[2] = __builtin_amdgcn_mfma_f32_4x4x1f32(r.uh[I], hu, D[2], 0, 0, 0);
  D[0] = __builtin_amdgcn_mfma_f32_4x4x1f32(r.vl[I], lv, D[0], 0, 0, 0);
  D[1] = __builtin_amdgcn_mfma_f32_4x4x1f32(r.vl[I], hv, D[1], 0, 0, 0);
  D[2] = __builtin_amdgcn_mfma_f32_4x4x1f32(r.vh[I], hv, D[2], 0, 0, 0);
  if constexpr (I + 1 < P) quad_products<P, I + 1>(r, m00, m01, m11, v0, v1, cnt, D);
}

// The quads' normal equations summed over the wave: register 4 k + i of lane q
// (of any quad) is element (i, q) of block k of the quad's product.  On return
// d[j], j < 3, in the lanes of 16-lane row r holds register 6 (r / 2) + 3 (r % 2)
// + j summed over the wave's quads, column q = lane % 4.  Twelve values meet by
// lane swaps and row rotations, where 28 sums held one per thread took three
// times the steps.
__device__ __forceinline__ void wave_reduce12(float (&d)[12]) {
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(d[j]), __float_as_uint(d[j + 6]), false, false);
    d[j] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(d[j]), __float_as_uint(d[j + 3]), false, false);
    float v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    v += dpp_ror<8>(v);
    v += dpp_ror<4>(v);
    d[j] = v;
  }
}

// Words of a wave's partial sums in LDS: 12 registers x 4 columns in the robust
// mode, and where reduction slot v (H, b, the point count) lies among them.
constexpr int kWaveWords = 48;
__device__ __forceinline__ int wave_word(int v) {
  const int r = (v >= 6) + (v >= 11) + (v >= 15) + (v >= 18) + (v >= 20);
  int i = r, c = v - (6 * r - r * (r - 1) / 2) + r;  // H(i, c)
  if (v >= kSlotB) i = v - kSlotB, c = 6;            // b_i
  if (v >= kSlotE) i = 6, c = 7;                     // the count (slots without a value read it too)
  const int blk = i < 4 ? (c < 4 ? 0 : 1) : 2;
  return 4 * (4 * blk + (i & 3)) + (c & 3);
}

// The wave totals of the final pass's three sums, in every lane.
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_ror<8>(v);
  v += dpp_ror<4>(v);
  v += dpp_ror<2>(v);
  v += dpp_ror<1>(v);
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

}  // namespace dpt
