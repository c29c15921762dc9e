// Map-point selection (stand-in for the map points the indirect pipeline
// provides): the n candidates with the largest integer gradient score
// s = (I[y][x+1] - I[y][x-1])^2 + (I[y+1][x] - I[y-1][x])^2 inside the margin,
// ties to the smaller linear index, written in ascending index order.
//
// Three launches:
//   A  histogram of s >> 9 (s <= 2 * 255^2 < 2^17), per workgroup in LDS, summed
//      into a global 256-bin histogram with integer atomics (order-independent)
//   B  every workgroup finds the coarse bucket of the n-th largest score with
//      one wave, then the 512-bin histogram of the low bits inside it
//   C  every workgroup finds the exact threshold T and how many ties `need` to
//      keep, counts its chunk's scores > T and == T, publishes both in one word,
//      sums the words of the chunks before it and writes its selected indices;
//      the last chunk writes the count
// Candidate c is pixel (m + c % Wc, m + c / Wc): candidate order is index order.
//
// A small image's launch is bound by its chain of latencies (image, histogram,
// atomics), a large or batched one by the scores' arithmetic and the atomics
// that flush the histograms; so scores are loaded before the histograms they are
// compared with are waited for, four at a time from four words (any alignment),
// and each is a packed difference and a dot product.  752x480: 5 + 6 + 5 + 11 us in
// four launches, now 4 + 5 + 8 in three; 2047x1535 (rows at any alignment): 8 + 21
// + 8 + 18, now 6 + 10 + 11; 64 images of 752x480: 15 + 23 + 19 + 34, now 16 + 15 +
// 31, the image being read from beyond the L2 caches once per launch.
#include <cstdint>
#include <cstring>
#include <mutex>

#include "dpt_device.h"

namespace dpt {

constexpr int kSelThreads = 256, kHistThreads = 1024;

// Candidates per chunk of the write pass, of which a thread has chunk / 256 and a
// wave a contiguous quarter.  A workgroup's time is mostly its chain of waits
// (image, threshold, counts, the words of the chunks before it): chunks of 1024
// where they fill the chip at least once (352 at 752x480, where 88 of 4096 would
// leave most of it idle), larger ones where the launch would have to start its
// workgroups in several turns (64 images of 752x480: 50 us with 5312 chunks of
// 4096, 43 with 1408 of 16384, 31 since a thread keeps bits and not scores).  `pixels`: of a launch's images together.
int select_chunk(int64_t pixels) { return pixels <= (1 << 20) ? 1024 : pixels <= (1 << 23) ? 4096 : 16384; }

// Layout of the int32 scratch buffer.  Between runs the coarse histogram is zero.
// A clears kHist2 and the chunks' words, B leaves the coarse bucket at kCoarse, C
// clears kHist1: each what no workgroup of its own launch reads.
struct SelScratch {
  static constexpr int kHist1 = 0, kHist2 = 256, kCoarse = 768, kChunks = 772;
};

// Ints of scratch for an image of W x H: its chunks in a launch of its own, which are its smallest.
int64_t select_scratch_ints(int32_t W, int32_t H) {
  const int64_t px = (int64_t)W * H, chunk = select_chunk(px);
  return SelScratch::kChunks + (px + chunk - 1) / chunk + 1;
}

__device__ __forceinline__ int sel_score(const uint8_t* img, int pitch, int x, int y) {
  const uint8_t* p = img + (int64_t)y * pitch + x;
  const int dx = (int)gload(p + 1) - (int)gload(p - 1);
  const int dy = (int)gload(p + pitch) - (int)gload(p - pitch);
  return dx * dx + dy * dy;
}

// Row and column of candidate c: the float quotient (c < 2^24 is exact, and
// the product's error is far below one row) corrected by at most one row.
__device__ __forceinline__ void cand_xy(const SelGeom& g, int c, int* x, int* y) {
  int r = (int)((float)c * g.inv_wc);
  int q = c - r * g.Wc;
  if (q < 0) {
    --r;
    q += g.Wc;
  } else if (q >= g.Wc) {
    ++r;
    q -= g.Wc;
  }
  *x = q;
  *y = r;
}

__device__ __forceinline__ int cand_score(const SelGeom& g, int c) {
  int x, y;
  cand_xy(g, c, &x, &y);
  return sel_score(g.img, g.pitch, g.m + x, g.m + y);
}

struct __attribute__((packed)) Word4 {
  uint32_t w;
};
__device__ __forceinline__ uint32_t load4(const uint8_t* p) {  // from any address
  return ((const __attribute__((address_space(1))) Word4*)p)->w;
}

// Byte K of lo and of hi as two 16-bit numbers.
template <int K>
__device__ __forceinline__ uint32_t byte_pair(uint32_t hi, uint32_t lo) {
  return __builtin_amdgcn_perm(hi, lo, 0x0c000c00u | (uint32_t)(4 + K) << 16 | (uint32_t)K);
}

typedef short sel_short2 __attribute__((ext_vector_type(2)));

// dx^2 + dy^2 of byte K: (right, down) - (left, up), squared and summed.
template <int K>
__device__ __forceinline__ int score_of(uint32_t left, uint32_t right, uint32_t up, uint32_t dn) {
  const sel_short2 d = __builtin_bit_cast(sel_short2, byte_pair<K>(dn, right)) -
                       __builtin_bit_cast(sel_short2, byte_pair<K>(up, left));
  return __builtin_amdgcn_sdot2(d, d, 0, false);
}

// Candidates c .. c + 3 of the image, loaded and then scored (-2 past the last
// one).  Four of one row take four words (pixel and right neighbours overlap the
// next group's); those that span a row's end are taken one by one.
struct Cand4 {
  uint32_t left, right, up, dn;
  bool words;
};

__device__ __forceinline__ Cand4 cand_load4(const SelGeom& g, int c) {
  Cand4 q = {};
  int x, y;
  cand_xy(g, c, &x, &y);
  q.words = (c < g.C) & (x + 3 < g.Wc);
  if (q.words) {
    const uint8_t* p = g.img + (int64_t)(g.m + y) * g.pitch + (g.m + x);
    q.left = load4(p - 1), q.right = load4(p + 1), q.up = load4(p - g.pitch), q.dn = load4(p + g.pitch);
  }
  return q;
}

__device__ __forceinline__ int4 cand_score4(const SelGeom& g, int c, const Cand4& q) {
  if (q.words)
    return make_int4(score_of<0>(q.left, q.right, q.up, q.dn), score_of<1>(q.left, q.right, q.up, q.dn),
                     score_of<2>(q.left, q.right, q.up, q.dn), score_of<3>(q.left, q.right, q.up, q.dn));
  int4 s = make_int4(-2, -2, -2, -2);
  if (c < g.C) s.x = cand_score(g, c);
  if (c + 1 < g.C) s.y = cand_score(g, c + 1);
  if (c + 2 < g.C) s.z = cand_score(g, c + 2);
  if (c + 3 < g.C) s.w = cand_score(g, c + 3);
  return s;
}

// f(score) for this thread's share of the image's candidates in a histogram
// launch: groups of four in steps of the launch, the next one being loaded while
// one is counted; `q` is the thread's first.
template <class F>
__device__ __forceinline__ void for_scores(const SelGeom& g, Cand4 q, F&& f) {
  const int step = 4 * (int)(gridDim.x * kHistThreads);
  for (int c = 4 * (int)(blockIdx.x * kHistThreads + threadIdx.x); c < g.C; c += step) {
    const Cand4 next = cand_load4(g, c + step);
    __builtin_amdgcn_sched_barrier(0);
    const int4 v = cand_score4(g, c, q);
    f(v.x), f(v.y), f(v.z), f(v.w);
    q = next;
  }
}

// The selection of one image (`one`), or of image blockIdx.y of a batch (`many`
// non-null): every kernel below runs over (chunks, images) and a workgroup past
// its image's chunk count returns at once.
__device__ __forceinline__ SelJob sel_job(const SelJob& one, const SelJob* many) {
  return many ? many[blockIdx.y] : one;
}

__global__ __launch_bounds__(kSelThreads) void sel_clear(SelJob one, const SelJob* many) {
  const SelJob j = sel_job(one, many);
  for (int b = threadIdx.x; b < SelScratch::kChunks; b += blockDim.x) j.sc[b] = 0;
  if (j.G == 0 && threadIdx.x == 0) *j.count = 0;  // no candidates: nothing selected
}

__global__ __launch_bounds__(kHistThreads) void sel_hist_coarse(SelJob one, const SelJob* many) {
  const SelJob j = sel_job(one, many);
  const SelGeom& g = j.g;
  if ((int)blockIdx.x * 4 * kHistThreads >= g.C) return;
  int* __restrict__ sc = j.sc;
  __shared__ int h[256];
  const int t = threadIdx.x, first = blockIdx.x * kHistThreads + t;
  const Cand4 q = cand_load4(g, 4 * first);
  if (t < 256) h[t] = 0;
  if (blockIdx.x == 0 && t < 512) sc[SelScratch::kHist2 + t] = 0;
  for (int k = first; k < j.G; k += gridDim.x * kHistThreads) sc[SelScratch::kChunks + k] = 0;
  __syncthreads();
  // bin 0 (scores below 512, most of a frame) is not counted: it is the
  // candidate total minus the other bins, which spares its atomics
  for_scores(g, q, [&](int sv) {
    const int b = sv >> 9;
    if (b > 0) atomicAdd(&h[b], 1);
  });
  __syncthreads();
  if (t < 256 && h[t]) atomicAdd(&sc[SelScratch::kHist1 + t], h[t]);
}

// One wave: the largest bin b with sum_{b' >= b} h[b'] >= n over NB bins
// (NB / 64 per lane), given `above` candidates already counted in higher bins.
// total >= 0: bin 0 is not stored and holds total minus the other bins.
// Returns b (or -1 if the total is short of n) and the count above b.
template <int NB>
__device__ __forceinline__ int2 wave_find_bin(const int* __restrict__ h, int n, int above, int total = -1) {
  constexpr int PB = NB / 64;
  const int lane = threadIdx.x & 63;
  int v[PB], t = 0;
#pragma unroll
  for (int j = 0; j < PB; ++j) t += (v[j] = gload(h + lane * PB + j));
  if (total >= 0) {
    int rest = t;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) rest += __shfl_xor(rest, d, 64);
    if (lane == 0) {
      v[0] = total - rest;
      t += v[0];
    }
  }
  // suffix sum over the lanes above this one
  int suf = t;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int y = __shfl_down(suf, d, 64);
    if (lane + d < 64) suf += y;
  }
  int cum = above + suf - t;  // candidates in bins above this lane's
  int found = -1, cum_at = 0;
  if (cum < n && cum + t >= n) {
#pragma unroll
    for (int j = PB - 1; j >= 0; --j) {
      if (found < 0 && cum + v[j] >= n) found = lane * PB + j, cum_at = cum;
      if (found < 0) cum += v[j];
    }
  }
  const unsigned long long hit = __ballot(found >= 0);
  if (hit == 0) return make_int2(-1, 0);
  const int src = __ffsll((long long)hit) - 1;
  return make_int2(__shfl(found, src, 64), __shfl(cum_at, src, 64));
}

// Coarse bucket B and the count above it (B = -1: take every candidate).
__device__ __forceinline__ int2 coarse_bucket(const SelGeom& g, const int* sc) {
  if (g.C <= g.n) return make_int2(-1, 0);
  return wave_find_bin<256>(sc + SelScratch::kHist1, g.n, 0, g.C);
}

__global__ __launch_bounds__(kHistThreads) void sel_hist_fine(SelJob one, const SelJob* many) {
  const SelJob j = sel_job(one, many);
  const SelGeom& g = j.g;
  if ((int)blockIdx.x * 4 * kHistThreads >= g.C) return;
  int* __restrict__ sc = j.sc;
  __shared__ int h[512];
  __shared__ int sB;
  const int t = threadIdx.x;
  const Cand4 q = cand_load4(g, 4 * (int)(blockIdx.x * kHistThreads + t));
  if (t < 64) {
    const int2 r = coarse_bucket(g, sc);
    if (t == 0) {
      sB = r.x;
      if (blockIdx.x == 0) sc[SelScratch::kCoarse] = r.x, sc[SelScratch::kCoarse + 1] = r.y;
    }
  }
  if (t < 512) h[t] = 0;
  __syncthreads();
  const int B = sB;
  if (B < 0) return;
  for_scores(g, q, [&](int sv) {
    if ((sv >> 9) == B) atomicAdd(&h[sv & 511], 1);
  });
  __syncthreads();
  if (t < 512 && h[t]) atomicAdd(&sc[SelScratch::kHist2 + t], h[t]);
}

// A chunk's word: valid, candidates above the threshold, ties at it.
__device__ __forceinline__ uint32_t chunk_word(int gt, int eq) { return 0x80000000u | (uint32_t)gt << 15 | (uint32_t)eq; }

// The word of chunk k, published by its workgroup in this launch.  Workgroups
// start in order, so those before this one are running or done; should one not
// publish for long all the same, its chunk is counted here instead: no wait
// without an end, whatever else runs on the device or in the scratch.
template <int CHUNK>
__device__ __forceinline__ uint32_t chunk_word_of(const SelGeom& g, int* sc, int k, int T) {
  uint32_t w = 0;
  for (int spin = 0; spin < 20000; ++spin) {
    w = (uint32_t)__hip_atomic_load(&sc[SelScratch::kChunks + k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (w) return w;
    __builtin_amdgcn_s_sleep(1);
  }
  int gt = 0, eq = 0;
  for (int c = k * CHUNK; c < (k + 1) * CHUNK && c < g.C; ++c) {
    const int sv = cand_score(g, c);
    gt += sv > T, eq += sv == T;
  }
  return chunk_word(gt, eq);
}

__device__ __forceinline__ int lanes_below(unsigned long long m, int add) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)add));
}

template <int CHUNK>
__global__ __launch_bounds__(kSelThreads, 6) void sel_write(SelJob one, const SelJob* many) {
  const SelJob j = sel_job(one, many);
  if ((int)blockIdx.x >= j.G) return;
  const SelGeom& g = j.g;
  int* __restrict__ sc = j.sc;
  constexpr int NW = kSelThreads / 64, R = CHUNK / (4 * kSelThreads);  // waves; groups of four per thread
  __shared__ int sT, sNeed, s_gt[NW], s_eq[NW], s_bgt[NW], s_beq[NW];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int c0 = (int)blockIdx.x * CHUNK + wave * (CHUNK / NW) + 4 * lane;
  constexpr int L = R < 4 ? R : 4;  // groups loaded together
  Cand4 q[L];
#pragma unroll
  for (int r = 0; r < L; ++r) q[r] = cand_load4(g, c0 + 256 * r);
  __builtin_amdgcn_sched_barrier(0);
  if (t < 64) {  // the threshold T and the ties at it to keep (T = -1: take everything)
    const int B = gload(sc + SelScratch::kCoarse), over = gload(sc + SelScratch::kCoarse + 1);
    const int2 f = B < 0 ? make_int2(0, g.n) : wave_find_bin<512>(sc + SelScratch::kHist2, g.n, over);
    if (t == 0) sT = B < 0 ? -1 : B * 512 + f.x, sNeed = g.n - f.y;
  }
  if (blockIdx.x == 0) sc[SelScratch::kHist1 + t] = 0;
  __syncthreads();
  const int T = sT, need = sNeed;
  // of each group four bits above the threshold and four at it (scores held
  // instead would leave fewer waves on a compute unit)
  uint32_t above[(R + 7) / 8] = {}, at[(R + 7) / 8] = {};
  int gt = 0, eq = 0;
#pragma unroll
  for (int r0 = 0; r0 < R; r0 += L) {
    if (r0 > 0) {
#pragma unroll
      for (int r = 0; r < L; ++r) q[r] = cand_load4(g, c0 + 256 * (r0 + r));
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int r = 0; r < L; ++r) {
      const int k = r0 + r;
      const int4 v = cand_score4(g, c0 + 256 * k, q[r]);
      above[k / 8] |= (uint32_t)((v.x > T) | (v.y > T) << 1 | (v.z > T) << 2 | (v.w > T) << 3) << (4 * (k & 7));
      at[k / 8] |= (uint32_t)((v.x == T) | (v.y == T) << 1 | (v.z == T) << 2 | (v.w == T) << 3) << (4 * (k & 7));
    }
  }
#pragma unroll
  for (int k = 0; k < (R + 7) / 8; ++k) gt += __popc(above[k]), eq += __popc(at[k]);
  gt = gt << 16 | eq;  // at most 4096 of each in a wave
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) gt += __shfl_xor(gt, d, 64);
  eq = gt & 0xffff, gt >>= 16;
  if (lane == 0) s_gt[wave] = gt, s_eq[wave] = eq;
  __syncthreads();
  // the waves before this one and the chunk's totals
  int wgt = 0, weq = 0, cgt = 0, ceq = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    wgt += w < wave ? s_gt[w] : 0, weq += w < wave ? s_eq[w] : 0;
    cgt += s_gt[w], ceq += s_eq[w];
  }
  if (t == 0)
    __hip_atomic_store(&sc[SelScratch::kChunks + blockIdx.x], (int)chunk_word(cgt, ceq), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  // the chunks before this one
  int bgt = 0, beq = 0;
  for (int k = t; k < (int)blockIdx.x; k += kSelThreads) {
    const uint32_t w = chunk_word_of<CHUNK>(g, sc, k, T);
    bgt += (int)(w >> 15 & 32767u), beq += (int)(w & 32767u);
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) bgt += __shfl_xor(bgt, d, 64), beq += __shfl_xor(beq, d, 64);
  if (lane == 0) s_bgt[wave] = bgt, s_beq[wave] = beq;
  __syncthreads();
  bgt = beq = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) bgt += s_bgt[w], beq += s_beq[w];
  // ties before a place are kept up to `need`
  int tie = beq + weq, pos = bgt + wgt + min(need, tie);
  if ((int)blockIdx.x == j.G - 1 && t == 0) *j.count = bgt + cgt + min(need, beq + ceq);
  int32_t* __restrict__ idx = j.idx;
  for (int r = 0; r < R; ++r) {
    const uint32_t ab = above[r / 8] >> (4 * (r & 7)) & 15u, eb = at[r / 8] >> (4 * (r & 7)) & 15u;
    if (!__any(ab | eb)) continue;
    unsigned long long ties[4], sel[4];
    int te = tie, p = pos;
#pragma unroll
    for (int k = 0; k < 4; ++k) te = lanes_below(ties[k] = __ballot(eb >> k & 1u), te);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t e = eb >> k & 1u;
      sel[k] = __ballot((ab >> k & 1u) | (e & (uint32_t)(te < need)));
      te += (int)e;
      p = lanes_below(sel[k], p);
    }
    int x, y;
    cand_xy(g, c0 + 256 * r, &x, &y);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (sel[k] >> lane & 1) idx[p++] = (g.m + y) * g.W + (g.m + x);
      if (++x == g.Wc) x = 0, ++y;
      tie += __popcll(ties[k]), pos += __popcll(sel[k]);
    }
  }
}

SelJob make_sel_job(const uint8_t* img, int32_t W, int32_t H, int32_t margin, int32_t n, int32_t* idx,
                    int32_t* count, int32_t* scratch, int chunk) {
  SelJob j;
  j.g.img = img;
  j.g.W = W;
  j.g.m = margin;
  j.g.Wc = W - 2 * margin;
  const int Hc = H - 2 * margin;
  j.g.C = (j.g.Wc > 0 && Hc > 0) ? j.g.Wc * Hc : 0;
  j.g.n = n;
  j.g.inv_wc = j.g.Wc > 0 ? 1.0f / (float)j.g.Wc : 0.0f;
  j.g.pitch = W;
  j.g.pad = 0;
  j.sc = scratch;
  j.idx = idx;
  j.count = count;
  j.G = (j.g.C + chunk - 1) / chunk;
  j.pad = 0;
  return j;
}

// The pipeline for one image (many == nullptr) or for n_img images whose
// chunk counts are at most G_max.  The write pass leaves the histograms
// cleared, so sel_clear runs only where an image has no candidates (its count
// must still be written); the coarse histogram starts zeroed (a fresh scratch by
// its owner).
static hipError_t run_select(const SelJob& one, const SelJob* many, int n_img, int G_max, int chunk, bool any_empty,
                             hipStream_t s) {
  // Histogram workgroups: as many as have a group of four per thread, but at most
  // 256 in all (and at least 8 for each image): every one flushes its bins with
  // atomics on the same few lines, and past a compute unit each more of them
  // cost more than they took off the counting.
  const int h_max = (int)(((int64_t)G_max * chunk + 4 * kHistThreads - 1) / (4 * kHistThreads));
  const int h_cap = n_img * 8 > 256 ? 8 : 256 / n_img;
  const dim3 hist(h_max < h_cap ? h_max : h_cap, n_img), grid(G_max, n_img);
  if (any_empty) hipLaunchKernelGGL(sel_clear, dim3(1, n_img), dim3(kSelThreads), 0, s, one, many);
  if (G_max > 0) {
    hipLaunchKernelGGL(sel_hist_coarse, hist, dim3(kHistThreads), 0, s, one, many);
    hipLaunchKernelGGL(sel_hist_fine, hist, dim3(kHistThreads), 0, s, one, many);
    if (chunk == 1024)
      hipLaunchKernelGGL(sel_write<1024>, grid, dim3(kSelThreads), 0, s, one, many);
    else if (chunk == 4096)
      hipLaunchKernelGGL(sel_write<4096>, grid, dim3(kSelThreads), 0, s, one, many);
    else
      hipLaunchKernelGGL(sel_write<16384>, grid, dim3(kSelThreads), 0, s, one, many);
  }
  return hipGetLastError();
}

hipError_t launch_select(const uint8_t* img, int32_t W, int32_t H, int32_t margin, int32_t n, int32_t* idx,
                         int32_t* count, int32_t* scratch, hipStream_t s) {
  const int chunk = select_chunk((int64_t)W * H);
  const SelJob j = make_sel_job(img, W, H, margin, n, idx, count, scratch, chunk);
  return run_select(j, nullptr, 1, j.G, chunk, j.G == 0, s);
}

hipError_t launch_select_batch(const SelJob* d_jobs, int n_img, int G_max, int chunk, bool any_empty, hipStream_t s) {
  SelJob none;
  std::memset(&none, 0, sizeof none);
  return run_select(none, d_jobs, n_img, G_max, chunk, any_empty, s);
}

// ---------------------------------------------------------------- selection without allocation

// Histograms, coarse bucket and the chunks' words of one selection of an
// image of up to kNoAllocSelectPixels pixels, for callers that cannot allocate.
// Every device holds its own copy for the life of the process; all calls on a
// device share it (calls that overlap on one device race).
// At most 2048 chunks of 4096, 1024 of 1024 or of 16384.
constexpr int64_t kNoAllocSelectInts = SelScratch::kChunks + 2048 + 1;
static_assert(kNoAllocSelectPixels <= 2048 * (int64_t)16384, "chunks of the static scratch");
static __device__ __align__(256) int32_t g_select_scratch[kNoAllocSelectInts];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
int32_t* g_scratch_ptr[kMaxDevices] = {};  // device address of g_select_scratch, per device

// The device address of the current device's copy of g_select_scratch, looked
// up once per device (the array's name in host code is not that address).
hipError_t select_scratch_ptr(int32_t** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if ((e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_select_scratch))) != hipSuccess) return e;
    g_scratch_ptr[dev] = static_cast<int32_t*>(p);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}
}  // namespace

hipError_t launch_select_noalloc(const uint8_t* img, int32_t W, int32_t H, int64_t pitch, int32_t margin, int32_t n,
                                 int32_t* idx, int32_t* count, hipStream_t s) {
  if ((int64_t)W * H > kNoAllocSelectPixels || pitch < W || pitch > INT32_MAX) return hipErrorInvalidValue;
  int32_t* sc = nullptr;
  hipError_t e = select_scratch_ptr(&sc);
  if (e != hipSuccess) return e;
  const int chunk = select_chunk((int64_t)W * H);
  SelJob j = make_sel_job(img, W, H, margin, n, idx, count, sc, chunk);
  j.g.pitch = (int32_t)pitch;
  // the histograms start at zero: cleared by a kernel (no memset node, so the
  // call can also be captured into a graph);
  // sel_clear also writes the count of an image without candidates
  hipLaunchKernelGGL(sel_clear, dim3(1, 1), dim3(kSelThreads), 0, s, j, nullptr);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return run_select(j, nullptr, 1, j.G, chunk, false, s);
}

}  // namespace dpt
