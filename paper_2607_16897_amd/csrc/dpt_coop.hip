// Cooperative multi-workgroup track: every camera stream's map is split into
// chunks, one workgroup each, with one or two threads per point (four for patterns
// other than the 8-pixel one), and all chunks of all streams run in one co-resident
// launch that covers every level and iteration of the frame.
//
// Per Gauss-Newton iteration the chunks of a stream exchange their 32 partial
// sums through a double-buffered global array.  Each partial is one 64-bit
// word holding an epoch tag above the float's bits, so a reader knows from the
// word alone whether it is current: a chunk publishes its partials and polls
// the stream's words until every chunk's carry the tag, with no counter, no
// fence and no second read.  Every word is stored twice: a group-scope copy,
// which stays in the L2 of the chunk's XCD, and a device-scope copy, written
// through to memory.  A stream's chunks share one XCD (the work list places
// them so), where a device-scope poll finds the first copy in the shared L2 in
// about half the round trip of the second; every eighth poll reads the second
// copies instead, so a chunk that the dispatcher placed on another XCD is still
// seen.  Every chunk then sums the partials in one fixed order
// and solves the 6x6 system across the lanes of every 16-lane row: all rows of all
// chunks of a stream compute bitwise-identical poses, so one exchange per iteration
// suffices and the result is reproducible.  Waits are bounded: a chunk that
// polls longer than `spin_limit` times gives up and reports a timeout instead
// of hanging.
#include <atomic>
#include <climits>
#include <cstring>
#include <type_traits>

#include "dpt_device.h"

namespace dpt {

// Chunk words read per round trip while polling (one load each in flight).
constexpr int kPollBatch = 8;

// Polls of the L2 copies between two polls of the device-scope copies, minus one.
constexpr int kSlowPollMask = 7;

// Publish one partial word: the group-scope store (kept in the XCD's L2, no
// write-through) to `fast`, the device-scope one to `slow`.
__device__ __forceinline__ void publish_word(__attribute__((address_space(1))) uint64_t* fast,
                                             __attribute__((address_space(1))) uint64_t* slow, uint64_t w) {
  asm volatile("global_store_dwordx2 %0, %1, off sc0" : : "v"(fast), "v"(w) : "memory");
  __hip_atomic_store(slow, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The value lane (lane ^ D) holds, D = 16 or 32, moved within the register
// file (v_permlane16_swap / v_permlane32_swap exchange the rows, or the
// halves, of two registers) instead of through the LDS crossbar.
template <int D>
__device__ __forceinline__ uint32_t lane_xor_u(uint32_t u) {
  static_assert(D == 16 || D == 32, "row or half swap");
  if constexpr (D == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return (threadIdx.x & 32) ? r[0] : r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return (threadIdx.x & 16) ? r[0] : r[1];
  }
}

template <int D>
__device__ __forceinline__ float lane_xor(float x) {
  return __uint_as_float(lane_xor_u<D>(__float_as_uint(x)));
}

// Row rotation within 16 lanes (DPP row_ror:K) of an integer.
template <int K>
__device__ __forceinline__ int dpp_ror_i(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x120 + K, 0xf, 0xf, false);
}

// The wave's minimum of lo and maximum of hi, in every lane: DPP rotations
// within each 16-lane row, then the row and half-wave swaps, with no LDS
// round trip between the steps.  All 64 lanes active.
__device__ __forceinline__ void wave_min_max(int& lo, int& hi) {
  lo = min(lo, dpp_ror_i<8>(lo)), hi = max(hi, dpp_ror_i<8>(hi));
  lo = min(lo, dpp_ror_i<4>(lo)), hi = max(hi, dpp_ror_i<4>(hi));
  lo = min(lo, dpp_ror_i<2>(lo)), hi = max(hi, dpp_ror_i<2>(hi));
  lo = min(lo, dpp_ror_i<1>(lo)), hi = max(hi, dpp_ror_i<1>(hi));
  lo = min(lo, (int)lane_xor_u<16>((uint32_t)lo)), hi = max(hi, (int)lane_xor_u<16>((uint32_t)hi));
  lo = min(lo, (int)lane_xor_u<32>((uint32_t)lo)), hi = max(hi, (int)lane_xor_u<32>((uint32_t)hi));
}

// Where a lane of wave 0 finds its words when it polls the chunks of a stream:
// the wave's 64 / NV lane groups read consecutive ranges of the chunks (group q
// the q-th range, lane v word v), kPollBatch chunks per batch.  The offsets and
// the marks of the words past the range's end are the same in every exchange of
// a launch, so they are formed once: a poll round is its loads and two or three
// instructions per word.  (Forming them in the round cost 105 instructions, 420
// cycles of issue per round; the loads' latency is about 700.)
struct PollLanes {
  uint32_t off[kPollBatch];  // bytes from the buffer's start, first batch
  float in[kPollBatch];      // 1: the word belongs to the range, 0: a repeat of its last chunk
  int cb, ce;                // the range
};

template <int NV>
__device__ __forceinline__ PollLanes poll_lanes(int nch) {
  constexpr int G = 64 / NV;
  const int lane = threadIdx.x & 63, q = lane / NV, v = lane % NV;
  PollLanes p;
  const int per = (nch + G - 1) / G;
  p.cb = q * per;
  p.ce = p.cb + per < nch ? p.cb + per : nch;
#pragma unroll
  for (int j = 0; j < kPollBatch; ++j) {
    // an empty range (fewer chunks than groups) re-reads the last chunk, marked out
    const int c = max(0, min(min(p.cb + j, p.ce - 1), nch - 1));
    p.off[j] = (uint32_t)(c * 32 + v) * 8u;
    p.in[j] = p.cb + j < p.ce ? 1.0f : 0.0f;
  }
  return p;
}

// A pointer that is the same in every lane, held in scalar registers.
__device__ __forceinline__ uint64_t* uniform_ptr(uint64_t* p) {
  const uint64_t u = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u), hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
  return (uint64_t*)(((uint64_t)hi << 32) | lo);
}

// Wave 0 only.  Publish this chunk's column sums (`mine`, lanes < NV) under
// `tag`, wait until all nch chunks of the stream published theirs, and return
// the stream totals (lanes < NV).  False on timeout.  A chunk's words are 32
// apart whatever NV is.  pl: poll_lanes<NV>(nch).  The lane groups' sums meet
// in a fixed tree, the same in every chunk of the stream.
template <bool KAHAN, int NV>
__device__ __forceinline__ bool exchange_partials(uint64_t* partials, const PollLanes& pl, int chunk, int nch,
                                                  uint32_t tag, float mine, int spin_limit, float* total,
                                                  int* polls = nullptr) {
  constexpr int G = 64 / NV;
  static_assert(G == 2 || G == 4, "32 or 16 values per chunk");
  static_assert(!(KAHAN && G != 2), "compensated sums use 32 values");
  const int lane = threadIdx.x & 63, q = lane / NV, v = lane % NV;
  // global-memory pointers: global loads and stores, which unlike flat ones
  // leave the LDS counter alone and skip the aperture check
  using gptr = __attribute__((address_space(1))) uint64_t*;
  using gbytes = __attribute__((address_space(1))) char*;
  const uint32_t half = (uint32_t)nch * 256u;  // bytes of one copy of one parity
  const gbytes buf = (gbytes)partials + (tag & 1u) * half;
  const uint64_t hi = (uint64_t)tag << 32;
  if (lane < NV) {
    const uint32_t o = (uint32_t)(chunk * 32 + lane) * 8u;
    publish_word((gptr)(buf + o), (gptr)(buf + 2u * half + o), hi | __float_as_uint(mine));
  }
  for (int t = 0; t < spin_limit; ++t) {
    const gbytes rb = buf + ((t & kSlowPollMask) == kSlowPollMask ? 2u * half : 0u);
    // a batch of loads in flight, then the checks, with no branch between the
    // loads: past its range's end a lane re-reads the range's last chunk and
    // leaves the word out
    uint64_t w[kPollBatch];
#pragma unroll
    for (int j = 0; j < kPollBatch; ++j)
      w[j] = __hip_atomic_load((gptr)(rb + pl.off[j]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // every load issued before the first wait: the scheduler otherwise starts
    // on the first words before the last load, a second latency per round
    __builtin_amdgcn_sched_barrier(0);
    float s = 0.0f, comp = 0.0f;
    uint32_t stale = 0;
    auto add = [&](uint64_t word, float in) {
      stale |= (uint32_t)(word >> 32) ^ tag;
      const float x = __uint_as_float((uint32_t)word);
      if (KAHAN) {
        const float y = x - comp;
        const float u = s + y;
        const float cn = (u - s) - y;
        s = in != 0.0f ? u : s;
        comp = in != 0.0f ? cn : comp;
      } else {
        s = fmaf(x, in, s);
      }
    };
#pragma unroll
    for (int j = 0; j < kPollBatch; ++j) add(w[j], pl.in[j]);
    for (int c0 = pl.cb + kPollBatch; c0 < pl.ce; c0 += kPollBatch) {
#pragma unroll
      for (int j = 0; j < kPollBatch; ++j)
        w[j] = __hip_atomic_load((gptr)(rb + (uint32_t)(min(c0 + j, pl.ce - 1) * 32 + v) * 8u), __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < kPollBatch; ++j) add(w[j], c0 + j < pl.ce ? 1.0f : 0.0f);
    }
    if (__all(stale == 0)) {
      if constexpr (G == 4) s += lane_xor<16>(s);  // (g0 + g1), (g2 + g3)
      if constexpr (KAHAN) {  // the two compensated sums: (s0 - c0) + (s1 - c1)
        const float ps = lane_xor<32>(s), pc = lane_xor<32>(comp);
        const float lo_s = q == 0 ? s : ps, lo_c = q == 0 ? comp : pc;
        const float hi_s = q == 0 ? ps : s, hi_c = q == 0 ? pc : comp;
        const float y = hi_s - (lo_c + hi_c);
        s = lo_s + y;
      } else {
        s += lane_xor<32>(s);
      }
      *total = s;
      if (kCycleProfile && polls) *polls = t + 1;
      return true;
    }
    // no sleep between rounds: a round is already a memory round trip, and
    // the next one starts as soon as this one has shown a word missing
  }
  return false;
}

// Polling by the whole workgroup, for streams of more than kPollBatch chunks:
// thread t reads value t % 32 of chunks c = t / 32 (mod blockDim / 32 groups),
// four loads in flight, and sums them in chunk order; the groups' sums meet in
// LDS (sh_grp, blockDim floats) and are added in group order, a fixed order
// shared by every chunk of the stream.  All threads; false on timeout.
template <bool KAHAN, int NV>
__device__ __forceinline__ bool exchange_wide(const uint64_t* partials, int nch, uint32_t tag, int spin_limit,
                                              float* sh_grp, float* sh_tot, int2 place) {
  const int t = threadIdx.x, v = t & 31, q = t >> 5, G = blockDim.x >> 5;
  // global-memory pointers, no branch between a batch's loads and no sleep
  // between rounds, as in exchange_partials: past the last chunk a lane
  // re-reads it and drops the word
  using gptr = const __attribute__((address_space(1))) uint64_t*;
  const gptr buf = (gptr)(partials + (size_t)(tag & 1u) * nch * 32);
  const gptr slow = (gptr)(partials + (size_t)(2 + (tag & 1u)) * nch * 32);
  float s = 0.0f, comp = 0.0f;
  bool ok = true;
  if (v < NV) {
    ok = false;
    for (int it = 0; it < spin_limit && !ok; ++it) {
      const gptr rb = (it & kSlowPollMask) == kSlowPollMask ? slow : buf;
      s = 0.0f, comp = 0.0f;
      ok = true;
      for (int c0 = q; c0 < nch; c0 += 4 * G) {
        uint64_t w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
          w[j] = __hip_atomic_load(&rb[min(c0 + j * G, nch - 1) * 32 + v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bool in = c0 + j * G < nch;
          ok &= !in | ((uint32_t)(w[j] >> 32) == tag);
          const float x = __uint_as_float((uint32_t)w[j]);
          if (KAHAN) {
            const float y = x - comp;
            const float u = s + y;
            const float cn = (u - s) - y;
            s = in ? u : s;
            comp = in ? cn : comp;
          } else {
            const float u = s + x;
            s = in ? u : s;
          }
        }
      }
    }
    sh_grp[q * NV + v] = s;
  }
  const int bad = __syncthreads_or(!ok);
  if (t < NV) {
    float tot = 0.0f, c2 = 0.0f;
    for (int g = 0; g < G; ++g) {
      const float x = sh_grp[g * NV + t];
      if (KAHAN) {
        const float y = x - c2;
        const float u = tot + y;
        c2 = (u - tot) - y;
        tot = u;
      } else {
        tot += x;
      }
    }
    sh_tot[place.x] = tot;
    sh_tot[place.y] = tot;
  }
  return bad == 0;
}

// What a thread takes from the stream totals: its lane's row of (H | b) with
// the diagonal entry (robust mode) or b_i alone in row[6] (fixed H), i = lane %
// 16 capped at 5, and the counts.
struct LaneTotals {
  float row[7], diag;
  float E, pts;
};

// Wave 0's sum over the workgroup's NW waves of the words at sh_red + w * stride
// + word: all reads in flight at once, then the sum in wave order.
template <bool KAHAN, int NW>
__device__ __forceinline__ float sum_waves(const float* sh_red, int stride, int word) {
  float part[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) part[w] = sh_red[w * stride + word];
  __builtin_amdgcn_sched_barrier(0);
  float s = part[0], comp = 0.0f;
#pragma unroll
  for (int w = 1; w < NW; ++w) {
    if (KAHAN) {
      const float y = part[w] - comp;
      const float u = s + y;
      comp = (u - s) - y;
      s = u;
    } else {
      s += part[w];
    }
  }
  return s;
}

// The stream totals of the workgroup's column sums: `mine` (wave 0, lane v < NV:
// slot v) exchanged across the stream's chunks; the totals land in sh_tot
// (kTotals floats, the layout of the lane-parallel solve) and the lane's share
// of them in tot.  Returns false on timeout (same value in every thread).  NV =
// 32 or 16.  place: total_place of lane % 32.  WIDE: streams of more than
// kPollBatch chunks are polled by the whole workgroup (exchange_wide, sh_grp:
// blockDim floats of LDS); otherwise wave 0 polls alone.
template <bool KAHAN, int NV, bool WIDE>
__device__ __forceinline__ bool stream_total(float mine, float* sh_tot, int2 place, uint64_t* partials,
                                             const PollLanes& pl, int chunk, int nch, uint32_t tag, int spin_limit,
                                             float* sh_grp, LaneTotals& tot, int* polls = nullptr) {
  const int lane = threadIdx.x & 63;
  const bool wide = WIDE && nch > kPollBatch;
  if (threadIdx.x < 64) {
    if (wide) {  // publish; the whole workgroup polls below
      if (lane < NV)
        publish_word((__attribute__((address_space(1))) uint64_t*)&partials[(size_t)(tag & 1u) * nch * 32 + chunk * 32 + lane],
                     (__attribute__((address_space(1))) uint64_t*)&partials[(size_t)(2 + (tag & 1u)) * nch * 32 +
                                                                           chunk * 32 + lane],
                     ((uint64_t)tag << 32) | __float_as_uint(mine));
    } else {
      float total = mine;
      bool ok = true;
      if (nch > 1) ok = exchange_partials<KAHAN, NV>(partials, pl, chunk, nch, tag, mine, spin_limit, &total, polls);
      if (lane < NV) sh_tot[place.x] = total, sh_tot[place.y] = total;
      if (lane == 0) sh_tot[kTotOk] = ok ? 1.0f : 0.0f;
    }
  }
  bool ok = true;
  if (wide) ok = exchange_wide<KAHAN, NV>(partials, nch, tag, spin_limit, sh_grp, sh_tot, place);
  __syncthreads();
  // every total requested with the verdict, before any test of either: left to
  // itself the compiler reads each behind the branch that first needs it, one
  // LDS round trip per test on the iteration's path
  const int i = min(lane & 15, 5);
  const float4 cnt = *reinterpret_cast<const float4*>(sh_tot + kTotE);
  if constexpr (NV == 32) {
    const float4 h0 = *reinterpret_cast<const float4*>(sh_tot + 8 * i), h1 = *reinterpret_cast<const float4*>(sh_tot + 8 * i + 4);
    tot.row[0] = h0.x, tot.row[1] = h0.y, tot.row[2] = h0.z, tot.row[3] = h0.w;
    tot.row[4] = h1.x, tot.row[5] = h1.y, tot.row[6] = h1.z;
    tot.diag = sh_tot[9 * i];
  } else {
    tot.row[6] = sh_tot[8 * i + kTotB];
  }
  tot.E = cnt.x, tot.pts = cnt.z;
  asm volatile("" ::: "memory");
  return wide ? ok : cnt.w != 0.0f;
}

// 3x4 rigid transforms (row-major [R | t]) in FP64, one output element per
// thread t < 12: out = A B, and out = A^-1 = [R^T | -R^T t].
__device__ __forceinline__ double compose34_elem(const double* A, const double* B, int t) {
  const int r = t >> 2, c = t & 3;
  double v = A[4 * r] * B[c] + A[4 * r + 1] * B[4 + c] + A[4 * r + 2] * B[8 + c];
  return c == 3 ? v + A[4 * r + 3] : v;
}

__device__ __forceinline__ double invert34_elem(const double* A, int t) {
  const int r = t >> 2, c = t & 3;
  if (c < 3) return A[4 * c + r];
  return -(A[r] * A[3] + A[4 + r] * A[7] + A[8 + r] * A[11]);
}

// The pose arithmetic between frames runs in one wave, an element per lane
// (lanes t < 12), its operands in LDS: a wave's LDS accesses keep their order,
// so the steps need no workgroup barrier.  It runs beside the final pass's
// exchange (about ten LDS round trips against the exchange's memory round
// trips); with the start slot and the stream's descriptor read in one go, nine
// frames of 2000 points take 412 instead of 422 us (two threads per point; one
// thread 466 instead of 483), one frame of 500 points 51.5 instead of 52.4.
__device__ __forceinline__ void wave_step() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// One step of orthonormalize34 on T across the lanes: the same products and sums per
// element, so the same result.  M: 12 doubles of scratch.  Whether an entry of R^T R
// was more than 1e-7 off the identity's (the step leaves 3/8 of the square).
__device__ __forceinline__ bool orthonormalize_step(double* T, double* M, int t) {
  const int r = (t >> 2) & 3, c = t & 3;
  const bool rot = t < 12 && c < 3;
  wave_step();
  // 3I - R^T R, element (r, c)
  const double rtr = T[r] * T[c] + T[4 + r] * T[4 + c] + T[8 + r] * T[8 + c];
  const double m = (r == c ? 3.0 : 0.0) - rtr;
  if (rot) M[t] = m;
  wave_step();
  const int q = min(r, 2);
  const double v = 0.5 * (T[4 * q] * M[c] + T[4 * q + 1] * M[4 + c] + T[4 * q + 2] * M[8 + c]);
  wave_step();
  if (rot) T[t] = v;
  wave_step();
  return __any(rot & (fabs(rtr - (r == c ? 1.0 : 0.0)) > 1e-7));
}

// Constant-velocity start P1 P0^-1 P1 from the pose history (h1 = P1, h0i =
// P0^-1, in LDS), taken relative to the reference (P T_rw^-1, rwi = T_rw^-1), into
// T0: the two products (P1 P0^-1) and (P1 T_rw^-1) side by side, then theirs, and
// the rotation back on SO(3): two steps, as the host takes for a given pose, where the
// first began more than 1e-7 off.  A caller's history may hold poses rounded to a few
// decimals (off by 1e-2, one step leaves 1e-4, two 1e-8); the products of tracked poses
// are rotations to FP64 rounding, and two steps for each took a window of nine frames
// from 396 to 401 us.  The second is a turn of a loop, not a second copy of cold code.
// One wave, t its lane.  m1, m2: 12 doubles of scratch each.
__device__ __forceinline__ void predict_wave(double* T0, const double* rwi, const double* h0i, const double* h1,
                                             double* m1, double* m2, int t) {
  wave_step();
  const int e = t & 15;
  if (e < 12 && t < 32) {
    const double v = compose34_elem(h1, t < 16 ? h0i : rwi, e);
    (t < 16 ? m1 : m2)[e] = v;
  }
  wave_step();
  double v = 0.0;
  if (t < 12) v = compose34_elem(m1, m2, t);
  if (t < 12) T0[t] = v;
#pragma unroll 1
  for (int it = 0; it < 2 && orthonormalize_step(T0, m2, t); ++it) {
  }
}

// Start pose relative to the reference for this launch: the given one, one
// in device memory (a learned proposal), or the constant-velocity prediction
// from the stream's pose history.  Block-wide;
// the result, the reference pose and the history land in LDS.
__device__ __forceinline__ void start_pose(const StartSlot& st, const double* __restrict__ hist, double* T0, double* rw,
                                           double* rwi, double* h0, double* h0i, double* h1, double* m1, double* m2) {
  const int t = threadIdx.x;
  if (t < 64) {
    const double mode = st.mode;
    if (t < 12) {
      const double older = gload(hist + t), newer = gload(hist + 12 + t);
      // kStartDevice: the proposal an earlier launch on this stream wrote
      T0[t] = mode > 1.5 ? gload(st.dev_rel + t) : st.T_rel[t];
      rw[t] = st.T_rw[t];
      rwi[t] = invert34_elem(st.T_rw, t);
      h0[t] = older;
      h1[t] = newer;
    }
    wave_step();
    if (t < 12) h0i[t] = invert34_elem(h0, t);
    if (mode > 0.5 && mode < 1.5) predict_wave(T0, rwi, h0i, h1, m1, m2, t);
  }
  __syncthreads();
}

// ---------------------------------------------------------------- cycle split (DPT_CYCLE_PROFILE builds)

#ifdef DPT_CYCLE_PROFILE
constexpr int kCycFields = DPT_CYCLE_FIELDS;
__device__ uint64_t g_cycles[kCycleSlots * kCycFields];
#endif

// Where this workgroup runs: XCC id << 32 | HW_ID (CU, SIMD, shader engine).
__device__ __forceinline__ uint64_t hw_place() {
#ifdef DPT_CYCLE_PROFILE
  uint32_t xcc, hw;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_HW_ID)" : "=s"(hw));
  return ((uint64_t)xcc << 32) | hw;
#else
  return 0;
#endif
}

// Thread 0's phase sums of one launch into the slot's totals.
__device__ __forceinline__ void cycles_flush(const uint64_t (&cy)[4], uint64_t iters, uint64_t t_start,
                                             uint64_t rt_start, uint64_t polls, const uint64_t (&fr)[5]) {
#ifdef DPT_CYCLE_PROFILE
  if (threadIdx.x != 0 || blockIdx.x >= (unsigned)kCycleSlots) return;
  uint64_t* o = g_cycles + (size_t)blockIdx.x * kCycFields;
  for (int k = 0; k < 4; ++k) atomicAdd((unsigned long long*)&o[k], (unsigned long long)cy[k]);
  atomicAdd((unsigned long long*)&o[DPT_CYCLE_ITERATIONS], (unsigned long long)iters);
  atomicAdd((unsigned long long*)&o[DPT_CYCLE_LAUNCHES], 1ull);
  atomicAdd((unsigned long long*)&o[DPT_CYCLE_KERNEL], (unsigned long long)(clock64() - t_start));
  atomicAdd((unsigned long long*)&o[DPT_CYCLE_REALTIME], (unsigned long long)(wall_clock64() - rt_start));
  atomicAdd((unsigned long long*)&o[DPT_CYCLE_POLLS], (unsigned long long)polls);
  for (int k = 0; k < 5; ++k) atomicAdd((unsigned long long*)&o[DPT_CYCLE_FRAME_START + k], (unsigned long long)fr[k]);
  o[DPT_CYCLE_PLACE] = hw_place();
#else
  (void)cy, (void)iters, (void)t_start, (void)rt_start, (void)polls, (void)fr;
#endif
}

hipError_t read_cycle_profile(uint64_t* host, int n_slots, bool reset) {
#ifdef DPT_CYCLE_PROFILE
  if (n_slots < 1 || n_slots > kCycleSlots) return hipErrorInvalidValue;
  hipError_t e = hipDeviceSynchronize();
  if (e != hipSuccess) return e;
  if ((e = hipMemcpyFromSymbol(host, HIP_SYMBOL(g_cycles), sizeof(uint64_t) * kCycFields * n_slots)) != hipSuccess)
    return e;
  if (reset) {
    static uint64_t zeros[kCycleSlots * kCycFields] = {};
    if ((e = hipMemcpyToSymbol(HIP_SYMBOL(g_cycles), zeros, sizeof zeros)) != hipSuccess) return e;
  }
  return hipDeviceSynchronize();
#else
  (void)host, (void)n_slots, (void)reset;
  return hipErrorNotSupported;
#endif
}

// ---------------------------------------------------------------- LDS tiles of the current level

// Bytes of a level a workgroup stages in LDS (every kernel with its templates in
// registers): levels of up to the small tile's size whole, larger ones as the band of
// rows its points' taps span, cut to the tile.  With the small tile and the kernel's
// own 3 to 4 KB a workgroup stays within 64 KB, so two share a compute unit's 160 KB;
// with the large one a workgroup has a compute unit to itself (coop_large_tile).
// A level is not copied whole because the large tile would hold it: bands took a window
// of nine 752x480 frames of 2000 points from 393 to 381 us.
constexpr int kTileSmall = 60 * 1024, kTileLarge = 144 * 1024;
constexpr int kTilePad = 16;  // the last pair of words read past the last byte
// Rows kept around the band at the level's start pose: the pose moves during the
// level's iterations.  Points whose taps leave the band are read from global
// memory (their whole wave).
constexpr int kBandMargin = 4;

// Whether a pattern's taps (a row and a column past its last sample, read as pairs
// of words) fit either tile's allocation from anywhere in its first granule, at a
// level of W bytes a row.
__device__ __forceinline__ bool tile_spans(const PatRegs& pat, int W) {
  return ((int)pat.dy_max - (int)pat.dy_min + 1) * W + (int)pat.dx_max - (int)pat.dx_min + 16 + 8 <= kTileSmall + kTilePad;
}

// Stage level g of the current frame (img = its first byte) in the workgroup's
// LDS tile: the whole level if it fits, else the rows the taps of the usable
// points span at pose T, widened by kBandMargin and cut to the tile's size.
// Copies the 16-byte granules that overlap those rows (each holds at least one
// byte of them, so none crosses into a page the level does not touch).
// Block-wide (NW waves); the caller has finished every read of the previous
// tile.  can: the thread's point may be valid (its validity at this level is
// still being loaded with its template: the band does not wait for it).
template <int NW, class PIX, class PR>
__device__ __forceinline__ Tile8 stage_tile(const IterParams& a, const PatRegs& pat, const LevelGeom& g,
                                            const PIX* img, const float* T, const PR& pr, bool can,
                                            uint8_t* tile_mem, bool large, int* sh_band) {
  const int W = g.W, H = g.H, row = W * (int)sizeof(PIX);
  const int rows_fit = ((large ? kTileLarge : kTileSmall) - 32) / row;
  int lo = 0, hi = H - 1;
  if (row * H > kTileSmall - 32) {
    float X, Y, Z;
    transform(T, pr.X0, pr.Y0, pr.Z0, X, Y, Z);
    const float iz = __builtin_amdgcn_rcpf(Z);
    const float u = fmaf(g.fx * X, iz, g.cx), v = fmaf(g.fy * Y, iz, g.cy);
    const bool ok = can & (Z > a.z_min) & inside(g, pat, u, v);
    const int iv = (int)floorf(ok ? v : 0.0f);
    int rlo = ok ? iv + (int)pat.dy_min : INT_MAX, rhi = ok ? iv + (int)pat.dy_max + 1 : INT_MIN;
    wave_min_max(rlo, rhi);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) sh_band[2 * wave] = rlo, sh_band[2 * wave + 1] = rhi;
    __syncthreads();
    rlo = INT_MAX, rhi = INT_MIN;
#pragma unroll
    for (int w = 0; w < NW; ++w) rlo = min(rlo, sh_band[2 * w]), rhi = max(rhi, sh_band[2 * w + 1]);
    if (rlo <= rhi) {
      lo = max(0, rlo - kBandMargin);
      hi = min(H - 1, rhi + kBandMargin);
    }
    if (hi - lo + 1 > rows_fit) hi = lo + rows_fit - 1;  // the rows below are read from global memory
  }
  const uintptr_t sa = reinterpret_cast<uintptr_t>(img + (int64_t)lo * W), s0 = sa & ~(uintptr_t)15;
  const int delta = (int)(sa - s0);
  const int ng = (delta + (hi - lo + 1) * row + 15) >> 4;
  // Global memory straight into LDS (global_load_lds_dwordx4): each wave moves
  // 64 consecutive granules per instruction, every load in flight at once and
  // no registers held.  The caller waits for all of them (s_waitcnt 0, then a
  // workgroup barrier) before the tile is read.
  const int lane = threadIdx.x & 63;
  for (int q0 = (int)(threadIdx.x & ~63u); q0 < ng; q0 += blockDim.x) {
    const int q = q0 + lane;
    if (q < ng)
      __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint32_t*>(s0 + 16 * (uintptr_t)q),
                                       (__attribute__((address_space(3))) void*)(tile_mem + 16 * q0), 16, 0, 0);
  }
  Tile8 t;
  t.lds = (const __attribute__((address_space(3))) uint8_t*)(tile_mem);
  t.lo = lo, t.hi = hi, t.delta = delta, t.spans = tile_spans(pat, row);
  return t;
}

// The pattern offsets of this thread's samples: all 8, or (NS = 4) the half
// `sub` of a point's pair takes.
template <int NS>
__device__ __forceinline__ void lane_offsets(const PatRegs& pat, int W, int sub, int (&off)[NS]) {
  int all[8];
  pattern_offsets(pat, W, all);
#pragma unroll
  for (int k = 0; k < NS; ++k) off[k] = NS == 8 ? all[k] : (sub ? all[NS + k] : all[k]);
}

// A tile that holds no row of a level of W bytes a row: every usable point reads
// global memory.
__device__ __forceinline__ Tile8 no_tile(uint8_t* tile_mem, const PatRegs& pat, int W) {
  Tile8 t;
  t.lds = (const __attribute__((address_space(3))) uint8_t*)(tile_mem);
  t.lo = 1, t.hi = 0, t.delta = 0, t.spans = tile_spans(pat, W);
  return t;
}

// MIXED: FP16 reference cache, Kahan-compensated FP32 sums across waves and
// chunks, FP64 solve, exponential and pose state.
// FIXED: fixed-H mode (FP32): unweighted residuals, only b, the cost and the
// counts are reduced and exchanged (16 slots), and the inverse of each level's
// constant H comes from the precompute.
// GENERIC: any pattern K (four lanes per point, CH / 4 points per chunk) on
// uint8 levels or (PIX = float) the floating-point Gaussian pyramid; 2: K up to
// kMaxSlotPattern, the templates in registers and the levels in LDS tiles like
// the 8-pixel kernels'; 1: larger patterns, both read from global memory in
// every iteration.
//
// LPP = 2 (8-pixel pattern only): two threads per point, four samples each;
// a chunk of CH threads holds CH / 2 points.
template <int CH, bool MIXED, bool FIXED, int GENERIC = 0, class PIX = uint8_t, bool WIN = false, int LPP = 1>
__global__ __launch_bounds__(CH, 2) void coop_track_kernel(const CoopStream* __restrict__ streams,
                                                           const int2* __restrict__ work,
                                                           const StartSlot* __restrict__ start,
                                                           TrackOut* __restrict__ out_ring, int slot, int n_out,
                                                           int n_frames, uint32_t seq0, uint32_t tag_base,
                                                           int spin_limit, int large_tile) {
  static_assert(!(MIXED && FIXED), "the fixed-H mode computes in FP32");
  static_assert(!(MIXED && GENERIC) && (GENERIC || std::is_same<PIX, uint8_t>::value), "variant");
  static_assert(LPP == 1 || (LPP == 2 && !GENERIC), "two threads per point: the 8-pixel kernels");
  using PR8 = typename std::conditional<MIXED, PointRegsH, PointRegs>::type;
  using PR4 = typename std::conditional<MIXED, PointRegsH4, PointRegs4>::type;
  using PR = typename std::conditional<
      GENERIC == 1, PointGeo,
      typename std::conditional<GENERIC == 2, PointRegsQ, typename std::conditional<LPP == 2, PR4, PR8>::type>::type>::type;
  constexpr bool TILED = GENERIC != 1;  // templates in registers, levels in LDS tiles
  constexpr bool FLOAT_PYR = std::is_same<PIX, float>::value;
  constexpr int TPP = GENERIC ? kLanesPerPoint : LPP;  // threads per point
  constexpr int PPC = CH / TPP;                        // points per chunk
  constexpr int NS = GENERIC ? kQuadSlots : 8 / LPP;   // samples per thread (TILED)
  constexpr int NV = FIXED ? kFixSlots : 32;
  __shared__ CoopStream ss;
  __shared__ double sh_T0[12], sh_rw[12], sh_rwi[12], sh_h0[12], sh_h0i[12], sh_h1[12], sh_Tf[12], sh_m1[12], sh_m2[12];
  __shared__ __align__(16) float sh_tot[kTotals];
  constexpr int NW = CH / 64;
  __shared__ __align__(16) float sh_red[NW * kWaveWords];
  __shared__ float sh_grp[GENERIC ? CH : 1];  // the whole-workgroup exchange of many-chunk streams
  __shared__ int sh_band[2 * (CH / 64)];
  extern __shared__ __align__(16) uint8_t sh_tile[];  // the tile and kTilePad (TILED), else none
  __shared__ __align__(16) StartSlot sh_start;
  const int2 w = work[blockIdx.x];
  if (w.x < 0) return;  // padding slot of the XCD-aware work list
  {
    // the stream's descriptor and the start slot, every word requested at once:
    // the slot lies in host memory, where each dependent read is a round trip of
    // more than a microsecond
    if (threadIdx.x < sizeof(StartSlot) / 4)
      reinterpret_cast<uint32_t*>(&sh_start)[threadIdx.x] = gload(reinterpret_cast<const uint32_t*>(start + w.x) + threadIdx.x);
    const uint32_t* src = reinterpret_cast<const uint32_t*>(streams + w.x);
    for (int j = threadIdx.x; j < (int)(sizeof(CoopStream) / 4); j += blockDim.x)
      reinterpret_cast<uint32_t*>(&ss)[j] = gload(src + j);
  }
  __syncthreads();
  if (sh_start.bank) {  // the stream's second reference bank, and its window pyramids
    for (int j = threadIdx.x; j < (int)(sizeof(RefCache) / 4); j += blockDim.x)
      reinterpret_cast<uint32_t*>(&ss.a.ref)[j] = reinterpret_cast<const uint32_t*>(&ss.ref_alt)[j];
    if (threadIdx.x == 0) ss.win = ss.win_alt;
  }
  start_pose(sh_start, ss.hist, sh_T0, sh_rw, sh_rwi, sh_h0, sh_h0i, sh_h1, sh_m1, sh_m2);
  const uint8_t* const l0 = sh_start.l0;  // level 0 of the window's frames, or null
  const int64_t l0_stride = sh_start.l0_stride;
  const TrackArgs& a = ss.a;
  const IterParams ip(a);
  const PatRegs pregs = pattern_regs(a.pat);
  // the same in every thread: scalar registers
  const int chunk = __builtin_amdgcn_readfirstlane(w.y), nch = __builtin_amdgcn_readfirstlane(ss.n_chunks);
  uint64_t* const partials = uniform_ptr(ss.partials);
  const int i = chunk * PPC + (int)threadIdx.x / TPP;
  const int sub = (int)threadIdx.x % TPP;
  const int nf = WIN ? n_frames : 1;
  const int2 place = total_place<NV>(threadIdx.x & 31);
  const PollLanes pl = poll_lanes<NV>(nch);
  const int li = threadIdx.x & 15;  // the lane's row of the system, its element of the pose
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int sE = FIXED ? kFixE : kSlotE, sP = FIXED ? kFixPts : kSlotPts;
  // where wave 0's lane finds its slot in a wave's partial sums: in an iteration
  // (wave_word, or in order for the fixed H) and in the final pass (cost, count, 0)
  const int word = FIXED ? min(lane, NV - 1) : wave_word(lane & 31);
  const int slot_v = lane % NV, word_final = slot_v == sE ? 0 : slot_v == sP ? 1 : 2;
  const int K = GENERIC ? a.pat.K : 8;
  // the point, the same for every level and frame
  PR pr;
  int j0;
  const bool can = load_geometry_once(a, i, pr, &j0);
  float ju[6], jv[6];
  warp_rows(pr.X0, pr.Y0, pr.Z0, ju, jv);
  const auto sample_offsets = [&](int W, int(&off)[NS]) {
    if constexpr (GENERIC)
      quad_offsets(a.pat, W, sub, off);
    else
      lane_offsets<NS>(pregs, W, sub, off);
  };
  // this thread's sums at pose T: its slots of the point, or the quad's all
  const int filled = GENERIC ? (K - sub + kLanesPerPoint - 1) / kLanesPerPoint : NS;
  const auto sample = [&](auto cost_only, const LevelGeom& g, const PIX* img, const Tile8& tile, const int(&off)[NS],
                          const float(&T)[12]) {
    constexpr bool C = decltype(cost_only)::value;
    PointSums ps;
    if constexpr (GENERIC == 2) {
      // up to 28 samples (a 5x5 patch) fill seven slots
      ps = K <= 7 * kLanesPerPoint ? sample_point<C, FIXED, PIX, 7>(ip, pregs, off, g, img, tile, T, pr, filled)
                                   : sample_point<C, FIXED, PIX, NS>(ip, pregs, off, g, img, tile, T, pr, filled);
    } else if constexpr (GENERIC == 1) {
      ps = sample_point_generic<C, FIXED, PIX>(a, a.pat, g, img, T, pr, sub);
    } else {
      ps = sample_point<C, FIXED, PIX, NS>(ip, pregs, off, g, img, tile, T, pr);
    }
    if constexpr (GENERIC) quad_sums<C, FIXED>(ps);
    return ps;
  };
  constexpr int QP = 4 / TPP;  // points per quad
  QuadRows<FIXED ? 1 : QP> rows;
  if constexpr (!FIXED) quad_rows_of<QP, 0>(ju, jv, rows);
  using Pose = typename std::conditional<MIXED, double, float>::type;
  uint32_t tag = tag_base;
  uint64_t cy[4] = {0, 0, 0, 0}, cy_iters = 0, cy_t0 = 0, cy_rt0 = 0, cy_polls = 0;
  uint64_t cy_fr[5] = {0, 0, 0, 0, 0};  // frame start, level starts, final pass, frames, frame end
  if constexpr (kCycleProfile) cy_t0 = clock64(), cy_rt0 = wall_clock64();
  // WIN: the frames of the launch in order, each from the constant-velocity
  // prediction of the history the previous one extended.  Every chunk keeps its
  // own copy of the history in LDS: the poses are bitwise identical in all
  // chunks of a stream, so no exchange is needed between frames.  Each start is
  // computed beside the previous frame's final pass.
  for (int f = 0; f < nf; ++f) {
    uint64_t cf0 = 0;
    if constexpr (kCycleProfile) cf0 = clock64();
    const PIX* cur = WIN        ? reinterpret_cast<const PIX*>(ss.win + f * ss.win_stride)
                     : FLOAT_PYR ? reinterpret_cast<const PIX*>(a.curf)
                                 : reinterpret_cast<const PIX*>(a.cur);
    // level 0 of the frame: from the source frames themselves when the window
    // pyramids were built without it
    const PIX* cur0 = WIN && l0 ? reinterpret_cast<const PIX*>(l0 + f * l0_stride) : cur + a.lv[0].off;
    // pose state, identical in every 16-lane row of every chunk of the stream:
    // one element per lane, and every element for the points' transforms
    Pose Tl = (Pose)sh_T0[min(li, 11)];
    float T[12];
    spread_pose((float)Tl, T);
    int status = 0, iterations = 0;
    int ipl[kMaxLevels];
#pragma unroll
    for (int j = 0; j < kMaxLevels; ++j) ipl[j] = 0;
    int64_t samples = 0;
    bool stop = false, timed_out = false;
    LaneTotals tot = {};
    // the level-0 tile and point registers, reused by the final pass when the
    // levels ran down to 0
    Tile8 tile0 = no_tile(sh_tile, pregs, a.lv[0].W);
    bool at0 = false;
    if constexpr (kCycleProfile) cy_fr[0] += clock64() - cf0, ++cy_fr[3];
    for (int l = a.levels - 1; l >= 0 && !stop; --l) {
      uint64_t cl0 = 0;
      if constexpr (kCycleProfile) cl0 = clock64();
      const LevelGeom g = a.lv[l];
      const PIX* img = WIN && l == 0 ? cur0 : cur + g.off;
      Tile8 tile;
      int offs[NS];
      const int64_t e = (int64_t)l * a.ref.cap + j0;
      const uint8_t vb = gload(a.ref.valid + e);
      if constexpr (!TILED) {
        pr.s0 = e * K;
      } else {
        load_template(a, e, sub, pr);
        sample_offsets(g.W, offs);
        tile = stage_tile<NW>(ip, pregs, g, img, T, pr, can, sh_tile, large_tile != 0, sh_band);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (l == 0) tile0 = tile, at0 = true;
      }
      pr.ok = can & (vb != 0);
      float hinv[6], hlo[6];  // fixed H: the lane's row of the level's H^-1, in two floats
      int hbad = 0;
      if constexpr (FIXED) {
        const FixedH* fh = a.ref.fixed + l;
#pragma unroll
        for (int j = 0; j < 6; ++j)
          hinv[j] = gload(fh->inv + 6 * min(li, 5) + j), hlo[j] = gload(fh->inv_lo + 6 * min(li, 5) + j);
        hbad = gload(&fh->bad);
      }
      bool converged = false;
      const int it0 = iterations;
      if constexpr (kCycleProfile) cy_fr[1] += clock64() - cl0;
      for (int it = 0; it < ip.max_iters; ++it) {
        uint64_t c0 = 0, c1 = 0, c2 = 0;
        if constexpr (kCycleProfile) c0 = clock64();
        const PointSums ps = sample(std::false_type{}, g, img, tile, offs, T);
        if constexpr (kCycleProfile) c1 = clock64();
        if constexpr (FIXED) {
          // b = -(ju v0 + jv v1) of the thread's samples (of a generic quad: once)
          const bool use = ps.ok & (!GENERIC | (sub == 0));
          const float v0 = use ? g.fx * ps.v0 : 0.0f, v1 = use ? g.fy * ps.v1 : 0.0f;
          float acc[kFixSlots];
#pragma unroll
          for (int r = 0; r < kFixSlots; ++r) acc[r] = r < 6 ? -fmaf(ju[min(r, 5)], v0, jv[min(r, 5)] * v1) : 0.0f;
          acc[kFixPts] = (ps.ok & (sub == 0)) ? 1.0f : 0.0f;
          wave_reduce16(acc);
          if ((lane & 15) == 0)
            *reinterpret_cast<float4*>(sh_red + wave * kWaveWords + 4 * (lane >> 4)) = make_float4(acc[0], acc[1], acc[2], acc[3]);
        } else {
          float m00 = g.fx * g.fx * ps.m00, m01 = g.fx * g.fy * ps.m01, m11 = g.fy * g.fy * ps.m11;
          float v0 = g.fx * ps.v0, v1 = g.fy * ps.v1;
          if constexpr (LPP == 2) {  // the point's sums: both threads' of the pair
            m00 += dpp_quad<0xB1>(m00), m01 += dpp_quad<0xB1>(m01), m11 += dpp_quad<0xB1>(m11);
            v0 += dpp_quad<0xB1>(v0), v1 += dpp_quad<0xB1>(v1);
          }
          f32x4 D[3] = {};
          quad_products<QP, 0>(rows, m00, m01, m11, v0, v1, ps.ok ? 1.0f : 0.0f, D);
          float d[12] = {D[0][0], D[0][1], D[0][2], D[0][3], D[1][0], D[1][1],
                         D[1][2], D[1][3], D[2][0], D[2][1], D[2][2], D[2][3]};
          wave_reduce12(d);
          if ((lane & 12) == 0) {
            float* o = sh_red + wave * kWaveWords + 24 * (lane >> 5) + 12 * ((lane >> 4) & 1) + (lane & 3);
            o[0] = d[0], o[4] = d[1], o[8] = d[2];
          }
        }
        __syncthreads();
        if constexpr (kCycleProfile) c2 = clock64();
        int polls = 0;
        const float mine = wave == 0 ? sum_waves<MIXED, NW>(sh_red, kWaveWords, word) : 0.0f;
        if (!stream_total<MIXED, NV, GENERIC != 0>(mine, sh_tot, place, partials, pl, chunk, nch, tag, spin_limit, sh_grp, tot,
                                              &polls)) {
          timed_out = stop = true;
          break;
        }
        uint64_t c3 = 0;
        if constexpr (kCycleProfile) c3 = clock64();
        ++tag;
        samples += (int64_t)K * (int)tot.pts;  // counts < 2^24: exact
        if (__builtin_expect((int)tot.pts < ip.min_points, 0)) {
          status = 2;  // too few points
          stop = true;
          break;
        }
        bool bad;
        Pose delta, step = 0;
        if constexpr (FIXED) {
          bad = hbad != 0;
          const float b[6] = {row_bcast<0>(tot.row[6]), row_bcast<1>(tot.row[6]), row_bcast<2>(tot.row[6]),
                              row_bcast<3>(tot.row[6]), row_bcast<4>(tot.row[6]), row_bcast<5>(tot.row[6])};
          const auto half = [&](const float (&m)[6], int j) { return fmaf(m[j], b[j], fmaf(m[j + 1], b[j + 1], m[j + 2] * b[j + 2])); };
          delta = (half(hinv, 0) + half(hinv, 3)) + (half(hlo, 0) + half(hlo, 3));
        } else {
          Pose row[7];
#pragma unroll
          for (int j = 0; j < 7; ++j) row[j] = (Pose)tot.row[j];
          delta = solve_rows(row, (Pose)tot.diag, (Pose)(MIXED ? 1e-12 : 1e-6), li, &bad);
        }
        if (__builtin_expect(!bad, 1)) {
          Tl = update_lanes(Tl, delta, &step);
          spread_pose((float)Tl, T);
        }
        if constexpr (kCycleProfile) {
          const uint64_t c4 = clock64();
          cy[0] += c1 - c0, cy[1] += c2 - c1, cy[2] += c3 - c2, cy[3] += c4 - c3, ++cy_iters, cy_polls += polls;
        }
        if (__builtin_expect(bad, 0)) {
          status = 3;  // not positive definite
          stop = true;
          break;
        }
        ++iterations;
        // the same in every lane; as a vote the compiler knows it, and the loop's
        // branches and counters stay scalar
        if (__any(step < (Pose)ip.step_eps)) {
          converged = true;
          break;
        }
      }
#pragma unroll
      for (int j = 0; j < kMaxLevels; ++j) ipl[j] = j == l ? iterations - it0 : ipl[j];
      if (!stop && l == 0 && !converged) status = 1;  // iteration cap at level 0
    }
    uint64_t cp0 = 0;
    if constexpr (kCycleProfile) cp0 = clock64();
    // What follows a frame's last update, in one wave while wave 0 exchanges the
    // final cost: the pose's rotation back on SO(3), the history extended by the
    // frame's estimate T_cw = T_rel T_rw, and the next frame's start.
    const auto finish_pose = [&] {
      if (lane < 12) sh_Tf[lane] = (double)Tl, sh_h0i[lane] = invert34_elem(sh_h1, lane), sh_h0[lane] = sh_h1[lane];
      orthonormalize_step(sh_Tf, sh_m2, lane), orthonormalize_step(sh_Tf, sh_m2, lane);
      if (lane < 12) sh_h1[lane] = compose34_elem(sh_Tf, sh_rw, lane);
      if (WIN && f + 1 < nf) predict_wave(sh_T0, sh_rwi, sh_h0i, sh_h1, sh_m1, sh_m2, lane);
      wave_step();
    };
    if (!timed_out) {  // final cost-only pass at level 0
      const LevelGeom g = a.lv[0];
      if (!at0) {  // the levels stopped above 0: level 0's registers, taps from global memory
        pr.ok = can & (gload(a.ref.valid + j0) != 0);
        if constexpr (TILED) load_template(a, j0, sub, pr);
      }
      if constexpr (!TILED) pr.s0 = (int64_t)j0 * K, pr.ok = can & (gload(a.ref.valid + j0) != 0);
      int offs[NS];
      if constexpr (TILED) sample_offsets(g.W, offs);
      PointSums ps = sample(std::true_type{}, g, WIN ? cur0 : cur + g.off, tile0, offs, T);
      if (GENERIC) ps.E = sub == 0 ? ps.E : 0.0f;
      const float E = wave_sum(ps.E), n = wave_sum((ps.ok & (sub == 0)) ? 1.0f : 0.0f);
      if (lane == 0) *reinterpret_cast<float4*>(sh_red + wave * kWaveWords) = make_float4(E, n, 0.0f, 0.0f);
      __syncthreads();
      if (wave == NW - 1) finish_pose();
      const float mine = wave == 0 ? sum_waves<MIXED, NW>(sh_red, kWaveWords, word_final) : 0.0f;
      if (!stream_total<MIXED, NV, GENERIC != 0>(mine, sh_tot, place, partials, pl, chunk, nch, tag, spin_limit, sh_grp, tot))
        timed_out = true;
      ++tag;
    }
    else {
      if (wave == NW - 1) finish_pose();
      __syncthreads();
    }
    uint64_t ct0 = 0;
    if constexpr (kCycleProfile) ct0 = clock64(), cy_fr[2] += ct0 - cp0;
    // the results, written by a wave that no exchange waits for first
    if (chunk == 0 && wave == NW - 1) {
      TrackOut* o = out_ring + (size_t)(WIN ? (slot + f) % kRing : slot) * n_out + w.x;
      if (lane < 12) {
        o->T[lane] = (float)Tl;
        o->Td[lane] = sh_Tf[lane];
      }
      if (lane == 16) {
        o->E = tot.E;
        o->n = (float)K * tot.pts;
        o->iterations = iterations;
        for (int j = 0; j < kMaxLevels; ++j) o->iters_per_level[j] = ipl[j];
        o->n_valid_points = (int)tot.pts;
        o->status = timed_out ? kStatusTimeout : status;
        o->samples = samples + (int64_t)K * (int)tot.pts;
        // a chunk gave up: so do the frames after this one
        if (WIN && timed_out)
          for (int q = f + 1; q < nf; ++q) out_ring[(size_t)((slot + q) % kRing) * n_out + w.x].status = kStatusTimeout;
      }
      // the fields reach the host before the sequence number: a system-scope
      // release (no acquire, so the L2 keeps the reference data it holds)
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
      if (lane == 16) {
        o->seq = seq0 + f;
        if (WIN && timed_out)
          for (int q = f + 1; q < nf; ++q) out_ring[(size_t)((slot + q) % kRing) * n_out + w.x].seq = seq0 + q;
      }
    }
    if constexpr (kCycleProfile) cy_fr[4] += clock64() - ct0;
    if (timed_out) break;
  }
  // the stream's history for the next launch (every chunk read it at its start,
  // before its first exchange)
  if (chunk == 0 && threadIdx.x < 12) {
    ss.hist[threadIdx.x] = sh_h0[threadIdx.x];
    ss.hist[12 + threadIdx.x] = sh_h1[threadIdx.x];
  }
  if constexpr (kCycleProfile) cycles_flush(cy, cy_iters, cy_t0, cy_rt0, cy_polls, cy_fr);
}

// The kernel of a variant (kCoop* bits); WIN: the window form.  Null for a
// combination that does not exist (a generic variant at another chunk size,
// window tracking of the floating-point pyramid).
template <int CH, bool WIN>
static const void* coop_fn(int variant) {
  if (variant & kCoopGeneric) {
    if (CH != kGenericThreads) return nullptr;
    constexpr int G = kGenericThreads;
    switch (variant & (kCoopFixedH | kCoopFloatPyr | kCoopSlots)) {
      case 0: return reinterpret_cast<const void*>(&coop_track_kernel<G, false, false, 1, uint8_t, WIN>);
      case kCoopFixedH: return reinterpret_cast<const void*>(&coop_track_kernel<G, false, true, 1, uint8_t, WIN>);
      case kCoopSlots: return reinterpret_cast<const void*>(&coop_track_kernel<G, false, false, 2, uint8_t, WIN>);
      case kCoopSlots | kCoopFixedH:
        return reinterpret_cast<const void*>(&coop_track_kernel<G, false, true, 2, uint8_t, WIN>);
      default: break;
    }
    if constexpr (!WIN) {  // no window tracking of the floating-point pyramid
      switch (variant & (kCoopFixedH | kCoopSlots)) {
        case 0: return reinterpret_cast<const void*>(&coop_track_kernel<G, false, false, 1, float>);
        case kCoopFixedH: return reinterpret_cast<const void*>(&coop_track_kernel<G, false, true, 1, float>);
        case kCoopSlots: return reinterpret_cast<const void*>(&coop_track_kernel<G, false, false, 2, float>);
        default: return reinterpret_cast<const void*>(&coop_track_kernel<G, false, true, 2, float>);
      }
    }
    return nullptr;
  }
  if (variant & kCoopPairs) {
    if (CH == 64) return nullptr;  // a pair chunk holds 64 or 128 points
    switch (variant & ~kCoopPairs) {
      case kCoopFP32:
        return reinterpret_cast<const void*>(&coop_track_kernel<CH, false, false, 0, uint8_t, WIN, 2>);
      case kCoopMixed:
        return reinterpret_cast<const void*>(&coop_track_kernel<CH, true, false, 0, uint8_t, WIN, 2>);
      case kCoopFixedH:
        return reinterpret_cast<const void*>(&coop_track_kernel<CH, false, true, 0, uint8_t, WIN, 2>);
      default: return nullptr;
    }
  }
  switch (variant) {
    case kCoopFP32: return reinterpret_cast<const void*>(&coop_track_kernel<CH, false, false, 0, uint8_t, WIN>);
    case kCoopMixed: return reinterpret_cast<const void*>(&coop_track_kernel<CH, true, false, 0, uint8_t, WIN>);
    case kCoopFixedH: return reinterpret_cast<const void*>(&coop_track_kernel<CH, false, true, 0, uint8_t, WIN>);
    default: return nullptr;
  }
}

// Whether a variant stages its levels in LDS tiles.
static bool tiled(int variant) { return !(variant & kCoopGeneric) || (variant & kCoopSlots); }

// Dynamic LDS that the co-residency is counted with.
static size_t coop_tile_lds(int variant) { return tiled(variant) ? kTileSmall + kTilePad : 0; }

// Whether a launch takes the large tile.  At most eight chunks on an XCD (work items
// are dealt to the eight XCDs in turn): four launches at once, as many as the hardware
// queues of a process run, then still fit an XCD's 32 compute units with any mix of
// tiles: k of them with the large one hold 8 k units, and the others' 16 chunks each
// share the rest in twos.  Of those launches, the ones whose chunks' points span more
// of the levels than the small tile holds: maps in no order (2000 points at 752x480
// 73.8 us a frame, 75.8 with the small tile; 320x240 65.9, 70.6) and maps in index order
// of so few points that a chunk's band of level 1 is past the large tile too (200 points
// at 1280x720 53.1, 55.1).  Others wait longer for the larger copy (1111 points at
// 641x479, fixed H, a window of nine 390 us, 382 with the small tile; 1111 at 1280x720
// 66.1, 63.4 a frame).  band: of level 1 in bytes, the widest stream's; INT64_MAX for
// maps in no order.
static bool coop_large_tile(int variant, int n_work, int64_t band) {
  return tiled(variant) && n_work <= 64 && band > kTileLarge;
}

// Co-resident workgroups per CU: the least over every variant at this chunk size.
template <int CH>
static int coop_blocks_per_cu() {
  static int nb = -1;
  if (nb < 0) {
    const int vs[] = {kCoopFP32,
                      kCoopMixed,
                      kCoopFixedH,
                      kCoopPairs,
                      kCoopPairs | kCoopMixed,
                      kCoopPairs | kCoopFixedH,
                      kCoopGeneric,
                      kCoopGeneric | kCoopFixedH,
                      kCoopGeneric | kCoopFloatPyr,
                      kCoopGeneric | kCoopFixedH | kCoopFloatPyr,
                      kCoopGeneric | kCoopSlots,
                      kCoopGeneric | kCoopSlots | kCoopFixedH,
                      kCoopGeneric | kCoopSlots | kCoopFloatPyr,
                      kCoopGeneric | kCoopSlots | kCoopFixedH | kCoopFloatPyr};
    int best = 1 << 30;
    for (int v : vs)
      for (const void* f : {coop_fn<CH, false>(v), coop_fn<CH, true>(v)}) {
        if (!f) continue;
        int k = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&k, f, CH, coop_tile_lds(v)) != hipSuccess) {
          (void)hipGetLastError();
          k = 0;
        }
        best = std::min(best, k);
      }
    nb = best;
  }
  return nb;
}

int coop_max_blocks(int chunk) {
  static int cu_count[64] = {};  // per device, queried once
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
    (void)hipGetLastError();
    return 0;
  }
  int cus = cu_count[dev];
  if (cus == 0) {
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
      (void)hipGetLastError();
      return 0;
    }
    cu_count[dev] = cus;
  }
  switch (chunk) {
    case 64: return coop_blocks_per_cu<64>() * cus;
    case 128: return coop_blocks_per_cu<128>() * cus;
    case 256: return coop_blocks_per_cu<256>() * cus;
    default: return 0;
  }
}

// The chunks of a stream wait for each other, so all workgroups of the grid
// must be resident together.  A grid of at most a quarter of the device's
// co-resident capacity is launched as an ordinary kernel: it is resident as
// soon as the device has that much room, which leaves room for three more such
// launches running concurrently on other streams (on the XCD that a stream's
// chunks are packed to as well: at most 16 of its 64 places each), and it avoids
// the cooperative launch's extra per-launch cost (about 15 us here).  Larger grids
// use the cooperative launch, which guarantees co-residency.  Either way every
// wait is bounded by spin_limit, so a chunk that cannot be scheduled turns
// into a reported timeout, not a hang.
template <int CH>
static hipError_t coop_launch_k(const CoopStream* d_streams, const int2* d_work, int n_work, const StartSlot* start,
                                TrackOut* out_ring, int slot, int n_out, int n_frames, uint32_t seq0, uint32_t tag_base,
                                int variant, int64_t band, int spin_limit, hipStream_t s) {
  const void* fn = n_frames > 0 ? coop_fn<CH, true>(variant) : coop_fn<CH, false>(variant);
  if (!fn) return hipErrorInvalidValue;
  const bool plain = 4 * n_work <= coop_max_blocks(CH);
  int large = coop_large_tile(variant, n_work, band);
  const size_t dyn = large ? kTileLarge + kTilePad : coop_tile_lds(variant);
  if (large) {  // past the default limit: raised once per kernel and device
    static std::atomic<bool> raised[64][2][64];  // zeroed; one array per chunk size
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::atomic<bool>& r = raised[dev][n_frames > 0][variant & 63];
    if (!r.load(std::memory_order_acquire)) {
      if ((e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn)) != hipSuccess) return e;
      r.store(true, std::memory_order_release);
    }
  }
  void* args[] = {(void*)&d_streams, (void*)&d_work,   (void*)&start,    (void*)&out_ring,   (void*)&slot,
                  (void*)&n_out,     (void*)&n_frames, (void*)&seq0,     (void*)&tag_base,   (void*)&spin_limit,
                  (void*)&large};
  if (plain) return hipLaunchKernel(fn, dim3(n_work), dim3(CH), args, dyn, s);
  return hipLaunchCooperativeKernel(fn, dim3(n_work), dim3(CH), args, dyn, s);
}

hipError_t launch_coop_track(const CoopStream* d_streams, const int2* d_work, int n_work, const StartSlot* start,
                             TrackOut* out_ring, int slot, int n_out, int n_frames, uint32_t seq0, uint32_t tag_base,
                             int chunk, int variant, int64_t band, int spin_limit, hipStream_t s) {
  if (slot < 0 || slot >= kRing || n_frames < 0 || n_frames > kRing) return hipErrorInvalidValue;
  switch (chunk) {
    case 64:
      return coop_launch_k<64>(d_streams, d_work, n_work, start, out_ring, slot, n_out, n_frames, seq0, tag_base,
                               variant, band, spin_limit, s);
    case 128:
      return coop_launch_k<128>(d_streams, d_work, n_work, start, out_ring, slot, n_out, n_frames, seq0, tag_base,
                                variant, band, spin_limit, s);
    case 256:
      return coop_launch_k<256>(d_streams, d_work, n_work, start, out_ring, slot, n_out, n_frames, seq0, tag_base,
                                variant, band, spin_limit, s);
    default: return hipErrorInvalidValue;
  }
}

// ---------------------------------------------------------------- engine (host)

hipError_t CoopEngine::init(int n_streams, const int* max_points, int chunk_, int ppc_, bool xcd, hipStream_t s) {
  release();
  n = n_streams;
  chunk = chunk_;
  ppc = ppc_;
  xcd_pack = xcd;
  stream = s;
  h_streams.assign(n, CoopStream{});
  max_chunks.resize(n);
  partial_words = 0;
  for (int k = 0; k < n; ++k) {
    max_chunks[k] = (max_points[k] + ppc - 1) / ppc;
    partial_words += (size_t)4 * max_chunks[k] * 32;  // two parities, each an L2 and a device-scope copy
  }
  if (partial_words == 0) partial_words = 64;
  hipError_t e;
  if ((e = hipMalloc(&d_streams, sizeof(CoopStream) * n)) != hipSuccess) return e;
  if ((e = hipMalloc(&d_partials, sizeof(uint64_t) * partial_words)) != hipSuccess) return e;
  if ((e = hipMemset(d_partials, 0, sizeof(uint64_t) * partial_words)) != hipSuccess) return e;
  tag_base = 1;
  // coherent (uncached on the device) pinned host memory: the kernel reads the
  // start slots and writes the results over the host link
  const unsigned fl = hipHostMallocMapped | hipHostMallocCoherent;
  if ((e = hipHostMalloc((void**)&h_start, sizeof(StartSlot) * kRing * n, fl)) != hipSuccess) return e;
  if ((e = hipHostMalloc((void**)&h_out, sizeof(TrackOut) * kRing * n, fl)) != hipSuccess) return e;
  if ((e = hipHostGetDevicePointer((void**)&dv_start, h_start, 0)) != hipSuccess) return e;
  if ((e = hipHostGetDevicePointer((void**)&dv_out, h_out, 0)) != hipSuccess) return e;
  memset(h_start, 0, sizeof(StartSlot) * kRing * n);
  memset(h_out, 0, sizeof(TrackOut) * kRing * n);
  size_t off = 0;
  for (int k = 0; k < n; ++k) {
    h_streams[k].partials = d_partials + off;
    off += (size_t)4 * max_chunks[k] * 32;
  }
  dirty = true;
  return hipSuccess;
}

void CoopEngine::release() {
  for (void* p : {(void*)d_streams, (void*)d_work, (void*)d_partials})
    if (p) (void)hipFree(p);
  if (h_start) (void)hipHostFree(h_start);
  if (h_out) (void)hipHostFree(h_out);
  d_streams = nullptr, d_work = nullptr, d_partials = nullptr;
  h_start = nullptr, h_out = nullptr, dv_start = nullptr, dv_out = nullptr;
  work_cap = 0;
  partial_words = 0;
}

void CoopEngine::set_stream(int k, const TrackArgs& a, const RefCache& alt, double* hist, const uint8_t* win,
                            const uint8_t* win_alt, int64_t win_stride) {
  CoopStream& c = h_streams[k];
  c.a = a;
  c.a.out = nullptr;  // results go to the launch's slot of h_out
  c.ref_alt = alt;
  c.hist = hist;
  c.win = win;
  c.win_alt = win_alt;
  c.win_stride = win_stride;
  const int n = std::max(a.ref.n, alt.n);  // the chunks cover the larger bank; the other leaves some idle
  c.n_chunks = n > 0 ? (n + ppc - 1) / ppc : 1;
  dirty = true;
}

// Work list: chunk slots of every stream.  With xcd_pack, the chunks of a stream
// go to block indices of one residue mod 8 (workgroups are dealt to the eight
// XCDs round robin), so a stream's partial sums stay within one XCD's L2;
// streams are assigned to XCDs largest first, each to the least loaded one.
hipError_t CoopEngine::upload() {
  h_work.clear();
  if (xcd_pack) {
    std::vector<std::vector<int2>> lists(8);
    std::vector<int> order(n), load(8, 0);
    for (int k = 0; k < n; ++k) order[k] = k;
    std::sort(order.begin(), order.end(),
              [&](int p, int q) { return h_streams[p].n_chunks > h_streams[q].n_chunks; });
    for (int k : order) {
      int x = (int)(std::min_element(load.begin(), load.end()) - load.begin());
      for (int c = 0; c < h_streams[k].n_chunks; ++c) lists[x].push_back(make_int2(k, c));
      load[x] += h_streams[k].n_chunks;
    }
    size_t depth = 0;
    for (auto& L : lists) depth = std::max(depth, L.size());
    for (size_t j = 0; j < depth; ++j)
      for (int x = 0; x < 8; ++x) h_work.push_back(j < lists[x].size() ? lists[x][j] : make_int2(-1, 0));
    while (!h_work.empty() && h_work.back().x < 0) h_work.pop_back();
  } else {
    for (int k = 0; k < n; ++k)
      for (int c = 0; c < h_streams[k].n_chunks; ++c) h_work.push_back(make_int2(k, c));
  }
  hipError_t e;
  if ((int)h_work.size() > work_cap) {
    if (d_work) (void)hipFree(d_work);
    d_work = nullptr;
    work_cap = (int)h_work.size();
    if ((e = hipMalloc(&d_work, sizeof(int2) * work_cap)) != hipSuccess) return e;
  }
  if ((e = hipMemcpyAsync(d_work, h_work.data(), sizeof(int2) * h_work.size(), hipMemcpyHostToDevice, stream)) !=
      hipSuccess)
    return e;
  if ((e = hipMemcpyAsync(d_streams, h_streams.data(), sizeof(CoopStream) * n, hipMemcpyHostToDevice, stream)) !=
      hipSuccess)
    return e;
  // the pageable sources above are consumed before the call returns only after a sync
  if ((e = hipStreamSynchronize(stream)) != hipSuccess) return e;
  dirty = false;
  return hipSuccess;
}

int CoopEngine::grid() const { return (int)h_work.size(); }

hipError_t CoopEngine::launch(int spin_limit, int slot, bool in_order, int n_frames) {
  hipError_t e;
  if (slot < 0 || slot >= kRing || n_frames < 0 || n_frames > kRing) return hipErrorInvalidValue;
  if (dirty && (e = upload()) != hipSuccess) return e;
  // tags used by this launch: at most levels * max_iters + 1 epochs per stream and frame
  uint32_t span = 1;
  for (const CoopStream& c : h_streams) span = std::max(span, (uint32_t)(c.a.levels * c.a.max_iters + 1));
  span *= (uint32_t)std::max(n_frames, 1);
  if (tag_base > 0xFFFFFFFFu - span) {  // wrap: restart the tags on cleared words
    if ((e = clear_partials()) != hipSuccess) return e;
  }
  const int nf = std::max(n_frames, 1);
  if (seq_next > 0xFFFFFFFFu - (uint32_t)nf) seq_next = 1;  // 0 never marks a result
  const uint32_t seq0 = seq_next;
  seq_next += (uint32_t)nf;
  for (int f = 0; f < nf; ++f) slot_seq[(slot + f) % kRing] = seq0 + (uint32_t)f;
  int64_t band = in_order ? 0 : INT64_MAX;
  for (const CoopStream& c : h_streams) {  // rows of level 1 under a chunk's points, with the tile's margins
    const LevelGeom& g = c.a.lv[std::min(1, c.a.levels - 1)];
    const int64_t pts = std::max(std::max(c.a.ref.n, c.ref_alt.n), 1);
    const int64_t rows = std::min<int64_t>(g.H, g.H * std::min<int64_t>(ppc, pts) / pts + 16);
    band = std::max(band, rows * g.W * ((variant & kCoopFloatPyr) ? 4 : 1));
  }
  e = launch_coop_track(d_streams, d_work, grid(), dv_start + (size_t)slot * n, dv_out, slot, n, n_frames, seq0,
                        tag_base, chunk, variant, band, spin_limit, stream);
  tag_base += span;
  return e;
}

bool CoopEngine::done(int slot) const {
  const TrackOut* o = h_out + (size_t)slot * n;
  for (int k = 0; k < n; ++k)
    if (__atomic_load_n(&o[k].seq, __ATOMIC_ACQUIRE) != slot_seq[slot]) return false;
  return true;
}

hipError_t CoopEngine::clear_partials() {
  tag_base = 1;
  return hipMemsetAsync(d_partials, 0, sizeof(uint64_t) * partial_words, stream);
}

// ---------------------------------------------------------------- pose history

struct HistoryArgs {
  double T[24];  // two 3x4 poses: older, newer
};

__global__ void set_history_kernel(double* hist, HistoryArgs h) {
  if (threadIdx.x < 24) hist[threadIdx.x] = h.T[threadIdx.x];
}

// Histories of n streams: vals[s] = (older 3x4, newer 3x4) into hists[s].
__global__ void set_history_batch_kernel(double* const* hists, const double* vals, int n) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= 24 * n) return;
  hists[e / 24][e % 24] = vals[e];
}

hipError_t launch_set_history_batch(double* const* d_hists, const double* d_vals, int n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(set_history_batch_kernel, dim3((24 * n + 255) / 256), dim3(256), 0, s, d_hists, d_vals, n);
  return hipGetLastError();
}

hipError_t launch_set_history(double* hist, const double* T0, const double* T1, hipStream_t s) {
  HistoryArgs h;
  for (int j = 0; j < 12; ++j) h.T[j] = T0[j], h.T[12 + j] = T1[j];
  hipLaunchKernelGGL(set_history_kernel, dim3(1), dim3(32), 0, s, hist, h);
  return hipGetLastError();
}

// ---------------------------------------------------------------- batched pyramid

template <int TILE>
__global__ __launch_bounds__(256) void pyramid_batch_kernel(const PyrJob* __restrict__ jobs) {
  const PyrJob& j = jobs[blockIdx.z];
  if ((int)blockIdx.x * TILE >= j.g.W[0] || (int)blockIdx.y * TILE >= j.g.H[0]) return;
  if constexpr (TILE == 64)
    pyramid_tile64v(j.src, j.pitch, j.dst, j.g);
  else
    pyramid_tile<TILE>(j.src, j.pitch, j.dst, j.g, j.vec4);
}

// As pyramid_batch_kernel, with job z's source and pitch taken from the kernel
// arguments (no table upload per call) and the vector paths chosen here.
template <int TILE>
__global__ __launch_bounds__(256) void pyramid_batch_args_kernel(const PyrJob* __restrict__ jobs, PyrSrcArgs srcs) {
  const int z = blockIdx.z;
  const PyrJob& j = jobs[z];
  if ((int)blockIdx.x * TILE >= j.g.W[0] || (int)blockIdx.y * TILE >= j.g.H[0]) return;
  const uint8_t* src = srcs.src[z];
  const int64_t pitch = srcs.pitch[z];
  if constexpr (TILE == 64) {
    pyramid_tile64v(src, pitch, j.dst, j.g);
  } else {
    const uintptr_t sa = reinterpret_cast<uintptr_t>(src), da = reinterpret_cast<uintptr_t>(j.dst);
    pyramid_tile<TILE>(src, pitch, j.dst, j.g,
                       ((pitch % 4) == 0 && (sa % 4) == 0 && (j.g.W[0] % 4) == 0 && (da % 4) == 0) ? 1 : 0);
  }
}

// pyramid_block over a batch: blockIdx.y = image, one thread per block.
template <int LV>
__global__ __launch_bounds__(256) void pyramid_batch_block_kernel(const PyrJob* __restrict__ jobs, PyrSrcArgs srcs) {
  constexpr int B = 1 << (LV - 1);
  const int z = blockIdx.y;
  const PyrJob& j = jobs[z];
  const int nbx = j.g.W[0] / B, t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nbx * (j.g.H[0] / B)) return;
  pyramid_block<LV>(srcs.src[z], srcs.pitch[z], j.dst, j.g, t % nbx, t / nbx, true);
}

hipError_t launch_pyramid_batch_args(const PyrJob* d_static, const PyrSrcArgs& srcs, int n_jobs, int max_w,
                                     int max_h, int levels, bool block, hipStream_t s) {
  if (n_jobs > kPyrArgJobs) return hipErrorInvalidValue;
  if (block) {  // every image passed pyramid_block_ok
    const int B = 1 << (levels - 1), n = (max_w / B) * (max_h / B);
    if (levels == 4)
      hipLaunchKernelGGL(pyramid_batch_block_kernel<4>, dim3((n + 255) / 256, n_jobs), dim3(256), 0, s, d_static, srcs);
    else
      hipLaunchKernelGGL(pyramid_batch_block_kernel<3>, dim3((n + 255) / 256, n_jobs), dim3(256), 0, s, d_static, srcs);
    return hipGetLastError();
  }
  if (levels <= 7)
    hipLaunchKernelGGL(pyramid_batch_args_kernel<64>, dim3((max_w + 63) / 64, (max_h + 63) / 64, n_jobs), dim3(256),
                       0, s, d_static, srcs);
  else
    hipLaunchKernelGGL(pyramid_batch_args_kernel<128>, dim3((max_w + 127) / 128, (max_h + 127) / 128, n_jobs),
                       dim3(256), 0, s, d_static, srcs);
  return hipGetLastError();
}

// Window pyramids: blockIdx.z = stream * n_frames + frame; a workgroup builds
// up to `tiles` consecutive tiles of a tile row.
template <int TILE>
__global__ __launch_bounds__(256) void pyramid_window_kernel(const WinJob* __restrict__ jobs, PyrWinSrc srcs,
                                                             int n_frames, int tiles) {
  const int z = blockIdx.z, js = z / n_frames, f = z - js * n_frames;
  const WinJob& j = jobs[js];
  const int oy = blockIdx.y * TILE;
  if (oy >= j.g.H[0]) return;
  const uint8_t* src = srcs.src[js] + f * srcs.stride[js];
  uint8_t* dst = j.dst + f * j.dst_stride;
  const int64_t pitch = srcs.pitch[js];
  const bool write_l0 = srcs.write_l0[js] != 0;
  const int W0 = j.g.W[0];
  for (int t = 0; t < tiles; ++t) {  // the tile's LDS is free again when the previous call returns
    const int ox = ((int)blockIdx.x * tiles + t) * TILE;
    if (ox >= W0) break;
    if constexpr (TILE == 64) {
      pyramid_tile64v_at(src, pitch, dst, j.g, ox, oy, write_l0);
    } else {
      const uintptr_t sa = reinterpret_cast<uintptr_t>(src), da = reinterpret_cast<uintptr_t>(dst);
      const int v4 = ((pitch % 4) == 0 && (sa % 4) == 0 && (W0 % 4) == 0 && (da % 4) == 0) ? 1 : 0;
      pyramid_tile_at<TILE>(src, pitch, dst, j.g, v4, ox, oy, write_l0);
    }
  }
}

// pyramid_block over the frames of a window: blockIdx.y = stream * n_frames + frame.
template <int LV>
__global__ __launch_bounds__(256) void pyramid_window_block_kernel(const WinJob* __restrict__ jobs, PyrWinSrc srcs,
                                                                   int n_frames) {
  constexpr int B = 1 << (LV - 1);
  const int z = blockIdx.y, js = z / n_frames, f = z - js * n_frames;
  const WinJob& j = jobs[js];
  const int nbx = j.g.W[0] / B, t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nbx * (j.g.H[0] / B)) return;
  pyramid_block<LV>(srcs.src[js] + f * srcs.stride[js], srcs.pitch[js], j.dst + f * j.dst_stride, j.g, t % nbx, t / nbx,
                    srcs.write_l0[js] != 0);
}

hipError_t launch_pyramid_window(const WinJob* d_jobs, const PyrWinSrc& srcs, int n_streams, int n_frames, int max_w,
                                 int max_h, int levels, bool block, hipStream_t s) {
  if (n_streams < 1 || n_streams > kPyrArgJobs || n_frames < 1 || (int64_t)n_streams * n_frames > 65535)
    return hipErrorInvalidValue;
  if (block) {  // every stream passed pyramid_block_ok for every frame
    const int B = 1 << (levels - 1), n = (max_w / B) * (max_h / B);
    if (levels == 4)
      hipLaunchKernelGGL(pyramid_window_block_kernel<4>, dim3((n + 255) / 256, n_streams * n_frames), dim3(256), 0, s,
                         d_jobs, srcs, n_frames);
    else
      hipLaunchKernelGGL(pyramid_window_block_kernel<3>, dim3((n + 255) / 256, n_streams * n_frames), dim3(256), 0, s,
                         d_jobs, srcs, n_frames);
    return hipGetLastError();
  }
  // several tiles of a row per workgroup where one each is many turns of the chip:
  // four, or two where four would leave places idle in a row.  5 levels, 9 frames a
  // stream, in us with one, two and four tiles: 752x480, 2 streams (1728 tiles) 6.5,
  // 7.0, 10.0; 5 (4320) 14.7, 13.2, 12.9; 8 19.8, 18.0, 17.4.  1001x700, one (1584)
  // 9.0, 7.8, 10.5; 2 (3168) 17.6, 13.5, 12.8.  320x240 (rows of 5 tiles), 24 (4320)
  // 13.0, 12.9, 13.9; 64 23.5, 22.2, 28.4.
  const int T = levels <= 7 ? 64 : 128, nx = (max_w + T - 1) / T, ny = (max_h + T - 1) / T, nz = n_streams * n_frames;
  const int tiles = (int64_t)nx * ny * nz <= 3072 ? 1 : 8 * ((nx + 3) / 4 * 4 - nx) <= nx ? 4 : 2;
  const dim3 grid((nx + tiles - 1) / tiles, ny, nz);
  if (levels <= 7)
    hipLaunchKernelGGL(pyramid_window_kernel<64>, grid, dim3(256), 0, s, d_jobs, srcs, n_frames, tiles);
  else
    hipLaunchKernelGGL(pyramid_window_kernel<128>, grid, dim3(256), 0, s, d_jobs, srcs, n_frames, tiles);
  return hipGetLastError();
}

hipError_t launch_pyramid_batch(const PyrJob* d_jobs, int n_jobs, int max_w, int max_h, int levels, hipStream_t s) {
  if (levels <= 7)
    hipLaunchKernelGGL(pyramid_batch_kernel<64>, dim3((max_w + 63) / 64, (max_h + 63) / 64, n_jobs), dim3(256), 0, s,
                       d_jobs);
  else
    hipLaunchKernelGGL(pyramid_batch_kernel<128>, dim3((max_w + 127) / 128, (max_h + 127) / 128, n_jobs), dim3(256),
                       0, s, d_jobs);
  return hipGetLastError();
}

}  // namespace dpt
