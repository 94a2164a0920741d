// The per-step sweep of Alg. 1: score every unexplored configuration
// (Sect. 3.6, score equation), normalise and quantise the scores
// (score-normalisation equation), and draw the next configuration by an
// exact integer inverse-CDF search (Sect. 3.7).
//
// Data layout (all over valid indices l):
//   P[c][stride]   model predictions, float32, one contiguous row per counter
//   explored       bitmask, bit l % 32 of word l / 32
//   s[stride]      float32 scores of the current step
//   bsum[n_blocks] uint64 sums of the quantised weights of each block of
//                  2^block_log2 configurations
//   acc[2][64]     per-step min / max / count accumulators, two sets used by
//                  alternate steps (the step using one set clears the other)
//
// Kernels per step (three launches up to the first draw; spaces of up to
// 32,768 configurations and restricted steps of up to 8,192 neighbours have
// all of it in one, small_step and nb_step below):
//   score_pass    4 configurations per thread, float4 loads of up to 8
//                 counter rows issued before any arithmetic; float32 with
//                 every operation rounded (this file is built without
//                 contraction): t = (x - a) / (a + x); s = s + dpc * t,
//                 counters ascending; the profiled configuration counts as
//                 explored.  Per-workgroup min / max of s over unexplored
//                 configurations go to one of 64 accumulator slots with
//                 order-preserving uint32 atomics.
//   weight_pass   one workgroup per block: q = rint(w * 2^23) and the block
//                 sum (plain stores; the kernel boundary publishes them to
//                 every XCD, which a device-scope handoff inside one launch
//                 would pay for with an L2 write-back per workgroup)
//   draw          one workgroup per draw; the step's first draw also marks the
//                 profiled configuration explored.
// A draw: one scan of the block sums gives Q and the block holding
// r = mulhi64(U, Q); recompute that block's q and scan it to l with
// prefix_l <= r < prefix_l + q_l; mark l explored and subtract q_l from its
// block sum (Alg. 1 zeroes S_l before the next draw of the iteration).  The
// result goes to pinned host memory in words that carry the draw's sequence
// number, which the host polls.  Every phase issues all of its loads before
// the first use, so a draw costs about two dependent memory round trips.
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "expert.h"

namespace cgs {

namespace {

constexpr int kScoreThreads = 256;
constexpr int kWeightThreads = 256;
constexpr int kDrawThreads = 256;
constexpr int kRowsInFlight = 8;
constexpr uint32_t kScoreGrid = 2048; // 8 workgroups of 256 threads per CU

// Combines the kAccSlots accumulator slots: wave 0 loads one slot per lane
// and reduces across the wave; the result is broadcast through LDS.  Every
// thread of the block must call it (it contains a barrier).
__device__ __forceinline__ StepAccSums reduce_slots(const StepAcc *__restrict__ slots) {
  static_assert(kAccSlots == kWave, "one slot per lane");
  __shared__ StepAccSums shared_sums;
  if (threadIdx.x < kWave) {
    const StepAcc a = slots[threadIdx.x];
    const uint32_t mn = wave_umin(a.min_key), mx = wave_umax(a.max_key);
    const uint32_t n = wave_sum(a.n_unexplored);
    if (threadIdx.x == 0) shared_sums = StepAccSums{mn, mx, n};
  }
  __syncthreads();
  return shared_sums;
}

template <bool kStream> __device__ __forceinline__ float4 load_row(const float *p) {
  if constexpr (kStream) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    const f4 v = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(p));
    return make_float4(v.x, v.y, v.z, v.w);
  } else {
    return *reinterpret_cast<const float4 *>(p);
  }
}

// Scores the 4 configurations of this thread in `tile` (4 * kScoreThreads
// configurations per tile) and folds the unexplored ones into the running
// min / max keys and count.  Counters ctr[0..n) with changes delta[].
// kStream: the rows are loaded past the caches.
template <int RIF = kRowsInFlight, bool kStream = false>
__device__ __forceinline__ void score_tile(const float *__restrict__ P, uint64_t stride,
                                           uint32_t profile, int n, const uint32_t *ctr,
                                           const float *delta,
                                           const uint32_t *__restrict__ explored,
                                           uint32_t n_valid, float *__restrict__ s_out,
                                           uint32_t tile, uint32_t &kmin, uint32_t &kmax,
                                           uint32_t &cnt) {
  const uint32_t l0 = 4u * (tile * kScoreThreads + threadIdx.x);
  if (l0 >= n_valid) return;
  float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;
  const uint32_t word = explored[l0 >> 5];
  uint32_t ex4 = (word >> (l0 & 31u)) & 0xfu;
  // configurations past the end and the profiled one count as explored
  const uint32_t tail = n_valid - l0;
  if (tail < 4u) ex4 |= (0xfu << tail) & 0xfu;
  if (profile - l0 < 4u) ex4 |= 1u << (profile - l0);
  const float *__restrict__ col = P + l0;
  for (int j0 = 0; j0 < n; j0 += RIF) {
    float4 x[RIF];
    float av[RIF];
#pragma unroll
    for (int u = 0; u < RIF; ++u) {
      if (j0 + u < n) {
        const size_t row = (size_t)ctr[j0 + u] * stride;
        x[u] = load_row<kStream>(col + row);
        av[u] = P[row + profile];
      }
    }
#pragma unroll
    for (int u = 0; u < RIF; ++u) {
      if (j0 + u < n && av[u] != 0.0f) { // a_p == 0: counter not in PC_used
        const float ap = av[u];
        const float d = delta[j0 + u];
        {
          const float t = (x[u].x - ap) / (ap + x[u].x);
          s0 = (x[u].x != 0.0f) ? s0 + d * t : s0;
        }
        {
          const float t = (x[u].y - ap) / (ap + x[u].y);
          s1 = (x[u].y != 0.0f) ? s1 + d * t : s1;
        }
        {
          const float t = (x[u].z - ap) / (ap + x[u].z);
          s2 = (x[u].z != 0.0f) ? s2 + d * t : s2;
        }
        {
          const float t = (x[u].w - ap) / (ap + x[u].w);
          s3 = (x[u].w != 0.0f) ? s3 + d * t : s3;
        }
      }
    }
  }
  *reinterpret_cast<float4 *>(s_out + l0) = make_float4(s0, s1, s2, s3);
  const float sv[4] = {s0, s1, s2, s3};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (!((ex4 >> e) & 1u)) {
      const uint32_t k = float_key(sv[e]);
      kmin = min(kmin, k);
      kmax = max(kmax, k);
      ++cnt;
    }
  }
}

// Block-wide reduction of the min / max keys and count; thread 0 adds them
// to accumulator slot `slot` (skipped when nothing was unexplored).
__device__ __forceinline__ void flush_acc(uint32_t kmin, uint32_t kmax, uint32_t cnt,
                                          StepAcc *slot) {
  __shared__ uint32_t red[3][kScoreThreads / kWave];
  kmin = wave_umin(kmin);
  kmax = wave_umax(kmax);
  cnt = wave_sum(cnt);
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) {
    red[0][wave] = kmin;
    red[1][wave] = kmax;
    red[2][wave] = cnt;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kScoreThreads / kWave; ++w) {
      kmin = min(kmin, red[0][w]);
      kmax = max(kmax, red[1][w]);
      cnt += red[2][w];
    }
    if (cnt != 0u) {
      atomicMin(&slot->min_key, kmin);
      atomicMax(&slot->max_key, kmax);
      atomicAdd(&slot->n_unexplored, cnt);
    }
  }
}

// Scores 4 configurations per thread over tiles of 4 * kScoreThreads
// configurations, grid-stride, so few workgroups update the accumulators.
// With prof_dev, the profiled configuration is read from device memory
// (written there by the previous step's draw) instead of `profile`.
template <bool kStream>
__global__ __launch_bounds__(kScoreThreads) void score_pass(
    const float *__restrict__ P, uint64_t stride, uint32_t profile,
    const uint32_t *__restrict__ prof_dev, ActiveCounters act,
    const uint32_t *__restrict__ explored, uint32_t n_valid, float *__restrict__ s_out,
    StepAcc *__restrict__ acc) {
  if (prof_dev) profile = *prof_dev;
  uint32_t kmin = 0xffffffffu, kmax = 0u, cnt = 0u;
  const int n = profile < n_valid ? act.n : 0;
  const uint32_t n_tiles = (n_valid + 4u * kScoreThreads - 1) / (4u * kScoreThreads);
  for (uint32_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x)
    score_tile<kRowsInFlight, kStream>(P, stride, profile, n, act.ctr, act.delta, explored, n_valid,
                                       s_out, tile, kmin, kmax, cnt);
  flush_acc(kmin, kmax, cnt, acc + (blockIdx.x & (kAccSlots - 1)));
}

// Folds the accumulator slot each lane of wave 0 loaded into the step's
// min / max / count and leaves them in `out` (LDS).  No barrier: the caller
// publishes `out` with its next one.
__device__ __forceinline__ void reduce_slot_values(const StepAcc &slot, StepAccSums *out) {
  if (threadIdx.x < kWave) {
    const uint32_t mn = wave_umin(slot.min_key), mx = wave_umax(slot.max_key);
    const uint32_t n = wave_sum(slot.n_unexplored);
    if (threadIdx.x == 0) *out = StepAccSums{mn, mx, n};
  }
}

// Sources of quantised weights for a draw.  A thread weighs runs of
// kRunWeights consecutive positions: load() issues every load of a run (from
// clamped addresses, so that no branch separates them; their arrays are
// padded to whole runs), weigh() turns it into weights, 0 for the positions
// of `out` (bit e: first + e) and past the end.  The step's s_min / s_max
// come from its accumulator slots in three stages, so a draw can overlap
// their load with its first loads: stage_load (every thread), stage_reduce
// (after the caller's own loads), then a barrier, then stage_read.
constexpr uint32_t kRunWeights = 16;

// Positions first .. first + kRunWeights - 1 at or past n.
__device__ __forceinline__ uint32_t past_end(uint32_t first, uint32_t n) {
  return first >= n ? 0xffffu : n - first < kRunWeights ? (0xffffu << (n - first)) & 0xffffu : 0u;
}

// The scores of a full step; explored configurations and the profiled one
// weigh 0.
struct ScoreWeights {
  const float *s;
  uint32_t *explored;
  uint32_t n;
  uint32_t profile;
  const StepAcc *acc;
  float gamma, w_min;
  StepNorm nm{};
  StepAcc slot{};
  struct Run {
    float4 s[kRunWeights / 4];
    uint4 raw[kRunWeights / 4];
    uint32_t mask;
  };
  __device__ void stage_load() {
    if (threadIdx.x < kWave) slot = acc[threadIdx.x];
  }
  __device__ void stage_reduce(StepAccSums *sh) const { reduce_slot_values(slot, sh); }
  __device__ void stage_read(const StepAccSums *sh) {
    nm = step_norm(key_float(sh->min_key), key_float(sh->max_key), gamma, w_min);
  }
  __device__ uint32_t operator()(uint32_t l) const {
    if (l >= n) return 0u;
    return quantized_weight(s[l], explored_bit(explored, l) || l == profile, nm);
  }
  __device__ void load(uint32_t first, const uint32_t *idx, Run &r) const {
    const uint32_t f = first < n ? first : 0u;
    r.mask = explored[f >> 5];
#pragma unroll
    for (uint32_t k = 0; k < kRunWeights / 4; ++k) {
      r.s[k] = reinterpret_cast<const float4 *>(s + f)[k];
      // the raw indices arrive with the scores: the pick's costs no further
      // round trip
      r.raw[k] = reinterpret_cast<const uint4 *>(idx + f)[k];
    }
  }
  __device__ void weigh(uint32_t first, const Run &r, uint32_t out,
                        uint32_t (&q)[kRunWeights]) const {
    uint32_t ex = out | past_end(first, n) | (r.mask >> (first & 31u) & 0xffffu);
    if (profile - first < kRunWeights) ex |= 1u << (profile - first);
    auto all = [&](auto wide) { // the choice of division path is made once
#pragma unroll
      for (uint32_t k = 0; k < kRunWeights / 4; ++k) {
        const float v[4] = {r.s[k].x, r.s[k].y, r.s[k].z, r.s[k].w};
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e)
          q[4 * k + e] =
              quantized_weight_t<decltype(wide)::value>(v[e], (ex >> (4 * k + e)) & 1u, nm);
      }
    };
    if (nm.wide) all(std::true_type{});
    else all(std::false_type{});
  }
  __device__ uint32_t raw_at(const Run &r, uint32_t e, uint32_t, const uint32_t *) const {
    uint32_t v = 0;
#pragma unroll
    for (uint32_t k = 0; k < kRunWeights / 4; ++k) {
      const uint32_t w[4] = {r.raw[k].x, r.raw[k].y, r.raw[k].z, r.raw[k].w};
#pragma unroll
      for (uint32_t i = 0; i < 4; ++i) v = e == 4 * k + i ? w[i] : v;
    }
    return v;
  }
  __device__ void remove(uint32_t l) const { atomicOr(&explored[l >> 5], 1u << (l & 31u)); }
  __device__ uint32_t valid_of(uint32_t l) const { return l; }
};
// Caller-given weights.
struct ArrayWeights {
  uint32_t *q;
  uint32_t n;
  struct Run {
    uint4 q[kRunWeights / 4];
  };
  __device__ void stage_load() {}
  __device__ void stage_reduce(StepAccSums *) const {}
  __device__ void stage_read(const StepAccSums *) {}
  __device__ void load(uint32_t first, const uint32_t *, Run &r) const {
    const uint32_t f = first < n ? first : 0u;
#pragma unroll
    for (uint32_t k = 0; k < kRunWeights / 4; ++k) r.q[k] = reinterpret_cast<const uint4 *>(q + f)[k];
  }
  __device__ void weigh(uint32_t first, const Run &r, uint32_t out,
                        uint32_t (&w)[kRunWeights]) const {
    const uint32_t ex = out | past_end(first, n);
#pragma unroll
    for (uint32_t k = 0; k < kRunWeights / 4; ++k) {
      const uint32_t v[4] = {r.q[k].x, r.q[k].y, r.q[k].z, r.q[k].w};
#pragma unroll
      for (uint32_t e = 0; e < 4; ++e) w[4 * k + e] = (ex >> (4 * k + e)) & 1u ? 0u : v[e];
    }
  }
  __device__ uint32_t raw_at(const Run &, uint32_t, uint32_t l, const uint32_t *) const { return l; }
  __device__ void remove(uint32_t l) const { q[l] = 0u; }
  __device__ uint32_t valid_of(uint32_t l) const { return l; }
};
// Quantised weights of a restricted step's candidates (position l in
// candidate order): drawing candidate l removes it and marks its
// configuration nb[l] explored.
struct NbWeights : ArrayWeights {
  const uint32_t *nb;
  uint32_t *explored;
  __device__ uint32_t raw_at(const Run &, uint32_t, uint32_t l, const uint32_t *idx) const {
    return idx[nb[l]];
  }
  __device__ void remove(uint32_t l) const {
    q[l] = 0u;
    atomicOr(&explored[nb[l] >> 5], 1u << (nb[l] & 31u));
  }
  __device__ uint32_t valid_of(uint32_t l) const { return nb[l]; }
};

// The draw result lives in mapped, coherent pinned host memory: four 64-bit
// words, each carrying 32 bits of the result and the draw's sequence number,
// stored with system scope.  The host (which polls instead of waiting for
// the stream) takes the result once all four words carry the number, so the
// stores need no order among them and the device no release fence, whose
// write-back of the L2 cost about 1 us of every draw.
__device__ __forceinline__ void publish(DrawResult *res, uint32_t valid, uint32_t raw,
                                        uint64_t total, uint64_t seq) {
  const uint32_t part[4] = {valid, raw, (uint32_t)total, (uint32_t)(total >> 32)};
#pragma unroll
  for (int i = 0; i < 4; ++i)
    __hip_atomic_store(&res->word[i], (uint64_t)part[i] << 32 | (uint32_t)seq, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

static_assert(kNoIndex == kNoProfile, "a draw without a pick leaves no profile");

// n draws, one after another, by one workgroup of NT threads; draw i uses
// u64[i] and publishes into res[i] under sequence number seq0 + i.
//  1. Thread t owns the contiguous run of block sums [t * per, t * per + per);
//     one exclusive scan over the run totals gives Q and, for the thread
//     whose run holds r, the block b with prefix_b <= r < prefix_b + bsum_b.
//  2. Every thread takes 2^block_log2 / NT consecutive configurations of
//     block b; a second scan finds l with prefix_l <= r' < prefix_l + q_l.
// The winner removes l; the run's owner subtracts q_l.
// Bound: the dependent round trips to memory of one workgroup (block sums,
// then scores with their raw indices; a further draw of a series waits for
// scores only, the run totals stay in registers) and its instruction issue:
// with 1,024 threads the two scans alone put 16 waves' instructions on four
// SIMDs, so a draw has 256 threads of 16 configurations.  The barriers order
// LDS only: removals are in flight across them, and the series keeps its own
// picks out of later draws.
// Measured (a draw launch): 5.6 us on 4.0M configurations and 5.2 us on
// 7,616, four further draws of one series 14.5 us; 7.9, 7.7 and 28 us with
// 1,024 threads, scans through the LDS crossbar, __syncthreads, the raw
// index fetched after the pick and a releasing store per result.  16 block
// sums in the first round trip: 6.0, 5.7 and 15.9 us (more instructions for
// the few sums there are).  Of spaces with more than 2,048 blocks the further
// sums are loaded 16 bytes at a time: the 64 lanes of a load lie in 64 cache
// lines, so the loads themselves bound it (a draw and its host turn, 8 bytes a
// load -> 16: 16,384 blocks 20.1 -> 17.3 us, 65,536 45.4 -> 30.9; 21.3 and 43.1
// with 1,024 threads; 32 sums a round trip 20.5 and 45.3).  Larger blocks: 2^13
// configurations 13.5 us (16.1 with 1,024 threads), 2^16 42 (56), 2^20 513
// (1,055) on 16.8M configurations.
template <int NT, typename W>
__device__ void draw_series(W &wsrc, int block_log2, uint64_t *__restrict__ bsum,
                            uint32_t n_blocks, int n, const uint64_t *u64,
                            const uint32_t *__restrict__ idx, DrawResult *__restrict__ res,
                            uint64_t seq0, uint32_t *__restrict__ prof_out = nullptr) {
  __shared__ uint64_t scratch[NT / kWave];
  __shared__ StepAccSums sums;
  __shared__ uint32_t found_block;
  __shared__ uint64_t found_rem;
  __shared__ uint32_t picked; // q of the pick, 0 without one
  __shared__ uint32_t pick_pos[kMaxDrawSeries], pick_valid[kMaxDrawSeries],
      pick_raw[kMaxDrawSeries];
  __shared__ uint64_t pick_total[kMaxDrawSeries];
  const uint32_t tid = threadIdx.x;

  wsrc.stage_load();
  constexpr uint32_t kChunk = 8; // block sums loaded per round trip
  uint32_t per = (n_blocks + NT - 1) / NT;
  if (per > kChunk) per = (per + 1u) & ~1u; // runs start at even blocks
  const uint32_t b0 = min(n_blocks, tid * per);
  const uint32_t b1 = min(n_blocks, b0 + per);
  uint64_t mine, run0[kChunk];   // the run's total and its first block sums
  auto load_sums = [&](uint32_t c, uint64_t (&v)[kChunk]) {
#pragma unroll
    for (uint32_t k = 0; k < kChunk; ++k) v[k] = bsum[min(c + k, n_blocks - 1)];
    uint64_t sum = 0;
#pragma unroll
    for (uint32_t k = 0; k < kChunk; ++k) {
      v[k] = c + k < b1 ? v[k] : 0ull;
      sum += v[k];
    }
    return sum;
  };
  // further sums two a load, as the lanes' loads of one instruction lie in as many
  // cache lines: the array is padded to an even number
  constexpr uint32_t kMore = 16;
  auto load_pairs = [&](uint32_t c, uint64_t (&v)[kMore]) {
    ulonglong2 w[kMore / 2];
#pragma unroll
    for (uint32_t k = 0; k < kMore / 2; ++k)
      w[k] = *reinterpret_cast<const ulonglong2 *>(bsum + min(c + 2 * k, (n_blocks - 1) & ~1u));
    uint64_t sum = 0;
#pragma unroll
    for (uint32_t k = 0; k < kMore; ++k) {
      v[k] = c + k < b1 ? (k & 1u ? w[k / 2].y : w[k / 2].x) : 0ull;
      sum += v[k];
    }
    return sum;
  };
  if (n_blocks != 0) {
    mine = load_sums(b0, run0);
    for (uint32_t c = b0 + kChunk; c < b1; c += kMore) {
      uint64_t v[kMore];
      mine += load_pairs(c, v);
    }
  } else {
    mine = 0;
  }
  wsrc.stage_reduce(&sums);
  for (int i = 0; i < n; ++i) {
    uint64_t Q;
    const uint64_t pre = block_excl_scan<NT, true>(mine, scratch, Q); // barriers publish sums
    if (i == 0) wsrc.stage_read(&sums);
    if (tid == 0) { // until the draw has a pick
      picked = 0;
      pick_pos[i] = kNoIndex;
      pick_valid[i] = kNoIndex;
      pick_raw[i] = kNoIndex;
      pick_total[i] = Q;
    }
    if (Q == 0) continue; // uniform
    const uint64_t r = __umul64hi(u64[i], Q);
    const bool owner = mine != 0 && pre <= r && r < pre + mine;
    if (owner) {
      uint64_t run = pre;
      uint32_t at = kNoIndex;
      uint64_t rem = 0;
      auto find = [&](uint32_t c, const auto &v) {
#pragma unroll
        for (uint32_t k = 0; k < sizeof(v) / sizeof(v[0]); ++k) {
          const bool hit = at == kNoIndex && r < run + v[k];
          rem = hit ? r - run : rem;
          at = hit ? c + k : at;
          run += v[k];
        }
      };
      find(b0, run0);
      for (uint32_t c = b0 + kChunk; c < b1 && at == kNoIndex; c += kMore) {
        uint64_t v[kMore];
        load_pairs(c, v);
        find(c, v);
      }
      found_block = at;
      found_rem = rem;
    }
    lds_barrier();
    const uint32_t blk = found_block;
    const uint64_t rem = found_rem;

    // 2^block_log2 / NT consecutive configurations per thread, kRunWeights
    // at a time; the weights of the first run stay in registers
    const uint32_t per2 = (1u << block_log2) / NT;
    const uint32_t first = (blk << block_log2) + tid * per2;
    auto weigh = [&](uint32_t f, const typename W::Run &run, uint32_t (&q)[kRunWeights]) {
      uint32_t out = 0; // this series' earlier picks
      for (int j = 0; j < i; ++j)
        if (pick_pos[j] - f < kRunWeights) out |= 1u << (pick_pos[j] - f);
      wsrc.weigh(f, run, out, q);
      uint64_t sum = 0;
#pragma unroll
      for (uint32_t e = 0; e < kRunWeights; ++e) sum += q[e];
      return sum;
    };
    typename W::Run run;
    uint32_t q[kRunWeights];
    wsrc.load(first, idx, run);
    const uint64_t sum0 = weigh(first, run, q);
    uint64_t mine2 = sum0;
    for (uint32_t c = kRunWeights; c < per2; c += kRunWeights) {
      typename W::Run more;
      uint32_t t[kRunWeights];
      wsrc.load(first + c, idx, more);
      mine2 += weigh(first + c, more, t);
    }
    uint64_t blk_total;
    const uint64_t pre2 = block_excl_scan<NT, true>(mine2, scratch, blk_total);
    if (mine2 != 0 && pre2 <= rem && rem < pre2 + mine2) {
      uint32_t f = first, at = kNoIndex, ql = 0;
      uint64_t below = pre2;
      auto find = [&]() {
#pragma unroll
        for (uint32_t e = 0; e < kRunWeights; ++e) {
          const bool hit = at == kNoIndex && rem < below + q[e];
          at = hit ? e : at;
          ql = hit ? q[e] : ql;
          below += q[e];
        }
      };
      find();
      for (uint32_t c = kRunWeights; at == kNoIndex && c < per2; c += kRunWeights) {
        f = first + c;
        wsrc.load(f, idx, run);
        weigh(f, run, q);
        find();
      }
      const uint32_t l = f + at;
      picked = ql;
      pick_pos[i] = l;
      pick_valid[i] = wsrc.valid_of(l);
      pick_raw[i] = wsrc.raw_at(run, at, l, idx);
      wsrc.remove(l);
    }
    lds_barrier();
    const uint32_t ql = picked;
    if (owner && ql != 0) {
      mine -= ql;
#pragma unroll
      for (uint32_t k = 0; k < kChunk; ++k)
        if (blk == b0 + k) run0[k] -= ql;
      bsum[blk] -= ql;
    }
  }
  // The results leave together, one thread each.  (No pick although Q > 0:
  // the block sums disagree with the weights.)
  lds_barrier();
  if (tid < (uint32_t)n) {
    if (prof_out && tid == 0) *prof_out = pick_valid[0]; // kNoIndex == kNoProfile
    publish(res + tid, pick_valid[tid], pick_raw[tid], pick_total[tid], seq0 + tid);
  }
}

// Sum of the quantised weights of block `blk` (2^block_log2 configurations),
// returned to every thread.  The step's accumulator slots and the block's
// first 4096 scores are loaded together; s_min / s_max are known once both
// have arrived.
__device__ __forceinline__ uint64_t weight_block_sum(const float *__restrict__ s,
                                                     const uint32_t *__restrict__ explored,
                                                     uint32_t n_valid, uint32_t profile,
                                                     const StepAcc *__restrict__ acc, float gamma,
                                                     float w_min, int block_log2, uint32_t blk) {
  __shared__ uint64_t scratch[kWeightThreads / kWave];
  __shared__ StepAccSums sums;
  constexpr uint32_t kRound = 16u * kWeightThreads; // 4 float4 per thread
  const uint32_t base = blk << block_log2;
  const uint32_t end = min(n_valid, base + (1u << block_log2));
  StepAcc slot{};
  if (threadIdx.x < kWave) slot = acc[threadIdx.x];
  float4 sv[4];
  uint32_t ex[4];
  auto load_round = [&](uint32_t r0) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t l0 = r0 + 4u * (threadIdx.x + k * kWeightThreads);
      if (l0 < end) {
        sv[k] = *reinterpret_cast<const float4 *>(s + l0);
        ex[k] = explored[l0 >> 5];
      } else { // past the block: weight 0, like explored configurations
        sv[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        ex[k] = 0xffffffffu;
      }
    }
  };
  load_round(base);
  reduce_slot_values(slot, &sums);
  __syncthreads();
  const StepNorm nm = step_norm(key_float(sums.min_key), key_float(sums.max_key), gamma, w_min);
  // the choice of division path is made once per block, outside the loop
  auto weigh = [&](auto wide) {
    uint64_t sum = 0;
    for (uint32_t r0 = base;;) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        // no per-configuration branches: positions past the end (and the
        // profiled configuration) count as explored and weigh 0
        const uint32_t l0 = r0 + 4u * (threadIdx.x + k * kWeightThreads);
        uint32_t ex4 = (ex[k] >> (l0 & 31u)) & 0xfu;
        const uint32_t tail = end - l0;
        if (tail < 4u) ex4 |= (0xfu << tail) & 0xfu;
        if (profile - l0 < 4u) ex4 |= 1u << (profile - l0);
        const float ss[4] = {sv[k].x, sv[k].y, sv[k].z, sv[k].w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          sum += quantized_weight_t<decltype(wide)::value>(ss[e], (ex4 >> e) & 1u, nm);
      }
      r0 += kRound;
      if (r0 >= end) break;
      load_round(r0);
    }
    return sum;
  };
  const uint64_t sum = nm.wide ? weigh(std::true_type{}) : weigh(std::false_type{});
  return block_sum<kWeightThreads>(sum, scratch); // its barriers also retire `sums`
}

__device__ __forceinline__ void clear_acc(StepAcc *acc_next) {
  if (threadIdx.x < kAccSlots) {
    acc_next[threadIdx.x].min_key = 0xffffffffu;
    acc_next[threadIdx.x].max_key = 0u;
    acc_next[threadIdx.x].n_unexplored = 0u;
  }
}

// One workgroup per block of 2^block_log2 configurations: block sums of q.
__global__ __launch_bounds__(kWeightThreads) void weight_pass(
    const float *__restrict__ s, const uint32_t *__restrict__ explored, uint32_t n_valid,
    uint32_t profile, const uint32_t *__restrict__ prof_dev, const StepAcc *__restrict__ acc,
    StepAcc *__restrict__ acc_next, float gamma, float w_min, int block_log2,
    uint64_t *__restrict__ bsum) {
  if (prof_dev) profile = *prof_dev;
  if (blockIdx.x == 0) clear_acc(acc_next); // the next step's accumulators
  const uint64_t total = weight_block_sum(s, explored, n_valid, profile, acc, gamma, w_min,
                                          block_log2, blockIdx.x);
  if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

// One draw.  `profile` (or kNoProfile; read from prof_dev when given) is
// excluded and, when `mark_profile`, marked explored once the draw is done.
// With prof_out, the pick's valid index (kNoProfile when there is none) is
// also stored there for the next step.
__global__ __launch_bounds__(kDrawThreads) void draw_scores(
    const float *__restrict__ s, uint32_t *__restrict__ explored, uint32_t n_valid,
    uint32_t profile, const uint32_t *__restrict__ prof_dev, int mark_profile,
    const StepAcc *__restrict__ acc, float gamma, float w_min, int block_log2,
    uint64_t *__restrict__ bsum, uint32_t n_blocks, uint64_t u64,
    const uint32_t *__restrict__ idx, DrawResult *__restrict__ res, uint64_t seq,
    uint32_t *__restrict__ prof_out) {
  if (prof_dev) profile = *prof_dev;
  ScoreWeights w{s, explored, n_valid, profile, acc, gamma, w_min};
  draw_series<kDrawThreads>(w, block_log2, bsum, n_blocks, 1, &u64, idx, res, seq, prof_out);
  __syncthreads();
  if (threadIdx.x == 0 && mark_profile && profile < n_valid)
    atomicOr(&explored[profile >> 5], 1u << (profile & 31u));
}

// Further draws of one step (after its first), made one after another by
// one workgroup, each removing its pick before the next exactly as separate
// launches of draw_scores would.
__global__ __launch_bounds__(kDrawThreads) void draw_many(
    const float *__restrict__ s, uint32_t *__restrict__ explored, uint32_t n_valid,
    const StepAcc *__restrict__ acc, float gamma, float w_min, int block_log2,
    uint64_t *__restrict__ bsum, uint32_t n_blocks, DrawSeries series,
    const uint32_t *__restrict__ idx, DrawResult *__restrict__ res, uint64_t seq0) {
  ScoreWeights w{s, explored, n_valid, kNoProfile, acc, gamma, w_min};
  draw_series<kDrawThreads>(w, block_log2, bsum, n_blocks, series.n, series.u64, idx, res, seq0);
}

// ------------------------------------------------------------ small spaces
// A whole step of a space of at most kSmallMaxValid configurations in one
// launch: 512 configurations a workgroup are scored, and the workgroup that
// finishes last weighs all of them, keeps the weights in LDS and makes the
// step's draws.
// Bound: latency.  As separate launches (score, weight, draw, further draws)
// such a step is four kernel starts, each with its own chain of dependent
// round trips, and every draw weighs a block again; here the draws after the
// weighing cost two LDS barriers and one LDS read each.
// The workgroups meet on one counter: each adds 1 with release once its
// scores and its min / max slot are written (every wave waits for its own
// stores first, stores_done), the one that brings it to the number of
// workgroups goes on after an acquire (no workgroup waits).
// 512 threads: with 256 the last workgroup's single wave per SIMD leaves its
// weighing waiting on its own latencies (2.6 against 1.5 us on 7,616
// configurations), with 1,024 every barrier of a draw costs more (0.62 to
// 1.2 us a draw).
// Measured on 7,616 configurations, 9 to 13 active counters: 10.1 us with one
// draw and 12.4 us with five, against 16.5 and 31 us for the separate launches'
// kernels alone; of one with a draw about a quarter to the scores, a sixth for
// the handoff, three eighths to load and weigh, the rest the draw, its result and
// the block sums.
// kSmallMaxValid: one accumulator slot per workgroup, and the weights fit in
// the last workgroup's LDS.  It is also where the two ways meet: steps
// enqueued ahead take 10.5 against 16.7 us on 8,192 configurations, 12.9
// against 16.6 us on 16,384, 16.5 against 16.8 us on 32,768.
constexpr int kSmallThreads = 512;
constexpr uint32_t kSmallPer = 64; // weights per thread of the last workgroup
// Workgroups of a step of a batch, split evenly over its sessions: the release
// of each writes back the L2 of its die, one after another.  64 sessions of
// 7,616 configurations, five draws: 28.7 us with one or two workgroups a
// session, 31.7 us with four, 43.6 us with eight, 50 us with fifteen.
constexpr uint32_t kBatchSmallGroups = 128;
static_assert(kSmallMaxValid == kSmallThreads * kSmallPer, "one run per thread");
static_assert(kSmallMaxValid <= kAccSlots * kSmallThreads, "one accumulator slot per workgroup");
static_assert(kSmallPer <= kWave && kSmallPer % 4 == 0, "a wave searches a run at once");
// Words between the runs of `per` weights in LDS: an odd number of 16-byte
// units, so that threads reading their runs start in different banks.
__host__ __device__ constexpr uint32_t small_ld(uint32_t per) { return per + (per & 4u ? 0u : 4u); }

// Score of configuration l against the profiled one: counters ctr[0..n) with
// changes delta[], the loads of RIF counters in flight together.
template <int RIF>
__device__ __forceinline__ float score_one(const float *__restrict__ P, uint64_t stride,
                                           uint32_t profile, int n, const uint32_t *ctr,
                                           const float *delta, uint32_t l) {
  float s = 0.0f;
  for (int j0 = 0; j0 < n; j0 += RIF) {
    float x[RIF], a[RIF];
#pragma unroll
    for (int u = 0; u < RIF; ++u) {
      const float *row = P + (size_t)ctr[min(j0 + u, n - 1)] * stride;
      x[u] = row[l];
      a[u] = row[profile];
    }
#pragma unroll
    for (int u = 0; u < RIF; ++u) {
      if (j0 + u < n && a[u] != 0.0f) { // a_p == 0: counter not in PC_used
        const float t = (x[u] - a[u]) / (a[u] + x[u]);
        s = (x[u] != 0.0f) ? s + delta[j0 + u] * t : s;
      }
    }
  }
  return s;
}

// The same for configurations l .. l + 3 (l a multiple of 4, the rows padded):
// 16-byte loads, for workgroups that score many configurations each.
template <int RIF>
__device__ __forceinline__ float4 score_four(const float *__restrict__ P, uint64_t stride,
                                             uint32_t profile, int n, const uint32_t *ctr,
                                             const float *delta, uint32_t l) {
  float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int j0 = 0; j0 < n; j0 += RIF) {
    float4 x[RIF];
    float a[RIF];
#pragma unroll
    for (int u = 0; u < RIF; ++u) {
      const float *row = P + (size_t)ctr[min(j0 + u, n - 1)] * stride;
      x[u] = *reinterpret_cast<const float4 *>(row + l);
      a[u] = row[profile];
    }
#pragma unroll
    for (int u = 0; u < RIF; ++u) {
      if (j0 + u < n && a[u] != 0.0f) {
        const float d = delta[j0 + u], v[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float t = (v[e] - a[u]) / (a[u] + v[e]);
          s[e] = (v[e] != 0.0f) ? s[e] + d * t : s[e];
        }
      }
    }
  }
  return make_float4(s[0], s[1], s[2], s[3]);
}

// One session's step as its workgroups see it; the counters and the uniforms
// stay where the launch put them.
struct SmallView {
  const float *P;
  uint64_t stride;
  uint32_t profile, n_valid;
  uint32_t *explored;
  float *s;
  StepAcc *acc, *acc_next;
  float gamma, w_min;
  int32_t block_log2;
  uint32_t n_blocks;
  uint64_t *bsum;
  const uint32_t *idx;
  DrawResult *res;
  uint64_t seq0;
  uint32_t *prof_out;
  uint32_t per;
  FastDiv per4;
  int n_act, n_draws;
  const uint32_t *ctr;
  const float *delta;
  const uint64_t *u64;
};

// The last workgroup's part: weighs the n_valid scores, makes the draws and
// leaves the block sums.  Thread t owns the run of a.per consecutive weights
// from t * per (LDS words q[t * ld ..]).
struct SmallPicks { // position (kNoIndex: none) and Q of every draw, in LDS
  uint32_t pos[kMaxDrawSeries];
  uint64_t total[kMaxDrawSeries];
};
__device__ __forceinline__ void small_draws(const SmallView &a, uint32_t *q, SmallPicks &picks) {
  __shared__ uint64_t scratch[kSmallThreads / kWave];
  __shared__ StepAccSums sums;
  uint32_t *pick_pos = picks.pos;
  uint64_t *pick_total = picks.total;
  constexpr uint32_t kBlocks = (kSmallMaxValid + 4095) >> 12; // blocks hold 4096 or more
  __shared__ unsigned long long blk_sum[kBlocks];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, n_valid = a.n_valid, profile = a.profile;
  const uint32_t per = a.per, ld = small_ld(per), first = tid * per;
  const uint32_t n_quads = kSmallThreads * (per / 4);
  StepAcc slot{};
  if (tid < kWave) slot = a.acc[tid];
  // scores four at a time, kInFlight loads per thread together; positions
  // past the end weigh 0
  constexpr uint32_t kInFlight = 4;
  float4 v[kInFlight];
  uint32_t ew[kInFlight];
  auto load = [&](uint32_t q0) {
#pragma unroll
    for (uint32_t k = 0; k < kInFlight; ++k) {
      const uint32_t f = 4u * (q0 + k * kSmallThreads + tid);
      const uint32_t fc = f < n_valid ? f : 0u;
      v[k] = *reinterpret_cast<const float4 *>(a.s + fc);
      ew[k] = a.explored[fc >> 5] >> (fc & 31u);
    }
  };
  load(0);
  reduce_slot_values(slot, &sums);
  if (tid < kBlocks) blk_sum[tid] = 0ull;
  if (tid < (uint32_t)a.n_draws) pick_pos[tid] = kNoIndex;
  lds_barrier();
  const StepNorm nm = step_norm(key_float(sums.min_key), key_float(sums.max_key), a.gamma, a.w_min);
  auto weigh = [&](auto wide) {
    for (uint32_t q0 = 0;;) {
#pragma unroll
      for (uint32_t k = 0; k < kInFlight; ++k) {
        const uint32_t quad = q0 + k * kSmallThreads + tid, f = 4u * quad;
        uint32_t ex4 = ew[k];
        if (f >= n_valid) ex4 = 0xfu;
        else if (n_valid - f < 4u) ex4 |= 0xfu << (n_valid - f);
        if (profile - f < 4u) ex4 |= 1u << (profile - f);
        const float sv[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
        uint32_t w[4];
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e)
          w[e] = quantized_weight_t<decltype(wide)::value>(sv[e], (ex4 >> e) & 1u, nm);
        const uint32_t run = fastdiv(quad, a.per4); // its thread
        if (quad < n_quads)
          *reinterpret_cast<uint4 *>(q + f + run * (ld - per)) = make_uint4(w[0], w[1], w[2], w[3]);
      }
      q0 += kInFlight * kSmallThreads;
      if (q0 >= n_quads) break;
      load(q0);
    }
  };
  if (nm.wide) weigh(std::true_type{});
  else weigh(std::false_type{});
  lds_barrier();
  uint64_t mine = 0;
  for (uint32_t e = 0; e < per; e += 4) {
    const uint4 w = *reinterpret_cast<const uint4 *>(q + tid * ld + e);
    mine += (uint64_t)w.x + w.y + w.z + w.w;
  }
  for (int i = 0; i < a.n_draws; ++i) {
    uint64_t Q;
    const uint64_t pre = block_excl_scan<kSmallThreads, true>(mine, scratch, Q);
    if (tid == 0) pick_total[i] = Q;
    const uint64_t r = __umul64hi(a.u64[i], Q); // 0 when Q == 0: no owner
    const bool owner = pre <= r && r < pre + mine;
    const uint64_t own = __ballot(owner);
    if (own != 0) { // the owner's wave looks through its run, one weight per lane
      const int o = __ffsll((unsigned long long)own) - 1;
      const uint32_t run = (tid & ~63u) + (uint32_t)o;
      const uint64_t rem = (uint64_t)__shfl((long long)(r - pre), o);
      const uint64_t w = lane < per ? q[run * ld + lane] : 0u;
      const uint64_t incl = wave_incl_scan(w);
      if (rem < incl && incl - w <= rem) { // one lane: prefix <= rem < prefix + w
        const uint32_t l = run * per + lane;
        q[run * ld + lane] = 0u;
        pick_pos[i] = l;
        atomicOr(&a.explored[l >> 5], 1u << (l & 31u));
      }
      const uint64_t hit = __ballot(rem < incl && incl - w <= rem);
      const uint64_t ql = (uint64_t)__shfl((long long)w, __ffsll((unsigned long long)hit) - 1);
      if (owner) mine -= ql;
    }
  }
  lds_barrier();
  if (a.res && tid < (uint32_t)a.n_draws) {
    const uint32_t l = pick_pos[tid];
    const uint32_t raw = l != kNoIndex ? a.idx[l] : kNoIndex;
    if (a.prof_out && tid == 0) *a.prof_out = l; // kNoIndex == kNoProfile
    publish(a.res + tid, l, raw, pick_total[tid], a.seq0 + tid);
  }
  // the block sums as the draws left them, for further draws of this step
  const uint32_t lg = (uint32_t)a.block_log2, b0 = first >> lg;
  uint64_t lower = mine; // the run's part in its first block
  if (first < n_valid && (first + per - 1) >> lg != b0) {
    lower = 0;
    for (uint32_t e = 0; e < per; e += 4) { // blocks start at multiples of 4
      const uint4 w = *reinterpret_cast<const uint4 *>(q + tid * ld + e);
      if ((first + e) >> lg == b0) lower += (uint64_t)w.x + w.y + w.z + w.w;
    }
  }
  if (__all(lower == mine && b0 == __shfl(b0, 0))) { // one block: one addition per wave
    const uint64_t sum = wave_sum(mine);
    if (lane == 0 && sum != 0) atomicAdd(&blk_sum[b0], (unsigned long long)sum);
  } else {
    if (lower != 0) atomicAdd(&blk_sum[b0], (unsigned long long)lower);
    if (mine != lower) atomicAdd(&blk_sum[b0 + 1], (unsigned long long)(mine - lower));
  }
  lds_barrier();
  if (tid < a.n_blocks) a.bsum[tid] = blk_sum[tid];
}

// One workgroup's part of the step: group `group` of n_groups takes every
// n_groups-th tile of 512 configurations (2,048 where groups take several),
// and the rest of the step when it arrives last.  A single group needs no meeting.
__device__ __forceinline__ void small_body(const SmallView &a, uint32_t group, uint32_t n_groups,
                                           uint32_t *small_q, SmallPicks &picks) {
  __shared__ uint32_t red[3][kSmallThreads / kWave];
  __shared__ uint32_t arrived;
  const uint32_t tid = threadIdx.x, n_valid = a.n_valid, profile = a.profile;
  const int n = profile < n_valid ? a.n_act : 0;
  uint32_t kmin = 0xffffffffu, kmax = 0u, cnt = 0u;
  auto fold = [&](float s, bool ex) {
    const uint32_t key = float_key(s);
    kmin = min(kmin, ex ? 0xffffffffu : key);
    kmax = max(kmax, ex ? 0u : key);
    cnt += (uint32_t)__popcll(__ballot(!ex));
  };
  if (n_groups * kSmallThreads >= n_valid) { // one configuration per thread
    const uint32_t l = group * kSmallThreads + tid, lc = min(l, n_valid - 1);
    const uint32_t word = a.explored[lc >> 5];
    const float s = score_one<16>(a.P, a.stride, profile, n, a.ctr, a.delta, lc);
    if (l < n_valid) a.s[l] = s;
    fold(s, l >= n_valid || l == profile || ((word >> (lc & 31u)) & 1u));
  } else {
    for (uint32_t l0 = 4 * group * kSmallThreads; l0 < n_valid;
         l0 += 4 * n_groups * kSmallThreads) {
      const uint32_t l = l0 + 4 * tid, lc = l < n_valid ? l : 0u;
      const uint32_t word = a.explored[lc >> 5] >> (lc & 31u);
      const float4 s = score_four<8>(a.P, a.stride, profile, n, a.ctr, a.delta, lc);
      if (l < n_valid) *reinterpret_cast<float4 *>(a.s + l) = s;
      const float v[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
      for (uint32_t e = 0; e < 4; ++e)
        fold(v[e], l + e >= n_valid || l + e == profile || ((word >> e) & 1u));
    }
  }
  kmin = wave_umin(kmin);
  kmax = wave_umax(kmax);
  if ((tid & 63u) == 0) {
    red[0][tid >> 6] = kmin;
    red[1][tid >> 6] = kmax;
    red[2][tid >> 6] = cnt;
  }
  if (n_groups > 1) stores_done(); // the scores, for the group that arrives last
  __syncthreads();
  if (tid == 0) {
    StepAcc slot{red[0][0], red[1][0], red[2][0], 0u};
#pragma unroll
    for (int w = 1; w < kSmallThreads / kWave; ++w) {
      slot.min_key = min(slot.min_key, red[0][w]);
      slot.max_key = max(slot.max_key, red[1][w]);
      slot.n_unexplored += red[2][w];
    }
    a.acc[group].min_key = slot.min_key;
    a.acc[group].max_key = slot.max_key;
    a.acc[group].n_unexplored = slot.n_unexplored;
    if (n_groups > 1) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      arrived = atomicAdd(&a.acc_next[0].pad, 1u);
    }
  }
  __syncthreads(); // also publishes a single group's scores within the workgroup
  if (n_groups > 1) {
    if (arrived != n_groups - 1) return; // uniform over the workgroup
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (tid == 0) a.acc_next[0].pad = 0u;
  }
  small_draws(a, small_q, picks);
  clear_acc(a.acc_next); // the next step's accumulators
  if (tid == 0 && profile < n_valid)
    atomicOr(&a.explored[profile >> 5], 1u << (profile & 31u));
}

__global__ __launch_bounds__(kSmallThreads) void small_step(SmallStep a) {
  extern __shared__ uint32_t small_q[];
  __shared__ SmallPicks picks;
  const uint32_t profile = a.prof_dev ? *a.prof_dev : a.profile;
  const SmallView v{a.P,    a.stride, profile,      a.n_valid,  a.explored, a.s,
                    a.acc,  a.acc_next, a.gamma,    a.w_min,    a.block_log2, a.n_blocks,
                    a.bsum, a.idx,    a.res,        a.seq0,     a.prof_out, a.per,
                    a.per4, a.act.n,  a.series.n,   a.act.ctr,  a.act.delta, a.series.u64};
  small_body(v, blockIdx.x, gridDim.x, small_q, picks);
}

// The same step in every session of a batch of small spaces, `groups`
// workgroups a session; a session with no draws to make rests.
__global__ __launch_bounds__(kSmallThreads) void batch_small(
    const BatchSess *__restrict__ sess, const SmallJob *__restrict__ jobs, uint32_t groups,
    DrawResult *__restrict__ res) {
  extern __shared__ uint32_t small_q[];
  __shared__ SmallPicks picks;
  const uint32_t si = blockIdx.x / groups;
  const BatchSess &d = sess[si];
  const SmallJob &j = jobs[si];
  if (j.n_draws == 0) return; // uniform over the session's workgroups
  const SmallView v{d.P, d.stride, j.profile, d.n_valid, d.explored, d.s,
                    d.acc + j.parity * kAccSlots, d.acc + (j.parity ^ 1) * kAccSlots,
                    d.gamma, d.w_min, d.block_log2, d.n_blocks, d.bsum, d.idx,
                    res + (size_t)si * kMaxDrawSeries, j.seq0, nullptr, d.per, d.per4,
                    j.n_act, j.n_draws, j.ctr, j.delta, j.u64};
  small_body(v, blockIdx.x - si * groups, groups, small_q, picks);
}

// Alg. 1 of one session per workgroup, iteration after iteration: the runs of
// a batch share nothing, and a single workgroup needs no meeting, so a run
// needs the host for nothing until it ends.  Per iteration: the current
// configuration is tested and profiled (one thread: the expert system is 60
// operations), the step and its draws are small_body's, the picks' runtimes
// decide the next configuration.  The explored bits live in LDS meanwhile.
// Every run ends: an iteration makes at least one test, of at most max_tests.
// Bound: one CU per run; an iteration of 7,616 configurations takes 28 us, of
// which the scores take half.  64 runs of 150 tests there: 2.92 ms with a
// launch of batch_small, a copy and a wait per iteration (28.7 us of the 104 of
// one are the kernel's) -> 1.04 ms, 0.72 of them this kernel's.
__global__ __launch_bounds__(kSmallThreads) void batch_tune(const BatchSess *__restrict__ sess,
                                                            TuneArgs t) {
  extern __shared__ uint32_t small_q[];
  __shared__ SmallPicks picks;
  __shared__ uint32_t explored[kSmallMaxValid / 32];
  __shared__ TuneRun r;
  __shared__ double pc[24];
  __shared__ uint64_t u64[kMaxDrawSeries];
  __shared__ uint32_t ctr[24];
  __shared__ float delta[24], runtime[kMaxDrawSeries];
  __shared__ int32_t n_act, n_draws;
  const uint32_t si = blockIdx.x, tid = threadIdx.x;
  const BatchSess &d = sess[si];
  const uint32_t n_words = (d.n_valid + 31) / 32;
  const uint64_t *uni = t.uniforms + (size_t)si * t.stride_u;
  uint32_t *tested = t.tested + (size_t)si * t.cap;
  uint8_t *profiled = t.profiled + (size_t)si * t.cap;
  for (uint32_t w = tid; w < n_words; w += kSmallThreads) explored[w] = d.explored[w];
  if (tid == 0) r = t.run[si];
  __syncthreads();
  // thread 0: true ends the run
  auto test = [&](uint32_t l, bool prof, float rt) {
    tested[r.nt] = l; // below cap: a configuration is drawn once and profiled once
    profiled[r.nt] = prof ? 1 : 0;
    ++r.nt;
    if (!r.found && (double)rt <= t.thresh) r.found = r.nt;
    return (t.stop_at_well && r.found) || r.nt >= t.max_tests;
  };
  for (uint32_t it = 0; it < t.max_iters && r.state <= kTuneRunning; ++it) { // uniform
    const bool start = r.state == kTuneStart;
    if (!start && tid < 24) pc[tid] = t.counters[(size_t)r.c * 24 + tid];
    if (!start && tid == 24) runtime[0] = t.runtime[r.c];
    __syncthreads();
    if (tid == 0) {
      n_act = 0;
      n_draws = 0; // no step
      r.late = 0;
      if (start) {
        u64[0] = uni[r.u++];
        n_draws = 1;
      } else if (test(r.c, true, runtime[0])) {
        r.state = kTuneEnded;
      } else {
        bool finite = true;
        for (int i = 0; i < 24; ++i) finite = finite && isfinite(pc[i]);
        if (!finite) {
          r.state = kTuneBadCounters;
        } else if (r.u >= t.n_uniforms) {
          r.state = kTuneNoNumbers;
        } else {
          double b[18], dc[24];
          expert::evaluate(pc, t.ep, b, dc);
          int n = 0;
#pragma unroll
          for (int i = 0; i < 24; ++i) {
            const float f = (float)dc[i];
            if (f == 0.0f) continue;
            ctr[n] = (uint32_t)i;
            delta[n++] = f;
          }
          n_act = n;
          int k = 0;
          for (; k < (int)t.draws && r.u < t.n_uniforms; ++k) u64[k] = uni[r.u++];
          n_draws = k;
        }
      }
    }
    __syncthreads();
    if (n_draws == 0) break; // uniform
    const uint32_t profile = start ? kNoProfile : r.c;
    const int parity = r.parity;
    const SmallView v{d.P, d.stride, profile, d.n_valid, explored, d.s,
                      d.acc + parity * kAccSlots, d.acc + (parity ^ 1) * kAccSlots,
                      d.gamma, d.w_min, d.block_log2, d.n_blocks, d.bsum, d.idx,
                      nullptr, 0, nullptr, d.per, d.per4, n_act, n_draws, ctr, delta, u64};
    small_body(v, 0, 1, small_q, picks);
    if (tid < (uint32_t)n_draws)
      runtime[tid] = picks.pos[tid] != kNoIndex ? t.runtime[picks.pos[tid]] : 0.0f;
    __syncthreads(); // also orders this step's scores and accumulators with the next
    if (tid == 0) {
      r.cur_acc = parity;
      r.parity = parity ^ 1;
      r.profile = profile;
      r.n_act = (uint32_t)n_act;
      r.last_total = picks.total[n_draws - 1];
      ++r.steps;
      ++r.iters;
      r.late = 1;
      for (int k = 0; k < n_draws; ++k)
        if (picks.total[k] != 0 && picks.pos[k] == kNoIndex) r.state = kTuneNoPick;
      if (start && r.state == kTuneStart) {
        r.state = picks.total[0] == 0 ? kTuneEnded : kTuneRunning;
        r.c = picks.pos[0];
      } else if (r.state == kTuneRunning) {
        float best = INFINITY;
        bool next = false, stop = false;
        uint32_t next_c = 0;
        for (int k = 0; k < n_draws && !stop; ++k) {
          if (picks.total[k] == 0) { // no configuration left: the draws after it were not needed
            r.u -= (uint64_t)(n_draws - 1 - k);
            break;
          }
          if (test(picks.pos[k], false, runtime[k])) {
            stop = true;
          } else {
            if (runtime[k] <= best) {
              best = runtime[k];
              next_c = picks.pos[k];
              next = true;
            }
            if (k + 1 == n_draws && n_draws < (int)t.draws) r.state = kTuneNoNumbers;
          }
        }
        if (r.state == kTuneRunning) {
          if (stop || !next) r.state = kTuneEnded;
          else r.c = next_c;
        }
      }
    }
    __syncthreads();
  }
  __syncthreads();
  for (uint32_t w = tid; w < n_words; w += kSmallThreads) d.explored[w] = explored[w];
  if (tid == 0) t.run[si] = r;
}

// ------------------------------------------------------------ batched
// Score tiles of every session, grid-stride over the concatenated tile list;
// a workgroup flushes its accumulators whenever the session changes.
// RIF: counter rows in flight per thread; WPE: waves per SIMD the compiler
// plans registers for (the autotuner's variants).
// kStream as in score_pass, chosen for the batch as a whole.
template <int RIF, int WPE, bool kStream>
__global__ __launch_bounds__(kScoreThreads)
__attribute__((amdgpu_waves_per_eu(WPE, 8))) void batch_score(const BatchSess *__restrict__ sess,
                                                              const BatchStep *__restrict__ step,
                                                              const uint16_t *__restrict__ tile_sess,
                                                              uint32_t total_tiles) {
  uint32_t kmin = 0xffffffffu, kmax = 0u, cnt = 0u;
  uint32_t cur = 0xffffffffu;
  for (uint32_t t = blockIdx.x; t < total_tiles; t += gridDim.x) {
    const uint32_t si = tile_sess[t];
    if (si != cur) {
      if (cur != 0xffffffffu)
        flush_acc(kmin, kmax, cnt,
                  sess[cur].acc + step[cur].parity * kAccSlots + (blockIdx.x & (kAccSlots - 1)));
      kmin = 0xffffffffu;
      kmax = 0u;
      cnt = 0u;
      cur = si;
    }
    const BatchSess &d = sess[si];
    const BatchStep &st = step[si];
    const int n = st.profile < d.n_valid ? st.n_act : 0;
    score_tile<RIF, kStream>(d.P, d.stride, st.profile, n, st.ctr, st.delta, d.explored, d.n_valid, d.s,
               t - d.tile0, kmin, kmax, cnt);
  }
  if (cur != 0xffffffffu)
    flush_acc(kmin, kmax, cnt,
              sess[cur].acc + step[cur].parity * kAccSlots + (blockIdx.x & (kAccSlots - 1)));
}

// Weight blocks of every session, grid-stride over the concatenated block list.
__global__ __launch_bounds__(kWeightThreads) void batch_weight(
    const BatchSess *__restrict__ sess, const BatchStep *__restrict__ step,
    const uint16_t *__restrict__ blk_sess, uint32_t total_blocks) {
  for (uint32_t b = blockIdx.x; b < total_blocks; b += gridDim.x) {
    const uint32_t si = blk_sess[b];
    const BatchSess &d = sess[si];
    const BatchStep &st = step[si];
    const uint32_t lb = b - d.blk0;
    if (lb == 0) clear_acc(d.acc + (st.parity ^ 1) * kAccSlots);
    const uint64_t total =
        weight_block_sum(d.s, d.explored, d.n_valid, st.profile, d.acc + st.parity * kAccSlots,
                         d.gamma, d.w_min, d.block_log2, lb);
    if (threadIdx.x == 0) d.bsum[lb] = total;
  }
}

// One workgroup per session: its draw, then its profile is marked explored.
__global__ __launch_bounds__(kDrawThreads) void batch_draw(const BatchSess *__restrict__ sess,
                                                           const BatchStep *__restrict__ step) {
  const BatchSess &d = sess[blockIdx.x];
  const BatchStep &st = step[blockIdx.x];
  if (!st.draw) return;
  ScoreWeights w{d.s, d.explored, d.n_valid, st.profile, d.acc + st.parity * kAccSlots, d.gamma,
                 d.w_min};
  draw_series<kDrawThreads>(w, d.block_log2, d.bsum, d.n_blocks, 1, &st.u64, d.idx, d.res, st.seq);
  __syncthreads();
  if (threadIdx.x == 0 && st.profile < d.n_valid)
    atomicOr(&d.explored[st.profile >> 5], 1u << (st.profile & 31u));
}

// ------------------------------------------------------------ neighbourhood
// The restricted step scores only candidates near the profiled configuration:
// one thread per candidate (before filtering) unranks it, keeps it if it is
// valid and unexplored, and scores it with the float32 chain of the full
// pass; one workgroup then compacts the kept candidates in candidate order,
// quantises their weights over the kept set and forms the block sums.
constexpr int kNbThreads = 256;
constexpr uint32_t kNbMaxSubsets = 32 + 32 * 31 / 2 + 32 * 31 * 30 / 6; // radius <= 3

// Raw index of candidate f: its subset of changed parameters (the last one
// whose first candidate <= f) by binary search of off, then the new digits.
__device__ __forceinline__ uint32_t nb_unrank(const NbStep &st, const uint32_t *off,
                                              const uint32_t *__restrict__ sub_code, uint32_t f) {
  uint32_t lo = 0, hi = st.n_subsets;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (off[mid] <= f) lo = mid;
    else hi = mid;
  }
  const uint32_t code = sub_code[lo];
  uint32_t u = f - off[lo];
  int64_t raw = st.profile_raw;
  // new digits of the changed parameters, the last one fastest; the
  // profile's own digit is skipped
  for (int k = (int)(code >> 24) - 1; k >= 0; --k) {
    const uint32_t j = (code >> (8 * k)) & 0xffu;
    const uint32_t alt = st.radix[j] - 1u;
    const uint32_t a = u % alt;
    u /= alt;
    const uint32_t pd = st.pdig[j];
    const uint32_t v = a < pd ? a : a + 1u;
    raw += ((int64_t)v - (int64_t)pd) * (int64_t)st.stride[j];
  }
  return (uint32_t)raw;
}
// Whether raw index rw is valid and unexplored; l receives its valid index
// when it is valid.
__device__ __forceinline__ bool nb_keep(uint32_t rw, const uint32_t *__restrict__ mask,
                                        const uint32_t *__restrict__ rank,
                                        const uint32_t *__restrict__ explored, uint32_t &l) {
  const uint32_t word = mask[rw >> 5], rk = rank[rw >> 5];
  if (!((word >> (rw & 31u)) & 1u)) return false;
  l = rk + (uint32_t)__popc(word & ((1u << (rw & 31u)) - 1u));
  return !((explored[l >> 5] >> (l & 31u)) & 1u);
}

__global__ __launch_bounds__(kNbThreads) void nb_score(
    NbStep st, const uint32_t *__restrict__ sub_off, const uint32_t *__restrict__ sub_code,
    const uint32_t *__restrict__ mask, const uint32_t *__restrict__ rank,
    const uint32_t *__restrict__ explored, const float *__restrict__ P, uint64_t stride,
    uint32_t *__restrict__ tmp_idx, float *__restrict__ tmp_s, StepAcc *__restrict__ acc) {
  __shared__ uint32_t off_lds[kNbMaxSubsets + 1];
  __shared__ float a_lds[CGS_MAX_COUNTERS];
  for (uint32_t i = threadIdx.x; i <= st.n_subsets; i += kNbThreads) off_lds[i] = sub_off[i];
  if (threadIdx.x < (uint32_t)st.act.n)
    a_lds[threadIdx.x] = P[(size_t)st.act.ctr[threadIdx.x] * stride + st.profile];
  __syncthreads();
  uint32_t kmin = 0xffffffffu, kmax = 0u, cnt = 0u;
  const uint32_t f = blockIdx.x * kNbThreads + threadIdx.x;
  if (f < st.total) {
    const uint32_t rw = nb_unrank(st, off_lds, sub_code, f);
    uint32_t l = 0;
    const bool keep = nb_keep(rw, mask, rank, explored, l);
    float s = 0.0f;
    if (keep) {
      for (int j0 = 0; j0 < st.act.n; j0 += kRowsInFlight) {
        float x[kRowsInFlight];
#pragma unroll
        for (int u2 = 0; u2 < kRowsInFlight; ++u2)
          if (j0 + u2 < st.act.n) x[u2] = P[(size_t)st.act.ctr[j0 + u2] * stride + l];
#pragma unroll
        for (int u2 = 0; u2 < kRowsInFlight; ++u2) {
          if (j0 + u2 < st.act.n && a_lds[j0 + u2] != 0.0f) {
            const float ap = a_lds[j0 + u2];
            const float t = (x[u2] - ap) / (ap + x[u2]);
            s = (x[u2] != 0.0f) ? s + st.act.delta[j0 + u2] * t : s;
          }
        }
      }
      const uint32_t k = float_key(s);
      kmin = k;
      kmax = k;
      cnt = 1;
    }
    tmp_idx[f] = keep ? l : 0xffffffffu;
    tmp_s[f] = s;
  }
  flush_acc(kmin, kmax, cnt, acc + (blockIdx.x & (kAccSlots - 1)));
}

constexpr int kNbFinishThreads = 1024;

__global__ __launch_bounds__(kNbFinishThreads) void nb_finish(
    uint32_t total, const uint32_t *__restrict__ tmp_idx, const float *__restrict__ tmp_s,
    StepAcc *__restrict__ acc, float gamma, float w_min, uint32_t *__restrict__ nb_idx,
    float *__restrict__ nb_s, uint32_t *__restrict__ nb_q, uint64_t *__restrict__ nb_bsum,
    NbStats *__restrict__ stats) {
  constexpr uint32_t kChunk = 8;
  __shared__ uint64_t scratch[kNbFinishThreads / kWave];
  __shared__ StepAccSums sums;
  __shared__ unsigned long long bsum_lds[kNbBlocks];
  const uint32_t tid = threadIdx.x;
  StepAcc slot{};
  if (tid < kWave) slot = acc[tid];
  if (tid < kNbBlocks) bsum_lds[tid] = 0ull;
  const uint32_t per = (total + kNbFinishThreads - 1) / kNbFinishThreads;
  const uint32_t f0 = min(total, tid * per), f1 = min(total, f0 + per);
  uint32_t kept = 0;
  for (uint32_t f = f0; f < f1; f += kChunk) {
    uint32_t v[kChunk];
#pragma unroll
    for (uint32_t k = 0; k < kChunk; ++k) v[k] = f + k < f1 ? tmp_idx[f + k] : 0xffffffffu;
#pragma unroll
    for (uint32_t k = 0; k < kChunk; ++k) kept += v[k] != 0xffffffffu;
  }
  reduce_slot_values(slot, &sums);
  uint64_t count;
  uint64_t pos = block_excl_scan<kNbFinishThreads>(kept, scratch, count); // barriers publish sums
  const StepNorm nm = step_norm(key_float(sums.min_key), key_float(sums.max_key), gamma, w_min);
  for (uint32_t f = f0; f < f1; f += kChunk) {
    uint32_t v[kChunk];
    float sv[kChunk];
#pragma unroll
    for (uint32_t k = 0; k < kChunk; ++k) {
      v[k] = f + k < f1 ? tmp_idx[f + k] : 0xffffffffu;
      sv[k] = f + k < f1 ? tmp_s[f + k] : 0.0f;
    }
#pragma unroll
    for (uint32_t k = 0; k < kChunk; ++k) {
      if (v[k] == 0xffffffffu) continue;
      const uint32_t q = quantized_weight(sv[k], false, nm);
      nb_idx[pos] = v[k];
      nb_s[pos] = sv[k];
      nb_q[pos] = q;
      atomicAdd(&bsum_lds[pos >> kNbBlockLog2], (unsigned long long)q);
      ++pos;
    }
  }
  __syncthreads();
  if (tid < kNbBlocks) nb_bsum[tid] = bsum_lds[tid];
  if (tid == 0) {
    uint64_t q_total = 0;
    for (uint32_t b = 0; b < kNbBlocks; ++b) q_total += bsum_lds[b];
    stats->count = (uint32_t)count;
    stats->total = q_total;
    stats->min_key = sums.min_key;
    stats->max_key = sums.max_key;
  }
  clear_acc(acc); // every slot was read before the scan's barriers
}

__global__ __launch_bounds__(kDrawThreads) void nb_draw(
    uint32_t *__restrict__ q, const uint32_t *__restrict__ nb, const NbStats *__restrict__ stats,
    uint64_t *__restrict__ bsum, uint32_t *__restrict__ explored, uint32_t profile,
    int mark_profile, uint32_t n_valid, uint64_t u64, const uint32_t *__restrict__ idx,
    DrawResult *__restrict__ res, uint64_t seq) {
  NbWeights w{{q, stats->count}, nb, explored};
  draw_series<kDrawThreads>(w, kNbBlockLog2, bsum, kNbBlocks, 1, &u64, idx, res, seq);
  __syncthreads();
  if (threadIdx.x == 0 && mark_profile && profile < n_valid)
    atomicOr(&explored[profile >> 5], 1u << (profile & 31u));
}

// A whole restricted step of at most kNbFusedMax neighbours in one launch:
// the candidates are scored, and the workgroup that finishes last compacts
// and weighs the kept ones and makes the step's first draw.
// Bound: latency.  The separate launches are three kernel starts with their
// chains of dependent round trips; and the gather of a candidate's counters
// touches one page of the predictions per counter and candidate, so two
// workgroups (476 candidates of radius 2 in a space of 16 parameters) wait on
// address translation in two of the eight dies.  Here LP threads share a
// candidate's counters (their terms meet in LDS and are added in counter
// order), which spreads the gather over LP times as many workgroups.
// The workgroups meet as those of small_step do.
// Measured (32 active counters, 27.7M configurations): 476 neighbours 13.1 us
// with 16 threads a candidate, 14.2 us with 8, 25.9 us as three launches
// (18.5 of them the scores on two workgroups); a step with its draw 21.8
// against 35.7 us, 19.8 against 28.1 us at radius 1, 39.9 against 42.0 us
// with 5,134 candidates (the one workgroup's compaction grows with them,
// hence the limit).
template <int LP>
__global__ __launch_bounds__(kNbThreads) void nb_step(NbFused a) {
  constexpr uint32_t kCands = kNbThreads / LP; // candidates per workgroup
  constexpr int kMine = CGS_MAX_COUNTERS / LP < 16 ? CGS_MAX_COUNTERS / LP : 16;
  extern __shared__ uint32_t nb_lds[];
  __shared__ float a_lds[CGS_MAX_COUNTERS];
  __shared__ uint32_t red[3][kNbThreads / kWave];
  __shared__ uint32_t arrived;
  __shared__ uint64_t scratch[kNbThreads / kWave];
  __shared__ StepAccSums sums;
  __shared__ unsigned long long blk_sum[kNbFusedBlocks];
  const NbStep &st = a.st;
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  const int n = st.act.n;
  // scoring: the subset tables, then one row of terms per candidate
  uint32_t *off = nb_lds, *code = off + st.n_subsets + 1;
  float *terms = reinterpret_cast<float *>(code + st.n_subsets);
  for (uint32_t i = tid; i <= st.n_subsets; i += kNbThreads) off[i] = a.sub_off[i];
  for (uint32_t i = tid; i < st.n_subsets; i += kNbThreads) code[i] = a.sub_code[i];
  if (tid < (uint32_t)n) a_lds[tid] = a.P[(size_t)st.act.ctr[tid] * a.stride + st.profile];
  __syncthreads();
  const uint32_t cand = tid / LP, part = tid % LP;
  const uint32_t f = blockIdx.x * kCands + cand;
  uint32_t l = 0;
  bool keep = false;
  if (f < st.total) keep = nb_keep(nb_unrank(st, off, code, f), a.mask, a.rank, a.explored, l);
  if (keep) {
    for (int j0 = (int)part; j0 < n; j0 += LP * kMine) {
      float x[kMine];
#pragma unroll
      for (int u = 0; u < kMine; ++u) {
        const int j = min(j0 + u * LP, n - 1);
        x[u] = a.P[(size_t)st.act.ctr[j] * a.stride + l];
      }
#pragma unroll
      for (int u = 0; u < kMine; ++u) {
        const int j = j0 + u * LP;
        if (j < n) {
          // a term outside PC_used is 0: the running sum is never -0, so
          // adding it changes nothing
          const float ap = a_lds[j];
          const float t = (x[u] - ap) / (ap + x[u]);
          terms[cand * (uint32_t)(n | 1) + j] =
              (ap != 0.0f && x[u] != 0.0f) ? st.act.delta[j] * t : 0.0f;
        }
      }
    }
  }
  lds_barrier();
  uint32_t kmin = 0xffffffffu, kmax = 0u;
  const bool scored = keep && part == 0;
  float s = 0.0f;
  if (scored) {
    for (int j = 0; j < n; ++j) s = s + terms[cand * (uint32_t)(n | 1) + j];
    kmin = kmax = float_key(s);
  }
  if (part == 0 && f < st.total) {
    a.tmp_idx[f] = keep ? l : kNoIndex;
    a.tmp_s[f] = s;
  }
  kmin = wave_umin(kmin);
  kmax = wave_umax(kmax);
  const uint32_t cnt = (uint32_t)__popcll(__ballot(scored));
  if (lane == 0) {
    red[0][tid >> 6] = kmin;
    red[1][tid >> 6] = kmax;
    red[2][tid >> 6] = cnt;
  }
  stores_done(); // the candidates, for the workgroup that arrives last
  __syncthreads();
  if (tid == 0) {
    StepAcc slot{red[0][0], red[1][0], red[2][0], 0u};
#pragma unroll
    for (int w = 1; w < kNbThreads / kWave; ++w) {
      slot.min_key = min(slot.min_key, red[0][w]);
      slot.max_key = max(slot.max_key, red[1][w]);
      slot.n_unexplored += red[2][w];
    }
    a.acc[blockIdx.x].min_key = slot.min_key;
    a.acc[blockIdx.x].max_key = slot.max_key;
    a.acc[blockIdx.x].n_unexplored = slot.n_unexplored;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    arrived = atomicAdd(&a.acc[0].pad, 1u);
  }
  __syncthreads();
  if (arrived != gridDim.x - 1) return; // uniform over the workgroup
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");

  // compaction: thread t takes the run of `per` candidates from t * per
  const uint32_t per = (st.total + kNbThreads - 1) / kNbThreads, ld = per | 1u;
  uint32_t *cq = nb_lds, *ci = cq + kNbThreads * ld; // the runs' weights and valid indices
  const uint32_t f0 = min(st.total, tid * per), f1 = min(st.total, f0 + per);
  StepAcc slot{};
  if (tid < kWave) slot = a.acc[tid];
  constexpr uint32_t kChunk = 8;
  uint32_t kept = 0;
  for (uint32_t c = 0; c < per; c += kChunk) {
    uint32_t v[kChunk];
    float sv[kChunk];
#pragma unroll
    for (uint32_t k = 0; k < kChunk; ++k) {
      const uint32_t at = min(f0 + c + k, st.total - 1);
      v[k] = a.tmp_idx[at];
      sv[k] = a.tmp_s[at];
    }
#pragma unroll
    for (uint32_t k = 0; k < kChunk; ++k) {
      if (c + k >= per) break;
      const bool in = f0 + c + k < f1 && v[k] != kNoIndex;
      ci[tid * ld + c + k] = in ? v[k] : kNoIndex;
      cq[tid * ld + c + k] = __float_as_uint(sv[k]); // its weight below
      kept += in;
    }
  }
  reduce_slot_values(slot, &sums);
  if (tid < kNbFusedBlocks) blk_sum[tid] = 0ull;
  uint64_t count;
  const uint32_t pos0 =
      (uint32_t)block_excl_scan<kNbThreads, true>(kept, scratch, count); // publishes sums
  const StepNorm nm =
      step_norm(key_float(sums.min_key), key_float(sums.max_key), a.gamma, a.w_min);
  uint64_t mine = 0;
  uint32_t pos = pos0;
  for (uint32_t k = 0; k < per; ++k) {
    const uint32_t v = ci[tid * ld + k];
    const float sv = __uint_as_float(cq[tid * ld + k]);
    const uint32_t q = quantized_weight(sv, v == kNoIndex, nm);
    cq[tid * ld + k] = q;
    if (v != kNoIndex) {
      a.nb_idx[pos] = v;
      a.nb_s[pos] = sv;
      mine += q;
      ++pos;
    }
  }
  uint64_t Q;
  const uint64_t pre = block_excl_scan<kNbThreads, true>(mine, scratch, Q);
  if (tid == 0) {
    a.stats->count = (uint32_t)count;
    a.stats->total = Q;
    a.stats->min_key = sums.min_key;
    a.stats->max_key = sums.max_key;
    a.acc[0].pad = 0u;
    if (a.draw && Q == 0) publish(a.res, kNoIndex, kNoIndex, 0, a.seq);
  }
  const uint64_t r = __umul64hi(a.u64, Q);
  const bool owner = a.draw && pre <= r && r < pre + mine;
  const uint64_t own = __ballot(owner);
  if (own != 0) { // the owner's wave looks through its run, one candidate per lane
    const int o = __ffsll((unsigned long long)own) - 1;
    const uint32_t run = (tid & ~63u) + (uint32_t)o;
    const uint64_t rem = (uint64_t)__shfl((long long)(r - pre), o);
    const uint64_t w = lane < per ? cq[run * ld + lane] : 0u;
    const uint32_t v = lane < per ? ci[run * ld + lane] : kNoIndex;
    const uint64_t incl = wave_incl_scan(w);
    const bool hit = rem < incl && incl - w <= rem; // one lane
    if (hit) {
      publish(a.res, v, a.idx[v], Q, a.seq);
      cq[run * ld + lane] = 0u;
      atomicOr(&a.explored[v >> 5], 1u << (v & 31u));
    }
    const uint64_t who = __ballot(hit);
    const uint64_t ql = (uint64_t)__shfl((long long)w, __ffsll((unsigned long long)who) - 1);
    if (owner) mine -= ql;
  }
  // the weights the draw left and their block sums, by position among the
  // kept
  const uint32_t b0 = pos0 >> kNbBlockLog2;
  uint64_t lower = 0;
  pos = pos0;
  for (uint32_t k = 0; k < per; ++k) {
    if (ci[tid * ld + k] == kNoIndex) continue;
    const uint32_t q = cq[tid * ld + k];
    a.nb_q[pos] = q;
    if (pos >> kNbBlockLog2 == b0) lower += q;
    ++pos;
  }
  if (lower) atomicAdd(&blk_sum[b0], (unsigned long long)lower);
  if (mine != lower) atomicAdd(&blk_sum[b0 + 1], (unsigned long long)(mine - lower));
  lds_barrier();
  if (tid < kNbBlocks) a.bsum[tid] = tid < kNbFusedBlocks ? blk_sum[tid] : 0ull;
  clear_acc(a.acc);
  if (tid == 0 && st.profile < a.n_valid)
    atomicOr(&a.explored[st.profile >> 5], 1u << (st.profile & 31u));
}

// Marks the profiled configuration explored (a step read without a draw).
__global__ __launch_bounds__(64) void mark_one(uint32_t *__restrict__ explored, uint32_t l,
                                               uint32_t n_valid) {
  if (threadIdx.x == 0 && l < n_valid) atomicOr(&explored[l >> 5], 1u << (l & 31u));
}

__global__ __launch_bounds__(kDrawThreads) void draw_array(uint32_t *__restrict__ q, uint32_t n,
                                                           int block_log2,
                                                           uint64_t *__restrict__ bsum,
                                                           uint32_t n_blocks, uint64_t u64,
                                                           DrawResult *__restrict__ res,
                                                           uint64_t seq) {
  ArrayWeights w{q, n};
  draw_series<kDrawThreads>(w, block_log2, bsum, n_blocks, 1, &u64, nullptr, res, seq);
}

__global__ __launch_bounds__(kWeightThreads) void array_block_sums(const uint32_t *__restrict__ q,
                                                                   uint32_t n, int block_log2,
                                                                   uint64_t *__restrict__ bsum) {
  __shared__ uint64_t scratch[kWeightThreads / kWave];
  const uint32_t B = 1u << block_log2;
  const uint32_t base = blockIdx.x << block_log2;
  uint64_t sum = 0;
  for (uint32_t off = threadIdx.x; off < B; off += kWeightThreads) {
    const uint32_t l = base + off;
    if (l < n) sum += q[l];
  }
  const uint64_t total = block_sum<kWeightThreads>(sum, scratch);
  if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

__global__ __launch_bounds__(256) void copy_weights(const float *__restrict__ s,
                                                    uint32_t *__restrict__ explored,
                                                    uint32_t n_valid,
                                                    const StepAcc *__restrict__ acc, float gamma,
                                                    float w_min, uint32_t first, uint32_t count,
                                                    uint32_t *__restrict__ q) {
  const StepAccSums a = reduce_slots(acc);
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  ScoreWeights w{s, explored, n_valid, kNoProfile, acc, gamma, w_min};
  w.nm = step_norm(key_float(a.min_key), key_float(a.max_key), gamma, w_min);
  q[i] = w(first + i);
}

__global__ __launch_bounds__(64) void reset_acc(StepAcc *__restrict__ acc, int n) {
  for (int i = threadIdx.x; i < n; i += 64) {
    acc[i].min_key = 0xffffffffu;
    acc[i].max_key = 0u;
    acc[i].n_unexplored = 0u;
    acc[i].pad = 0u;
  }
}

// A new session: nothing explored, scores 0, neutral accumulators.
__global__ __launch_bounds__(256) void session_init(uint32_t *__restrict__ explored,
                                                    uint64_t n_words, float *__restrict__ s,
                                                    uint64_t stride, StepAcc *__restrict__ acc,
                                                    int n_acc) {
  const uint64_t i0 = (uint64_t)blockIdx.x * 256 + threadIdx.x, step = (uint64_t)gridDim.x * 256;
  for (uint64_t i = i0; i < stride / 4; i += step) // stride is a multiple of 64
    reinterpret_cast<float4 *>(s)[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  for (uint64_t i = i0; i < n_words; i += step) explored[i] = 0u;
  for (uint64_t i = i0; i < (uint64_t)n_acc; i += step)
    acc[i] = StepAcc{0xffffffffu, 0u, 0u, 0u};
}

} // namespace

hipError_t launch_session_init(uint32_t *d_explored, uint64_t n_words, float *d_s,
                               uint64_t stride, StepAcc *d_acc, int n_acc, hipStream_t stream) {
  const uint64_t items = std::max<uint64_t>({stride / 4, n_words, (uint64_t)n_acc});
  const uint32_t grid = (uint32_t)std::min<uint64_t>(2048, (items + 255) / 256);
  hipLaunchKernelGGL(session_init, dim3(grid), dim3(256), 0, stream, d_explored, n_words, d_s,
                     stride, d_acc, n_acc);
  return hipGetLastError();
}

hipError_t launch_reset_acc(StepAcc *d_acc, int n, hipStream_t stream) {
  hipLaunchKernelGGL(reset_acc, dim3(1), dim3(64), 0, stream, d_acc, n);
  return hipGetLastError();
}

hipError_t launch_score_pass(const float *d_P, uint64_t stride, uint32_t profile,
                             const ActiveCounters &act, const uint32_t *d_explored,
                             uint32_t n_valid, float *d_s, StepAcc *d_acc, hipStream_t stream,
                             const uint32_t *d_prof) {
  const uint32_t n_tiles = (n_valid + 4u * kScoreThreads - 1) / (4u * kScoreThreads);
  if (n_tiles == 0) return hipSuccess;
  if (4ull * (uint64_t)act.n * n_valid > kStreamBytes)
    hipLaunchKernelGGL(score_pass<true>, dim3(n_tiles), dim3(kScoreThreads), 0, stream, d_P,
                       stride, profile, d_prof, act, d_explored, n_valid, d_s, d_acc);
  else
    hipLaunchKernelGGL(score_pass<false>, dim3(std::min<uint32_t>(n_tiles, kScoreGrid)),
                       dim3(kScoreThreads), 0, stream, d_P, stride, profile, d_prof, act,
                       d_explored, n_valid, d_s, d_acc);
  return hipGetLastError();
}

hipError_t launch_weight_pass(const float *d_s, const uint32_t *d_explored, uint32_t n_valid,
                              uint32_t profile, const StepAcc *d_acc, StepAcc *d_acc_next,
                              float gamma, float w_min, int block_log2, uint64_t *d_bsum,
                              uint32_t n_blocks, hipStream_t stream, const uint32_t *d_prof) {
  if (n_blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(weight_pass, dim3(n_blocks), dim3(kWeightThreads), 0, stream, d_s, d_explored,
                     n_valid, profile, d_prof, d_acc, d_acc_next, gamma, w_min, block_log2,
                     d_bsum);
  return hipGetLastError();
}

hipError_t launch_draw(const float *d_s, uint32_t *d_explored, uint32_t n_valid, uint32_t profile,
                       bool mark_profile, const StepAcc *d_acc, float gamma, float w_min,
                       int block_log2, uint64_t *d_bsum, uint32_t n_blocks, uint64_t u64,
                       const uint32_t *d_idx, DrawResult *d_res, uint64_t seq,
                       hipStream_t stream, const uint32_t *d_prof, uint32_t *d_prof_out) {
  hipLaunchKernelGGL(draw_scores, dim3(1), dim3(kDrawThreads), 0, stream, d_s, d_explored, n_valid,
                     profile, d_prof, mark_profile ? 1 : 0, d_acc, gamma, w_min, block_log2,
                     d_bsum, n_blocks, u64, d_idx, d_res, seq, d_prof_out);
  return hipGetLastError();
}

hipError_t launch_draw_many(const float *d_s, uint32_t *d_explored, uint32_t n_valid,
                            const StepAcc *d_acc, float gamma, float w_min, int block_log2,
                            uint64_t *d_bsum, uint32_t n_blocks, const DrawSeries &series,
                            const uint32_t *d_idx, DrawResult *d_res, uint64_t seq0,
                            hipStream_t stream) {
  if (series.n < 1 || series.n > kMaxDrawSeries) return hipErrorInvalidValue;
  hipLaunchKernelGGL(draw_many, dim3(1), dim3(kDrawThreads), 0, stream, d_s, d_explored, n_valid,
                     d_acc, gamma, w_min, block_log2, d_bsum, n_blocks, series, d_idx, d_res,
                     seq0);
  return hipGetLastError();
}

void small_shape(uint32_t n_valid, uint32_t *tiles, uint32_t *per, FastDiv *per4) {
  *tiles = (n_valid + kSmallThreads - 1) / kSmallThreads;
  *per = std::max<uint32_t>(4, (*tiles + 3u) & ~3u); // `tiles` weights per thread, in quads
  *per4 = make_fastdiv(*per / 4);
}

namespace {
constexpr size_t kSmallLds = small_ld(kSmallPer) * kSmallThreads * sizeof(uint32_t);
} // namespace

hipError_t launch_small_step(SmallStep &a, hipStream_t stream) {
  if (a.n_valid == 0 || a.n_valid > kSmallMaxValid || a.series.n < 0 ||
      a.series.n > kMaxDrawSeries || a.block_log2 < 12)
    return hipErrorInvalidValue;
  uint32_t grid;
  small_shape(a.n_valid, &grid, &a.per, &a.per4);
  const size_t lds = small_ld(a.per) * kSmallThreads * sizeof(uint32_t);
  const hipError_t e = allow_lds(small_step, lds, kSmallLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(small_step, dim3(grid), dim3(kSmallThreads), lds, stream, a);
  return hipGetLastError();
}

hipError_t launch_batch_small(const BatchSess *d_sess, const SmallJob *d_jobs, uint32_t n,
                              uint32_t max_tiles, uint32_t max_per, DrawResult *d_res,
                              hipStream_t stream) {
  if (n == 0) return hipSuccess;
  if (max_per > kSmallPer) return hipErrorInvalidValue;
  const uint32_t groups =
      std::max<uint32_t>(1, std::min<uint32_t>(std::min<uint32_t>(max_tiles, kAccSlots), kBatchSmallGroups / n));
  const size_t lds = small_ld(max_per) * kSmallThreads * sizeof(uint32_t);
  const hipError_t e = allow_lds(batch_small, lds, kSmallLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(batch_small, dim3(n * groups), dim3(kSmallThreads), lds, stream, d_sess,
                     d_jobs, groups, d_res);
  return hipGetLastError();
}

hipError_t launch_batch_tune(const BatchSess *d_sess, const TuneArgs &a, uint32_t n,
                             uint32_t max_per, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  if (max_per > kSmallPer || a.draws < 1 || a.draws > kMaxDrawSeries) return hipErrorInvalidValue;
  const size_t lds = small_ld(max_per) * kSmallThreads * sizeof(uint32_t);
  const hipError_t e = allow_lds(batch_tune, kSmallLds, kSmallLds); // its static part is 6 KB
  if (e != hipSuccess) return e;
  batch_tune<<<n, kSmallThreads, lds, stream>>>(d_sess, a);
  return hipGetLastError();
}

hipError_t launch_batch_score(const BatchSess *d_sess, const BatchStep *d_step,
                              const uint16_t *d_tile_sess, uint32_t total_tiles, uint32_t grid,
                              int variant, uint64_t row_bytes, hipStream_t stream) {
  if (total_tiles == 0 || grid == 0) return hipSuccess;
  const bool streamed = batch_streams(row_bytes);
#define CGS_BATCH_SCORE(RIF, WPE)                                                               \
  do {                                                                                          \
    if (streamed)                                                                               \
      hipLaunchKernelGGL((batch_score<RIF, WPE, true>), dim3(grid), dim3(kScoreThreads), 0,     \
                         stream, d_sess, d_step, d_tile_sess, total_tiles);                     \
    else                                                                                        \
      hipLaunchKernelGGL((batch_score<RIF, WPE, false>), dim3(grid), dim3(kScoreThreads), 0,    \
                         stream, d_sess, d_step, d_tile_sess, total_tiles);                     \
  } while (0)
  switch (variant) {
  case 1: CGS_BATCH_SCORE(4, 4); break;
  case 2: CGS_BATCH_SCORE(16, 2); break;
  case 3: CGS_BATCH_SCORE(8, 4); break;
  case 4: CGS_BATCH_SCORE(4, 8); break;
  default: CGS_BATCH_SCORE(8, 1); break; // the unconstrained kernel
  }
#undef CGS_BATCH_SCORE
  return hipGetLastError();
}

hipError_t launch_batch_weight(const BatchSess *d_sess, const BatchStep *d_step,
                               const uint16_t *d_blk_sess, uint32_t total_blocks, uint32_t grid,
                               hipStream_t stream) {
  if (total_blocks == 0 || grid == 0) return hipSuccess;
  hipLaunchKernelGGL(batch_weight, dim3(grid), dim3(kWeightThreads), 0, stream, d_sess, d_step,
                     d_blk_sess, total_blocks);
  return hipGetLastError();
}

hipError_t launch_batch_draw(const BatchSess *d_sess, const BatchStep *d_step, uint32_t n_sess,
                             hipStream_t stream) {
  if (n_sess == 0) return hipSuccess;
  hipLaunchKernelGGL(batch_draw, dim3(n_sess), dim3(kDrawThreads), 0, stream, d_sess, d_step);
  return hipGetLastError();
}

hipError_t launch_mark_one(uint32_t *d_explored, uint32_t l, uint32_t n_valid,
                           hipStream_t stream) {
  hipLaunchKernelGGL(mark_one, dim3(1), dim3(64), 0, stream, d_explored, l, n_valid);
  return hipGetLastError();
}

hipError_t launch_nb_step(const NbFused &a, hipStream_t stream) {
  const NbStep &st = a.st;
  if (st.total == 0 || st.total > kNbFusedMax || st.n_subsets > kNbMaxSubsets)
    return hipErrorInvalidValue;
  // as many threads per candidate as leave at most 64 workgroups (one
  // accumulator slot each)
  constexpr uint32_t kAll = kAccSlots * kNbThreads; // threads of 64 workgroups
  const int lp = st.total * 16 <= kAll ? 16 : st.total * 8 <= kAll ? 8 : 2;
  const uint32_t cands = kNbThreads / lp, grid = (st.total + cands - 1) / cands;
  const uint32_t per = (st.total + kNbThreads - 1) / kNbThreads;
  const size_t score = (2 * st.n_subsets + 1 + (size_t)cands * (st.act.n | 1)) * 4;
  const size_t lds = std::max(score, (size_t)2 * kNbThreads * (per | 1) * 4);
  auto kernel = lp == 16 ? nb_step<16> : lp == 8 ? nb_step<8> : nb_step<2>;
  // most: every subset of 32 parameters, and 128 candidates' terms of every counter
  constexpr size_t kNbLds = (2 * (size_t)kNbMaxSubsets + 1 + kNbThreads / 2 * (CGS_MAX_COUNTERS | 1)) * 4;
  static_assert(kNbLds >= (size_t)2 * kNbThreads * (kNbFusedMax / kNbThreads | 1) * 4, "the compaction's");
  const hipError_t e = allow_lds(kernel, lds, kNbLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(kNbThreads), lds, stream, a);
  return hipGetLastError();
}

hipError_t launch_nb_score(const NbStep &st, const uint32_t *d_sub_off, const uint32_t *d_sub_code,
                           const uint32_t *d_mask, const uint32_t *d_rank,
                           const uint32_t *d_explored, const float *d_P, uint64_t stride,
                           uint32_t *d_tmp_idx, float *d_tmp_s, StepAcc *d_nb_acc,
                           hipStream_t stream) {
  if (st.total == 0 || st.total > kNbMaxCandidates || st.n_subsets > kNbMaxSubsets)
    return hipErrorInvalidValue;
  const uint32_t grid = (st.total + kNbThreads - 1) / kNbThreads;
  hipLaunchKernelGGL(nb_score, dim3(grid), dim3(kNbThreads), 0, stream, st, d_sub_off, d_sub_code,
                     d_mask, d_rank, d_explored, d_P, stride, d_tmp_idx, d_tmp_s, d_nb_acc);
  return hipGetLastError();
}

hipError_t launch_nb_finish(uint32_t total, const uint32_t *d_tmp_idx, const float *d_tmp_s,
                            StepAcc *d_nb_acc, float gamma, float w_min, uint32_t *d_nb_idx,
                            float *d_nb_s, uint32_t *d_nb_q, uint64_t *d_nb_bsum,
                            NbStats *d_stats, hipStream_t stream) {
  if (total > kNbMaxCandidates) return hipErrorInvalidValue;
  hipLaunchKernelGGL(nb_finish, dim3(1), dim3(kNbFinishThreads), 0, stream, total, d_tmp_idx,
                     d_tmp_s, d_nb_acc, gamma, w_min, d_nb_idx, d_nb_s, d_nb_q, d_nb_bsum,
                     d_stats);
  return hipGetLastError();
}

hipError_t launch_nb_draw(uint32_t *d_nb_q, const uint32_t *d_nb_idx, const NbStats *d_stats,
                          uint64_t *d_nb_bsum, uint32_t *d_explored, uint32_t profile,
                          int mark_profile, uint32_t n_valid, uint64_t u64, const uint32_t *d_idx,
                          DrawResult *d_res, uint64_t seq, hipStream_t stream) {
  hipLaunchKernelGGL(nb_draw, dim3(1), dim3(kDrawThreads), 0, stream, d_nb_q, d_nb_idx, d_stats,
                     d_nb_bsum, d_explored, profile, mark_profile, n_valid, u64, d_idx, d_res, seq);
  return hipGetLastError();
}

hipError_t launch_copy_weights(const float *d_s, uint32_t *d_explored, uint32_t n_valid,
                               const StepAcc *d_acc, float gamma, float w_min, uint32_t first,
                               uint32_t count, uint32_t *d_q, hipStream_t stream) {
  if (count == 0) return hipSuccess;
  hipLaunchKernelGGL(copy_weights, dim3((count + 255) / 256), dim3(256), 0, stream, d_s,
                     d_explored, n_valid, d_acc, gamma, w_min, first, count, d_q);
  return hipGetLastError();
}

hipError_t launch_array_block_sums(const uint32_t *d_q, uint32_t n, int block_log2,
                                   uint64_t *d_bsum, hipStream_t stream) {
  const uint32_t n_blocks = (uint32_t)(((uint64_t)n + (1u << block_log2) - 1) >> block_log2);
  if (n_blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(array_block_sums, dim3(n_blocks), dim3(kWeightThreads), 0, stream, d_q, n,
                     block_log2, d_bsum);
  return hipGetLastError();
}

hipError_t launch_array_draw(uint32_t *d_q, uint32_t n, int block_log2, uint64_t *d_bsum,
                             uint32_t n_blocks, uint64_t u64, DrawResult *d_res, uint64_t seq,
                             hipStream_t stream) {
  hipLaunchKernelGGL(draw_array, dim3(1), dim3(kDrawThreads), 0, stream, d_q, n, block_log2,
                     d_bsum, n_blocks, u64, d_res, seq);
  return hipGetLastError();
}

} // namespace cgs
