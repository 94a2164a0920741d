// Device helpers shared by the libcgs kernels (wave64, gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"
#include "stepdiv.h"

namespace cgs {

constexpr int kWave = 64;

__device__ __forceinline__ uint32_t fastdiv(uint32_t n, FastDiv d) {
  const uint32_t t = __umulhi(d.m, n);
  return (t + ((n - t) >> (d.sh & 0xffu))) >> (d.sh >> 8);
}

// Mixed-radix decode of raw index k (parameter 0 most significant) into
// 4-bit digits: parameters 0..15 in `lo`, 16..31 in `hi`.
__device__ __forceinline__ void decode_packed(uint32_t k, const SpaceDev *__restrict__ sp,
                                              uint64_t &lo, uint64_t &hi) {
  lo = 0;
  hi = 0;
  const int n = sp->n_params;
  for (int j = n - 1; j >= 16; --j) {
    const uint32_t q = fastdiv(k, sp->div[j]);
    hi |= (uint64_t)(k - q * sp->radix[j]) << (4 * (j - 16));
    k = q;
  }
  for (int j = (n < 16 ? n : 16) - 1; j >= 0; --j) {
    const uint32_t q = fastdiv(k, sp->div[j]);
    lo |= (uint64_t)(k - q * sp->radix[j]) << (4 * j);
    k = q;
  }
}

__device__ __forceinline__ uint32_t digit_of(uint64_t lo, uint64_t hi, uint32_t j) {
  const uint64_t w = j < 16 ? (lo >> (4 * j)) : (hi >> (4 * (j - 16)));
  return (uint32_t)w & 15u;
}

__device__ __forceinline__ uint32_t uabs32(int32_t v) {
  return v < 0 ? (uint32_t)(-(int64_t)v) : (uint32_t)v;
}

// One constraint of kind `kind` for the values of its parameters.
__device__ __forceinline__ bool satisfies(uint32_t kind, int64_t bound, int32_t va, int32_t vb,
                                          int32_t vc) {
  switch (kind) {
  case CGS_DIV: {
    const uint32_t d = uabs32(vb);
    return d != 0 && (uabs32(va) % d) == 0;
  }
  case CGS_DIV2: {
    // |v| < 2^20, so |vb * vc| < 2^40; a divisor larger than |va| divides
    // only va == 0.
    const uint64_t d = (uint64_t)uabs32(vb) * (uint64_t)uabs32(vc);
    const uint32_t n = uabs32(va);
    return d != 0 && (d > n ? n == 0 : (n % (uint32_t)d) == 0);
  }
  case CGS_PROD_LE: return (int64_t)va * vb <= bound;
  case CGS_PROD3_LE: return (int64_t)va * vb * vc <= bound;
  case CGS_PROD_GE: return (int64_t)va * vb >= bound;
  default: return va <= vb; // CGS_LE
  }
}

// Order-preserving map float -> uint32 (a < b  <=>  key(a) < key(b) for
// non-NaN values), so min/max reduce with integer atomics.
__device__ __forceinline__ uint32_t float_key(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_float(uint32_t k) {
  const uint32_t u = (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
  return __uint_as_float(u);
}

// The constants of one step's normalisation: the divisors of positive
// scores (s_max) and of the others (-s_min) with their reciprocals
// (stepdiv.h), the cut-off and the smallest weight.  1 - s / s_min is
// formed as 1 + s / (-s_min): the same float, since IEEE division and
// rounding to nearest are symmetric under a change of sign.  A divisor that
// no unexplored configuration divides by (s_max <= 0: no positive score;
// s_min >= 0: only zero scores, whose quotient is 0 for any divisor) is
// replaced by 1.
struct StepNorm {
  StepDivisor pos, neg; // s_max and -s_min
  bool fast;            // both divisors in the fast path's range
  bool wide;            // fast, and both divisors >= kWideDivisorMin
  float gamma, w_min;
};
// The reciprocals are made opaque to the optimiser: it would otherwise
// turn the per-lane choice between two reciprocals back into one division
// per configuration.
__device__ __forceinline__ float opaque(float x) {
  asm volatile("" : "+v"(x));
  return x;
}
__device__ __forceinline__ StepNorm step_norm(float s_min, float s_max, float gamma, float w_min) {
  StepNorm nm{step_divisor(s_max > 0.0f ? s_max : 1.0f),
              step_divisor(s_min < 0.0f ? -s_min : 1.0f), false, false, gamma, w_min};
  nm.fast = nm.pos.fast && nm.neg.fast;
  nm.wide = nm.fast && nm.pos.d >= kWideDivisorMin && nm.neg.d >= kWideDivisorMin;
  nm.pos.r = opaque(nm.pos.r);
  nm.neg.r = opaque(nm.neg.r);
  return nm;
}

// Normalised weight of the score-normalisation equation, quantised to
// rint(w * 2^23):
//   s > 0: (1 + s/s_max)^8;  gamma < s <= 0: max(w_min, (1 - s/s_min)^8),
//   1 when s == 0;  s <= gamma: w_min;  explored: 0.
// The eighth power is three squarings.  With gamma <= 0 and w_min <= 1 (the
// session's parameters are checked for both) the cases fold into
//   y = 1 + s / D (D = s_max or -s_min by the sign of s),
//   w = s > gamma ? max(w_min, y^8) : w_min
// (for s > 0, y^8 >= 1 >= w_min): every value is the same float as the
// case-by-case form.  The division is correctly rounded through the step's
// reciprocal (stepdiv.h) wherever the fast path's operand range holds (the
// divisors are checked once per step; |s| <= D for every unexplored
// configuration, so only a non-zero |s| below 2^-60 leaves it) and the IEEE
// division otherwise.  When the step's divisors are both at least
// kWideDivisorMin (nm.wide, kWide = true) no score needs the division: below
// the range only 1 + s / D = 1 matters, which the sequence also gives
// (stepdiv.h), so the per-configuration range check goes too.
template <bool kWide>
__device__ __forceinline__ uint32_t quantized_weight_t(float s, bool explored, const StepNorm &nm) {
  const bool pos = s > 0.0f;
  const float d = pos ? nm.pos.d : nm.neg.d;
  float t;
  if (kWide) {
    t = div_fast_core(s, d, pos ? nm.pos.r : nm.neg.r);
  } else if (nm.fast) {
    t = div_fast_core(s, d, pos ? nm.pos.r : nm.neg.r); // +-0 for s == 0
    const uint32_t ab = __float_as_uint(s) & 0x7fffffffu;
    const bool slow = !explored && ab - 1u < 0x217fffffu; // 0 < |s| < 2^-60
    if (__any(slow)) t = slow ? s / d : t;
  } else {
    t = s == 0.0f ? 0.0f : s / d;
  }
  const float y = 1.0f + t;
  const float y2 = y * y;
  const float y4 = y2 * y2;
  const float y8 = y4 * y4;
  const float w = s > nm.gamma ? fmaxf(nm.w_min, y8) : nm.w_min;
  return explored ? 0u : (uint32_t)rintf(w * 8388608.0f);
}
__device__ __forceinline__ uint32_t quantized_weight(float s, bool explored, const StepNorm &nm) {
  return nm.wide ? quantized_weight_t<true>(s, explored, nm)
                 : quantized_weight_t<false>(s, explored, nm);
}

__device__ __forceinline__ bool explored_bit(const uint32_t *__restrict__ ex, uint32_t l) {
  return (ex[l >> 5] >> (l & 31u)) & 1u;
}

// ------------------------------------------------------------ wave / block
// Cross-lane moves of the integer scans and reductions are DPP operand
// modifiers of the VALU (a few cycles each) rather than ds_bpermute round
// trips through the LDS crossbar (~60 cycles, two per 64-bit value): a
// 64-lane 64-bit scan is 6 steps of two moves and one add.  The steps are the
// four in-row shifts by 1, 2, 4 and 8, then row 0 to row 1 and row 2 to row
// 3 (row_bcast15 into rows 1 and 3), then the lower half's last lane into
// rows 2 and 3 (row_bcast31).  A lane without a source gets `none`.
constexpr int kDppShr1 = 0x111, kDppShr2 = 0x112, kDppShr4 = 0x114, kDppShr8 = 0x118;
constexpr int kDppBcast15 = 0x142, kDppBcast31 = 0x143;

template <int kCtrl, int kRows>
__device__ __forceinline__ uint32_t dpp_move(uint32_t v, uint32_t none) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)v, kCtrl, kRows, 0xf, false);
}
template <int kCtrl, int kRows>
__device__ __forceinline__ uint64_t dpp_move(uint64_t v, uint64_t none) {
  const uint32_t lo = dpp_move<kCtrl, kRows>((uint32_t)v, (uint32_t)none);
  const uint32_t hi = dpp_move<kCtrl, kRows>((uint32_t)(v >> 32), (uint32_t)(none >> 32));
  return (uint64_t)hi << 32 | lo;
}
// Inclusive scan of v under `op` across the wave's 64 lanes (all of them
// active); lane 63 holds the reduction.
template <typename T, typename Op>
__device__ __forceinline__ T wave_scan(T v, T none, Op op) {
  v = op(v, dpp_move<kDppShr1, 0xf>(v, none));
  v = op(v, dpp_move<kDppShr2, 0xf>(v, none));
  v = op(v, dpp_move<kDppShr4, 0xf>(v, none));
  v = op(v, dpp_move<kDppShr8, 0xf>(v, none));
  v = op(v, dpp_move<kDppBcast15, 0xa>(v, none));
  return op(v, dpp_move<kDppBcast31, 0xc>(v, none));
}
__device__ __forceinline__ uint32_t last_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1);
}
__device__ __forceinline__ uint64_t last_lane(uint64_t v) {
  return (uint64_t)last_lane((uint32_t)(v >> 32)) << 32 | last_lane((uint32_t)v);
}
struct AddOp {
  template <typename T> __device__ T operator()(T a, T b) const { return a + b; }
};

// Sums, minima and maxima over the wave, in every lane.  The float sum keeps
// the butterfly order its results are defined by.
template <typename T> __device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
  return last_lane(wave_scan(v, 0u, AddOp{}));
}
__device__ __forceinline__ uint64_t wave_sum(uint64_t v) {
  return last_lane(wave_scan(v, (uint64_t)0, AddOp{}));
}
__device__ __forceinline__ uint32_t wave_umin(uint32_t v) {
  return last_lane(wave_scan(v, 0xffffffffu, [](uint32_t a, uint32_t b) { return min(a, b); }));
}
__device__ __forceinline__ uint32_t wave_umax(uint32_t v) {
  return last_lane(wave_scan(v, 0u, [](uint32_t a, uint32_t b) { return max(a, b); }));
}

// Inclusive scan across a wave.
__device__ __forceinline__ uint64_t wave_incl_scan(uint64_t v) {
  return wave_scan(v, (uint64_t)0, AddOp{});
}

// A barrier that orders LDS accesses only: loads and stores of global memory
// stay in flight across it (__syncthreads waits for all of them).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Waits until the L2 has this wave's stores of global memory.  Neither a
// barrier nor a release of one wave does that for the others (__syncthreads
// compiles to a wait for LDS, as the waves of a workgroup share a cache), and
// the write-back of an agent-scope release covers what has reached the L2.  So
// every wave waits before the barrier after which one thread releases the
// whole workgroup's stores to other workgroups.
__device__ __forceinline__ void stores_done() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Exclusive scan over the whole block (NT threads, NT % 64 == 0); `total`
// receives the block sum.  `scratch` holds NT / 64 entries.  Contains
// barriers (kLdsOnly: of LDS only): every thread must call it.
template <int NT, bool kLdsOnly = false>
__device__ __forceinline__ uint64_t block_excl_scan(uint64_t v, uint64_t *scratch, uint64_t &total) {
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  constexpr int NW = NT / kWave;
  const uint64_t incl = wave_incl_scan(v);
  kLdsOnly ? lds_barrier() : __syncthreads();
  if (lane == kWave - 1) scratch[wave] = incl;
  kLdsOnly ? lds_barrier() : __syncthreads();
  uint64_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const uint64_t t = scratch[w];
    before += (w < (int)wave) ? t : 0ull;
    all += t;
  }
  total = all;
  return before + incl - v;
}

template <int NT> __device__ __forceinline__ uint64_t block_sum(uint64_t v, uint64_t *scratch) {
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  constexpr int NW = NT / kWave;
  v = wave_sum(v);
  __syncthreads();
  if (lane == 0) scratch[wave] = v;
  __syncthreads();
  uint64_t all = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) all += scratch[w];
  return all;
}

} // namespace cgs
