// Regression-forest evaluation over every valid configuration (Sect. 3.4.2:
// internal nodes test a tuning parameter, leaves hold predicted counters).
//
// One thread per valid configuration, 256 per workgroup.  Each thread decodes
// its raw index once into packed 4-bit digits.  Trees are processed one at a
// time: the workgroup stages tree t's internal nodes (uint16: feature |
// threshold << 8) in LDS, every thread walks depth D levels out of LDS and
// parks its leaf id in LDS.  Then each thread gathers its T leaf vectors
// (float4 loads from the L2-resident leaf array), sums them in ascending t
// starting from tree 0, divides once by T, and writes the counters
// structure-of-arrays: P[c][l], so a row of P is contiguous over
// configurations and the sweep reads it coalesced.
#include <algorithm>

#include "device_common.h"
#include "models.h"

namespace cgs {

namespace {

constexpr int kForestThreads = 256;
constexpr int kForestBatch = 16; // loads in flight per thread (node staging, leaf gathers)

__global__ __launch_bounds__(kForestThreads) void forest_eval(
    const SpaceDev *__restrict__ sp, const uint32_t *__restrict__ idx, uint32_t first,
    uint32_t count, const uint16_t *__restrict__ nodes, const float *__restrict__ leaves,
    int n_trees, int depth, int n_counters, float *__restrict__ P, uint64_t stride,
    uint16_t *__restrict__ leaf_out) {
  extern __shared__ uint16_t smem[];
  const uint32_t n_int = (1u << depth) - 1u;
  const uint32_t n_int_pad = (n_int + 8u) & ~7u; // keep the leaf-id area 16-byte aligned
  uint16_t *lnodes = smem;
  uint16_t *lleaf = smem + n_int_pad; // [T][256]

  const uint32_t i = blockIdx.x * kForestThreads + threadIdx.x;
  const bool active = i < count;
  const uint32_t l = first + i;
  uint64_t lo = 0, hi = 0;
  if (active) decode_packed(idx[l], sp, lo, hi);

  for (int t = 0; t < n_trees; ++t) {
    __syncthreads();
    const uint16_t *tn = nodes + (size_t)t * n_int;
    // the tree's nodes, kForestBatch loads per thread issued before the
    // first LDS store (a plain loop waits for every load in turn)
    for (uint32_t j0 = threadIdx.x; j0 < n_int; j0 += kForestBatch * kForestThreads) {
      uint16_t v[kForestBatch];
#pragma unroll
      for (int b = 0; b < kForestBatch; ++b) {
        const uint32_t j = j0 + b * kForestThreads;
        v[b] = j < n_int ? tn[j] : (uint16_t)0;
      }
#pragma unroll
      for (int b = 0; b < kForestBatch; ++b) {
        const uint32_t j = j0 + b * kForestThreads;
        if (j < n_int) lnodes[j] = v[b];
      }
    }
    __syncthreads();
    uint32_t node = 0;
    for (int lev = 0; lev < depth; ++lev) {
      const uint32_t nd = lnodes[node];
      const uint32_t dig = digit_of(lo, hi, nd & 0xffu);
      node = 2u * node + 1u + (dig > (nd >> 8) ? 1u : 0u);
    }
    const uint32_t leaf = node - n_int;
    lleaf[t * kForestThreads + threadIdx.x] = (uint16_t)leaf;
    if (leaf_out != nullptr && active) leaf_out[(size_t)t * count + i] = (uint16_t)leaf;
  }
  if (!active) return;

  const uint32_t n_leaf = 1u << depth;
  const float t_div = (float)n_trees;
  if ((n_counters & 3) == 0) {
    // leaf vectors of kForestBatch / 2 trees in flight at once; the sums
    // still run in ascending tree order from tree 0
    constexpr int TB = kForestBatch / 2;
    for (int c = 0; c < n_counters; c += 4) {
      float4 acc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      for (int t0 = 0; t0 < n_trees; t0 += TB) {
        float4 v[TB];
#pragma unroll
        for (int u = 0; u < TB; ++u) {
          const int t = min(t0 + u, n_trees - 1);
          const uint32_t lf = lleaf[t * kForestThreads + threadIdx.x];
          v[u] = *reinterpret_cast<const float4 *>(leaves + ((size_t)t * n_leaf + lf) * n_counters +
                                                   c);
        }
#pragma unroll
        for (int u = 0; u < TB; ++u) {
          if (t0 + u >= n_trees) break;
          if (t0 + u == 0) {
            acc = v[0];
          } else {
            acc.x = acc.x + v[u].x;
            acc.y = acc.y + v[u].y;
            acc.z = acc.z + v[u].z;
            acc.w = acc.w + v[u].w;
          }
        }
      }
      P[(size_t)(c + 0) * stride + l] = acc.x / t_div;
      P[(size_t)(c + 1) * stride + l] = acc.y / t_div;
      P[(size_t)(c + 2) * stride + l] = acc.z / t_div;
      P[(size_t)(c + 3) * stride + l] = acc.w / t_div;
    }
  } else {
    for (int c = 0; c < n_counters; ++c) {
      float acc = leaves[(size_t)lleaf[threadIdx.x] * n_counters + c];
      for (int t = 1; t < n_trees; ++t) {
        const uint32_t lf = lleaf[t * kForestThreads + threadIdx.x];
        acc = acc + leaves[((size_t)t * n_leaf + lf) * n_counters + c];
      }
      P[(size_t)c * stride + l] = acc / t_div;
    }
  }
}

// Resident variant, for forests whose nodes fit in LDS together: each
// workgroup stages every
// tree once and then runs grid-stride over tiles of configurations, so the
// node tables cross L2 once per workgroup instead of once per 256
// configurations, and there is no barrier per tree.  A thread walks its
// configuration through all trees level by level (the T independent LDS
// reads of a level are in flight together), keeps the leaf ids in registers
// and gathers and sums the leaf vectors exactly as forest_eval does
// (ascending t from tree 0, one division by T).
//
// kBits, wherever the space's tests digit > threshold are at most 63 (the sum
// of the radices less one): every test has a bit in a 64-bit word of the
// configuration (digit d sets the lowest d bits of its parameter's), and a
// node is one byte, the place of its bit (63, never set, for a threshold that
// no digit exceeds).  A level is an LDS read and three instructions instead
// of ten, and twice the nodes fit.  The walk bounds deep forests with few
// counters, the leaf gathers the others (16 trees x 64 counters).  Which forests
// take it: byte_nodes_pay.
// Measured on 4.0M configurations of 12 parameters (42 tests), nodes as
// (feature, threshold) -> as bits: 16 trees of depth 12, 24 counters 674 -> 411
// us, 8 counters 559 -> 256; 4 trees of depth 8 188 -> 142; one tree of depth
// 12 112 -> 114.  Lanes side by side on the columns of one leaf, with the
// leaf ids and the results staged in LDS, took 594 us for the first and 270
// for the second: the six loads of a lane from one leaf vector meet in the
// vector cache anyway.
//
// A thread walks TM trees, whatever the number that exist, and holds their leaf
// ids: up to 32 trees in multiples of eight at 1,024 threads, 128 registers
// each; beyond, 512 threads (at 1,024 the leaf ids of 64 trees spill: 33 trees of
// depth 6 and 8 counters 495 us on 1M configurations, 220 with 40 walked by 512
// threads; 17 trees of depth 2 and 64 counters 436 us with 32 walked, 376 with 24).
constexpr int kResidentThreads = 1024;
constexpr int kResidentTrees = 16; // without kBits
constexpr size_t kResidentLds = 160 * 1024 - 1024;

template <int TM, bool kBits, int NT>
__global__ __launch_bounds__(NT) void forest_eval_resident(
    const SpaceDev *__restrict__ sp, const uint32_t *__restrict__ idx, uint32_t first,
    uint32_t count, const uint16_t *__restrict__ nodes, const float *__restrict__ leaves,
    int n_trees, int depth, int n_counters, float *__restrict__ P, uint64_t stride,
    uint16_t *__restrict__ leaf_out) {
  // [T][2^D - 1] feature | threshold << 8, or, one byte each, [T][2^D] with a tree's node n (from 1) at n
  extern __shared__ uint16_t lnodes[];
  uint8_t *bnodes = reinterpret_cast<uint8_t *>(lnodes);
  __shared__ uint32_t bit_base[CGS_MAX_PARAMS]; // | (radix - 1) << 8
  const int n_par = sp->n_params;
  if (kBits) {
    if (threadIdx.x < (uint32_t)n_par) {
      uint32_t b = 0;
      for (int j = n_par - 1; j > (int)threadIdx.x; --j) b += sp->radix[j] - 1u;
      bit_base[threadIdx.x] = b | (sp->radix[threadIdx.x] - 1u) << 8;
    }
    __syncthreads();
  }
  const uint32_t n_int = (1u << depth) - 1u;
  // kBits: over [T][2^D], whose entry 0 is not a node
  const uint32_t total = kBits ? (uint32_t)n_trees << depth : (uint32_t)n_trees * n_int;
  for (uint32_t j0 = threadIdx.x; j0 < total; j0 += kForestBatch * NT) {
    uint16_t v[kForestBatch];
#pragma unroll
    for (int b = 0; b < kForestBatch; ++b) {
      const uint32_t j = j0 + b * NT, n = j & n_int;
      const bool have = j < total && (!kBits || n > 0);
      v[b] = have ? nodes[kBits ? (j >> depth) * n_int + n - 1u : j] : (uint16_t)0;
    }
#pragma unroll
    for (int b = 0; b < kForestBatch; ++b) {
      const uint32_t j = j0 + b * NT;
      if (j >= total) continue;
      if (kBits) {
        const uint32_t base = bit_base[v[b] & 0xffu], thr = v[b] >> 8;
        bnodes[j] = (uint8_t)(thr < base >> 8 ? (base & 0xffu) + thr : 63u);
      } else {
        lnodes[j] = v[b];
      }
    }
  }
  __syncthreads();
  const uint32_t n_leaf = 1u << depth;
  // x / T; for T a power of two, x * (1 / T) is the same float (exact scaling)
  const float t_div = (float)n_trees;
  const bool pow2 = (n_trees & (n_trees - 1)) == 0;
  const float t_inv = 1.0f / t_div;
  const uint32_t n_tiles = (count + NT - 1) / NT;
  for (uint32_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    const uint32_t i = tile * NT + threadIdx.x;
    if (i >= count) break; // the last tile; no barrier follows
    const uint32_t l = first + i;
    uint64_t lo, hi = 0; // kBits: lo holds the tests' bits
    if (kBits) {
      lo = 0;
      uint32_t raw = idx[l], base = 0;
      for (int j = n_par - 1; j >= 0; --j) {
        const uint32_t q = fastdiv(raw, sp->div[j]), r = sp->radix[j];
        lo |= (uint64_t)((1u << (raw - q * r)) - 1u) << base;
        base += r - 1u;
        raw = q;
      }
    } else {
      decode_packed(idx[l], sp, lo, hi);
    }
    // walks of up to 8 trees interleaved level by level; leaf ids two per
    // register
    constexpr int TW = TM < 8 ? TM : 8;
    const uint32_t n_first = kBits ? n_leaf : n_int; // number of the first leaf
    uint32_t leafp[(TM + 1) / 2];
#pragma unroll
    for (int t0 = 0; t0 < TM; t0 += TW) {
      uint32_t nw[TW];
#pragma unroll
      for (int u = 0; u < TW; ++u) nw[u] = kBits ? 1u : 0u;
      for (int lev = 0; lev < depth; ++lev) {
#pragma unroll
        for (int u = 0; u < TW; ++u) {
          if (kBits) {
            const uint8_t *tn = bnodes + (min(t0 + u, n_trees - 1) << depth);
            nw[u] = 2u * nw[u] + ((uint32_t)(lo >> tn[nw[u]]) & 1u);
          } else if (t0 + u < n_trees) {
            const uint32_t nd = lnodes[(t0 + u) * n_int + nw[u]];
            nw[u] = 2u * nw[u] + 1u + (digit_of(lo, hi, nd & 0xffu) > (nd >> 8) ? 1u : 0u);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < TW; u += 2)
        leafp[(t0 + u) / 2] = (nw[u] - n_first) | (u + 1 < TW ? (nw[u + 1] - n_first) << 16 : 0u);
    }
    auto leaf_of = [&](int t) { return (leafp[t >> 1] >> (16 * (t & 1))) & 0xffffu; };
    if (leaf_out != nullptr) {
#pragma unroll
      for (int t = 0; t < TM; ++t)
        if (t < n_trees) leaf_out[(size_t)t * count + i] = (uint16_t)leaf_of(t);
    }
    auto store = [&](int c, float acc) {
      P[(size_t)c * stride + l] = pow2 ? acc * t_inv : acc / t_div;
    };
    if ((n_counters & 3) == 0) {
      // leaf vectors of up to 8 trees in flight (more would spill at 1024
      // threads); the sum runs in ascending t from tree 0
      constexpr int TB = TM < 8 ? TM : TM > 16 ? 4 : 8;
      for (int c = 0; c < n_counters; c += 4) {
        float4 acc;
#pragma unroll
        for (int t0 = 0; t0 < TM; t0 += TB) {
          float4 v[TB];
#pragma unroll
          for (int u = 0; u < TB; ++u)
            if (t0 + u < n_trees)
              v[u] = *reinterpret_cast<const float4 *>(
                  leaves + ((size_t)(t0 + u) * n_leaf + leaf_of(t0 + u)) * n_counters + c);
          if (t0 == 0) acc = v[0];
#pragma unroll
          for (int u = (t0 == 0 ? 1 : 0); u < TB; ++u) {
            if (t0 + u < n_trees) {
              acc.x = acc.x + v[u].x;
              acc.y = acc.y + v[u].y;
              acc.z = acc.z + v[u].z;
              acc.w = acc.w + v[u].w;
            }
          }
        }
        store(c, acc.x);
        store(c + 1, acc.y);
        store(c + 2, acc.z);
        store(c + 3, acc.w);
      }
    } else {
      for (int c = 0; c < n_counters; ++c) {
        float acc = leaves[(size_t)leaf_of(0) * n_counters + c];
#pragma unroll
        for (int t = 1; t < TM; ++t)
          if (t < n_trees) acc = acc + leaves[((size_t)t * n_leaf + leaf_of(t)) * n_counters + c];
        store(c, acc);
      }
    }
  }
}

// Partial sums of squared prediction differences over sampled valid
// configurations: one double per workgroup.  DENSE_A: Pa holds the sampled
// configurations' predictions in sample order (column i for sample i).
template <bool DENSE_A>
__global__ __launch_bounds__(256) void sq_diff(const float *__restrict__ Pa,
                                               const float *__restrict__ Pb, uint64_t stride_a,
                                               uint64_t stride_b, int n_counters,
                                               const uint32_t *__restrict__ sample, uint32_t n,
                                               double *__restrict__ partial) {
  __shared__ double red[4];
  double acc = 0.0;
  for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    const uint32_t l = sample[i];
    for (int c = 0; c < n_counters; ++c) {
      const double d = (double)Pa[(size_t)c * stride_a + (DENSE_A ? i : l)] -
                       (double)Pb[(size_t)c * stride_b + l];
      acc += d * d;
    }
  }
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// Predictions of listed valid configurations: out[i][c] = P[c][idx[i]].
__global__ __launch_bounds__(256) void gather_rows(const float *__restrict__ P, uint64_t stride,
                                                   int n_counters,
                                                   const uint32_t *__restrict__ idx, uint32_t n,
                                                   float *__restrict__ out) {
  const uint64_t e = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (uint64_t)n * n_counters) return;
  const uint32_t i = (uint32_t)(e / n_counters);
  const int c = (int)(e % n_counters);
  out[e] = P[(size_t)c * stride + idx[i]];
}

} // namespace

hipError_t launch_gather_rows(const float *P, uint64_t stride, int n_counters,
                              const uint32_t *d_idx, uint32_t n, float *d_out,
                              hipStream_t stream) {
  const uint64_t total = (uint64_t)n * n_counters;
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(gather_rows, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, P,
                     stride, n_counters, d_idx, n, d_out);
  return hipGetLastError();
}

hipError_t launch_sq_diff(const float *Pa, const float *Pb, uint64_t stride_a, uint64_t stride_b,
                          int n_counters, const uint32_t *sample, uint32_t n, double *partial,
                          uint32_t grid, hipStream_t stream) {
  hipLaunchKernelGGL(sq_diff<false>, dim3(grid), dim3(256), 0, stream, Pa, Pb, stride_a, stride_b,
                     n_counters, sample, n, partial);
  return hipGetLastError();
}

hipError_t launch_sq_diff_dense(const float *Pa, const float *Pb, uint64_t stride_a,
                                uint64_t stride_b, int n_counters, const uint32_t *sample,
                                uint32_t n, double *partial, uint32_t grid, hipStream_t stream) {
  hipLaunchKernelGGL(sq_diff<true>, dim3(grid), dim3(256), 0, stream, Pa, Pb, stride_a, stride_b,
                     n_counters, sample, n, partial);
  return hipGetLastError();
}

// Whether a forest of T trees of depth D with C counters takes byte nodes where
// the space allows them.  Microseconds on 1M configurations, (feature,
// threshold) nodes -> bytes: the walks of one or two shallow trees are too short
// to pay for the configuration's bits (1 x depth 1 x 5 20.6 -> 21.5, x depth 8 24.9
// -> 22.5; 2 x 4 x 8 25.6 -> 27.4, 2 x 8 x 8 31.8 -> 28.8, 2 x 8 x 24 44.2 -> 46.1).
// From three trees on every depth gains (3 x 1 x 24 52.4 -> 51.3, 16 x 11 x 8 220 ->
// 104), up to 32 trees.  Beyond, few waves are in flight for the leaf gathers, so
// their loads per tree decide: two always pay (33 x 2 x 8 193 -> 179, 40 x 11 x 8
// 508 -> 344), six only where nearly all of the 64 trees walked exist (48 x 6 x 24
// 639 -> 696, 57 x 6 x 24 862 -> 828), sixteen hardly (57 x 6 x 64 1,979 -> 2,118).
bool byte_nodes_pay(int T, int D, int C) {
  if (T == 1) return D >= 4;
  if (T == 2) return D >= 8 && C <= 8;
  if (T <= 32) return true;
  const int loads = C % 4 ? C : C / 4; // of a leaf vector, 16 bytes each where they can be
  return loads <= 2 || (T > 56 && loads <= 6);
}

// Evaluates valid configurations [first, first + count).  With d_leaf_out
// set, also writes leaf ids [T][count] and skips nothing else.
hipError_t launch_forest_eval(const SpaceDev *d_space, const uint32_t *d_idx, uint32_t n_valid,
                              const uint16_t *d_nodes, const float *d_leaves, int n_trees,
                              int depth, int n_counters, int n_bits, float *d_P, uint64_t stride,
                              uint16_t *d_leaf_out, uint32_t leaf_first, uint32_t leaf_count,
                              hipStream_t stream) {
  const uint32_t first = d_leaf_out ? leaf_first : 0u;
  const uint32_t count = d_leaf_out ? leaf_count : n_valid;
  if (count == 0) return hipSuccess;
  const uint32_t n_int = (1u << depth) - 1u;
  const bool bits = n_bits <= 63 && byte_nodes_pay(n_trees, depth, n_counters);
  const size_t res_lds =
      bits ? (size_t)n_trees << depth : (size_t)n_trees * n_int * sizeof(uint16_t);
  const bool resident =
      n_trees <= (bits ? CGS_MAX_TREES : kResidentTrees) && res_lds <= kResidentLds;
  if (resident) {
    // as many workgroups as fit on the device at once (LDS-bound), at most
    // one per tile
    int dev = 0, n_cu = 256;
    if (hipGetDevice(&dev) == hipSuccess)
      hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
    const uint32_t per_cu = (uint32_t)std::max<size_t>(1, std::min<size_t>(2, kResidentLds / std::max<size_t>(res_lds, 1)));
    auto grid_of = [&](uint32_t threads) {
      const uint32_t tiles = (count + threads - 1) / threads;
      return std::max<uint32_t>(1, std::min<uint32_t>(tiles, (uint32_t)n_cu * per_cu));
    };
#define CGS_FOREST_RES(TMV, BV, NT)                                                             \
  do {                                                                                          \
    const hipError_t e = allow_lds(forest_eval_resident<TMV, BV, NT>, res_lds, kResidentLds);       \
    if (e != hipSuccess) return e;                                                              \
    hipLaunchKernelGGL((forest_eval_resident<TMV, BV, NT>), dim3(grid_of(NT)), dim3(NT),         \
                       res_lds, stream, d_space, d_idx, first, count, d_nodes, d_leaves,        \
                       n_trees, depth, n_counters, d_P, stride, d_leaf_out);                    \
  } while (0)
    constexpr int kN = kResidentThreads;
    if (bits) {
      if (n_trees <= 1) CGS_FOREST_RES(1, true, kN);
      else if (n_trees <= 2) CGS_FOREST_RES(2, true, kN);
      else if (n_trees <= 4) CGS_FOREST_RES(4, true, kN);
      else if (n_trees <= 8) CGS_FOREST_RES(8, true, kN);
      else if (n_trees <= 16) CGS_FOREST_RES(16, true, kN);
      else if (n_trees <= 24) CGS_FOREST_RES(24, true, kN);
      else if (n_trees <= 32) CGS_FOREST_RES(32, true, kN);
      else if (n_trees <= 40) CGS_FOREST_RES(40, true, kN / 2);
      else if (n_trees <= 48) CGS_FOREST_RES(48, true, kN / 2);
      else CGS_FOREST_RES(64, true, kN / 2);
    } else {
      if (n_trees <= 1) CGS_FOREST_RES(1, false, kN);
      else if (n_trees <= 2) CGS_FOREST_RES(2, false, kN);
      else if (n_trees <= 4) CGS_FOREST_RES(4, false, kN);
      else if (n_trees <= 8) CGS_FOREST_RES(8, false, kN);
      else CGS_FOREST_RES(16, false, kN);
    }
#undef CGS_FOREST_RES
    return hipGetLastError();
  }
  const uint32_t n_int_pad = (n_int + 8u) & ~7u;
  const size_t lds = (size_t)(n_int_pad + (uint32_t)n_trees * kForestThreads) * sizeof(uint16_t);
  const uint32_t grid = (count + kForestThreads - 1) / kForestThreads;
  hipLaunchKernelGGL(forest_eval, dim3(grid), dim3(kForestThreads), lds, stream, d_space, d_idx,
                     first, count, d_nodes, d_leaves, n_trees, depth, n_counters, d_P, stride,
                     d_leaf_out);
  return hipGetLastError();
}

// Predictions given per configuration, src[l][C], into the model layout
// P[c][stride].
__global__ void rows_to_columns(const float *__restrict__ src, uint32_t n, int C,
                                float *__restrict__ P, uint64_t stride) {
  for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < (uint64_t)n * C;
       e += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t l = e / C, c = e - l * C;
    P[c * stride + l] = src[e];
  }
}

hipError_t launch_rows_to_columns(const float *d_src, uint32_t n, int C, float *d_P,
                                  uint64_t stride, hipStream_t stream) {
  const uint64_t total = (uint64_t)n * C;
  const uint32_t grid = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(8192, (total + 255) / 256));
  rows_to_columns<<<grid, 256, 0, stream>>>(d_src, n, C, d_P, stride);
  return hipGetLastError();
}

// ------------------------------------------------------- model inputs
// The values a caller gives are checked where they land: 1.57M leaf values
// pass in 3.5 us, after an upload that is needed anyway; the
// same check in a host loop, one value at a time up to the first bad one,
// took about 1.2 ms before anything was uploaded (loading the forest of 16
// depth-12 trees on 4.0M configurations: 2.28 -> 1.12 ms).
__global__ __launch_bounds__(64) void check_begin(unsigned long long *first) {
  if (threadIdx.x == 0) *first = ~0ull;
}
__global__ __launch_bounds__(256) void check_floats(const float *__restrict__ x, uint64_t n,
                                                    int nonneg, unsigned long long *first) {
  uint64_t bad = ~0ull;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * 256) {
    const float v = x[i];
    const bool ok = isfinite(v) && (!nonneg || v >= 0.0f);
    if (!ok && i < bad) bad = i;
  }
  if (bad != ~0ull) atomicMin(first, (unsigned long long)bad);
}
hipError_t launch_check_floats(const float *x, uint64_t n, bool nonneg, uint64_t *first,
                               hipStream_t stream) {
  unsigned long long *f = reinterpret_cast<unsigned long long *>(first);
  check_begin<<<1, 64, 0, stream>>>(f);
  const uint32_t grid = (uint32_t)std::min<uint64_t>(2048, (n + 1023) / 1024);
  if (grid) check_floats<<<grid, 256, 0, stream>>>(x, n, nonneg ? 1 : 0, f);
  return hipGetLastError();
}

// At most 63 columns per row are padding; clearing the whole array first
// cost a pass over it (47 us for 385 MB).
__global__ __launch_bounds__(64) void clear_columns(float *__restrict__ P, uint64_t stride,
                                                    uint64_t from) {
  for (uint64_t l = from + threadIdx.x; l < stride; l += 64)
    P[(uint64_t)blockIdx.x * stride + l] = 0.0f;
}
hipError_t launch_clear_columns(float *P, uint64_t stride, int C, uint64_t from,
                                hipStream_t stream) {
  if (from >= stride) return hipSuccess;
  clear_columns<<<C, 64, 0, stream>>>(P, stride, from);
  return hipGetLastError();
}

} // namespace cgs
