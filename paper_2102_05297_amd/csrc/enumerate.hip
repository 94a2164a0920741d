// Tuning-space enumeration with constraint pruning and stable compaction
// (Sect. 1: the space is the cross product of the parameters' value sets
// restricted by a-priori constraints; Alg. 1 takes it as the array TS).
//
// Three passes over the raw index range [0, n_raw), in tiles of 2048 raw
// indices per 256-thread workgroup (4 waves x 8 rows of 64):
//   mark     decode + constraints (from truth tables a small launch writes
//            first) -> one ballot per row of 64; the ballot is the validity
//            bitmask (two uint32 words); per-tile valid count
//   scan     one workgroup: exclusive scan of the tile counts -> tile offsets
//            and the number of valid configurations
//   compact  per tile: re-read the bitmask, rank set bits with popcounts and
//            write the raw indices, ascending, and the rank of every mask
//            word (valid configurations before it), so that a raw index
//            maps to its valid index with one load and a popcount
// Integer-only; the output is independent of scheduling.
#include <algorithm>

#include "device_common.h"

namespace cgs {

namespace {

constexpr int kEnumThreads = 256;
constexpr int kRowsPerWave = 8;
constexpr uint32_t kTile = kEnumTile;
static_assert(kTile == kEnumThreads * kRowsPerWave, "a row of 64 per wave and step");
constexpr uint32_t kTruth = CGS_MAX_RADIX * CGS_MAX_RADIX;
constexpr uint32_t kMaxLow = 1024; // 16 KB of LDS
constexpr uint32_t kMaxMid = 256;  // 4 KB

// The tables of one space: truth[c * 256 + 16 da + db], bit dc: constraint c
// holds for digits da, db, dc of its parameters; low[r]: the packed digits of
// raw index r < n_low, the product of the last parameters' radices; low[n_low +
// m]: those of raw index m n_low, m < n_mid, the product of the radices before
// them.  Workgroups 0 .. n_cons - 1 write one constraint each, the others `low`.
__global__ __launch_bounds__(kEnumThreads) void enum_tables(const SpaceDev *__restrict__ sp,
                                                            uint32_t n_low, uint32_t n_mid,
                                                            uint32_t *__restrict__ truth,
                                                            ulonglong2 *__restrict__ low) {
  const uint32_t n_cons = (uint32_t)sp->n_cons, tid = threadIdx.x;
  if (blockIdx.x >= n_cons) {
    const uint32_t r = (blockIdx.x - n_cons) * kEnumThreads + tid;
    if (r >= n_low + n_mid) return;
    uint64_t lo, hi;
    decode_packed(r < n_low ? r : (r - n_low) * n_low, sp, lo, hi);
    low[r] = make_ulonglong2(lo, hi);
    return;
  }
  const uint32_t c = blockIdx.x, code = sp->cons_code[c];
  const uint32_t a = (code >> 8) & 0xffu, b = (code >> 16) & 0xffu, cc = code >> 24;
  const uint32_t da = tid / CGS_MAX_RADIX, db = tid % CGS_MAX_RADIX;
  uint32_t bits = 0;
  if (da < sp->radix[a] && db < sp->radix[b])
    for (uint32_t dc = 0; dc < sp->radix[cc]; ++dc)
      bits |= (uint32_t)satisfies(code & 0xffu, sp->cons_bound[c],
                                  sp->table[a * CGS_MAX_RADIX + da],
                                  sp->table[b * CGS_MAX_RADIX + db],
                                  sp->table[cc * CGS_MAX_RADIX + dc])
              << dc;
  truth[c * kTruth + tid] = bits;
}

// Bound: the instructions per configuration, about a tenth of what decoding
// every parameter and evaluating every constraint takes (a division for each
// parameter and for each divisibility constraint): the 64 configurations of a
// row share their high digits (at most two values, as n_low >= 64 unless it
// is the whole space); the low digits are one LDS read per configuration, those
// above them are decoded with scalar instructions, about once per tile; a
// constraint is one LDS read of its truth table.  kMid: the high digits would
// change too often (n_low < 512), so the middle ones have a table too.
// Measured on 2^24 configurations of 12 parameters, 6 constraints: 87 us (3 us
// for the tables); a decode and the constraints themselves per configuration
// 205 us; decoding the high digits for every row 387 us.  Without the middle
// table, n_low = 128 (the last radices 16, 16 and 8) came near that: 2^31 raw
// indices, 2 constraints 13.5 ms, 6.9 with it; on n_low = 1,024 (2^30) it would
// take 3.1 -> 3.4.
template <bool kMid>
__global__ __launch_bounds__(kEnumThreads) void enum_mark(
    const SpaceDev *__restrict__ sp, const uint32_t *__restrict__ truth_in,
    const ulonglong2 *__restrict__ low_in, uint32_t n_low, FastDiv div_low, uint32_t n_tiles,
    uint32_t *__restrict__ mask, uint32_t *__restrict__ tile_count, uint32_t n_mid,
    FastDiv div_mid) {
  extern __shared__ ulonglong2 low[]; // [n_low], [n_mid], then the truth tables
  __shared__ uint32_t wave_cnt[kEnumThreads / kWave];
  const uint32_t n_raw = sp->n_raw, n_words = sp->n_words, n_cons = (uint32_t)sp->n_cons;
  const ulonglong2 *mid = low + n_low;
  uint32_t *truth = reinterpret_cast<uint32_t *>(low + n_low + n_mid);
  for (uint32_t e = threadIdx.x; e < n_low + n_mid; e += kEnumThreads) low[e] = low_in[e];
  for (uint32_t e = threadIdx.x; e < n_cons * kTruth; e += kEnumThreads) truth[e] = truth_in[e];
  __syncthreads();

  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t n_both = n_low * (kMid ? n_mid : 1u);
  uint32_t have = ~0u; // the value whose digits are lo0, hi0 (the next one's: lo1, hi1)
  uint64_t lo0 = 0, hi0 = 0, lo1 = 0, hi1 = 0;
  for (uint32_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    const uint64_t wave_base = (uint64_t)tile * kTile + (uint64_t)wave * (kWave * kRowsPerWave);
    uint64_t lo[kRowsPerWave], hi[kRowsPerWave];
    uint32_t ok[kRowsPerWave], cnt = 0;
#pragma unroll
    for (int row = 0; row < kRowsPerWave; ++row) {
      const uint64_t row_base = min(wave_base + (uint64_t)row * kWave, (uint64_t)(n_raw - 1));
      const uint32_t q = fastdiv((uint32_t)row_base, div_low), h = kMid ? fastdiv(q, div_mid) : q;
      if (h != have) {
        have = h;
        decode_packed(h * n_both, sp, lo0, hi0);
        const uint64_t next = (uint64_t)(h + 1) * n_both;
        if (next < n_raw) decode_packed((uint32_t)next, sp, lo1, hi1);
      }
      uint32_t r = (uint32_t)row_base - q * n_low + lane;
      const bool wrap = r >= n_low;
      if (wrap) r -= n_low;
      const bool in = wave_base + (uint64_t)row * kWave + lane < n_raw;
      ulonglong2 d = low[in ? r : 0u];
      bool over = wrap; // past the value of lo0, hi0
      if (kMid) {
        const uint32_t m = q - h * n_mid + (wrap ? 1u : 0u);
        over = m >= n_mid;
        const ulonglong2 e = mid[over ? 0u : m];
        d.x |= e.x;
        d.y |= e.y;
      }
      lo[row] = d.x | (over ? lo1 : lo0);
      hi[row] = d.y | (over ? hi1 : hi0);
      ok[row] = in ? 1u : 0u;
    }
    for (uint32_t c = 0; c < n_cons; ++c) {
      const uint32_t code = sp->cons_code[c];
      const uint32_t *t = truth + c * kTruth;
#pragma unroll
      for (int row = 0; row < kRowsPerWave; ++row) {
        const uint32_t da = digit_of(lo[row], hi[row], (code >> 8) & 0xffu),
                       db = digit_of(lo[row], hi[row], (code >> 16) & 0xffu),
                       dc = digit_of(lo[row], hi[row], code >> 24);
        ok[row] &= t[da * CGS_MAX_RADIX + db] >> dc;
      }
    }
#pragma unroll
    for (int row = 0; row < kRowsPerWave; ++row) {
      const uint64_t bal = __ballot(ok[row] & 1u);
      const uint64_t w = (wave_base >> 5) + 2 * row;
      if (lane < 2 && w + lane < n_words) mask[w + lane] = (uint32_t)(bal >> (32 * lane));
      cnt += (uint32_t)__popcll(bal);
    }
    __syncthreads();
    if (lane == 0) wave_cnt[wave] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t t = 0;
      for (int w = 0; w < kEnumThreads / kWave; ++w) t += wave_cnt[w];
      tile_count[tile] = t;
    }
  }
}

constexpr int kScanThreads = 1024;

__global__ __launch_bounds__(kScanThreads) void enum_scan(const uint32_t *__restrict__ tile_count,
                                                          uint32_t n_tiles,
                                                          uint32_t *__restrict__ tile_off,
                                                          uint64_t *__restrict__ total) {
  __shared__ uint64_t scratch[kScanThreads / kWave];
  const uint32_t per = (n_tiles + kScanThreads - 1) / kScanThreads;
  const uint32_t begin = min(n_tiles, threadIdx.x * per);
  const uint32_t end = min(n_tiles, begin + per);
  uint64_t local = 0;
  for (uint32_t i = begin; i < end; ++i) local += tile_count[i];
  uint64_t all;
  uint64_t run = block_excl_scan<kScanThreads>(local, scratch, all);
  for (uint32_t i = begin; i < end; ++i) {
    tile_off[i] = (uint32_t)run;
    run += tile_count[i];
  }
  if (threadIdx.x == 0) *total = all;
}

__global__ __launch_bounds__(kEnumThreads) void enum_compact(const SpaceDev *__restrict__ sp,
                                                             const uint32_t *__restrict__ mask,
                                                             const uint32_t *__restrict__ tile_off,
                                                             uint32_t *__restrict__ idx,
                                                             uint32_t *__restrict__ word_rank) {
  __shared__ uint32_t wave_cnt[kEnumThreads / kWave];
  const uint32_t n_words = sp->n_words;
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  const uint64_t wave_base = (uint64_t)blockIdx.x * kTile + (uint64_t)wave * (kWave * kRowsPerWave);
  const uint64_t w0 = wave_base >> 5; // 16 words per wave
  uint32_t c = 0;
  if (lane < 2 * kRowsPerWave && w0 + lane < n_words) c = (uint32_t)__popc(mask[w0 + lane]);
  c = wave_sum(c);
  if (lane == 0) wave_cnt[wave] = c;
  __syncthreads();
  uint32_t off = tile_off[blockIdx.x];
  for (uint32_t w = 0; w < wave; ++w) off += wave_cnt[w];
  for (int row = 0; row < kRowsPerWave; ++row) {
    const uint64_t wi = w0 + 2 * row;
    const uint64_t lo = wi < n_words ? mask[wi] : 0u;
    const uint64_t hi = wi + 1 < n_words ? mask[wi + 1] : 0u;
    const uint64_t bits = lo | (hi << 32);
    if (lane == 0 && wi < n_words) word_rank[wi] = off;
    if (lane == 1 && wi + 1 < n_words) word_rank[wi + 1] = off + (uint32_t)__popc((uint32_t)lo);
    if ((bits >> lane) & 1ull) {
      const uint32_t rank = (uint32_t)__popcll(bits & ((1ull << lane) - 1ull));
      idx[off + rank] = (uint32_t)(wave_base + (uint64_t)row * kWave + lane);
    }
    off += (uint32_t)__popcll(bits);
  }
}

// raw[i] = idx[pos[i]]; every pos[i] lies within the list.
__global__ __launch_bounds__(256) void gather_idx(const uint32_t *__restrict__ idx,
                                                  const uint32_t *__restrict__ pos, uint32_t n,
                                                  uint32_t *__restrict__ raw) {
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256)
    raw[i] = idx[pos[i]];
}

} // namespace

hipError_t launch_gather_idx(const uint32_t *d_idx, const uint32_t *d_pos, uint32_t n,
                             uint32_t *d_raw, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  gather_idx<<<std::min<uint32_t>((n + 255) / 256, 4096), 256, 0, stream>>>(d_idx, d_pos, n, d_raw);
  return hipGetLastError();
}

size_t enumeration_table_bytes() {
  return (kMaxLow + kMaxMid) * sizeof(ulonglong2) + CGS_MAX_CONSTRAINTS * kTruth * sizeof(uint32_t);
}

uint32_t enumeration_tiles(uint32_t n_raw) {
  return (uint32_t)(((uint64_t)n_raw + kTile - 1) / kTile);
}

// phase 0: mark + scan (then the host reads *d_total); phase 1: compact and
// word ranks.
hipError_t launch_enumeration(const SpaceDev &space, const SpaceDev *d_space, void *d_tables,
                              uint32_t *d_mask, uint32_t *d_tile_count, uint32_t *d_tile_off,
                              uint64_t *d_total, uint32_t *d_idx, uint32_t *d_rank, int phase,
                              hipStream_t stream) {
  const uint32_t n_raw = space.n_raw;
  const uint32_t n_tiles = enumeration_tiles(n_raw);
  if (n_tiles == 0) return hipSuccess;
  if (phase == 0) {
    uint32_t n_low = 1; // 64 or more, or the whole space: no radix is above 16
    int j = space.n_params - 1;
    for (; j >= 0 && n_low * space.radix[j] <= kMaxLow; --j) n_low *= space.radix[j];
    uint32_t n_mid = 1; // 17 or more, or what is left
    for (; n_low < 512 && j >= 0 && n_mid * space.radix[j] <= kMaxMid; --j)
      n_mid *= space.radix[j];
    const uint32_t n_cons = (uint32_t)space.n_cons;
    ulonglong2 *low = static_cast<ulonglong2 *>(d_tables);
    uint32_t *truth = reinterpret_cast<uint32_t *>(low + kMaxLow + kMaxMid);
    enum_tables<<<n_cons + (n_low + n_mid + kEnumThreads - 1) / kEnumThreads, kEnumThreads, 0,
                  stream>>>(d_space, n_low, n_mid, truth, low);
    const size_t lds = (n_low + n_mid) * sizeof(ulonglong2) + n_cons * kTruth * sizeof(uint32_t);
    // up to eight workgroups per CU; more tiles than that share the tables
    (n_mid > 1 ? enum_mark<true> : enum_mark<false>)<<<std::min<uint32_t>(n_tiles, 2048),
                                                       kEnumThreads, lds, stream>>>(
        d_space, truth, low, n_low, make_fastdiv(n_low), n_tiles, d_mask, d_tile_count, n_mid,
        make_fastdiv(n_mid));
    hipLaunchKernelGGL(enum_scan, dim3(1), dim3(kScanThreads), 0, stream, d_tile_count, n_tiles,
                       d_tile_off, d_total);
  } else {
    hipLaunchKernelGGL(enum_compact, dim3(n_tiles), dim3(kEnumThreads), 0, stream, d_space,
                       d_mask, d_tile_off, d_idx, d_rank);
  }
  return hipGetLastError();
}

} // namespace cgs
