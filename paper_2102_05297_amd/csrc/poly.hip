// Least-squares polynomial counter models per binary subspace (Sect. 3.4.1).
//
// The binary parameters' digits select a subspace; within it every counter is
// a polynomial in the non-binary parameters: products of their features over
// all parameter sets up to the chosen order (main effects and interactions),
// plus squares.  Feature x_j = (2 v - v_max - v_min) / (v_max - v_min).
//
// Fit: F[i][t] (float64) for every measured point and basis term, with the
// point's counters appended as columns T..T+C-1; per subspace the Gram matrix
// of those columns gives F^T F and F^T Y; a ridge 1e-9 trace / T is added and
// one workgroup per subspace factors it (Cholesky, packed lower triangle in
// LDS, panels of 16 columns) and solves for every counter.  Evaluation,
// float32: the terms summed once per combination of all but the last
// parameters' digits, then one thread per valid configuration (nested); or
// every term per configuration, coefficients of a group of subspaces in LDS.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "device_common.h"
#include "models.h"

namespace cgs {

namespace {

constexpr int kPolyThreads = 256;
constexpr int kGB = 32;        // Gram block edge
constexpr int kGramChunk = 128; // points staged per round of the Gram kernel
constexpr int kEvalThreads = 1024; // one workgroup per CU holds the coefficients
constexpr double kRidge = 1e-9;

__device__ __forceinline__ uint32_t term_count(uint32_t d) { return d & 7u; }
__device__ __forceinline__ uint32_t term_var(uint32_t d, uint32_t i) {
  return (d >> (3 + 5 * i)) & 31u;
}

__device__ __forceinline__ uint32_t subspace_of(const PolyDev *pd, uint64_t lo, uint64_t hi) {
  uint32_t s = 0;
  for (int i = 0; i < pd->B; ++i) s |= digit_of(lo, hi, pd->bin_params[i]) << i;
  return s;
}

// Exclusive prefix sums of in[0..n) in one workgroup.
__global__ __launch_bounds__(1024) void poly_excl_scan(const uint64_t *__restrict__ in,
                                                       uint64_t *__restrict__ out, uint32_t n) {
  __shared__ uint64_t scratch[16];
  const uint32_t t = threadIdx.x, per = (n + 1023) / 1024;
  const uint32_t a = min(n, t * per), b = min(n, a + per);
  uint64_t mine = 0;
  for (uint32_t i = a; i < b; ++i) mine += in[i];
  uint64_t tot;
  uint64_t run = block_excl_scan<1024>(mine, scratch, tot);
  for (uint32_t i = a; i < b; ++i) {
    const uint64_t v = in[i];
    out[i] = run;
    run += v;
  }
}

// ---------------------------------------------------------------- design
__device__ __forceinline__ bool in_design(const SpaceDev *sp, const uint32_t *allowed,
                                          uint32_t raw) {
  uint64_t lo, hi;
  decode_packed(raw, sp, lo, hi);
  bool ok = true;
  for (int j = 0; j < sp->n_params; ++j) ok = ok && ((allowed[j] >> digit_of(lo, hi, j)) & 1u);
  return ok;
}

__global__ __launch_bounds__(kPolyThreads) void poly_design_count(
    const SpaceDev *__restrict__ sp, const uint32_t *__restrict__ idx, uint32_t nv,
    const uint32_t *__restrict__ allowed, uint64_t *__restrict__ cnt) {
  __shared__ uint64_t scratch[kPolyThreads / 64];
  for (uint32_t tile = blockIdx.x; (uint64_t)tile * kPolyThreads < nv; tile += gridDim.x) {
    const uint32_t l = tile * kPolyThreads + threadIdx.x;
    const uint64_t f = (l < nv && in_design(sp, allowed, idx[l])) ? 1ull : 0ull;
    const uint64_t s = block_sum<kPolyThreads>(f, scratch);
    if (threadIdx.x == 0) cnt[tile] = s;
  }
}

__global__ __launch_bounds__(kPolyThreads) void poly_design_write(
    const SpaceDev *__restrict__ sp, const uint32_t *__restrict__ idx, uint32_t nv,
    const uint32_t *__restrict__ allowed, const uint64_t *__restrict__ off,
    uint32_t *__restrict__ out) {
  __shared__ uint64_t scratch[kPolyThreads / 64];
  for (uint32_t tile = blockIdx.x; (uint64_t)tile * kPolyThreads < nv; tile += gridDim.x) {
    const uint32_t l = tile * kPolyThreads + threadIdx.x;
    const bool f = l < nv && in_design(sp, allowed, idx[l]);
    uint64_t tot;
    const uint64_t r = block_excl_scan<kPolyThreads>(f ? 1ull : 0ull, scratch, tot);
    if (f) out[off[tile] + r] = l;
  }
}

// ---------------------------------------------------------------- fit
// sub[i]: the subspace of point i, S where it is outside the valid list.  Here
// and not on the host, where the divisions of the points' indices by the
// radices took 0.65 ms for 20,736 points of 12 parameters.
__global__ __launch_bounds__(kPolyThreads) void poly_subspaces(
    const PolyDev *__restrict__ pd, const SpaceDev *__restrict__ sp,
    const uint32_t *__restrict__ idx, uint32_t nv, const uint32_t *__restrict__ pts, uint32_t n,
    uint32_t *__restrict__ sub) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t p = pts[i];
    uint64_t lo = 0, hi = 0;
    if (p < nv) decode_packed(idx[p], sp, lo, hi);
    sub[i] = p < nv ? subspace_of(pd, lo, hi) : (uint32_t)pd->S;
  }
}

// F[i][t]: basis term t of point i for t < T, its counter t - T for t >= T.
// err bit 0: a point outside the valid list, bit 1: a non-finite target.
__global__ __launch_bounds__(kPolyThreads) void poly_features(
    const PolyDev *__restrict__ pd, const SpaceDev *__restrict__ sp,
    const uint32_t *__restrict__ idx, uint32_t nv, const uint32_t *__restrict__ pts,
    const float *__restrict__ Y, uint32_t n, double *__restrict__ F,
    uint32_t *__restrict__ err) {
  const uint32_t T = pd->T, C = pd->C, Ta = T + C;
  for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < (uint64_t)n * Ta;
       e += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t i = (uint32_t)(e / Ta), t = (uint32_t)(e - (uint64_t)i * Ta);
    const uint32_t p = pts[i];
    uint64_t lo = 0, hi = 0;
    if (p < nv) decode_packed(idx[p], sp, lo, hi);
    else if (t == 0) atomicOr(err, 1u);
    double v;
    if (t < T) {
      const uint32_t d = pd->terms[t];
      v = 1.0;
      for (uint32_t q = 0; q < term_count(d); ++q) {
        const uint32_t j = term_var(d, q);
        v *= pd->xv64[j * CGS_MAX_RADIX + digit_of(lo, hi, j)];
      }
    } else {
      const float y = Y[(uint64_t)i * C + (t - T)];
      if (!isfinite(y)) atomicOr(err, 2u);
      v = isfinite(y) ? (double)y : 0.0;
    }
    F[e] = v;
  }
}

// Gram matrix [F | Y]^T [F | Y] of one subspace's points, one 32 x 32 block
// of it per workgroup: blockIdx.x = subspace, blockIdx.y = block pair
// (a-block <= b-block), blockIdx.z = part: part q of gridDim.z sums the q-th
// contiguous share of list[off[s] .. off[s + 1]) (the subspace's points in
// input order) into G + q * S * Ta^2; poly_gram_sum adds the parts in order,
// so the sums are the same on every run.  The rows of a chunk of points are
// staged in LDS with all loads in flight.
__global__ __launch_bounds__(kPolyThreads) void poly_gram(const PolyDev *__restrict__ pd,
                                                          const double *__restrict__ F,
                                                          const uint32_t *__restrict__ list,
                                                          const uint32_t *__restrict__ off,
                                                          const uint32_t *__restrict__ pairs,
                                                          double *__restrict__ G) {
  extern __shared__ double gl[]; // fa[kGramChunk][kGB + 1], fb[kGramChunk][kGB + 1]
  double(*fa)[kGB + 1] = reinterpret_cast<double(*)[kGB + 1]>(gl);
  double(*fb)[kGB + 1] = reinterpret_cast<double(*)[kGB + 1]>(gl + kGramChunk * (kGB + 1));
  const uint32_t T = pd->T, Ta = T + pd->C, s = blockIdx.x;
  const uint32_t pr = pairs[blockIdx.y];
  const uint32_t a0 = (pr & 0xffffu) * kGB, b0 = (pr >> 16) * kGB;
  const uint32_t t = threadIdx.x;
  const uint32_t ra = (t / (kGB / 2)) * 2, cb = (t % (kGB / 2)) * 2; // 2 x 2 outputs
  const uint32_t q0 = off[s], len = off[s + 1] - q0;
  const uint32_t p0 = q0 + (uint32_t)((uint64_t)len * blockIdx.z / gridDim.z);
  const uint32_t p1 = q0 + (uint32_t)((uint64_t)len * (blockIdx.z + 1) / gridDim.z);
  double acc[2][2] = {{0.0, 0.0}, {0.0, 0.0}};
  constexpr int kB = 8;
  for (uint32_t base = p0; base < p1; base += kGramChunk) {
    const uint32_t m = min((uint32_t)kGramChunk, p1 - base);
    __syncthreads();
    for (uint32_t e0 = t; e0 < m * kGB; e0 += kB * kPolyThreads) {
      double va[kB], vb[kB];
#pragma unroll
      for (int u = 0; u < kB; ++u) {
        const uint32_t e = min(e0 + u * kPolyThreads, m * kGB - 1);
        const uint32_t p = e / kGB, c = e % kGB;
        const double *row = F + (uint64_t)list[base + p] * Ta;
        va[u] = a0 + c < Ta ? row[a0 + c] : 0.0;
        vb[u] = b0 + c < Ta ? row[b0 + c] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < kB; ++u) {
        const uint32_t e = e0 + u * kPolyThreads;
        if (e < m * kGB) {
          fa[e / kGB][e % kGB] = va[u];
          fb[e / kGB][e % kGB] = vb[u];
        }
      }
    }
    __syncthreads();
    for (uint32_t p = 0; p < m; ++p) {
      const double x0 = fa[p][ra], x1 = fa[p][ra + 1], y0 = fb[p][cb], y1 = fb[p][cb + 1];
      acc[0][0] += x0 * y0;
      acc[0][1] += x0 * y1;
      acc[1][0] += x1 * y0;
      acc[1][1] += x1 * y1;
    }
  }
  double *Gs = G + ((uint64_t)blockIdx.z * gridDim.x + s) * Ta * Ta;
  for (int u = 0; u < 2; ++u)
    for (int v = 0; v < 2; ++v) {
      const uint32_t a = a0 + ra + u, b = b0 + cb + v;
      if (a < Ta && b < Ta) {
        Gs[(uint64_t)a * Ta + b] = acc[u][v];
        Gs[(uint64_t)b * Ta + a] = acc[u][v];
      }
    }
}

// G[e] = sum of the parts' entries e, parts in order (Gp: [parts][S Ta^2]).
__global__ __launch_bounds__(256) void poly_gram_sum(const double *__restrict__ Gp,
                                                     uint64_t total, uint32_t parts,
                                                     double *__restrict__ G) {
  for (uint64_t e = (uint64_t)blockIdx.x * 256 + threadIdx.x; e < total;
       e += (uint64_t)gridDim.x * 256) {
    double x = Gp[e];
    for (uint32_t q = 1; q < parts; ++q) x += Gp[(uint64_t)q * total + e];
    G[e] = x;
  }
}

__device__ __forceinline__ uint32_t pk(uint32_t i, uint32_t j) { return i * (i + 1) / 2 + j; }

// One workgroup per subspace: (G + lam I) beta = R by Cholesky in LDS
// (packed lower triangle), then the two triangular solves for CC counters at
// a time, in panels of 16 terms: a panel's columns are factored with a row
// per lane in registers, then taken off the rest of the triangle at once; the
// solves take a block of 16 rows per counter in one thread's registers, then
// take it off the other rows.  Every element has the same multiply-adds in
// the same order as column by column.
// Bound: the chains of square roots and divisions (one of each per term, and
// a division per term in each solve).  Column by column, with three barriers
// per column and four per row of the solves, it took 502 us on 139 terms and
// 24 counters; in panels 248 us, of which a third was
// saved by keeping the loops over a panel's columns rolled (unrolled: 300 us).
constexpr int kSolveThreads = 512;
constexpr uint32_t kSolveNB = 16; // columns per panel

__device__ __forceinline__ double lane_value(double v, int lane) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
  return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

__global__ __launch_bounds__(kSolveThreads) void poly_solve(const PolyDev *__restrict__ pd,
                                                            const double *__restrict__ G,
                                                            uint32_t CC,
                                                            double *__restrict__ beta64,
                                                            float *__restrict__ beta32,
                                                            uint32_t *__restrict__ err) {
  extern __shared__ double L[]; // packed lower triangle, then z[T][CC]
  __shared__ double s_lam;
  constexpr uint32_t NB = kSolveNB;
  const uint32_t T = pd->T, C = pd->C, Ta = T + C, s = blockIdx.x, t = threadIdx.x;
  const uint32_t lane = t & 63u, wave = t >> 6;
  const double *Gs = G + (uint64_t)s * Ta * Ta;
  double *z = L + (uint64_t)T * (T + 1) / 2;
  double *b64 = beta64 + (uint64_t)s * T * C;
  float *b32 = beta32 + (uint64_t)s * T * C;
  if (Gs[0] == 0.0) { // no point in this subspace (the constant column sums to n_s)
    for (uint32_t e = t; e < T * C; e += kSolveThreads) {
      b64[e] = 0.0;
      b32[e] = 0.0f;
    }
    return;
  }
  // G's lower triangle into L by the whole workgroup, 8 loads per thread in
  // flight (one thread per row would wait for up to T loads in turn)
  constexpr int kB = 8;
  const uint32_t nt = T * T;
  for (uint32_t e0 = t; e0 < nt; e0 += kB * kSolveThreads) {
    double v[kB];
#pragma unroll
    for (int u = 0; u < kB; ++u) {
      const uint32_t e = min(e0 + u * kSolveThreads, nt - 1);
      v[u] = Gs[(uint64_t)(e / T) * Ta + e % T];
    }
#pragma unroll
    for (int u = 0; u < kB; ++u) {
      const uint32_t e = e0 + u * kSolveThreads, i = e / T, j = e % T;
      if (e < nt && j <= i) L[pk(i, j)] = v[u];
    }
  }
  __syncthreads();
  if (t == 0) { // the trace in index order
    double tr = 0.0;
#pragma unroll 8
    for (uint32_t i = 0; i < T; ++i) tr += L[pk(i, i)];
    s_lam = kRidge * tr / (double)T;
  }
  __syncthreads();
  for (uint32_t i = t; i < T; i += kSolveThreads) L[pk(i, i)] += s_lam;
  for (uint32_t j0 = 0; j0 < T; j0 += NB) {
    const uint32_t nb = min(NB, T - j0), j1 = j0 + nb;
    __syncthreads();
    // the panel, one row per lane: the diagonal block in lanes 0 .. 15 of every
    // wave that has rows, 48 of the rows below it in the others
    const uint32_t row = lane < NB ? (lane < nb ? j0 + lane : T) : j1 + 48 * wave + lane - NB;
    const bool work = wave == 0 || j1 + 48 * wave < T;
    double a[NB];
    if (work) {
#pragma unroll
      for (uint32_t c = 0; c < NB; ++c) {
        const uint32_t j = j0 + c;
        a[c] = c < nb && row < T && j <= row ? L[pk(row, j)] : 0.0;
      }
    }
    __syncthreads(); // every wave has the diagonal block
    if (work) {
      // rolled, with the columns moving down by one: unrolled sixteen times the
      // code is longer than its first pass through the instruction cache allows
      const bool mine = row < T && (lane >= NB || wave == 0);
#pragma unroll 1
      for (uint32_t c = 0; c < nb; ++c) {
        double d = lane_value(a[0], c);
        if (!(d > 0.0)) {
          if (t == 0) atomicOr(err, 4u);
          d = s_lam;
        }
        d = sqrt(d);
        const double x = lane == c ? d : a[0] / d;
        if (mine && j0 + c <= row) L[pk(row, j0 + c)] = x;
        // columns past the panel take rows below it, and are never reached
#pragma unroll
        for (uint32_t k = 1; k < NB; ++k) a[k - 1] = a[k] - x * lane_value(x, c + k);
      }
    }
    __syncthreads();
    // the panel's columns off the rest of the triangle (nb == NB wherever there is any)
    for (uint32_t i = j1 + t / 16; i < T; i += kSolveThreads / 16) {
      double li[NB];
#pragma unroll
      for (uint32_t c = 0; c < NB; ++c) li[c] = L[pk(i, j0) + c];
      for (uint32_t k = j1 + t % 16; k <= i; k += 16) {
        double v = L[pk(i, k)];
        const double *lk = L + pk(k, j0);
#pragma unroll
        for (uint32_t c = 0; c < NB; ++c) v -= li[c] * lk[c];
        L[pk(i, k)] = v;
      }
    }
  }
  // L z = R, then L^T beta = z, CC counters at a time: a block of rows by one
  // thread per counter, then off the other rows by all
  const uint32_t last = (T - 1) / NB * NB;
  for (uint32_t c0 = 0; c0 < C; c0 += CC) {
    const uint32_t cc = min(CC, C - c0);
    __syncthreads();
    for (uint32_t e0 = t; e0 < T * cc; e0 += kB * kSolveThreads) {
      double v[kB];
#pragma unroll
      for (int u = 0; u < kB; ++u) {
        const uint32_t e = min(e0 + u * kSolveThreads, T * cc - 1);
        v[u] = Gs[(uint64_t)(e / cc) * Ta + T + c0 + e % cc];
      }
#pragma unroll
      for (int u = 0; u < kB; ++u) {
        const uint32_t e = e0 + u * kSolveThreads;
        if (e < T * cc) z[(e / cc) * CC + e % cc] = v[u];
      }
    }
    double x[NB];
    for (uint32_t j0 = 0; j0 < T; j0 += NB) {
      const uint32_t nb = min(NB, T - j0), j1 = j0 + nb;
      __syncthreads();
      if (t < cc) {
#pragma unroll
        for (uint32_t k = 0; k < NB; ++k) x[k] = k < nb ? z[(j0 + k) * CC + t] : 0.0;
#pragma unroll 1
        for (uint32_t i = 0; i < nb; ++i) {
          const double v = x[0] / L[pk(j0 + i, j0 + i)];
          z[(j0 + i) * CC + t] = v;
          // rows past the block are never reached
#pragma unroll
          for (uint32_t k = 1; k < NB; ++k) x[k - 1] = x[k] - L[pk(min(j0 + i + k, j1 - 1), j0 + i)] * v;
        }
      }
      __syncthreads();
      for (uint32_t e = t; e < (T - j1) * cc; e += kSolveThreads) {
        const uint32_t k = j1 + e / cc, c = e % cc;
        const double *lk = L + pk(k, j0), *zi = z + j0 * CC + c; // nb == NB here
        double v = z[k * CC + c];
#pragma unroll
        for (uint32_t i = 0; i < NB; ++i) v -= lk[i] * zi[i * CC];
        z[k * CC + c] = v;
      }
    }
    for (uint32_t j0 = last + NB; j0 > 0;) {
      j0 -= NB;
      const uint32_t nb = min(NB, T - j0);
      __syncthreads();
      if (t < cc) {
#pragma unroll
        for (uint32_t k = 0; k < NB; ++k) x[k] = k < nb ? z[(j0 + nb - 1 - k) * CC + t] : 0.0;
#pragma unroll 1
        for (uint32_t i = j0 + nb; i-- > j0;) {
          const double v = x[0] / L[pk(i, i)];
          z[i * CC + t] = v;
#pragma unroll
          for (uint32_t k = 1; k < NB; ++k) x[k - 1] = x[k] - L[pk(i, i >= j0 + k ? i - k : j0)] * v;
        }
      }
      __syncthreads();
      for (uint32_t e = t; e < j0 * cc; e += kSolveThreads) {
        const uint32_t k = e / cc, c = e % cc;
        const double *lk = L + pk(j0, k), *zi = z + j0 * CC + c;
        double l[NB], x1[NB], v = z[k * CC + c];
#pragma unroll
        for (uint32_t i = 0; i < NB; ++i) { // row j0 + i starts i j0 + i (i + 1) / 2 further on
          const uint32_t u = min(i, nb - 1);
          l[i] = lk[u * j0 + u * (u + 1) / 2];
          x1[i] = zi[u * CC];
        }
#pragma unroll
        for (uint32_t u = 0; u < NB; ++u)
          if (NB - 1 - u < nb) v -= l[NB - 1 - u] * x1[NB - 1 - u];
        z[k * CC + c] = v;
      }
    }
    __syncthreads();
    for (uint32_t e = t; e < T * cc; e += kSolveThreads) {
      const uint32_t i = e / cc, c = e % cc;
      const double v = z[i * CC + c];
      b64[(uint64_t)i * C + c0 + c] = v;
      b32[(uint64_t)i * C + c0 + c] = (float)v;
    }
  }
}

// ---------------------------------------------------------------- evaluate
// P[c][l] for the valid configurations whose subspace lies in this
// workgroup's group of SG subspaces (group blockIdx.x / per_group, part
// blockIdx.x % per_group of the valid list): coefficients of the group,
// padded with zeros to CB counters so every multiply-add runs unguarded on
// vector loads, feature table and term descriptors staged in LDS.
template <int CB>
__global__ __launch_bounds__(kEvalThreads) void poly_eval(const PolyDev *__restrict__ pd,
                                                          const SpaceDev *__restrict__ sp,
                                                          const uint32_t *__restrict__ idx,
                                                          uint32_t nv,
                                                          const float *__restrict__ beta32,
                                                          uint32_t SG, uint32_t per_group,
                                                          float *__restrict__ P, uint64_t stride) {
  extern __shared__ float lds[]; // [SG][T][CB] coefficients
  __shared__ float xv[CGS_MAX_PARAMS * CGS_MAX_RADIX];
  __shared__ uint32_t terms[kPolyMaxTerms];
  const uint32_t T = pd->T, C = pd->C, S = pd->S, t = threadIdx.x;
  const uint32_t group = blockIdx.x / per_group, part = blockIdx.x % per_group;
  const uint32_t g0 = group * SG, g1 = min(S, g0 + SG);
  // 16 coefficient loads per thread in flight before the first LDS store (a
  // plain loop waits for every load in turn)
  constexpr int kB = 16;
  const uint32_t n_co = (g1 - g0) * T * CB;
  for (uint32_t e0 = t; e0 < n_co; e0 += kB * kEvalThreads) {
    float v[kB];
#pragma unroll
    for (int b = 0; b < kB; ++b) {
      const uint32_t e = e0 + b * kEvalThreads;
      const uint32_t c = e % CB, st = e / CB; // st = (s - g0) * T + term
      v[b] = (e < n_co && c < C) ? beta32[((uint64_t)g0 * T + st) * C + c] : 0.0f;
    }
#pragma unroll
    for (int b = 0; b < kB; ++b) {
      const uint32_t e = e0 + b * kEvalThreads;
      if (e < n_co) lds[e] = v[b];
    }
  }
  for (uint32_t e = t; e < CGS_MAX_PARAMS * CGS_MAX_RADIX; e += kEvalThreads) xv[e] = pd->xv32[e];
  for (uint32_t e = t; e < T; e += kEvalThreads) terms[e] = pd->terms[e];
  __syncthreads();
  // product of the features of term d for the configuration with digits lo, hi
  auto feature = [&](uint32_t d, uint64_t lo, uint64_t hi) {
    float f = 1.0f;
    for (uint32_t q = 0; q < term_count(d); ++q) {
      const uint32_t j = term_var(d, q);
      f *= xv[j * CGS_MAX_RADIX + digit_of(lo, hi, j)];
    }
    return f;
  };
  auto one = [&](uint32_t l, uint64_t lo, uint64_t hi, uint32_t s) {
    const float *bs = lds + (uint64_t)(s - g0) * T * CB;
    float acc[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) acc[c] = 0.0f;
    for (uint32_t k = 0; k < T; ++k) {
      const float f = feature(terms[k], lo, hi);
      const float4 *bk = reinterpret_cast<const float4 *>(bs + k * CB);
#pragma unroll
      for (int c4 = 0; c4 < CB / 4; ++c4) {
        const float4 b = bk[c4];
        acc[4 * c4] += f * b.x;
        acc[4 * c4 + 1] += f * b.y;
        acc[4 * c4 + 2] += f * b.z;
        acc[4 * c4 + 3] += f * b.w;
      }
    }
#pragma unroll
    for (int c = 0; c < CB; ++c)
      if ((uint32_t)c < C) P[(uint64_t)c * stride + l] = fmaxf(acc[c], 0.0f); // counters >= 0
  };
  if constexpr (CB > 32) { // two accumulator sets would not fit in registers
    for (uint32_t l = part * kEvalThreads + t; l < nv; l += per_group * kEvalThreads) {
      uint64_t lo, hi;
      decode_packed(idx[l], sp, lo, hi);
      const uint32_t s = subspace_of(pd, lo, hi);
      if (s >= g0 && s < g1) one(l, lo, hi, s);
    }
    return;
  }
  // two consecutive configurations per thread: when they share a subspace
  // (consecutive ones mostly do) each coefficient read from LDS serves both
  for (uint32_t l0 = 2 * (part * kEvalThreads + t); l0 < nv;
       l0 += 2 * per_group * kEvalThreads) {
    const uint32_t l1 = l0 + 1;
    uint64_t lo0, hi0, lo1 = 0, hi1 = 0;
    decode_packed(idx[l0], sp, lo0, hi0);
    const uint32_t s0 = subspace_of(pd, lo0, hi0);
    uint32_t s1 = ~0u;
    if (l1 < nv) {
      decode_packed(idx[l1], sp, lo1, hi1);
      s1 = subspace_of(pd, lo1, hi1);
    }
    const bool in0 = s0 >= g0 && s0 < g1, in1 = s1 >= g0 && s1 < g1;
    if (in0 && in1 && s0 == s1) {
      const float *bs = lds + (uint64_t)(s0 - g0) * T * CB;
      float a0[CB], a1[CB];
#pragma unroll
      for (int c = 0; c < CB; ++c) a0[c] = a1[c] = 0.0f;
      for (uint32_t k = 0; k < T; ++k) {
        const uint32_t d = terms[k];
        const float f0 = feature(d, lo0, hi0), f1 = feature(d, lo1, hi1);
        const float4 *bk = reinterpret_cast<const float4 *>(bs + k * CB);
#pragma unroll
        for (int c4 = 0; c4 < CB / 4; ++c4) {
          const float4 b = bk[c4];
          a0[4 * c4] += f0 * b.x;
          a0[4 * c4 + 1] += f0 * b.y;
          a0[4 * c4 + 2] += f0 * b.z;
          a0[4 * c4 + 3] += f0 * b.w;
          a1[4 * c4] += f1 * b.x;
          a1[4 * c4 + 1] += f1 * b.y;
          a1[4 * c4 + 2] += f1 * b.z;
          a1[4 * c4 + 3] += f1 * b.w;
        }
      }
#pragma unroll
      for (int c = 0; c < CB; ++c)
        if ((uint32_t)c < C)
          *reinterpret_cast<float2 *>(P + (uint64_t)c * stride + l0) =
              make_float2(fmaxf(a0[c], 0.0f), fmaxf(a1[c], 0.0f)); // counters >= 0
    } else {
      if (in0) one(l0, lo0, hi0, s0);
      if (in1) one(l1, lo1, hi1, s1);
    }
  }
}

// Nested evaluation.  Consecutive configurations share the digits of all but
// the last parameters.  With the last (non-binary) parameters of a space as
// the inner ones, a polynomial is, for fixed outer digits, a polynomial in
// the inner features alone: its coefficient of inner monomial m is
//   g_m = sum over the terms t with inner part m of beta_t * outer part of t,
// formed once per combination of outer digits, and a configuration costs M
// multiply-adds per counter instead of T (139 terms in 11 inner monomials
// for the last three parameters of four values of the 12-parameter space).
// A workgroup takes runs of consecutive tiles of consecutive combinations.
// Per tile it forms the outer parts of the terms, then g as float32 matrix
// products on the matrix cores: rows are combinations of one subspace (the
// tile's, put in order of subspace), columns counters, and each inner
// monomial has its own run of terms, filled up to eights.  A wave keeps its
// share of the coefficients in registers from tile to tile while its subspace
// stays the same.  Then each thread evaluates one of the tile's valid
// configurations.  Three barriers per tile; two workgroups per CU fill each
// other's waits.
// Measured on the 4.0M configurations of the 12-parameter space, 139 terms, 24
// counters: 276 us; every configuration by itself (poly_eval) 982 us.  g takes
// a third of it; writing the 385 MB alone takes 77 us.
typedef float v4f __attribute__((ext_vector_type(4)));
constexpr int kNestThreads = 512;
constexpr uint32_t kNestTile = 32; // combinations per tile at most
constexpr uint32_t kNestRows = 16; // combinations per matrix product
constexpr uint32_t kNestRun = 4;   // consecutive tiles of one workgroup
constexpr uint32_t kNestLdx = 35;  // features of a combination, then 1 and 0

template <int CB>
__global__ __launch_bounds__(kNestThreads, CB <= 32 ? 4 : 2) void poly_eval_nested(
    const PolyDev *__restrict__ pd, const PolyNest *__restrict__ pn,
    const SpaceDev *__restrict__ sp, const uint32_t *__restrict__ idx,
    const uint32_t *__restrict__ mask, const uint32_t *__restrict__ rank, uint32_t nv,
    const float *__restrict__ beta32, uint32_t tile_n, float *__restrict__ P, uint64_t stride) {
  extern __shared__ float4 nest_lds[]; // g [tile_n + 1][M][CB], then the parts below
  __shared__ float xf[kNestTile * kNestLdx];
  __shared__ float xv[CGS_MAX_PARAMS * CGS_MAX_RADIX];
  __shared__ uint32_t slots[kNestMaxPadded];
  __shared__ uint32_t sub[kNestTile], perm[kNestTile], group[kNestTile + 1], n_group;
  const uint32_t T = pd->T, C = pd->C, B = pd->B, tid = threadIdx.x, lane = tid & 63u;
  const uint32_t M = pn->M, r_in = pn->r_in, ldv = M | 1u, K = pn->K, ldp = K | 1u;
  const uint32_t n_slot = pn->n_slot, n_par = pn->first;
  float *g = reinterpret_cast<float *>(nest_lds);
  const uint32_t spare = tile_n * M * CB;
  float *part = g + (size_t)(tile_n + 1) * M * CB;          // [tile_n][ldp] outer parts
  float *inner = part + (size_t)tile_n * ldp + kNestSlack;  // [r_in][ldv] inner monomials
  for (uint32_t e = tid; e < CGS_MAX_PARAMS * CGS_MAX_RADIX; e += kNestThreads) xv[e] = pd->xv32[e];
  for (uint32_t e = tid; e < K; e += kNestThreads) slots[e] = pn->slots[e];
  for (uint32_t e = tid; e < kNestSlack; e += kNestThreads) part[(size_t)tile_n * ldp + e] = 0.0f;
  for (uint32_t e = tid; e < kNestTile; e += kNestThreads) {
    xf[e * kNestLdx + 32] = 1.0f;
    xf[e * kNestLdx + 33] = 0.0f;
  }
  __syncthreads();
  for (uint32_t e = tid; e < r_in * M; e += kNestThreads) {
    const uint32_t i = e / M, m = e - i * M, d = pn->inner[m];
    uint64_t lo, hi;
    decode_packed(i, sp, lo, hi); // raw index i: outer digits 0, inner digits those of i
    float f = 1.0f;
    for (uint32_t q = 0; q < term_count(d); ++q) {
      const uint32_t j = term_var(d, q);
      f *= xv[j * CGS_MAX_RADIX + digit_of(lo, hi, j)];
    }
    inner[i * ldv + m] = f;
  }
  // valid configurations before raw index k
  const uint32_t n_raw = sp->n_raw;
  auto rank_of = [&](uint32_t k) -> uint32_t {
    const uint32_t w = min(k, n_raw - 1) >> 5;
    const uint32_t r = rank[w], b = mask[w];
    return k >= n_raw ? nv : r + (uint32_t)__popc(b & ((1u << (k & 31u)) - 1u));
  };
  const uint32_t n_outer = n_raw / r_in;
  // the matrix products of this wave: half h of the steps, counters 16 n ..
  constexpr int kN = (CB + 15) / 16;
  constexpr bool kKeep = CB <= 32; // room for the coefficients beside the accumulators
  const uint32_t row = lane & 15u, k4 = lane >> 4;
  float bv[2 * kNestPairs];
  uint32_t have = ~0u; // (subspace, n, h) of bv
#pragma unroll
  for (int u = 0; u < 2 * kNestPairs; ++u) bv[u] = 0.0f;

  uint32_t bit[2] = {32u, 32u}; // subspace bits of parameters tid % 16 and that + 16
  for (uint32_t b = 0; b < B; ++b)
    for (uint32_t u = 0; u < 2; ++u)
      if (pd->bin_params[b] == tid % 16 + 16 * u) bit[u] = b;
  const uint32_t span = kNestRun * tile_n;
  for (uint32_t s0 = blockIdx.x * span; s0 < n_outer; s0 += gridDim.x * span) {
    const uint32_t s1 = min(n_outer, s0 + span);
    uint32_t l0 = rank_of(s0 * r_in);
    uint32_t l1 = rank_of(min(s0 + tile_n, s1) * r_in);
    uint32_t raw = l0 < l1 ? idx[min(l0 + tid, l1 - 1)] : 0u;
    for (uint32_t p0 = s0; p0 < s1; p0 += tile_n) {
      const uint32_t np = min(tile_n, s1 - p0);
      // the next tile's range (its first index is loaded once this is here)
      const uint32_t l2 = p0 + tile_n < s1 ? rank_of(min(p0 + 2 * tile_n, s1) * r_in) : l1;
      uint32_t raw_next = 0;
      if (l0 < l1) { // uniform: the tile has valid configurations
        // 16 threads per combination: the features of its outer digits
        for (uint32_t i = tid / 16; i < np; i += kNestThreads / 16) {
          uint64_t lo, hi;
          decode_packed((p0 + i) * r_in, sp, lo, hi);
          uint32_t s = 0;
#pragma unroll
          for (uint32_t u = 0; u < 2; ++u) {
            const uint32_t j = tid % 16 + 16 * u, digit = digit_of(lo, hi, j);
            if (j < n_par) xf[i * kNestLdx + j] = xv[j * CGS_MAX_RADIX + digit];
            s |= bit[u] < 32u ? digit << bit[u] : 0u;
          }
#pragma unroll
          for (int o = 1; o < 16; o <<= 1) s |= (uint32_t)__shfl_xor((int)s, o, 16);
          if (tid % 16 == 0) sub[i] = s;
        }
        lds_barrier();
        if (tid < 64) { // in order of subspace, in groups of up to kNestRows of one
          const uint32_t mine = lane < np ? sub[lane] : ~0u;
          uint32_t pos = 0, same = 0; // same: earlier ones of the same subspace
#pragma unroll
          for (uint32_t k = 0; k < kNestTile; ++k) {
            const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)mine, k);
            const uint32_t before = other == mine && k < lane;
            same += before;
            pos += other < mine ? 1u : before;
          }
          if (lane < np) perm[pos] = lane;
          // positions that start a group, as bits
          uint32_t starts = lane < np && same % kNestRows == 0 ? 1u << pos : 0u;
#pragma unroll
          for (int o = 1; o < 64; o <<= 1) starts |= (uint32_t)__shfl_xor((int)starts, o, 64);
          if (lane < np && (starts >> lane & 1u))
            group[__popc(starts & ((1u << lane) - 1u))] = lane;
          if (lane == 0) {
            const uint32_t n = (uint32_t)__popc(starts);
            group[n] = np;
            n_group = n;
          }
        }
        for (uint32_t i = tid / 16; i < np; i += kNestThreads / 16) {
          const float *x = xf + i * kNestLdx;
#pragma unroll 4
          for (uint32_t t = tid % 16; t < K; t += 16) {
            const uint32_t d = slots[t];
            float f = x[d & 255u];
            for (uint32_t q = 1; q < n_slot; ++q) f *= x[d >> (8 * q) & 255u];
            part[i * ldp + t] = f;
          }
        }
        lds_barrier();
        const uint32_t n_role = (uint32_t)__builtin_amdgcn_readfirstlane((int)n_group) * kN * 2;
        const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid / 64));
        for (uint32_t role = wave; role < n_role; role += kNestThreads / 64) {
          const uint32_t h = role & 1u, n = (role >> 1) % kN, q = (role >> 1) / kN;
          const uint32_t r0 = group[q], rows = group[q + 1] - r0;
          const uint32_t s = (uint32_t)__builtin_amdgcn_readfirstlane((int)sub[perm[r0]]);
          const uint32_t pair0 = h ? pn->split : 0u;
          const uint32_t pairs = (h ? K / 8 : pn->split) - pair0;
          const uint32_t key = (s * kN + n) * 2 + h, c = 16 * n + row;
          if (!kKeep || key != have) {
            have = key;
            const float *b = beta32 + (size_t)s * T * C + min(c, C - 1);
#pragma unroll
            for (int u = 0; u < 2 * kNestPairs; ++u) {
              // the term in the low byte, or bit 31: none (a zero, whatever the value read)
              const int32_t t = pn->order[min(8 * pair0 + 4 * u + k4, K - 1)];
              bv[u] = __int_as_float(__float_as_int(b[(t & 255) * C]) & ~(t >> 31));
            }
          }
          const float *a = part + perm[r0 + min(row, rows - 1)] * ldp + 8 * pair0 + k4;
          float *out[4]; // rows that do not exist are written to the spare row
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const uint32_t i = 4 * k4 + r;
            out[r] = g + (i < rows && c < CB ? perm[r0 + i] * M * CB + c : spare) +
                     (h ? pn->split_m : 0u) * CB;
          }
          const uint32_t ends = (uint32_t)__builtin_amdgcn_readfirstlane(
              (int)(uint32_t)(pn->ends >> pair0)); // last pairs of the monomials
          v4f acc0 = v4f{0.0f, 0.0f, 0.0f, 0.0f}, acc1 = acc0;
#pragma unroll
          for (int u0 = 0; u0 < kNestPairs; u0 += 4) {
            if ((uint32_t)u0 >= pairs) break;
            float av[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) av[u] = a[8 * u0 + 4 * u];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(av[2 * u], bv[2 * (u0 + u)], acc0, 0, 0, 0);
              acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(av[2 * u + 1], bv[2 * (u0 + u) + 1], acc1,
                                                          0, 0, 0);
              if (ends >> (u0 + u) & 1u) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                  *out[r] = acc0[r] + acc1[r];
                  out[r] += CB;
                }
                acc0 = acc1 = v4f{0.0f, 0.0f, 0.0f, 0.0f};
              }
            }
          }
        }
        if (l1 < l2) raw_next = idx[min(l1 + tid, l2 - 1)];
        lds_barrier();
        for (uint32_t l = l0 + tid; l < l1; l += kNestThreads) {
          const uint32_t q = fastdiv(raw, pn->div_in);
          const float *v = inner + (raw - q * r_in) * ldv;
          const float4 *gp = reinterpret_cast<const float4 *>(g + (size_t)(q - p0) * M * CB);
          if (l + kNestThreads < l1) raw = idx[l + kNestThreads];
          float acc[CB];
#pragma unroll
          for (int c = 0; c < CB; ++c) acc[c] = 0.0f;
          for (uint32_t m = 0; m < M; ++m) {
            const float f = v[m];
#pragma unroll
            for (int c4 = 0; c4 < CB / 4; ++c4) {
              const float4 b = gp[m * (CB / 4) + c4];
              acc[4 * c4] += f * b.x;
              acc[4 * c4 + 1] += f * b.y;
              acc[4 * c4 + 2] += f * b.z;
              acc[4 * c4 + 3] += f * b.w;
            }
          }
          // the loads in flight are waited for here, so that no wait falls behind the stores
          asm volatile("" ::"v"(raw), "v"(raw_next));
#pragma unroll
          for (int c = 0; c < CB; ++c)
            if ((uint32_t)c < C) P[(uint64_t)c * stride + l] = fmaxf(acc[c], 0.0f); // counters >= 0
        }
      } else if (l1 < l2) {
        raw_next = idx[min(l1 + tid, l2 - 1)];
      }
      l0 = l1;
      l1 = l2;
      raw = raw_next;
    }
  }
}

constexpr size_t kEvalLds = 144 * 1024;
constexpr size_t kSolveLds = 156 * 1024;

} // namespace

// LDS of the solve: the packed factor, then as many counters' right-hand
// sides as fit in the rest of 160 KB (at least one).
uint32_t poly_solve_cc(int T, int C) {
  const size_t tri = (size_t)T * (T + 1) / 2 * 8;
  const size_t room = tri < kSolveLds ? kSolveLds - tri : 0;
  return (uint32_t)std::max<size_t>(1, std::min<size_t>(C, room / ((size_t)T * 8)));
}
size_t poly_solve_lds(int T, int C) {
  return ((size_t)T * (T + 1) / 2 + (size_t)T * poly_solve_cc(T, C)) * 8;
}

hipError_t launch_poly_design(const SpaceDev *d_space, const uint32_t *d_idx, uint32_t nv,
                              const uint32_t *d_allowed, uint64_t *d_tile_cnt,
                              uint64_t *d_tile_off, uint32_t *d_out, hipStream_t stream) {
  const uint32_t tiles = (nv + kPolyThreads - 1) / kPolyThreads;
  const uint32_t grid = std::max<uint32_t>(1, std::min<uint32_t>(tiles, 4096));
  poly_design_count<<<grid, kPolyThreads, 0, stream>>>(d_space, d_idx, nv, d_allowed, d_tile_cnt);
  poly_excl_scan<<<1, 1024, 0, stream>>>(d_tile_cnt, d_tile_off, tiles);
  poly_design_write<<<grid, kPolyThreads, 0, stream>>>(d_space, d_idx, nv, d_allowed, d_tile_off,
                                                      d_out);
  return hipGetLastError();
}

uint32_t poly_gram_parts(int S, uint32_t n_pairs) {
  const uint64_t wgs = (uint64_t)S * n_pairs;
  return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(8, 1024 / std::max<uint64_t>(wgs, 1)));
}

hipError_t launch_poly_subspaces(const PolyDev *d_pd, const SpaceDev *d_space,
                                 const uint32_t *d_idx, uint32_t nv, const uint32_t *d_pts,
                                 uint32_t n, uint32_t *d_sub, hipStream_t stream) {
  const uint32_t grid = std::min<uint32_t>(4096, (n + kPolyThreads - 1) / kPolyThreads);
  poly_subspaces<<<grid, kPolyThreads, 0, stream>>>(d_pd, d_space, d_idx, nv, d_pts, n, d_sub);
  return hipGetLastError();
}

hipError_t launch_poly_fit(const PolyDev *d_pd, int T, int C, int S, const SpaceDev *d_space,
                           const uint32_t *d_idx, uint32_t nv, const uint32_t *d_pts,
                           const float *d_Y, uint32_t n, double *d_F,
                           const uint32_t *d_list, const uint32_t *d_off,
                           const uint32_t *d_pairs, uint32_t n_pairs, double *d_G, double *d_Gp,
                           double *d_beta64, float *d_beta32, uint32_t *d_err,
                           hipStream_t stream) {
  const uint64_t fe = (uint64_t)n * (T + C);
  const uint32_t gf = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(8192, (fe + 255) / 256));
  poly_features<<<gf, kPolyThreads, 0, stream>>>(d_pd, d_space, d_idx, nv, d_pts, d_Y, n, d_F,
                                                 d_err);
  const size_t gram_lds = (size_t)2 * kGramChunk * (kGB + 1) * sizeof(double);
  hipError_t e = allow_lds(poly_gram, gram_lds, gram_lds);
  if (e != hipSuccess) return e;
  // few (subspace, block pair) workgroups: each subspace's points in parts
  const uint32_t parts = d_Gp ? poly_gram_parts(S, n_pairs) : 1u;
  poly_gram<<<dim3(S, n_pairs, parts), kPolyThreads, gram_lds, stream>>>(
      d_pd, d_F, d_list, d_off, d_pairs, parts > 1 ? d_Gp : d_G);
  if (parts > 1) {
    const uint64_t total = (uint64_t)S * (T + C) * (T + C);
    const uint32_t g = (uint32_t)std::min<uint64_t>(4096, (total + 255) / 256);
    poly_gram_sum<<<g, 256, 0, stream>>>(d_Gp, total, parts, d_G);
  }
  const size_t lds = poly_solve_lds(T, C);
  e = allow_lds(poly_solve, lds, kSolveLds);
  if (e != hipSuccess) return e;
  poly_solve<<<S, kSolveThreads, lds, stream>>>(d_pd, d_G, poly_solve_cc(T, C), d_beta64,
                                               d_beta32, d_err);
  return hipGetLastError();
}

namespace {

constexpr size_t kNestLds = (160 - 10) * 1024; // 10 KB: the kernel's own arrays

// Outer combinations per tile of the nested evaluation: the most that leave
// room for two workgroups in a CU's LDS, or for one (0: not even eight).
uint32_t nest_tile(int CB, const PolyNest &n, size_t *lds) {
  if (n.M == 0) return 0;
  const size_t fixed = ((size_t)n.r_in * (n.M | 1) + kNestSlack + (size_t)n.M * CB) * 4;
  const size_t per = ((size_t)n.M * CB + (n.K | 1)) * 4;
  for (size_t room : {kNestLds - 80 * 1024, kNestLds})
    for (uint32_t tile = kNestTile; tile >= 8; tile /= 2)
      if (fixed + tile * per <= room) {
        *lds = fixed + tile * per;
        return tile;
      }
  return 0;
}

// Whether the nested evaluation is expected to be clearly faster.  Its tiles are
// a chain of short phases whose cost hardly depends on how many of a tile's
// configurations are valid, while a configuration by itself costs T terms: few
// terms, few valid configurations or a short tile leave nothing to gain.  The
// microseconds below were fitted to 567 spaces (3 to 16 values, 64 to 16.8M
// valid configurations of 0.01 % to all raw ones, 5 to 101 terms, 1 to 64
// counters), where each form was timed: by itself, terms and counters per valid
// configuration; nested, a workgroup's run of tiles times the launch's waves of
// workgroups, for the tiles that hold anything.  They are within a third, and
// 1.4 keeps what is not clear by itself.  Taken wherever a tile fits, the nested
// form was slower on 334 of them, down to a quarter of the speed (5 x 16 values,
// 17 % valid, 21 terms, 64 counters 30 -> 130 us); with this rule on one by more
// than 5 % (70 against 56 us).  For the space above it says 759 and 163 us.
bool nested_pays(int T, int CB, const PolyNest &n, uint32_t tile, size_t lds, uint32_t n_raw,
                 uint32_t nv) {
  const double m = 1e-6 * nv, MC = (double)n.M * CB;
  const double single = 5.0 + 0.6 * T + m * (0.03 * T * CB + (CB > 32 ? 0.2 : 0.4) * T + 0.5 * CB);
  const uint32_t n_outer = n_raw / n.r_in, tiles = (n_outer + tile - 1) / tile;
  const double groups = (tiles + kNestRun - 1) / kNestRun, at_once = lds <= kNestLds - 80 * 1024 ? 512 : 256;
  const double serial = std::min(tiles, kNestRun) * std::max(1.0, groups / at_once);
  const double per_tile = (double)nv / tiles, held = std::min(1.0, per_tile);
  const double eval = std::max(1.0, per_tile / kNestThreads) * (0.0024 * MC + 0.07 * CB);
  const double form = tile / 32.0 * n.K * (0.0016 + 0.0007 * ((CB + 15) / 16));
  const double nested = 13.0 + 0.006 * n.M * n.r_in + serial * (1.7 + held * (0.7 + eval + form)) +
                        m * 0.64 * CB;
  return nested * 1.4 < single;
}

int counters_padded(int C) {
  return C <= 8 ? 8 : C <= 16 ? 16 : C <= 24 ? 24 : C <= 32 ? 32 : C <= 48 ? 48 : 64;
}

} // namespace

bool poly_is_nested(int T, int C, const PolyNest &nest, uint32_t n_raw, uint32_t nv) {
  size_t lds = 0;
  const int CB = counters_padded(C);
  const uint32_t tile = nest_tile(CB, nest, &lds);
  return tile && nested_pays(T, CB, nest, tile, lds, n_raw, nv);
}

// Nested where the model was found to be (poly_is_nested); otherwise every
// configuration by itself.
hipError_t launch_poly_eval(const PolyDev *d_pd, int T, int C, int S, const PolyNest &nest,
                            const PolyNest *d_nest, const SpaceDev *d_space, uint32_t n_raw,
                            const uint32_t *d_idx, const uint32_t *d_mask,
                            const uint32_t *d_rank, uint32_t nv, const float *d_beta32,
                            float *d_P, uint64_t stride, hipStream_t stream) {
  const int CB = counters_padded(C);
  hipError_t e = hipSuccess;
  size_t nest_lds = 0;
  if (const uint32_t tile = nest_tile(CB, nest, &nest_lds)) { // nest.M == 0: none
    const uint32_t n_outer = n_raw / nest.r_in;
    const uint32_t span = kNestRun * tile;
    const uint32_t grid = std::min<uint32_t>((n_outer + span - 1) / span, 1u << 20);
#define CGS_POLY_NEST(CBV)                                                                      \
  do {                                                                                          \
    e = allow_lds(poly_eval_nested<CBV>, nest_lds, kNestLds);                                   \
    if (e == hipSuccess)                                                                        \
      poly_eval_nested<CBV><<<grid, kNestThreads, nest_lds, stream>>>(                          \
          d_pd, d_nest, d_space, d_idx, d_mask, d_rank, nv, d_beta32, tile, d_P, stride);       \
  } while (0)
    switch (CB) {
    case 8: CGS_POLY_NEST(8); break;
    case 16: CGS_POLY_NEST(16); break;
    case 24: CGS_POLY_NEST(24); break;
    case 32: CGS_POLY_NEST(32); break;
    case 48: CGS_POLY_NEST(48); break;
    default: CGS_POLY_NEST(64); break;
    }
#undef CGS_POLY_NEST
    return e != hipSuccess ? e : hipGetLastError();
  }
  const size_t per = (size_t)T * CB * 4;
  const uint32_t SG = (uint32_t)std::max<size_t>(1, std::min<size_t>(S, kEvalLds / per));
  const uint32_t groups = (S + SG - 1) / SG;
  const size_t lds = SG * per;
  const uint32_t grid = std::max<uint32_t>(
      1, std::min<uint32_t>(1024, (nv + kEvalThreads - 1) / kEvalThreads));
#define CGS_POLY_EVAL(CBV)                                                                      \
  do {                                                                                          \
    e = allow_lds(poly_eval<CBV>, lds, kEvalLds);                                               \
    if (e == hipSuccess)                                                                        \
      poly_eval<CBV><<<grid * groups, kEvalThreads, lds, stream>>>(                             \
          d_pd, d_space, d_idx, nv, d_beta32, SG, grid, d_P, stride);                           \
  } while (0)
  switch (CB) {
  case 8: CGS_POLY_EVAL(8); break;
  case 16: CGS_POLY_EVAL(16); break;
  case 24: CGS_POLY_EVAL(24); break;
  case 32: CGS_POLY_EVAL(32); break;
  case 48: CGS_POLY_EVAL(48); break;
  default: CGS_POLY_EVAL(64); break;
  }
#undef CGS_POLY_EVAL
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

} // namespace cgs
