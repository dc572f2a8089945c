// Exact filtered kNN over the full-precision vectors: the exact top-k over
// the predicate-passing rows that Section 3.1 takes as ground truth, and the
// pre-filtering baseline (i) of Section 3.2.  A row's distance is
//   d = sum_{j<D} (x_j - q_j)^2,
// summed in j order from +0 in fp32 with the difference, its square and each
// addition rounded separately; rows rank by (d, original id).
//
// Two plans, chosen per batch by the host:
//  * direct: every selected row of a query is scored exactly
//    (exact_rerank_kernel over the query's row interval, its selection
//    bitmap masking residual clauses);
//  * screened, for batches whose queries share rows (wide intervals, or an
//    unclustered index where every query spans all rows): a bf16 matrix-core
//    pass computes dd = |x|^2 + |q|^2 - 2 x.q for 32 queries x 32 rows per
//    tile.  eps(q) bounds |dd - d| for every row (bf16 rounding of x and q,
//    fp32 accumulation, and the fp32 rounding of d itself).  Pass 1 reads a
//    sample (every S-th tile of a wavefront) and keeps,
//    per (query, wavefront, chunk, group of R lanes), the smallest dd of the
//    rows it saw (R is chosen so that a query's interval spans several times
//    k such bins); these come from distinct rows, so the k-th smallest of
//    them, v_k, has k rows with d <= v_k + eps, and every row of the exact
//    top k has dd <= v_k + 2 eps.  Pass 2 lists the rows under that bound, and only
//    those are scored exactly.  Both plans end in the same exact scoring and
//    merge, so results are identical.
#include <hip/hip_runtime.h>
#include <cfloat>
#include <climits>
#include <cmath>

#include "exact_bound.h"
#include "ifvs_internal.h"
#include "topk_device.h"

namespace ifvs {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr int kExWaves = 8;        // wavefronts per screening workgroup
constexpr int kExKC = 8;           // K steps (16 dims each) loaded per round
// Row lengths of up to kExKeep K steps (128 dimensions) keep the query tile's
// fragments and the next row tile's in registers: 8 VGPRs a step beside about
// 60, which fills the 128 of sixteen wavefronts per CU at 8 steps (pass 2 then
// spills five).  Longer rows load both in the loop.  4M rows, 256 queries of 10% / 50%, us
// with the loads in the loop -> held (one run, eps from 2^-8 for every value and an
// atomic per candidate on both sides): 16 dimensions 323 / 540 -> 314 / 417, 32:
// 318 / 591 -> 283 / 537, 64: 352 / 639 -> 322 / 638, 112: 501 / 963 -> 459 /
// 914, 128: 558 / 1096 -> 529 / 1073.
constexpr int kExKeep = 8;

// fp32 -> bf16 bits, round to nearest even (finite inputs).
__device__ __forceinline__ uint32_t bf16_bits(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// How far that rounding moves a value (infinite where it overflows).
__device__ __forceinline__ double bf16_error(float f) {
  return static_cast<double>(f) - static_cast<double>(__uint_as_float(bf16_bits(f) << 16));
}

// Eight consecutive values of a row (zero past `dim`) as one MFMA fragment.
__device__ __forceinline__ uint4 pack_fragment(const float* __restrict__ row, int dim, int k0) {
  uint32_t w[4];
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    const int k = k0 + 2 * h;
    const uint32_t lo = k < dim ? bf16_bits(row[k]) : 0u;
    const uint32_t hi = k + 1 < dim ? bf16_bits(row[k + 1]) : 0u;
    w[h] = lo | (hi << 16);
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// ---------------------------------------------------------------- staging
// One thread per physical row: the fp32 copies (64-row tiles,
// xt[(r / 64 * dim + j) * 64 + r % 64], for scans of consecutive rows, and
// row-major, xr[r * dim + j], for scattered rows), |x|^2 (fp32, summed in j
// order) and the
// bf16 fragments of its 32-row tile (xb[(tile32 * ks + s) * 64 + lane]: lane
// l holds row l % 32, dims s * 16 + (l / 32) * 8 .. + 8).  Also the largest
// norm and, after it, the largest movement by the rounding to bf16 (as fp32
// bits; both are non-negative) and a count of non-finite values.
__global__ __launch_bounds__(256) void exact_stage_kernel(const float* __restrict__ x, int64_t n, int dim,
                                                          int ks, const int32_t* __restrict__ perm,
                                                          float* __restrict__ xt, float* __restrict__ xr,
                                                          uint4* __restrict__ xb,
                                                          float* __restrict__ xn, unsigned* __restrict__ max_norm_bits,
                                                          unsigned long long* __restrict__ bad) {
  const int64_t r = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t n32 = (n + 31) / 32 * 32;
  if (r >= n32) return;
  const bool real = r < n;
  const float* src = real ? x + static_cast<size_t>(perm ? perm[r] : r) * dim : nullptr;
  float acc = 0.0f;
  double moved = 0.0;
  unsigned nonfinite = 0;
  if (real) {
    for (int j = 0; j < dim; ++j) {
      const float v = src[j];
      const double by = bf16_error(v);
      moved += by * by;
      xt[(static_cast<size_t>(r >> 6) * dim + j) * 64 + (r & 63)] = v;
      xr[static_cast<size_t>(r) * dim + j] = v;
      acc = __fadd_rn(acc, __fmul_rn(v, v));
      nonfinite += isfinite(v) ? 0u : 1u;
    }
  }
  xn[r] = acc;
  const int64_t t32 = r >> 5;
  const int lane_lo = static_cast<int>(r & 31);
  for (int s = 0; s < ks; ++s)
    for (int h = 0; h < 2; ++h) {
      const uint4 f = real ? pack_fragment(src, dim, s * 16 + h * 8) : make_uint4(0, 0, 0, 0);
      xb[(static_cast<size_t>(t32) * ks + s) * 64 + h * 32 + lane_lo] = f;
    }
  if (real) {
    atomicMax(max_norm_bits, __float_as_uint(sqrtf(acc)));
    atomicMax(max_norm_bits + 1, __float_as_uint(static_cast<float>(sqrt(moved) * (1.0 + 0x1p-22))));
    if (nonfinite) atomicAdd(bad, static_cast<unsigned long long>(nonfinite));
  }
}

// ------------------------------------------------------------ query prep
// One wavefront per query position p (original query qorder[p]): its bf16
// fragments in 32-query tiles, |q|^2, and eps(p) (exact_eps), computed in fp64
// from the rows' largest norm and rounding and the query's, and rounded up.
// Also clears the position's candidate count.
__global__ __launch_bounds__(64) void exact_query_kernel(const float* __restrict__ q, int dim, int ks, int nq,
                                                         const int32_t* __restrict__ qorder,
                                                         const unsigned* __restrict__ max_norm_bits,
                                                         uint4* __restrict__ qb, float* __restrict__ qn,
                                                         float* __restrict__ eps, int32_t* __restrict__ cand_n) {
  const int p = blockIdx.x;
  const int lane = threadIdx.x;
  const int t = p / 32, lane_lo = p % 32;
  const bool real = p < nq;
  const float* row = real ? q + static_cast<size_t>(qorder[p]) * dim : nullptr;
  for (int s = lane; s < 2 * ks; s += 64) {
    const int step = s >> 1, h = s & 1;
    const uint4 f = real ? pack_fragment(row, dim, step * 16 + h * 8) : make_uint4(0, 0, 0, 0);
    qb[(static_cast<size_t>(t) * ks + step) * 64 + h * 32 + lane_lo] = f;
  }
  if (!real) return;
  double s2 = 0.0, moved = 0.0;
  float acc = 0.0f;
  if (lane == 0) {
    for (int j = 0; j < dim; ++j) {
      const double by = bf16_error(row[j]);
      acc = __fadd_rn(acc, __fmul_rn(row[j], row[j]));
      s2 += static_cast<double>(row[j]) * row[j];
      moved += by * by;
    }
    const double qnorm = sqrt(s2);
    const double X = static_cast<double>(__uint_as_float(*max_norm_bits));
    qn[p] = acc;
    eps[p] = exact_eps(dim, X, __uint_as_float(max_norm_bits[1]), qnorm, sqrt(moved));
    cand_n[p] = 0;
  }
}

// --------------------------------------------------------------- screening
struct ScreenArgs {
  const uint4* xb;            // row fragments
  const float* xn;            // [n32] |x|^2
  const uint4* qb;            // query fragments
  const float* qn;            // [positions] |q|^2
  const float* thr;           // [positions] pass 2: keep rows with dd <= thr
  const int32_t* qorder;
  const int64_t* iv;          // [nq original][2]
  const DevPred* preds;       // residual_mask per original query
  const uint64_t* bitmap;     // [nq original][stride64] physical order
  int64_t stride64;
  int nq, ks;
  int64_t chunk_rows;         // rows per workgroup chunk (multiple of 32 * kExWaves)
  int splits;                 // chunks per query tile
  int step;                   // pass 1: a wavefront's every step-th tile
  int bin_lanes;              // R: lanes whose minima share one bin (1, 2, ..., 32)
  float* bins;                // pass 1: [positions][splits * kExWaves * 32 / R]
  int32_t* cand;              // pass 2: [positions][cand_cap]
  int32_t* cand_n;
  int64_t cand_cap;
};

struct QueryInfo {
  int64_t iv0, iv1;
  float qn, thr;
  int32_t orig, resid;
};

// What a (row, query) cell is tested against (rows fit 31 bits; an empty
// interval has width 0).
struct alignas(16) ScreenCell {
  uint32_t row0, width;
  float bound;                  // pass 2: rows whose |x|^2 - 2 x.q exceeds this are no candidates
  uint32_t resid;
};

// grid.x = splits * query tiles.  Each workgroup scores the rows of one
// chunk of its 32-query tile's hull (the smallest row range holding all 32
// intervals); wavefront w takes the chunk's 32-row tiles w, w + 8, ...
//
// Bound by the row fragments' way from L2 and by the test of 16 (row, query)
// cells a lane: the queries' fragments stay in registers (kExKeep), the next
// tile's rows are loaded while this one is tested, and a cell's test is one
// 16-byte LDS read, a subtraction, a multiply-add and two comparisons.  10M x
// 96 dimensions, 256 queries of 10%: pass 1 690 -> 123 us (an eighth of the
// tiles), pass 2 820 -> 660 (3.3 GB of fragments, 5 TB/s).
template <int PASS, int KS>
__global__ __launch_bounds__(kExWaves * 64) __attribute__((amdgpu_waves_per_eu(KS > 0 && KS <= kExKeep ? 4 : 2)))
void exact_screen_kernel(const ScreenArgs a) {
  __shared__ QueryInfo s_q[32];
  __shared__ ScreenCell s_cell[32];
  __shared__ int64_t s_hull[2];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int qt = blockIdx.x / a.splits, chunk = blockIdx.x % a.splits;
  const int ks = KS > 0 ? KS : a.ks;
  if (threadIdx.x < 32) {
    const int p = qt * 32 + threadIdx.x;
    QueryInfo qi{0, 0, 0.0f, -1.0f, -1, 0};
    if (p < a.nq) {
      const int o = a.qorder[p];
      qi.iv0 = a.iv[2 * o];
      qi.iv1 = a.iv[2 * o + 1];
      qi.qn = a.qn[p];
      qi.thr = PASS == 2 ? a.thr[p] : 0.0f;
      qi.orig = o;
      qi.resid = a.preds[o].residual_mask != 0;
      if (qi.iv1 <= qi.iv0) qi.iv0 = qi.iv1 = 0;
    }
    s_q[threadIdx.x] = qi;
    s_cell[threadIdx.x] = ScreenCell{static_cast<uint32_t>(qi.iv0), static_cast<uint32_t>(qi.iv1 - qi.iv0),
                                     PASS == 2 ? __fsub_rn(qi.thr, qi.qn) : 0.0f, static_cast<uint32_t>(qi.resid)};
    // hull of the tile's non-empty intervals
    int64_t lo = qi.iv1 > qi.iv0 ? qi.iv0 : INT64_MAX, hi = qi.iv1 > qi.iv0 ? qi.iv1 : 0;
    bool res = qi.resid != 0;
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) {
      lo = min(lo, static_cast<int64_t>(__shfl_xor(lo, o, 32)));
      hi = max(hi, static_cast<int64_t>(__shfl_xor(hi, o, 32)));
      const int other = __shfl_xor(static_cast<int>(res), o, 32);   // every lane shuffles
      res = res || other != 0;
    }
    if (threadIdx.x == 0) {
      s_hull[0] = lo;
      s_hull[1] = hi;
    }
    if (threadIdx.x == 0) s_q[0].resid |= res ? 2 : 0;   // bit 1: some query of the tile has residual clauses
  }
  __syncthreads();
  const bool any_resid = (s_q[0].resid & 2) != 0;
  const int64_t hull_lo = s_hull[0], hull_hi = s_hull[1];
  int64_t r_begin = hull_lo + static_cast<int64_t>(chunk) * a.chunk_rows;
  int64_t r_end = min(hull_hi, r_begin + a.chunk_rows);
  if (hull_hi <= hull_lo) r_begin = r_end = 0;
  // 32-row tiles of the chunk (rows outside [r_begin, r_end) are masked)
  const int64_t t_begin = r_begin >> 5, t_end = (r_end + 31) >> 5;

  // This lane's 16 output cells: query m(i) = 8 (i / 4) + 4 (lane / 32) + i % 4,
  // row lane % 32 of the tile.
  const int half = lane >> 5;
  float run_min[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) run_min[i] = __builtin_inff();
  const uint4* a_frag = a.qb + static_cast<size_t>(qt) * ks * 64;
  constexpr bool kKeepA = KS > 0 && KS <= kExKeep;
  uint4 ka[kKeepA ? KS : 1];
  if constexpr (kKeepA) {
#pragma unroll
    for (int u = 0; u < KS; ++u) ka[u] = a_frag[u * 64 + lane];
  }

  const int64_t step = static_cast<int64_t>(kExWaves) * (PASS == 1 ? a.step : 1);
  uint4 nb[kKeepA ? KS : 1];
  float nx = 0.0f;
  // (past the end: the last tile again, unused)
  auto load_rows = [&](int64_t t) {
    if constexpr (kKeepA) {
      const int64_t tc = t < t_end ? t : t_end - 1;
      const uint4* b_frag = a.xb + static_cast<size_t>(tc) * ks * 64;
#pragma unroll
      for (int u = 0; u < KS; ++u) nb[u] = b_frag[u * 64 + lane];
      nx = a.xn[tc * 32 + (lane & 31)];
    }
  };
  if (t_begin + wave < t_end) load_rows(t_begin + wave);
  for (int64_t t = t_begin + wave; t < t_end; t += step) {
    f32x16 acc = {};
    float xr = nx;
    if constexpr (kKeepA) {
#pragma unroll
      for (int u = 0; u < KS; ++u)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(&ka[u]),
                                                        *reinterpret_cast<const bf16x8*>(&nb[u]), acc, 0, 0, 0);
      load_rows(t + step);
    } else {
      const uint4* b_frag = a.xb + static_cast<size_t>(t) * ks * 64;
      xr = a.xn[t * 32 + (lane & 31)];
      for (int s0 = 0; s0 < ks; s0 += kExKC) {
        uint4 bv[kExKC], av[kExKC];
#pragma unroll
        for (int u = 0; u < kExKC; ++u)
          if (KS > 0 ? (s0 + u < KS) : (s0 + u < ks)) {
            bv[u] = b_frag[(s0 + u) * 64 + lane];
            av[u] = a_frag[(s0 + u) * 64 + lane];
          }
#pragma unroll
        for (int u = 0; u < kExKC; ++u)
          if (KS > 0 ? (s0 + u < KS) : (s0 + u < ks))
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(&av[u]),
                                                            *reinterpret_cast<const bf16x8*>(&bv[u]), acc, 0, 0, 0);
      }
    }
    const uint32_t row = static_cast<uint32_t>(t * 32) + (lane & 31);
    const bool in_chunk = row >= static_cast<uint32_t>(r_begin) && row < static_cast<uint32_t>(r_end);
    uint32_t hits = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int m = 8 * (i >> 2) + 4 * half + (i & 3);
      const ScreenCell cell = s_cell[m];
      bool sel = in_chunk && row - cell.row0 < cell.width;
      if (any_resid && sel && (cell.resid & 1))
        sel = (a.bitmap[static_cast<size_t>(s_q[m].orig) * a.stride64 + (row >> 6)] >> (row & 63)) & 1ull;
      const float dd = __fmaf_rn(-2.0f, acc[i], xr);      // without |q|^2
      if (PASS == 1) {
        if (sel) run_min[i] = fminf(run_min[i], dd);
      } else {
        // (not `<=`: where |x|^2, |q|^2 or x.q overflow, dd or the bound is NaN,
        // and the row has to be scored)
        hits |= (sel && !(dd > cell.bound) ? 1u : 0u) << i;
      }
    }
    // Candidates are rare where intervals are long: a lane's loop over its own
    // cells (16 inlined appends would not fit the registers).  Where a short
    // interval lies within the error bound most rows are: one atomic per query
    // and half wavefront (2682 queries of 0.3% of 200K x 400 dimensions: the
    // lane loop 1215 us, this 286; on 10M x 96, 10%, the lane loop is 2% faster).
    const uint64_t with_hits = PASS == 2 ? __ballot(hits != 0) : 0ull;
    if (__popcll(with_hits) > 8) {
#pragma unroll 1
      for (int i = 0; i < 16; ++i) {
        const bool hit = (hits >> i) & 1u;
        const uint64_t both = __ballot(hit);
        if (both == 0) continue;
        const uint32_t mine = static_cast<uint32_t>(half ? both >> 32 : both);
        const int first = mine != 0 ? __builtin_ctz(mine) : 0;
        const int p = qt * 32 + 8 * (i >> 2) + 4 * half + (i & 3);
        int pos = 0;
        if (hit && (lane & 31) == first) pos = atomicAdd(&a.cand_n[p], __popc(mine));
        pos = __shfl(pos, 32 * half + first, 64) + __popc(mine & ((1u << (lane & 31)) - 1u));
        if (hit && pos < a.cand_cap) a.cand[static_cast<size_t>(p) * a.cand_cap + pos] = static_cast<int32_t>(row);
      }
    } else if (with_hits != 0) {
      while (hits != 0) {
        const int i = __builtin_ctz(hits);
        hits &= hits - 1;
        const int p = qt * 32 + 8 * (i >> 2) + 4 * half + (i & 3);
        const int pos = atomicAdd(&a.cand_n[p], 1);
        if (pos < a.cand_cap) a.cand[static_cast<size_t>(p) * a.cand_cap + pos] = static_cast<int32_t>(row);
      }
    }
  }
  if (PASS == 1) {
    // One value per (query, wavefront, chunk, group of R lanes): the smallest
    // over the R lanes' rows.
    const int R = a.bin_lanes, per = 32 / R;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      float v = run_min[i];
      for (int o = 1; o < R; o <<= 1) v = fminf(v, __shfl_xor(v, o, 32));
      run_min[i] = v;
    }
    if ((lane & (R - 1)) == 0) {
      const size_t n_bins = static_cast<size_t>(a.splits) * kExWaves * per;
      const size_t slot = static_cast<size_t>(chunk * kExWaves + wave) * per + (lane & 31) / R;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int p = qt * 32 + 8 * (i >> 2) + 4 * half + (i & 3);
        if (p < a.nq) a.bins[static_cast<size_t>(p) * n_bins + slot] = __fadd_rn(run_min[i], s_q[p - qt * 32].qn);
      }
    }
  }
}

// ---------------------------------------------------------------- threshold
// One wavefront per query position: v_k = k-th smallest bin value, and the
// candidate bound thr = v_k + 2 eps (+inf while fewer than k bins hold a
// row, NaN without a finite eps: neither leaves a row out).
__global__ __launch_bounds__(64) void exact_threshold_kernel(const float* __restrict__ bins, int64_t n_bins, int k,
                                                             int kpl, const float* __restrict__ eps,
                                                             float* __restrict__ thr) {
  extern __shared__ uint64_t pool[];
  const int p = blockIdx.x;
  const int lane = threadIdx.x;
  const float* src = bins + static_cast<size_t>(p) * n_bins;
  int cnt = 0;
  uint64_t kth = kNoKey;
  for (int64_t b = 0; b < n_bins; b += 64) {
    const int64_t i = b + lane;
    const float v = i < n_bins ? src[i] : __builtin_inff();
    const bool ok = fabsf(v) < __builtin_inff();       // (-inf: an overflowed sum, no bound)
    const uint64_t key = (static_cast<uint64_t>(ordered_bits(v)) << 32) | static_cast<uint32_t>(i);
    pool_push(pool, cnt, kth, key, ok && key < kth, k, kpl);
  }
  pool_compact(pool, cnt, kth, k, kpl);
  if (lane == 0) {
    float t = __builtin_inff();
    if (kth != kNoKey) {
      const double bound = static_cast<double>(from_ordered_bits(static_cast<uint32_t>(kth >> 32))) +
                           2.0 * static_cast<double>(eps[p]);
      t = static_cast<float>(bound * (1.0 + 0x1p-20) + 1e-30);
    }
    thr[p] = t;
  }
}

// ------------------------------------------------------------------ rerank
constexpr int kStageDims = 64;     // dimensions of 64 rows staged in LDS per step

struct RerankArgs {
  const float* xt;            // fp32 rows in 64-row tiles, physical order
  const float* xr;            // fp32 rows, row-major, physical order
  int dim;
  const float* q;             // [nq original][dim]
  const int32_t* qorder;
  const int64_t* iv;
  const DevPred* preds;
  const uint64_t* bitmap;
  int64_t stride64;
  const int32_t* perm;
  const int32_t* cand;        // screened: [positions][cand_cap]
  const int32_t* cand_n;      // null: direct plan
  int64_t cand_cap;
  int k, kpl, chunks;
  uint64_t* partials;         // [positions][chunks][k]
};

// grid = (chunks, positions), one wavefront each: chunk c of the query's
// work -- its candidate list (LISTED: screened plan, list not overflowed) or
// its row interval (direct plan, or a list that overflowed) -- scored
// exactly, the k best keys written to partials.
//  * Consecutive rows (an interval): each lane reads its own row from the
//    64-row tiles, one coalesced 256-byte load per dimension for the wave.
//  * Scattered rows (a candidate list): the 64 lanes' rows are staged in
//    LDS 64 dimensions at a time from the row-major copy, one coalesced
//    256-byte load per row, then each lane reads its own row.
// Either way each lane adds its row's terms in j order.
template <bool LISTED>
__global__ __launch_bounds__(64) void exact_rerank_kernel(const RerankArgs a) {
  extern __shared__ uint64_t smem_r[];
  uint64_t* pool = smem_r;
  const int dim_pad = (a.dim + kStageDims - 1) / kStageDims * kStageDims;
  float* s_q = reinterpret_cast<float*>(smem_r + 64 * a.kpl);
  float* s_x = s_q + dim_pad;                     // LISTED: [64 rows][kStageDims + 1]
  const int c = blockIdx.x, p = blockIdx.y;
  const int lane = threadIdx.x;
  const int o = a.qorder[p];
  for (int j = lane; j < dim_pad; j += 64) s_q[j] = j < a.dim ? a.q[static_cast<size_t>(o) * a.dim + j] : 0.0f;
  __syncthreads();
  const int64_t iv0 = a.iv[2 * o], iv1 = a.iv[2 * o + 1];
  const bool resid = a.preds[o].residual_mask != 0;
  const bool listed = LISTED && a.cand_n[p] <= a.cand_cap;
  int cnt = 0;
  uint64_t thr = kNoKey;
  auto offer = [&](int64_t row, bool ok, float d) {
    uint64_t key = kNoKey;
    if (ok) {
      const uint32_t id = a.perm ? static_cast<uint32_t>(a.perm[row]) : static_cast<uint32_t>(row);
      key = (static_cast<uint64_t>(ordered_bits(d)) << 32) | id;
    }
    pool_push(pool, cnt, thr, key, ok && key < thr, a.k, a.kpl);
  };
  if (listed) {
    const int64_t n_items = a.cand_n[p];
    const int64_t per = (n_items + a.chunks - 1) / a.chunks;
    const int64_t i0 = static_cast<int64_t>(c) * per, i1 = min(n_items, i0 + per);
    const int32_t* list = a.cand + static_cast<size_t>(p) * a.cand_cap;
    for (int64_t b = i0; b < i1; b += 64) {
      const int64_t i = b + lane;
      const bool ok = i < i1;
      const int32_t row = ok ? list[i] : 0;
      const uint64_t okm = __ballot(ok);
      float d = 0.0f;
      for (int j0 = 0; j0 < a.dim; j0 += kStageDims) {
        const int nj = min(kStageDims, a.dim - j0);
#pragma unroll
        for (int r0 = 0; r0 < 64; r0 += 16) {
          float v[16];
#pragma unroll
          for (int u = 0; u < 16; ++u) {
            const int ri = __builtin_amdgcn_readlane(row, r0 + u);
            const bool live = ((okm >> (r0 + u)) & 1) && lane < nj;
            v[u] = live ? a.xr[static_cast<size_t>(ri) * a.dim + j0 + lane] : 0.0f;
          }
#pragma unroll
          for (int u = 0; u < 16; ++u) s_x[(r0 + u) * (kStageDims + 1) + lane] = v[u];
        }
        wave_lds_fence();
        if (ok) {
          const float* xrow = s_x + lane * (kStageDims + 1);
          for (int j = 0; j < nj; ++j) {
            const float e = __fsub_rn(xrow[j], s_q[j0 + j]);
            d = __fadd_rn(d, __fmul_rn(e, e));
          }
        }
        wave_lds_fence();
      }
      offer(row, ok, d);
    }
  } else if (iv1 > iv0) {
    // 64-row tiles of the interval, dealt out in contiguous runs
    const int64_t t0 = iv0 >> 6, t1 = (iv1 + 63) >> 6;
    const int64_t per = (t1 - t0 + a.chunks - 1) / a.chunks;
    const int64_t ta = t0 + static_cast<int64_t>(c) * per, tb = min(t1, ta + per);
    for (int64_t t = ta; t < tb; ++t) {
      const int64_t row = t * 64 + lane;
      bool ok = row >= iv0 && row < iv1;
      if (ok && resid) ok = (a.bitmap[static_cast<size_t>(o) * a.stride64 + t] >> lane) & 1ull;
      float d = 0.0f;
      if (ok) {
        const float* xr = a.xt + static_cast<size_t>(t) * a.dim * 64 + lane;
        // 16 values in flight, then added in j order
        int j = 0;
        for (; j + 16 <= a.dim; j += 16) {
          float v[16];
#pragma unroll
          for (int u = 0; u < 16; ++u) v[u] = xr[static_cast<size_t>(j + u) * 64];
#pragma unroll
          for (int u = 0; u < 16; ++u) {
            const float e = __fsub_rn(v[u], s_q[j + u]);
            d = __fadd_rn(d, __fmul_rn(e, e));
          }
        }
        for (; j < a.dim; ++j) {
          const float e = __fsub_rn(xr[static_cast<size_t>(j) * 64], s_q[j]);
          d = __fadd_rn(d, __fmul_rn(e, e));
        }
      }
      offer(row, ok, d);
    }
  }
  pool_compact(pool, cnt, thr, a.k, a.kpl);
  uint64_t* dst = a.partials + (static_cast<size_t>(p) * a.chunks + c) * a.k;
  for (int e = lane; e < a.k; e += 64) dst[e] = pool[e];
}

template <int KS>
const void* screen_symbol(int pass) {
  return pass == 1 ? reinterpret_cast<const void*>(&exact_screen_kernel<1, KS>)
                   : reinterpret_cast<const void*>(&exact_screen_kernel<2, KS>);
}

// Reconstruction from the codes (the reconstruct-then-exact baseline (ii) of
// Section 3.2): physical row r, dimension m * dsub + j, is codeword
// C_PQ[m][code_r[m]][j]; one thread per (row, subspace).
__global__ __launch_bounds__(256) void decode_kernel(const uint32_t* __restrict__ codes_t, int64_t n, int M, int mw,
                                                     int dsub, const float* __restrict__ cpq, float* __restrict__ x) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n * M) return;
  const int64_t r = i / M;
  const int m = static_cast<int>(i % M);
  const uint32_t word = codes_t[((r >> 6) * mw + (m >> 2)) * 64 + (r & 63)];
  const int code = static_cast<int>((word >> (8 * (m & 3))) & 0xFFu);
  const float* c = cpq + (static_cast<size_t>(m) * kKsub + code) * dsub;
  float* dst = x + static_cast<size_t>(r) * M * dsub + static_cast<size_t>(m) * dsub;
  for (int j = 0; j < dsub; ++j) dst[j] = c[j];
}

}  // namespace

hipError_t launch_decode(const uint32_t* codes_t, int64_t n, int m, int mw, int dsub, const float* cpq, float* x,
                         hipStream_t s) {
  const int64_t total = n * m;
  decode_kernel<<<static_cast<unsigned>((total + 255) / 256), 256, 0, s>>>(codes_t, n, m, mw, dsub, cpq, x);
  return hipGetLastError();
}

int exact_ksteps(int dim) { return (dim + 15) / 16; }

hipError_t launch_exact_stage(const float* x, int64_t n, int dim, const int32_t* perm, float* xt, float* xr,
                              uint4* xb, float* xn, unsigned* max_norm_bits, unsigned long long* bad, hipStream_t s) {
  const int64_t n32 = (n + 31) / 32 * 32;
  const unsigned blocks = static_cast<unsigned>((n32 + 255) / 256);
  exact_stage_kernel<<<blocks, 256, 0, s>>>(x, n, dim, exact_ksteps(dim), perm, xt, xr, xb, xn, max_norm_bits,
                                            bad);
  return hipGetLastError();
}

hipError_t launch_exact_queries(const float* q, int dim, int nq, const int32_t* qorder, const unsigned* max_norm_bits,
                                uint4* qb, float* qn, float* eps, int32_t* cand_n, hipStream_t s) {
  const int padded = (nq + 31) / 32 * 32;
  exact_query_kernel<<<padded, 64, 0, s>>>(q, dim, exact_ksteps(dim), nq, qorder, max_norm_bits, qb, qn, eps,
                                          cand_n);
  return hipGetLastError();
}

hipError_t launch_exact_screen(const ExactScreen& e, int pass, hipStream_t s) {
  ScreenArgs a{};
  a.xb = e.xb;
  a.xn = e.xn;
  a.qb = e.qb;
  a.qn = e.qn;
  a.thr = e.thr;
  a.qorder = e.qorder;
  a.iv = e.iv;
  a.preds = e.preds;
  a.bitmap = e.bitmap;
  a.stride64 = e.stride64;
  a.nq = e.nq;
  a.ks = exact_ksteps(e.dim);
  a.chunk_rows = e.chunk_rows;
  a.splits = e.splits;
  a.step = e.step;
  a.bin_lanes = e.bin_lanes;
  a.bins = e.bins;
  a.cand = e.cand;
  a.cand_n = e.cand_n;
  a.cand_cap = e.cand_cap;
  const void* fn = nullptr;
  switch (a.ks) {
    case 1: fn = screen_symbol<1>(pass); break;
    case 2: fn = screen_symbol<2>(pass); break;
    case 3: fn = screen_symbol<3>(pass); break;
    case 4: fn = screen_symbol<4>(pass); break;
    case 5: fn = screen_symbol<5>(pass); break;
    case 6: fn = screen_symbol<6>(pass); break;
    case 7: fn = screen_symbol<7>(pass); break;
    case 8: fn = screen_symbol<8>(pass); break;
    default: fn = screen_symbol<0>(pass); break;
  }
  const int n_qtiles = (e.nq + 31) / 32;
  void* args[] = {&a};
  return hipLaunchKernel(fn, dim3(static_cast<unsigned>(n_qtiles * e.splits)), dim3(kExWaves * 64), args, 0, s);
}

hipError_t launch_exact_threshold(const float* bins, int64_t n_bins, int nq, int k, const float* eps, float* thr,
                                  hipStream_t s) {
  const int kpl = pool_kpl(k);
  exact_threshold_kernel<<<nq, 64, static_cast<size_t>(64 * kpl) * sizeof(uint64_t), s>>>(bins, n_bins, k, kpl, eps,
                                                                                         thr);
  return hipGetLastError();
}

int64_t exact_bins_per_query(int splits, int bin_lanes) {
  return static_cast<int64_t>(splits) * kExWaves * (32 / bin_lanes);
}
int64_t exact_chunk_quantum() { return 32 * kExWaves; }

hipError_t launch_exact_rerank(const ExactRerank& e, hipStream_t s) {
  RerankArgs a{};
  a.xt = e.xt;
  a.xr = e.xr;
  a.dim = e.dim;
  a.q = e.q;
  a.qorder = e.qorder;
  a.iv = e.iv;
  a.preds = e.preds;
  a.bitmap = e.bitmap;
  a.stride64 = e.stride64;
  a.perm = e.perm;
  a.cand = e.cand;
  a.cand_n = e.cand_n;
  a.cand_cap = e.cand_cap;
  a.k = e.k;
  a.kpl = pool_kpl(e.k);
  a.chunks = e.chunks;
  a.partials = e.partials;
  const bool listed = e.cand_n != nullptr;
  const int dim_pad = (e.dim + kStageDims - 1) / kStageDims * kStageDims;
  const size_t lds = static_cast<size_t>(64 * a.kpl) * sizeof(uint64_t) +
                     (static_cast<size_t>(dim_pad) + (listed ? 64 * (kStageDims + 1) : 0)) * sizeof(float);
  if (lds > static_cast<size_t>(kLdsBudget)) return hipErrorInvalidValue;
  const void* fn = listed ? reinterpret_cast<const void*>(&exact_rerank_kernel<true>)
                          : reinterpret_cast<const void*>(&exact_rerank_kernel<false>);
  hipError_t err = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  if (err != hipSuccess) return err;
  void* args[] = {&a};
  return hipLaunchKernel(fn, dim3(static_cast<unsigned>(e.chunks), static_cast<unsigned>(e.nq)), dim3(64), args, lds, s);
}

}  // namespace ifvs
