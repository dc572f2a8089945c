// Filter stage (Section 2, stage 1): evaluate each query's conjunctive
// predicate over the attribute columns and emit the candidate pool P as a
// selection bitmap, plus the pool size.
//
// A clause lo <= v < hi only distinguishes values by where they lie among the
// clause bounds of the batch, so the batch's clauses on one column cut its
// values into classes (at most two bounds per clause), and one 128-bit mask
// per class says which of 128 queries' clauses on that column the class
// passes.  A row's selection by all 128 queries is then the AND of one mask
// per column -- work per (row, column) instead of per (row, query, clause).
//  * filter_plan_kernel (one workgroup per 128 queries and column) sorts the
//    bounds, builds the class masks, and, where the bounds span few values, a
//    value -> class table.
//  * filter_class_kernel: lane L of a wavefront turns rows 32L .. 32L + 31 of a
//    2048-row block into classes (one table read, or a binary search of the
//    bounds), reads their masks word by word (32 queries) and transposes the
//    32 x 32 bits in registers, which leaves it with bitmap word L of the
//    block for each of the 32 queries: 32 coalesced stores.  The transposition is 8 VALU operations per 32
//    (row, query) pairs against 4 per single pair for compare-and-collect.
//    10M rows x 256 queries: 155 us with two clauses on two columns (3690 us
//    with the per-pair tests), 4M rows with one clause 57 us (161 us); the
//    stores alone (32 bytes per row) would take 47 us at 10M rows, the LDS
//    mask reads and the VALU work about as long each, overlapped only as far
//    as the 16 wavefronts per CU reach that 128 registers allow.
//  * filter_kernel<true>, the pair tests of one column, for batches of one
//    clause a query with few pairs: a wavefront stages 2048 values in LDS, lane
//    L walks rows 32L + 31 .. 32L and shifts each of 16 queries' compare bits
//    into a word of its own (three VALU operations per 64 pairs).
//  * filter_kernel<false>, the general pair tests, for batches whose clauses
//    name more than kFilterCols columns: per 64 rows and query one ballot, lane
//    i keeping step i's word.  Bound by its chain of loads and ballots: 16
//    queries take 420 us whether they have 10K rows or 200K.
// Pool sizes: each workgroup sums its popcounts in LDS and writes one partial
// count per query (no device-wide atomics); a small kernel adds the partials
// and leaves their exclusive prefix sums for the row-list compaction.
#include "ifvs_internal.h"
#include "topk_device.h"

namespace ifvs {

namespace {

constexpr int kFilterWaves = 4;                          // per-pair tests
constexpr int kRowsPerWave = 64 * 64;
static_assert(kFilterWaves * kRowsPerWave == kFilterPartRows, "one count partial per workgroup");
constexpr int kBlockRows = 2048;                         // rows a wavefront classifies
constexpr int kClassWaves = static_cast<int>(kFilterPartRows / kBlockRows);
constexpr int kPlanThreads = 1024;
constexpr int kGroupWords = kFilterGroup / 32;           // mask words per class

// Four words read together wherever they start (columns start at any row).
typedef uint32_t U32x4 __attribute__((ext_vector_type(4), aligned(4)));

// int32 values in unsigned order.
__device__ __forceinline__ uint32_t biased(int32_t v) { return static_cast<uint32_t>(v) ^ 0x80000000u; }

// Number of the n sorted keys that are <= v.
__device__ __forceinline__ int class_of(const uint32_t* __restrict__ keys, int n, uint32_t v) {
  int lo = 0, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (keys[mid] <= v) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// One workgroup per (column slot, query group): the sorted bounds of the
// group's clauses on the column, the class masks (class i: values from bound
// i - 1 up to bound i), the value table.  The first slot's masks also clear
// the queries that nothing satisfies.
__global__ __launch_bounds__(kPlanThreads) void filter_plan_kernel(const DevPred* __restrict__ preds, int nq,
                                                          int residual_only, FilterCols fc, FilterPlan* plans) {
  __shared__ __align__(16) uint32_t s_raw[kFilterBounds];
  __shared__ uint32_t s_key[kFilterBounds];
  __shared__ int s_rank[kFilterBounds];
  __shared__ int s_bounds;
  const int c = blockIdx.x, g = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  FilterPlan& out = plans[static_cast<size_t>(g) * kFilterCols + c];
  // Even wavefronts hold queries 0..63 of the group, odd ones 64..127; the
  // first two also list the bounds.
  const int half = wave & 1, q = g * kFilterGroup + half * 64 + lane;
  int n_clauses = -1;                             // on this column; -1: nothing passes
  uint32_t lo[kMaxClauses], width[kMaxClauses];   // clauses on other columns pass everything
#pragma unroll
  for (int j = 0; j < kMaxClauses; ++j) lo[j] = width[j] = 0;
  if (tid == 0) s_bounds = 0;
  for (int i = tid; i < kFilterBounds; i += blockDim.x) {
    s_raw[i] = ~0u;
    s_rank[i] = 0;
  }
  if (q < nq) {
    const DevPred& p = preds[q];
    const int nc = residual_only ? p.n_res : p.n_eff;
    int32_t col[kMaxClauses];
#pragma unroll
    for (int j = 0; j < kMaxClauses; ++j) {
      col[j] = residual_only ? p.res_col[j] : p.col[j];
      lo[j] = biased(residual_only ? p.res_lo[j] : p.lo[j]);
      width[j] = residual_only ? p.res_width[j] : p.width[j];
    }
    n_clauses = p.n_eff < 0 ? -1 : 0;
#pragma unroll
    for (int j = 0; j < kMaxClauses; ++j) {
      if (n_clauses >= 0 && j < nc && col[j] == fc.col[c]) ++n_clauses;
      else width[j] = 0;
    }
  }
  __syncthreads();
  if (wave < 2) {
#pragma unroll
    for (int j = 0; j < kMaxClauses; ++j) {
      const uint64_t have = __ballot(width[j] != 0);
      if (have == 0) continue;
      int at = 0;
      if (lane == 0) at = atomicAdd(&s_bounds, 2 * static_cast<int>(__popcll(have)));
      at = __builtin_amdgcn_readfirstlane(at) + 2 * static_cast<int>(__popcll(have & ((1ull << lane) - 1)));
      const uint32_t hi = lo[j] + width[j];       // (0: past the last value)
      if (width[j] != 0) {
        s_raw[at] = lo[j];
        s_raw[at + 1] = hi != 0 ? hi : ~0u;
      }
    }
  }
  __syncthreads();
  const int nb = s_bounds;
  // Sort by rank: the wavefronts share each bound's comparisons.
  const int per = (nb + 63) / 64 * 64;
  for (int e = tid; e < per * 16; e += blockDim.x) {
    const int i = e % per, from = e / per * (kFilterBounds / 16);
    if (from >= nb) continue;
    const uint32_t k = s_raw[i];
    int r = 0;
#pragma unroll 4
    for (int j = from; j < from + kFilterBounds / 16; j += 4) {
      if (j >= nb) break;
      const uint4 o = *reinterpret_cast<const uint4*>(s_raw + j);
      r += (o.x < k || (o.x == k && j < i)) + (o.y < k || (o.y == k && j + 1 < i)) +
           (o.z < k || (o.z == k && j + 2 < i)) + (o.w < k || (o.w == k && j + 3 < i));
    }
    if (i < nb && r > 0) atomicAdd(&s_rank[i], r);
  }
  __syncthreads();
  for (int i = tid; i < nb; i += blockDim.x) {
    s_key[s_rank[i]] = s_raw[i];
    out.bounds[s_rank[i]] = s_raw[i];
  }
  if (tid == 0) out.n_bounds = nb;
  __syncthreads();
  // Class masks: lane = query, one ballot per class and 64 queries.  (A class
  // whose bounds are equal holds no value; its mask is never read.)
  for (int cls = wave >> 1; cls <= nb; cls += kPlanThreads / 128) {
    const uint32_t v = cls == 0 ? 0u : s_key[cls - 1];
    bool pass = c > 0 || n_clauses >= 0;
#pragma unroll
    for (int j = 0; j < kMaxClauses; ++j) pass = pass && (width[j] == 0 || v - lo[j] < width[j]);
    const uint64_t word = __ballot(pass);
    if (lane < 2) out.masks[half * 2 + lane][cls] = static_cast<uint32_t>(word >> (32 * lane));
  }
  for (int e = tid; e < fc.direct[c]; e += blockDim.x)
    out.direct[e] = static_cast<uint16_t>(class_of(s_key, nb, fc.base[c] + static_cast<uint32_t>(e)));
}

// In-register transposition of 32 x 32 bits: bit q of r[i] to bit i of r[q].
__device__ __forceinline__ void transpose32(uint32_t (&r)[32]) {
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const uint32_t a = r[i], b = r[i + 16];
    r[i] = __builtin_amdgcn_perm(b, a, 0x05040100u);
    r[i + 16] = __builtin_amdgcn_perm(b, a, 0x07060302u);
  }
#pragma unroll
  for (int h = 0; h < 32; h += 16)
#pragma unroll
    for (int i = h; i < h + 8; ++i) {
      const uint32_t a = r[i], b = r[i + 8];
      r[i] = __builtin_amdgcn_perm(b, a, 0x06020400u);
      r[i + 8] = __builtin_amdgcn_perm(b, a, 0x07030501u);
    }
#pragma unroll
  for (int s = 4; s > 0; s >>= 1) {
    uint32_t m = s == 4 ? 0x0F0F0F0Fu : s == 2 ? 0x33333333u : 0x55555555u;
    asm("" : "+s"(m));   // (a mask the compiler does not know stays one bit-field insert)
#pragma unroll
    for (int h = 0; h < 32; h += 2 * s)
#pragma unroll
      for (int i = h; i < h + s; ++i) {
        const uint32_t a = r[i], b = r[i + s], up = b << s, down = a >> s;
        r[i] = up ^ (m & (a ^ up));
        r[i + s] = b ^ (m & (down ^ b));
      }
  }
}

// One halving step of add_counts: the lane keeps N of its 2N registers.
template <int N>
__device__ __forceinline__ void fold_counts(uint32_t (&c)[16], int lane, int o) {
  const bool up = (lane & o) != 0;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const uint32_t keep = up ? c[i + N] : c[i], send = up ? c[i] : c[i + N];
    c[i] = keep + static_cast<uint32_t>(__shfl_xor(static_cast<int>(send), o, 64));
  }
}

// Adds each lane's 32 counts (c[i]: count i in the low half, i + 16 in the
// high half, each at most 32) over the wavefront into dst[0..32).
__device__ __forceinline__ void add_counts(uint32_t (&c)[16], uint32_t* dst, int lane) {
  fold_counts<8>(c, lane, 32);
  fold_counts<4>(c, lane, 16);
  fold_counts<2>(c, lane, 8);
  fold_counts<1>(c, lane, 4);
  uint32_t v = c[0];
  v += static_cast<uint32_t>(__shfl_xor(static_cast<int>(v), 2, 64));
  v += static_cast<uint32_t>(__shfl_xor(static_cast<int>(v), 1, 64));
  if ((lane & 3) == 0) {
    // lane bits 5..2 chose among registers 8, 4, 2, 1 apart
    const int i = ((lane >> 5) & 1) * 8 + ((lane >> 4) & 1) * 4 + ((lane >> 3) & 1) * 2 + ((lane >> 2) & 1);
    atomicAdd(&dst[i], v & 0xFFFFu);
    atomicAdd(&dst[i + 16], v >> 16);
  }
}

// grid = (parts of kFilterPartRows rows, query groups x splits): workgroup
// (x, g * splits + w) does words w, w + splits, ... of group g.  Dynamic LDS: per
// column its class masks ([word][class]: neighbouring classes in different
// banks), then its value table or its bounds (sizes from fc).
template <int NC>
__global__ __launch_bounds__(kClassWaves * 64, NC <= 2 ? 4 : 2) void filter_class_kernel(
    const int32_t* __restrict__ attrs, int64_t n, FilterCols fc, const FilterPlan* __restrict__ plans, int nq,
    int splits, uint32_t* __restrict__ out, int64_t stride, uint32_t* __restrict__ count_parts) {
  extern __shared__ __align__(16) uint32_t smem_f[];
  __shared__ uint32_t s_cnt[kFilterGroup];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = __builtin_amdgcn_readfirstlane(static_cast<int>(blockIdx.y) / splits);
  const int w0 = static_cast<int>(blockIdx.y) - g * splits;
  const int q0 = g * kFilterGroup, qn = min(kFilterGroup, nq - q0);
  const FilterPlan* plan = plans + static_cast<size_t>(g) * kFilterCols;
  int mask_at[NC], table_at[NC];       // word offsets in smem_f
  int at = 0;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int nb = plan[c].n_bounds, stride_c = fc.max_bounds[c] + 1;
    mask_at[c] = at;
#pragma unroll
    for (int w = 0; w < kGroupWords; ++w)
      for (int i = tid; i <= nb; i += blockDim.x) smem_f[at + w * stride_c + i] = plan[c].masks[w][i];
    at += stride_c * kGroupWords;
    table_at[c] = at;
    const uint32_t* src = fc.direct[c] > 0 ? reinterpret_cast<const uint32_t*>(plan[c].direct) : plan[c].bounds;
    const int words = fc.direct[c] > 0 ? (fc.direct[c] + 1) / 2 : nb;
    for (int i = tid; i < words; i += blockDim.x) smem_f[at + i] = src[i];
    at += fc.direct[c] > 0 ? (fc.direct[c] + 1) / 2 : fc.max_bounds[c];
  }
  if (tid < kFilterGroup) s_cnt[tid] = 0;
  __syncthreads();
  const int64_t base = (static_cast<int64_t>(blockIdx.x) * kClassWaves + wave) * kBlockRows;
  if (base < n) {
    const int last = static_cast<int>(min(n - base, static_cast<int64_t>(kBlockRows))) - 1;
    uint32_t cls[NC][16];     // classes of rows 2i and 2i + 1 of the lane's 32
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int32_t* __restrict__ col = attrs + static_cast<int64_t>(fc.col[c]) * n + base;
      uint32_t v[32];
      if (last == kBlockRows - 1) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const U32x4 x = *reinterpret_cast<const U32x4*>(col + static_cast<uint32_t>(32 * lane + 4 * i));
          v[4 * i] = x.x;
          v[4 * i + 1] = x.y;
          v[4 * i + 2] = x.z;
          v[4 * i + 3] = x.w;
        }
      } else {
        // rows past n repeat the last row and are masked below
#pragma unroll
        for (int i = 0; i < 32; ++i) v[i] = static_cast<uint32_t>(col[static_cast<uint32_t>(min(32 * lane + i, last))]);
      }
      if (fc.direct[c] > 0) {
        const uint16_t* direct = reinterpret_cast<const uint16_t*>(smem_f + table_at[c]);
        const uint32_t lo = fc.base[c], hi = lo + static_cast<uint32_t>(fc.direct[c] - 1);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const uint32_t x = biased(static_cast<int32_t>(v[2 * i])), y = biased(static_cast<int32_t>(v[2 * i + 1]));
          cls[c][i] = direct[min(max(x, lo), hi) - lo] | (static_cast<uint32_t>(direct[min(max(y, lo), hi) - lo]) << 16);
        }
      } else {
        const uint32_t* keys = smem_f + table_at[c];
        const int nb = plan[c].n_bounds;
        int top = 1;
        while (2 * top <= nb) top *= 2;
#pragma unroll
        for (int h = 0; h < 32; h += 8) {
          int k[8] = {};
          for (int s = top; s > 0; s >>= 1) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              const int t = k[i] + s;
              if (t <= nb && keys[t - 1] <= biased(static_cast<int32_t>(v[h + i]))) k[i] = t;
            }
          }
#pragma unroll
          for (int i = 0; i < 4; ++i)
            cls[c][h / 2 + i] = static_cast<uint32_t>(k[2 * i]) | (static_cast<uint32_t>(k[2 * i + 1]) << 16);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    const int rows_left = last + 1 - 32 * lane;     // of this lane's 32 rows
    const uint32_t valid = rows_left >= 32 ? ~0u : rows_left <= 0 ? 0u : (1u << rows_left) - 1u;
    const uint32_t w32 = static_cast<uint32_t>(base / 32) + lane;
    const bool stores = w32 < stride;
    for (int w = w0; w * 32 < qn; w += splits) {
      uint32_t m[32];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const uint32_t* mask = smem_f + mask_at[c] + w * (fc.max_bounds[c] + 1);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const uint32_t a = mask[cls[c][i] & 0xFFFFu], b = mask[cls[c][i] >> 16];
          m[2 * i] = c == 0 ? a : m[2 * i] & a;
          m[2 * i + 1] = c == 0 ? b : m[2 * i + 1] & b;
        }
        __builtin_amdgcn_sched_barrier(0);   // one column's reads in flight at a time: registers
      }
      transpose32(m);
      if (last < kBlockRows - 1) {
#pragma unroll
        for (int i = 0; i < 32; ++i) m[i] &= valid;
      }
      auto dst = (__attribute__((address_space(1))) uint32_t*)(out + static_cast<int64_t>(q0 + 32 * w) * stride + w32);
      const int qw = stores ? min(32, qn - 32 * w) : 0;
#pragma unroll
      for (int i = 0; i < 32; ++i) {
        // (one pointer stepped along: the compiler would keep the 32 products
        // of the stride in registers and spill them)
        asm volatile("" : "+v"(dst));
        if (i < qw) *dst = m[i];
        dst += stride;
      }
      if (count_parts) {
        uint32_t cnt[16];
#pragma unroll
        for (int i = 0; i < 16; ++i)
          cnt[i] = static_cast<uint32_t>(__popc(m[i])) | (static_cast<uint32_t>(__popc(m[i + 16])) << 16);
        add_counts(cnt, s_cnt + 32 * w, lane);
      }
    }
  }
  if (count_parts) {
    __syncthreads();
    for (int i = tid; i < qn; i += blockDim.x)
      if (i / 32 % splits == w0)
        count_parts[static_cast<int64_t>(q0 + i) * gridDim.x + blockIdx.x] = s_cnt[i];
  }
}

// A predicate's clause list for one pass, as the kernel reads it from LDS.
struct PassClauses {
  int32_t nc;                 // clauses to test; -1: nothing passes
  int32_t col[kMaxClauses];
  uint32_t lo[kMaxClauses];
  uint32_t width[kMaxClauses];
};

constexpr int kBlockPad = kBlockRows + kBlockRows / 32;   // staged block, one pad word per 32 rows

// kOneClause (the launcher checks it): every query has one clause, all on
// column `col`.
template <bool kOneClause>
__global__ __launch_bounds__(kFilterWaves * 64) void filter_kernel(
    const int32_t* __restrict__ attrs, int64_t n, int col, const DevPred* __restrict__ preds, int nq, int residual_only,
    uint32_t* __restrict__ out, int64_t stride, uint32_t* __restrict__ count_parts) {
  __shared__ PassClauses sc[kFilterQueries];
  __shared__ uint32_t s_vals[kOneClause ? kFilterWaves * kBlockPad : 1];
  __shared__ uint32_t s_cnt[kFilterWaves][kFilterQueries];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int q0 = blockIdx.y * kFilterQueries;
  const int qn = min(kFilterQueries, nq - q0);
  // The clause list of each query of the group for this pass: all effective
  // clauses, or only the residual ones.
  if (threadIdx.x < qn) {
    const DevPred& p = preds[q0 + threadIdx.x];
    PassClauses c{};
    if (p.n_eff < 0) {
      c.nc = -1;
    } else {
      c.nc = residual_only ? p.n_res : p.n_eff;
      for (int j = 0; j < c.nc; ++j) {
        c.col[j] = residual_only ? p.res_col[j] : p.col[j];
        c.lo[j] = static_cast<uint32_t>(residual_only ? p.res_lo[j] : p.lo[j]);
        c.width[j] = residual_only ? p.res_width[j] : p.width[j];
      }
    }
    sc[threadIdx.x] = c;
  }
  __syncthreads();
  const int64_t base = (static_cast<int64_t>(blockIdx.x) * kFilterWaves + wave) * kRowsPerWave;
  // A wavefront past the last row does nothing but still joins the count
  // reduction's barrier.
  const bool active = base < n;
  uint32_t cnt[kFilterQueries];   // this lane's selected rows per query
#pragma unroll
  for (int qi = 0; qi < kFilterQueries; ++qi) cnt[qi] = 0;

  if constexpr (kOneClause) {
    if (active) {
      const int32_t* __restrict__ values = attrs + static_cast<int64_t>(col) * n;
      uint32_t lo[kFilterQueries], width[kFilterQueries];
#pragma unroll
      for (int qi = 0; qi < kFilterQueries; ++qi) {
        lo[qi] = qi < qn ? sc[qi].lo[0] : 0;
        width[qi] = qi < qn ? sc[qi].width[0] : 0;   // width 0: nothing passes
      }
      uint32_t* vals = s_vals + wave * kBlockPad;
      for (int blk = 0; blk < kRowsPerWave / kBlockRows; ++blk) {
        const int64_t bb = base + static_cast<int64_t>(blk) * kBlockRows;
        // Local row r at vals[r + r / 32] (rows past n repeat the last row and
        // are masked below).
#pragma unroll 8
        for (int j = 0; j < kBlockRows / 64; ++j) {
          const int r = 64 * j + lane;
          const int64_t i = bb + r;
          vals[r + (r >> 5)] = static_cast<uint32_t>(values[i < n ? i : n - 1]);
        }
        wave_lds_fence();
        // Lane L: rows 32L + 31 down to 32L, so row 32L + r lands in bit r.
        uint32_t word[kFilterQueries];
#pragma unroll
        for (int qi = 0; qi < kFilterQueries; ++qi) word[qi] = 0;
        const uint32_t* mine = vals + 33 * lane;
#pragma unroll 4
        for (int r = 31; r >= 0; --r) {
          const uint32_t v = mine[r];
#pragma unroll
          for (int qi = 0; qi < kFilterQueries; ++qi)
            word[qi] = word[qi] + word[qi] + (v - lo[qi] < width[qi] ? 1u : 0u);
        }
        const int64_t row0 = bb + 32 * lane;
        uint32_t valid = ~0u;
        if (row0 + 32 > n) valid = row0 >= n ? 0u : ((1u << static_cast<int>(n - row0)) - 1u);
        const int64_t w32 = bb / 32 + lane;
#pragma unroll
        for (int qi = 0; qi < kFilterQueries; ++qi) {
          if (qi < qn) {
            const uint32_t wd = word[qi] & valid;
            if (w32 < stride) out[static_cast<int64_t>(q0 + qi) * stride + w32] = wd;
            cnt[qi] += static_cast<uint32_t>(__popc(wd));
          }
        }
        // The next block overwrites vals only after every lane has read it.
        wave_lds_fence();
      }
    }
  } else if (active) {
    // held_{lo,hi}[qi] of lane L: the ballot word of step L for query qi.
    uint32_t held_lo[kFilterQueries], held_hi[kFilterQueries];
#pragma unroll
    for (int qi = 0; qi < kFilterQueries; ++qi) held_lo[qi] = held_hi[qi] = 0;
    for (int it = 0; it < 64; ++it) {
      const int64_t i = base + static_cast<int64_t>(it) * 64 + lane;
      const bool in = i < n;
      const int64_t ii = in ? i : n - 1;
      const bool mine = lane == it;
#pragma unroll
      for (int qi = 0; qi < kFilterQueries; ++qi) {
        if (qi < qn) {
          const int nc = sc[qi].nc;
          bool pass = in && nc >= 0;
          for (int c = 0; c < nc; ++c) {
            const int32_t v = attrs[static_cast<int64_t>(sc[qi].col[c]) * n + ii];
            pass &= static_cast<uint32_t>(v) - sc[qi].lo[c] < sc[qi].width[c];
          }
          const uint64_t word = __ballot(pass);
          held_lo[qi] = mine ? static_cast<uint32_t>(word) : held_lo[qi];
          held_hi[qi] = mine ? static_cast<uint32_t>(word >> 32) : held_hi[qi];
        }
      }
    }
    const int64_t w32 = base / 32 + 2 * lane;           // this lane's two 32-bit words
#pragma unroll
    for (int qi = 0; qi < kFilterQueries; ++qi) {
      if (qi < qn) {
        uint32_t* dst = out + static_cast<int64_t>(q0 + qi) * stride + w32;
        if (w32 < stride) dst[0] = held_lo[qi];
        if (w32 + 1 < stride) dst[1] = held_hi[qi];
        cnt[qi] = static_cast<uint32_t>(__popc(held_lo[qi]) + __popc(held_hi[qi]));
      }
    }
  }

  // Pool sizes: wavefront sums, then one partial per (workgroup, query).
  if (count_parts) {
#pragma unroll
    for (int qi = 0; qi < kFilterQueries; ++qi) {
      unsigned c = cnt[qi];
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off, 64);
      if (lane == 0) s_cnt[wave][qi] = c;
    }
    __syncthreads();
    if (threadIdx.x < qn) {
      uint32_t sum = 0;
#pragma unroll
      for (int w = 0; w < kFilterWaves; ++w) sum += s_cnt[w][threadIdx.x];
      count_parts[static_cast<int64_t>(q0 + threadIdx.x) * gridDim.x + blockIdx.x] = sum;
    }
  }
}

// counts[q] = sum of the q-th row of count_parts ([nq][parts]), and the
// row is turned into its exclusive prefix sums in place (the compaction
// kernel's output offsets; every count is below 2^31).  One wavefront per
// query.
__global__ __launch_bounds__(64) void reduce_counts_kernel(uint32_t* __restrict__ count_parts, int parts,
                                                           int nq, unsigned long long* __restrict__ counts) {
  const int q = blockIdx.x;
  if (q >= nq) return;
  const int lane = threadIdx.x;
  uint32_t* row = count_parts + static_cast<int64_t>(q) * parts;
  uint32_t carry = 0;
  for (int i0 = 0; i0 < parts; i0 += 64) {
    const int i = i0 + lane;
    const uint32_t v = i < parts ? row[i] : 0u;
    uint32_t incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t y = __shfl_up(incl, off, 64);
      if (lane >= off) incl += y;
    }
    if (i < parts) row[i] = carry + incl - v;
    carry += __shfl(incl, 63, 64);
  }
  if (lane == 0) counts[q] = carry;
}

// codes [n][m] bytes -> tiles of 64 rows: word j of physical row (64t + L) is
// stored at codes_t[(t*mw + j)*64 + L] and holds bytes 4j..4j+3 of original
// row perm[64t + L] (zero past m and past n), so a wavefront reading word j of
// a tile reads 256 contiguous bytes.
__global__ void relayout_kernel(const uint8_t* __restrict__ codes, int64_t n, int m, int mw,
                                const int32_t* __restrict__ perm, uint32_t* __restrict__ codes_t,
                                int64_t n_tiles) {
  const int64_t total = n_tiles * mw * 64;
  for (int64_t o = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; o < total;
       o += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int64_t lane = o & 63;
    const int64_t j = (o >> 6) % mw;
    const int64_t t = (o >> 6) / mw;
    const int64_t row = t * 64 + lane;
    uint32_t w = 0;
    if (row < n) {
      const int64_t src = perm ? perm[row] : row;
      for (int b = 0; b < 4; ++b) {
        const int64_t col = j * 4 + b;
        if (col < m) w |= static_cast<uint32_t>(codes[src * m + col]) << (8 * b);
      }
    }
    codes_t[o] = w;
  }
}

}  // namespace

hipError_t launch_relayout_codes(const uint8_t* codes, int64_t n, int m, int mw, const int32_t* perm,
                                 uint32_t* codes_t, int64_t n_tiles, hipStream_t s) {
  const int64_t total = n_tiles * mw * 64;
  const int64_t blocks = std::min<int64_t>((total + 255) / 256, 65536);
  relayout_kernel<<<dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s>>>(codes, n, m, mw, perm,
                                                                          codes_t, n_tiles);
  return hipGetLastError();
}

int64_t filter_count_parts(int64_t n) {
  const int64_t rows_per_block = static_cast<int64_t>(kFilterWaves) * kRowsPerWave;
  return (n + rows_per_block - 1) / rows_per_block;
}

namespace {

size_t filter_class_lds(const FilterCols& fc) {
  size_t words = 0;
  for (int c = 0; c < fc.n; ++c)
    words += static_cast<size_t>(fc.max_bounds[c] + 1) * kGroupWords +
             (fc.direct[c] > 0 ? (fc.direct[c] + 1) / 2 : fc.max_bounds[c]);
  return words * sizeof(uint32_t);
}

template <int NC>
hipError_t launch_filter_class(const int32_t* attrs, int64_t n, const FilterCols& fc, const FilterPlan* plans, int nq,
                               uint32_t* out, int64_t stride, uint32_t* count_parts, unsigned parts, unsigned groups,
                               hipStream_t s) {
  const size_t lds = filter_class_lds(fc);
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&filter_class_kernel<NC>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  if (e != hipSuccess) return e;
  // Few rows: the words of a group in workgroups of their own (a word takes
  // a wavefront about 3 us, mostly latency; classifying the rows again costs
  // less than waiting while the chip has room).
  const unsigned words = static_cast<unsigned>((std::min(nq, kFilterGroup) + 31) / 32);
  const unsigned splits = parts * groups * words <= 512 ? words : 1;
  filter_class_kernel<NC><<<dim3(parts, groups * splits), dim3(kClassWaves * 64), lds, s>>>(
      attrs, n, fc, plans, nq, static_cast<int>(splits), out, stride, count_parts);
  return hipGetLastError();
}

}  // namespace

// The classes serve any batch whose clauses name 1 to kFilterCols columns:
// their plan costs one small launch (6 us for 16 queries, 18 us for 256) whatever
// the row count, and bounds more than kFilterDirect values apart cost them a
// search.  Batches of exactly one clause a query on one column have the pair
// tests of a staged column, without a plan: the faster ones while the pairs are
// few, or no more than 2 us slower.  Whole calls, pair tests and classes: 45K
// rows, 8 queries 40 and 38 us (bounds 9000 apart 40 and 47), 32 queries 41 and 42
// (41 and 53), 128 queries 48 and 57 (48 and 72), 256 queries 49 and 58; 400K rows
// the same, 256 queries 59 and 59; 1M rows, 60 queries 43.7 and 44.6, 256 queries
// 76 and 66; 4M rows, 16 queries 45 and 42; 10M rows, 1 query 62 and 56, 256
// queries 392 and 177.  (Two clauses: classes 43 to 63 us at 10K rows, the
// general pair tests 209 to 374.)
// (One group's clauses have at most kFilterBounds bounds in all, which fit
// the LDS; groups that put that many on different columns may not.)
bool filter_has_classes(const FilterCols& fc) {
  return fc.n >= 1 && fc.n <= kFilterCols && filter_class_lds(fc) + kFilterGroup * sizeof(uint32_t) <= kLdsBudget;
}

constexpr int64_t kPairTests = 60'000'000;   // most (row, query) pairs and
constexpr int64_t kPairRows = 4'000'000;     // rows for the pair tests of one column

hipError_t launch_filter(const int32_t* attrs, int64_t n, const DevPred* preds, int nq, bool residual_only,
                         const FilterCols& fc, FilterPlan* plans, uint32_t* out, int64_t stride,
                         unsigned long long* counts, uint32_t* count_parts, hipStream_t s) {
  const unsigned parts = static_cast<unsigned>(filter_count_parts(n));
  uint32_t* cp = counts ? count_parts : nullptr;
  hipError_t e = hipSuccess;
  const bool few = fc.n == 1 && fc.one_clause && n <= kPairRows && n * nq <= kPairTests;
  if (!few && filter_has_classes(fc)) {
    const unsigned groups = static_cast<unsigned>((nq + kFilterGroup - 1) / kFilterGroup);
    filter_plan_kernel<<<dim3(static_cast<unsigned>(fc.n), groups), dim3(kPlanThreads), 0, s>>>(
        preds, nq, residual_only ? 1 : 0, fc, plans);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    switch (fc.n) {
      case 1: e = launch_filter_class<1>(attrs, n, fc, plans, nq, out, stride, cp, parts, groups, s); break;
      case 2: e = launch_filter_class<2>(attrs, n, fc, plans, nq, out, stride, cp, parts, groups, s); break;
      case 3: e = launch_filter_class<3>(attrs, n, fc, plans, nq, out, stride, cp, parts, groups, s); break;
      default: e = launch_filter_class<4>(attrs, n, fc, plans, nq, out, stride, cp, parts, groups, s); break;
    }
  } else {
    const unsigned gy = static_cast<unsigned>((nq + kFilterQueries - 1) / kFilterQueries);
    auto* fn = few ? &filter_kernel<true> : &filter_kernel<false>;
    fn<<<dim3(parts, gy), dim3(kFilterWaves * 64), 0, s>>>(attrs, n, fc.col[0], preds, nq, residual_only ? 1 : 0, out,
                                                           stride, cp);
    e = hipGetLastError();
  }
  if (e != hipSuccess || !counts) return e;
  reduce_counts_kernel<<<dim3(nq), dim3(64), 0, s>>>(count_parts, static_cast<int>(parts), nq, counts);
  return hipGetLastError();
}

}  // namespace ifvs
