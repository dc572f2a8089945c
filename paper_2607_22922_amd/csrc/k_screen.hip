// Rank stage (Section 2, stage 2) of a batch whose queries select largely the
// same rows: four queries are screened per table read, and only the rows that
// may enter a query's top k are scored.
//
// The tiled scan reads one 4-byte table entry per (row, query, subspace) and
// is bound by the LDS's random reads.  Here an LDS word holds one 6-bit entry
// of each of four queries, so a read serves four (row, query) pairs:
//  1. screen_seed_kernel   per query, an upper bound T of its k-th distance:
//     the exact distances of an evenly spaced sample of its rows, the k-th
//     smallest of the lanes' minima (distinct rows).
//  2. screen_pack_kernel   entry -> floor((entry - smallest of its subspace)
//     / step), at most 63, step = (T - sum of the smallest) / L: the sum of a
//     row's packed entries exceeding L proves that its distance exceeds T.
//     The four bytes of a word are the four queries of a group.
//  3. screen_kernel        per 64-row tile, four words (subspaces) are added
//     bytewise (4 x 63 < 256), then unpacked into 16-bit sums that start at
//     0x7FFF - L: bit 15 set means pruned.  A tile is left as soon as no lane
//     has a query alive.  Surviving rows go to their query's list.
//     Large batches run 2-4 over every 16th block of tiles first, for a T
//     close to the answer: the sums then pass it a subspace group earlier and
//     fewer rows survive.
//  4. screen_rerank_kernel the listed rows' distances exactly as the scan
//     sums them (fp32, m order), and the query's k best.
// Measured, 256 queries: 100M x 16-byte codes, 10% selected: 1310 us for the
// whole pass (LDS 80% busy, 10 reads a tile of 16), 300 us for the sample and
// the small kernels, against the scan's 5110; 4M x 48-byte codes, half of the
// rows masked: 1200 us (LDS 94% busy: 24 of 48 reads a tile at 6.3 CU-cycles
// each, 32 random reads on 32 banks) and 340, against 8570.
// Exactness: every entry is >= 0 (checked; other queries keep the scan), the
// quantization rounds down, T carries the fp32 rounding of M additions, and a
// row whose distance equals T survives.  A query whose list overflows, or
// whose sample holds fewer than k rows, keeps the scan too (mode 0).
#include <algorithm>

#include "ifvs_internal.h"
#include "topk_device.h"

namespace ifvs {

namespace {

constexpr int kXcds = 8;
constexpr int kSeedThreads = 1024;          // seed and rerank workgroups (16 wavefronts)
constexpr int kSeedWaves = kSeedThreads / 64;
constexpr int kQueue = 128;                 // survivors a wavefront holds before it appends them
constexpr int kTailWords = 8;               // code words loaded together past the prefetched ones
constexpr uint32_t kFields = 0x80008000u;

__device__ __forceinline__ float widen_s(float v) { return v; }
__device__ __forceinline__ float widen_s(__half v) { return __half2float(v); }

__device__ __forceinline__ uint64_t tile_interval(int64_t t, int64_t r0, int64_t r1) {
  const int64_t row0 = t * 64;
  const int64_t lo = max(r0 - row0, static_cast<int64_t>(0)), hi = min(r1 - row0, static_cast<int64_t>(64));
  if (hi <= lo) return 0;
  return (hi >= 64 ? ~0ull : ((1ull << hi) - 1)) & ~((1ull << lo) - 1);
}

// One query's table into LDS as fp32 [m][256]; true when an entry is negative
// or NaN (workgroup-wide after the caller's barrier through s_bad).
template <typename LutT>
__device__ __forceinline__ bool stage_table(const LutT* __restrict__ src, int m, float* s_tab) {
  constexpr int kVec = 16 / sizeof(LutT);
  bool bad = false;
  const uint4* v4 = reinterpret_cast<const uint4*>(src);
  for (int v = threadIdx.x; v < m * kKsub / kVec; v += kSeedThreads) {
    const uint4 x = v4[v];
    const LutT* xe = reinterpret_cast<const LutT*>(&x);
#pragma unroll
    for (int u = 0; u < kVec; ++u) {
      const float f = widen_s(xe[u]);
      bad = bad || !(f >= 0.0f);
      s_tab[v * kVec + u] = f;
    }
  }
  return bad;
}

// k-th smallest (1-based) of the workgroup's kSeedThreads words, by bisection
// on the value; every lane of the calling wavefront gets it.
__device__ __forceinline__ uint32_t kth_of_minima(const uint32_t* s_min, int k) {
  const int lane = threadIdx.x & 63;
  uint32_t v[kSeedWaves];
#pragma unroll
  for (int i = 0; i < kSeedWaves; ++i) v[i] = s_min[i * 64 + lane];
  uint32_t lo = 0x80000000u, hi = 0xFFFFFFFFu;   // the distances are >= 0
  while (lo < hi) {
    const uint32_t mid = lo + (hi - lo) / 2;
    int c = 0;
#pragma unroll
    for (int i = 0; i < kSeedWaves; ++i) c += __popcll(__ballot(v[i] <= mid));
    if (c >= k) hi = mid;
    else lo = mid + 1;
  }
  return lo;
}

// T (> 0 words of ordered bits) becomes the query's bound: the packed tables'
// scale, the sums' start, the scan's shared threshold.
__device__ __forceinline__ void set_bound(const ScreenBatch& a, int p, int q, uint32_t bits, double low) {
  const float T = from_ordered_bits(bits);
  // What is left of T above the smallest entries, with the rounding of the
  // fp32 sums (M additions, each within 2^-24) and a floor against underflow.
  const double rest = fmax(static_cast<double>(T) * (1.0 + (a.m + 8) * 0x1p-23) - low, 1e-30);
  if (!(rest < 3e38)) return;
  a.thr[p] = T;
  a.scale[p] = static_cast<float>(static_cast<double>(a.levels) / rest * (1.0 - 0x1p-20));
  a.level[p] = a.levels;
  // The bound also serves the scan, should the query fall back to it (rows at
  // this distance stay eligible: no id is as large).
  a.gthr[q] = (static_cast<uint64_t>(bits) << 32) | 0xFFFFFFFFull;
}

// One workgroup per query position.  Bound by the latency of its tile loop
// (sixteen wavefronts, tiles loaded one ahead); lanes drop out above the
// bound of the tiles before (recomputed after 1, 4 and 16 tiles a wavefront).
template <int P, typename LutT>
__global__ __launch_bounds__(kSeedThreads) void screen_seed_kernel(const ScreenBatch a) {
  extern __shared__ __align__(16) unsigned char smem[];
  float* s_tab = reinterpret_cast<float*>(smem);
  __shared__ uint32_t s_min[kSeedThreads];
  __shared__ uint32_t s_cut;
  __shared__ float s_low[256];
  __shared__ int s_bad;
  const int p = blockIdx.x;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int q = a.qorder[p];
  if (threadIdx.x == 0) {
    a.list_n[p] = 0;
    a.level[p] = -1;
    a.mode[q] = 0;
    s_bad = 0;
    s_cut = 0xFFFFFFFFu;
  }
  if (a.counts && a.counts[q] <= static_cast<unsigned long long>(a.list_rows)) return;   // left to the row lists
  const int64_t r0 = a.iv[2 * q], r1 = a.iv[2 * q + 1];
  if (r1 <= r0) return;                        // nothing selected: the scan writes the empty lists
  const bool resid = a.preds[q].residual_mask != 0;
  const uint64_t* bits = a.bitmap + static_cast<size_t>(q) * a.stride64;
  __syncthreads();
  if (stage_table(static_cast<const LutT*>(a.lut) + static_cast<size_t>(q) * a.m * kKsub, a.m, s_tab)) s_bad = 1;
  __syncthreads();
  if (s_bad) return;
  // Smallest entry of each subspace.
  for (int m = wave; m < a.m; m += kSeedWaves) {
    const float4 x = reinterpret_cast<const float4*>(s_tab + m * kKsub)[lane];
    float v = fminf(fminf(x.x, x.y), fminf(x.z, x.w));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fminf(v, __shfl_xor(v, o, 64));
    if (lane == 0) {
      s_low[m] = v;
      a.low[static_cast<size_t>(p) * a.mw * 4 + m] = v;
    }
  }
  // Sample: slots of evenly spaced tiles of the interval.
  const int64_t ft = r0 >> 6, span = ((r1 + 63) >> 6) - ft;
  const int slots = static_cast<int>(min(span, static_cast<int64_t>(a.seed_tiles)));
  auto slot_tile = [&](int i) -> int64_t { return ft + static_cast<int64_t>(i) * span / slots; };
  uint32_t nw[P];
  auto load = [&](int i) {
    const uint32_t* tile = a.codes_t + static_cast<size_t>(slot_tile(i < slots ? i : 0)) * a.mw * 64;
#pragma unroll
    for (int j = 0; j < P; ++j) nw[j] = tile[j * 64 + lane];
  };
  float best = __builtin_inff();
  float cut = __builtin_inff();
  load(wave);
  int next_check = 1;
  const int per_wave = (slots + kSeedWaves - 1) / kSeedWaves;
  for (int it = 0; it < per_wave; ++it) {
    if (it == next_check) {
      s_min[threadIdx.x] = ordered_bits(best);
      __syncthreads();
      if (wave == 0) {
        const uint32_t c = kth_of_minima(s_min, a.k);
        if (lane == 0) s_cut = c;
      }
      __syncthreads();
      cut = s_cut < 0xFF800000u ? from_ordered_bits(s_cut) : __builtin_inff();
      next_check *= 4;
    }
    const int i = it * kSeedWaves + wave;
    uint32_t w[P];
#pragma unroll
    for (int j = 0; j < P; ++j) w[j] = nw[j];
    load(i + kSeedWaves);
    if (i >= slots) continue;
    const int64_t t = slot_tile(i);
    uint64_t mk = tile_interval(t, r0, r1);
    if (resid && mk != 0) mk &= bits[t];
    if (mk == 0) continue;
    bool live = __builtin_amdgcn_inverse_ballot_w64(mk);
    float d = 0.0f;
    auto add_word = [&](int j, uint32_t word) {
      if (live) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (4 * j + u < a.m) d = __fadd_rn(d, s_tab[(4 * j + u) * kKsub + ((word >> (8 * u)) & 0xFFu)]);
        live = !(d > cut);
      }
    };
#pragma unroll
    for (int j = 0; j < P; ++j) add_word(j, w[j]);
    const uint32_t* tile = a.codes_t + static_cast<size_t>(t) * a.mw * 64;
    for (int j0 = P; j0 < a.mw && __ballot(live) != 0; j0 += kTailWords) {
      uint32_t tw[kTailWords];
#pragma unroll
      for (int u = 0; u < kTailWords; ++u) tw[u] = tile[min(j0 + u, a.mw - 1) * 64 + lane];
#pragma unroll
      for (int u = 0; u < kTailWords; ++u)
        if (j0 + u < a.mw) add_word(j0 + u, tw[u]);
    }
    if (live) best = fminf(best, d);
  }
  s_min[threadIdx.x] = ordered_bits(best);
  __syncthreads();
  if (wave != 0) return;
  const uint32_t kth = kth_of_minima(s_min, a.k);
  if (lane != 0 || kth >= 0xFF800000u) return;   // fewer than k sampled rows, or an infinite distance
  double low = 0.0;
  for (int m = 0; m < a.m; ++m) low += static_cast<double>(s_low[m]);
  set_bound(a, p, q, kth, low);
}

// grid = (groups, 4-subspace words), thread = codeword: the group's packed
// tables [group][word * 4 + u][256], byte i = query i's entry (63 where a
// query of the group is not screened; zero past M).
template <typename LutT>
__global__ __launch_bounds__(kKsub) void screen_pack_kernel(const ScreenBatch a) {
  const int g = blockIdx.x, j = blockIdx.y, c = threadIdx.x;
  uint32_t w[4] = {};
#pragma unroll
  for (int i = 0; i < kScreenGroup; ++i) {
    const int p = g * kScreenGroup + i;
    const bool on = p < a.nq && a.level[p] >= 0;
    const LutT* tab = static_cast<const LutT*>(a.lut) + static_cast<size_t>(on ? a.qorder[p] : 0) * a.m * kKsub;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int m = 4 * j + u;
      if (m >= a.m) break;
      uint32_t b = 63;
      if (on) {
        const float e = __fsub_rn(widen_s(tab[m * kKsub + c]), a.low[static_cast<size_t>(p) * a.mw * 4 + m]);
        b = static_cast<uint32_t>(fminf(__fmul_rn(e, a.scale[p]), 63.0f));
      }
      w[u] |= b << (8 * i);
    }
  }
#pragma unroll
  for (int u = 0; u < 4; ++u)
    a.tab[(static_cast<size_t>(g) * a.mw * 4 + 4 * j + u) * kKsub + c] = w[u];
}

// Workgroup = eight wavefronts on one chunk of a group's hull (the smallest
// row range that holds the four intervals); XCD x takes a contiguous run of
// groups and walks it chunk by chunk, so groups with nearby intervals read
// the same code tiles from its L2 at about the same time.  A wavefront takes
// blocks of up to 64 tiles: lane l works out the four selection words of tile
// l at once (intervals, and bitmap words loaded side by side), and the tiles
// with a row selected are then visited with the next one's first P code words
// in flight; the words after them are read only for tiles still alive.
template <int P, int kThreads>
__global__ __launch_bounds__(kThreads) void screen_kernel(const ScreenBatch a) {
  constexpr int kWaves = kThreads / 64;
  extern __shared__ __align__(16) uint32_t s_dyn[];
  uint32_t* s_tab = s_dyn;                                  // [mw * 4][256]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t* queue = s_dyn + a.mw * 4 * kKsub + wave * kQueue;
  const int groups = (a.nq + kScreenGroup - 1) / kScreenGroup;
  const int per_xcd = (groups + kXcds - 1) / kXcds;
  const int slot = blockIdx.x / kXcds;
  const int chunk = slot / per_xcd;
  const int g = static_cast<int>(blockIdx.x % kXcds) * per_xcd + slot % per_xcd;
  if (g >= groups) return;
  int64_t r0[kScreenGroup], r1[kScreenGroup];
  const uint64_t* bits[kScreenGroup];
  uint32_t start[kScreenGroup];
  int64_t lo = INT64_MAX, hi = 0;
#pragma unroll
  for (int i = 0; i < kScreenGroup; ++i) {
    const int p = g * kScreenGroup + i;
    r0[i] = r1[i] = 0;
    bits[i] = nullptr;
    start[i] = 0x8000u;
    if (p < a.nq && a.level[p] >= 0) {
      const int q = a.qorder[p];
      r0[i] = a.iv[2 * q];
      r1[i] = a.iv[2 * q + 1];
      start[i] = 0x7FFFu - static_cast<uint32_t>(a.level[p]);
      if (a.preds[q].residual_mask != 0) bits[i] = a.bitmap + static_cast<size_t>(q) * a.stride64;
      lo = min(lo, r0[i]);
      hi = max(hi, r1[i]);
    }
  }
  if (hi <= lo) return;
  const int t_lo = static_cast<int>(lo >> 6), t_hi = static_cast<int>((hi + 63) >> 6);
  const int cell_tiles = a.chunk_tiles * a.step;
  const int c_first = t_lo / cell_tiles, c_end = (t_hi + cell_tiles - 1) / cell_tiles;
  if (c_first + chunk >= c_end) return;
  {
    const uint4* src = reinterpret_cast<const uint4*>(a.tab + static_cast<size_t>(g) * a.mw * 4 * kKsub);
    for (int v = threadIdx.x; v < a.mw * kKsub; v += kThreads) reinterpret_cast<uint4*>(s_tab)[v] = src[v];
  }
  __syncthreads();
  const uint32_t s02 = start[0] | (start[2] << 16), s13 = start[1] | (start[3] << 16);
  const int bt = min(64, a.chunk_tiles / kWaves);           // tiles per block

  for (int cell = c_first + chunk; cell < c_end; cell += a.splits) {
    const int cell_t0 = cell * cell_tiles;
    const int tb = max(t_lo, cell_t0), te = min(t_hi, cell_t0 + cell_tiles);
    int qc = 0;
    // Queries whose list is full when this wavefront appends to it (bit i) are
    // not screened any further: the scan takes them.  Without this a query of
    // equal rows queues every one of them (16 such among 256 over 4M masked
    // rows of 48-byte codes: 24.7 ms -> 8.8; asking at the start of a cell
    // too costs the others 7-35%).
    uint32_t over = 0;
    auto flush = [&]() {
      wave_lds_fence();
      for (int e0 = 0; e0 < qc; e0 += 64) {
        const bool ok = e0 + lane < qc;
        const uint32_t v = ok ? queue[e0 + lane] : 0u;
#pragma unroll
        for (int i = 0; i < kScreenGroup; ++i) {
          const uint64_t mk = __ballot(ok && (v >> 30) == static_cast<uint32_t>(i));
          if (mk == 0) continue;
          const int p = g * kScreenGroup + i;
          int base = 0;
          if (lane == 0) base = atomicAdd(&a.list_n[p], static_cast<int>(__popcll(mk)));
          base = __builtin_amdgcn_readfirstlane(base);
          if (base + static_cast<int>(__popcll(mk)) > a.list_cap) over |= 1u << i;
          const int pos = base + lanes_below(mk);
          if (ok && (v >> 30) == static_cast<uint32_t>(i) && pos < a.list_cap)
            a.lists[static_cast<size_t>(p) * a.list_cap + pos] =
                static_cast<int32_t>(cell_t0 * 64 + static_cast<int>(v & 0x3FFFFFFFu));
        }
      }
      wave_lds_fence();
      qc = 0;
    };

    int blk = tb + wave * bt * a.step;                       // this wavefront's next block
    int blk0 = 0;
    uint64_t todo = 0;
    uint64_t lm[kScreenGroup];                               // lane's tile: selection words
#pragma unroll
    for (int i = 0; i < kScreenGroup; ++i) lm[i] = 0;
    // The next tile with a row selected (-1: none left), its words to bm.
    auto advance = [&](uint64_t (&bm)[kScreenGroup]) -> int {
      while (todo == 0) {
        if (blk >= te) return -1;
        blk0 = blk;
        blk += kWaves * bt * a.step;
        const int t = blk0 + lane;
        const bool in = lane < bt && t < te;
        uint64_t any = 0;
#pragma unroll
        for (int i = 0; i < kScreenGroup; ++i) {
          lm[i] = in && !((over >> i) & 1) ? tile_interval(t, r0[i], r1[i]) : 0ull;
          if (bits[i] && lm[i] != 0) lm[i] &= bits[i][t];
          any |= lm[i];
        }
        todo = __ballot(any != 0);
      }
      const int b = __builtin_ctzll(todo);
      todo &= todo - 1;
#pragma unroll
      for (int i = 0; i < kScreenGroup; ++i) {
        const uint32_t l = __builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(lm[i])), b);
        const uint32_t h = __builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(lm[i] >> 32)), b);
        bm[i] = (static_cast<uint64_t>(h) << 32) | l;
      }
      return blk0 + b;
    };
    uint64_t bn[kScreenGroup];
    uint32_t wn[P];
    auto load = [&](int t) {
      const uint32_t* tile = a.codes_t + static_cast<size_t>(t < 0 ? tb : t) * a.mw * 64;
#pragma unroll
      for (int j = 0; j < P; ++j) wn[j] = tile[j * 64 + lane];
    };
    int t_next = advance(bn);
    load(t_next);
    while (t_next >= 0) {
      const int t = t_next;
      uint32_t w[P];
#pragma unroll
      for (int j = 0; j < P; ++j) w[j] = wn[j];
      uint32_t s0 = __builtin_amdgcn_inverse_ballot_w64(bn[0]) ? s02 & 0xFFFFu : 0x8000u;
      uint32_t s1 = __builtin_amdgcn_inverse_ballot_w64(bn[1]) ? s13 & 0xFFFFu : 0x8000u;
      const uint32_t s2 = __builtin_amdgcn_inverse_ballot_w64(bn[2]) ? s02 & 0xFFFF0000u : 0x80000000u;
      const uint32_t s3 = __builtin_amdgcn_inverse_ballot_w64(bn[3]) ? s13 & 0xFFFF0000u : 0x80000000u;
      s0 |= s2;                                              // queries 0 and 2
      s1 |= s3;                                              // queries 1 and 3
      t_next = advance(bn);
      load(t_next);
      auto add_word = [&](const uint32_t* tab, uint32_t word) {
        uint32_t x = tab[word & 0xFFu] + tab[kKsub + ((word >> 8) & 0xFFu)];
        x += tab[2 * kKsub + ((word >> 16) & 0xFFu)];
        x += tab[3 * kKsub + (word >> 24)];
        s0 += x & 0x00FF00FFu;
        s1 += (x >> 8) & 0x00FF00FFu;
      };
      auto alive = [&]() { return __ballot((s0 & s1 & kFields) != kFields) != 0; };
      bool on = true;
#pragma unroll
      for (int j = 0; j < P; ++j) {
        if (on) {
          add_word(s_tab + j * 4 * kKsub, w[j]);
          if (j > 0 || P == 1) on = alive();
        }
      }
      if (on && P < a.mw) {
        const uint32_t* tile = a.codes_t + static_cast<size_t>(t) * a.mw * 64;
        for (int j0 = P; j0 < a.mw && on; j0 += kTailWords) {
          uint32_t tw[kTailWords];
#pragma unroll
          for (int u = 0; u < kTailWords; ++u) tw[u] = tile[min(j0 + u, a.mw - 1) * 64 + lane];
#pragma unroll
          for (int u = 0; u < kTailWords; ++u)
            if (on && j0 + u < a.mw) {
              add_word(s_tab + (j0 + u) * 4 * kKsub, tw[u]);
              if (u & 1) on = alive();
            }
        }
      }
      if (!on) continue;
      const uint32_t left[kScreenGroup] = {s0 & 0x8000u, s1 & 0x8000u, s0 & 0x80000000u, s1 & 0x80000000u};
#pragma unroll
      for (int i = 0; i < kScreenGroup; ++i) {
        const uint64_t al = __ballot(left[i] == 0);
        if (al == 0 || ((over >> i) & 1)) continue;
        const int cnt = __popcll(al);
        if (qc + cnt > kQueue) flush();
        if (left[i] == 0)
          queue[qc + lanes_below(al)] =
              (static_cast<uint32_t>(i) << 30) | static_cast<uint32_t>((t - cell_t0) * 64 + lane);
        qc += cnt;
      }
    }
    flush();
  }
}

// One workgroup per query position: its listed rows' exact distances, the k
// best of each wavefront, then those below the smallest k-th key sorted.
// kFinal: they are the answer.  Else (the sample's survivors) the k-th of them
// is the query's new bound, and its list starts again.
template <typename LutT, bool kFinal>
__global__ __launch_bounds__(kSeedThreads) void screen_rerank_kernel(const ScreenBatch a) {
  extern __shared__ __align__(16) unsigned char smem[];
  float* s_tab = reinterpret_cast<float*>(smem);
  uint64_t* s_sort = reinterpret_cast<uint64_t*>(smem);      // over the table, once the rows are scored
  uint64_t* pools = reinterpret_cast<uint64_t*>(smem + a.rerank_table_bytes);
  __shared__ unsigned long long s_thr;
  __shared__ int s_n;
  const int p = blockIdx.x;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (a.level[p] < 0) return;
  const int n = kFinal ? a.list_n[p] : min(a.list_n[p], a.list_cap);
  if (n > a.list_cap) return;                                // the scan takes the query (mode 0)
  const int q = a.qorder[p];
  if (threadIdx.x == 0) {
    if (kFinal) a.mode[q] = 2;
    s_thr = kNoKey;
    s_n = 0;
  }
  stage_table(static_cast<const LutT*>(a.lut) + static_cast<size_t>(q) * a.m * kKsub, a.m, s_tab);
  __syncthreads();
  uint64_t* pool = pools + static_cast<size_t>(wave) * a.pool_stride;
  int cnt = 0;
  uint64_t thr = kNoKey;
  const float T = a.thr[p];
  const int32_t* list = a.lists + static_cast<size_t>(p) * a.list_cap;
  for (int b = wave * 64; b < n; b += kSeedThreads) {
    const bool ok = b + lane < n;
    const int32_t row = ok ? list[b + lane] : list[b];
    const uint32_t* src = a.codes_t + static_cast<size_t>(row >> 6) * a.mw * 64 + (row & 63);
    const uint32_t* rm = a.codes_rm ? a.codes_rm + static_cast<size_t>(row) * a.rw : nullptr;
    float d = 0.0f;
    for (int j0 = 0; j0 < a.mw; j0 += kTailWords) {
      uint32_t w[kTailWords];
      if (rm) {
        // (16-byte rows: rw is a multiple of 4)
#pragma unroll
        for (int u = 0; u < kTailWords; u += 4) {
          const uint4 x = *reinterpret_cast<const uint4*>(rm + min(j0 + u, a.rw - 4));
          w[u] = x.x;
          w[u + 1] = x.y;
          w[u + 2] = x.z;
          w[u + 3] = x.w;
        }
      } else {
#pragma unroll
        for (int u = 0; u < kTailWords; ++u) w[u] = src[min(j0 + u, a.mw - 1) * 64];
      }
#pragma unroll
      for (int u = 0; u < kTailWords; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int m = 4 * (j0 + u) + v;
          if (m < a.m) d = __fadd_rn(d, s_tab[m * kKsub + ((w[u] >> (8 * v)) & 0xFFu)]);
        }
    }
    uint64_t key = kNoKey;
    const bool in = ok && d <= T;
    if (in) key = (static_cast<uint64_t>(ordered_bits(d)) << 32) | static_cast<uint32_t>(a.perm ? a.perm[row] : row);
    pool_push(pool, cnt, thr, key, in && key < thr, a.k, a.kpl);
  }
  pool_compact(pool, cnt, thr, a.k, a.kpl);
  if (lane == 0 && thr != kNoKey) atomicMin(&s_thr, static_cast<unsigned long long>(thr));
  __syncthreads();
  const uint64_t top = s_thr;
  for (int e = lane; e < cnt; e += 64) {
    const uint64_t key = pool[e];
    if (key <= top) s_sort[atomicAdd(&s_n, 1)] = key;
  }
  __syncthreads();
  const int have = s_n;
  int np = 2;
  while (np < have || np < a.k) np *= 2;
  for (int e = have + threadIdx.x; e < np; e += kSeedThreads) s_sort[e] = kNoKey;
  __syncthreads();
  for (int size = 2; size <= np; size <<= 1)
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      const int e = threadIdx.x;                             // np <= 2 * kSeedThreads: one pair a thread
      if (e < np / 2) {
        const int i = ((e & ~(stride - 1)) << 1) | (e & (stride - 1));
        const int j = i | stride;
        const uint64_t x = s_sort[i], y = s_sort[j];
        if (((i & size) == 0) == (x > y)) {
          s_sort[i] = y;
          s_sort[j] = x;
        }
      }
      __syncthreads();
    }
  if (!kFinal) {
    if (threadIdx.x == 0) {
      a.list_n[p] = 0;
      const uint64_t key = s_sort[a.k - 1];
      if (key != kNoKey) {
        double low = 0.0;
        for (int m = 0; m < a.m; ++m) low += static_cast<double>(a.low[static_cast<size_t>(p) * a.mw * 4 + m]);
        set_bound(a, p, q, static_cast<uint32_t>(key >> 32), low);
      }
    }
    return;
  }
  for (int e = threadIdx.x; e < a.k; e += kSeedThreads) {
    const uint64_t key = s_sort[e];
    const size_t o = static_cast<size_t>(q) * a.k + e;
    a.ids_out[o] = key == kNoKey ? -1 : static_cast<int32_t>(static_cast<uint32_t>(key));
    a.dist_out[o] = key == kNoKey ? __builtin_inff() : from_ordered_bits(static_cast<uint32_t>(key >> 32));
  }
}

size_t rerank_table_bytes(int m) {
  // the table, later kSeedWaves lists of up to kScreenMaxK keys
  return std::max(static_cast<size_t>(m) * kKsub * sizeof(float),
                  static_cast<size_t>(kSeedWaves) * kScreenMaxK * sizeof(uint64_t));
}
size_t seed_lds(int m) { return static_cast<size_t>(m) * kKsub * sizeof(float); }
size_t rerank_lds(int m, int k) {
  return rerank_table_bytes(m) + static_cast<size_t>(kSeedWaves) * pool_stride_for(k) * sizeof(uint64_t);
}
// Wavefronts per screening workgroup: eight while three workgroups' tables
// fit a CU, sixteen where one or two do.
int screen_waves(int mw) { return mw > 12 ? 16 : 8; }
size_t screen_lds(int mw) {
  return static_cast<size_t>(mw) * 4 * kKsub * 4 + static_cast<size_t>(screen_waves(mw)) * kQueue * 4;
}

template <typename LutT>
const void* pick_seed(int p) {
  switch (p) {
    case 1: return reinterpret_cast<const void*>(&screen_seed_kernel<1, LutT>);
    case 2: return reinterpret_cast<const void*>(&screen_seed_kernel<2, LutT>);
    case 3: return reinterpret_cast<const void*>(&screen_seed_kernel<3, LutT>);
    case 4: return reinterpret_cast<const void*>(&screen_seed_kernel<4, LutT>);
    case 5: return reinterpret_cast<const void*>(&screen_seed_kernel<5, LutT>);
    default: return reinterpret_cast<const void*>(&screen_seed_kernel<6, LutT>);
  }
}

const void* pick_screen(int mw) {
  switch (mw) {
    case 1: return reinterpret_cast<const void*>(&screen_kernel<1, 512>);
    case 2: return reinterpret_cast<const void*>(&screen_kernel<2, 512>);
    case 3: return reinterpret_cast<const void*>(&screen_kernel<3, 512>);
    case 4: return reinterpret_cast<const void*>(&screen_kernel<4, 512>);
    case 5: return reinterpret_cast<const void*>(&screen_kernel<5, 512>);
    default: break;
  }
  return screen_waves(mw) == 8 ? reinterpret_cast<const void*>(&screen_kernel<6, 512>)
                               : reinterpret_cast<const void*>(&screen_kernel<6, 1024>);
}

hipError_t launch_with_lds(const void* fn, dim3 grid, int threads, size_t lds, ScreenBatch& a, hipStream_t s) {
  const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  if (e != hipSuccess) return e;
  void* args[] = {&a};
  return hipLaunchKernel(fn, grid, dim3(static_cast<unsigned>(threads)), args, lds, s);
}

}  // namespace

// (the seed kernel's static arrays take 6 KB beside its table)
bool screen_supported(int m, int k) {
  const size_t budget = static_cast<size_t>(kLdsBudget);
  return k <= kScreenMaxK && m <= 256 && seed_lds(m) + 6144 <= budget && rerank_lds(m, k) + 64 <= budget &&
         screen_lds((m + 3) / 4) <= budget;
}

hipError_t launch_screen(ScreenBatch a, int lut_dtype, hipStream_t s) {
  const bool f16 = lut_dtype == 1;
  const int pre = std::min(a.mw, 6);
  const int groups = (a.nq + kScreenGroup - 1) / kScreenGroup;
  a.kpl = pool_kpl(a.k);
  a.pool_stride = pool_stride_for(a.k);
  a.rerank_table_bytes = rerank_table_bytes(a.m);
  hipError_t e = launch_with_lds(f16 ? pick_seed<__half>(pre) : pick_seed<float>(pre),
                                 dim3(static_cast<unsigned>(a.nq)), kSeedThreads, seed_lds(a.m), a, s);
  if (e != hipSuccess) return e;
  const dim3 pack(static_cast<unsigned>(groups), static_cast<unsigned>(a.mw));
  const unsigned per_xcd = static_cast<unsigned>((groups + kXcds - 1) / kXcds);
  // The sample's pass, then the whole one.
  for (int pass = a.sample > 1 ? 0 : 1; pass < 2; ++pass) {
    if (f16) screen_pack_kernel<__half><<<pack, kKsub, 0, s>>>(a);
    else screen_pack_kernel<float><<<pack, kKsub, 0, s>>>(a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    ScreenBatch b = a;
    b.step = pass == 0 ? a.sample : 1;
    if (pass == 0) {
      // (an eighth of the tiles per workgroup: its few tiles fill the GPU)
      b.chunk_tiles = std::max(64, a.chunk_tiles / 8 / 64 * 64);
      b.splits = a.splits * a.chunk_tiles / (b.chunk_tiles * a.sample) + 2;
    }
    e = launch_with_lds(pick_screen(a.mw), dim3(kXcds * per_xcd * static_cast<unsigned>(b.splits)),
                        screen_waves(a.mw) * 64, screen_lds(a.mw), b, s);
    if (e != hipSuccess) return e;
    const void* fn = f16 ? (pass == 0 ? reinterpret_cast<const void*>(&screen_rerank_kernel<__half, false>)
                                      : reinterpret_cast<const void*>(&screen_rerank_kernel<__half, true>))
                         : (pass == 0 ? reinterpret_cast<const void*>(&screen_rerank_kernel<float, false>)
                                      : reinterpret_cast<const void*>(&screen_rerank_kernel<float, true>));
    e = launch_with_lds(fn, dim3(static_cast<unsigned>(a.nq)), kSeedThreads, rerank_lds(a.m, a.k), b, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace ifvs
