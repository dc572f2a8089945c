// One training step of the filter-aware conditioning (Section 2, training
// paragraph): from the conditioned tables of a batch of training queries,
// the softmax cross-entropy of each query's candidate list (ground-truth
// positives first, then mined hard negatives; score = -distance / tau), the
// anchor regularizer lam * mean(Delta^2), and their gradients carried back
// through the tables and Delta = alpha . W into the memory bank and W, and
// to w_z.  Plain SGD.  C_PQ and the codes stay fixed.
//
// train_query_kernel (one workgroup per query):
//   1. the query's table into LDS; its candidates' distances, summed over
//      subspaces in order as the scan does;
//   2. softmax statistics in fp64; g_v = d(batch loss)/d(distance of v);
//   3. the table gradient g_lut[m][c] = sum over candidates v whose code in
//      subspace m is c of g_v, the candidates added in order by one
//      wavefront (lane = subspace), in the table's LDS;
//   4. one thread per codeword c (four groups of 256 threads, each a quarter
//      of the subspaces): for every subspace and sub-dimension j,
//      Delta, e = q - C_PQ - Delta, the Delta gradient
//        gd = g_lut * (-2 w e) + (2 lam / (M K d) / nq) Delta
//      (stored for the W update), and the reductions over c of gd * W
//      (alpha gradient) and g_lut * e^2 (w_f gradient): a wavefront
//      reduction each, the four wavefronts' partials added in wave order.
// The kernel is bound by latency: one workgroup per CU, so the candidates'
// code words are fetched side by side into LDS (a serial chain of loads per
// candidate before), sixteen wavefronts share the subspaces instead of four,
// and a subspace's W and Delta-gradient values stay in registers between their
// two uses (d of 2, 4 or 8 with r = 8).  256 queries, M = 48, d = 2, 42
// candidates: 340 -> 72 us.
// train_update_w: W -= lr * sum_q gd_q (x) alpha_q: a thread holds the r sums
// of one (subspace, codeword, sub-dimension), so a gradient is read once and
// not r times, over a quarter of the queries in order; the quarters are added
// in order (69 -> 33 us at that shape).
// train_update_bank: bank[row] -= lr * (sum of g_alpha over the (query, hash
// function) pairs that hit the row, in pair order; a row hit twice gets
// both), applied by the row's first pair.
// Every sum has a fixed order, so a step's results do not depend on
// scheduling: two identical steps give identical bits.
#include <cmath>

#include "ifvs_internal.h"

namespace ifvs {

namespace {

constexpr int kTrainThreads = 1024;
constexpr int kTrainWaves = kTrainThreads / 64;
constexpr int kTrainGroups = kTrainThreads / kKsub;

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ double wave_max_d(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

// Original id of a candidate slot, -1 when absent or out of range.
__device__ __forceinline__ int64_t cand_id(const TrainArgs& a, int qi, int v) {
  const int64_t id = a.cand[static_cast<int64_t>(qi) * a.n_cand + v];
  return (id >= 0 && id < a.n) ? id : -1;
}

// Code of physical row `row` in subspace mm.
__device__ __forceinline__ int code_of(const TrainArgs& a, int64_t row, int mm) {
  const uint32_t w = a.codes_t[((row >> 6) * a.mw + (mm >> 2)) * 64 + (row & 63)];
  return static_cast<int>((w >> (8 * (mm & 3))) & 0xFFu);
}

// D, R: the fixed sub-dimension and direction counts (0: any).
template <int D, int R>
__global__ __launch_bounds__(kTrainThreads) void train_query_kernel(const TrainArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int qi = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int M = a.m, d = D > 0 ? D : a.dsub, r = R > 0 ? R : a.r, mr = a.m * r;
  float* s_tab = reinterpret_cast<float*>(smem);                 // [M][256]: table, then its gradient
  float* s_v = s_tab + M * kKsub;                                 // [n_cand]: distances, then g_v
  float* s_gw = s_v + a.n_cand;                                   // [4][dim]: w_f gradient, per wavefront
  float* s_ga = s_gw + 4 * a.dim;                                 // [4][M*r]: alpha gradient, per wavefront
  // Reductions ([3][kTrainWaves]) use the table's LDS while it holds nothing:
  // after the distances, and after the gradients.
  double* s_red = reinterpret_cast<double*>(smem);
  static_assert(3 * kTrainWaves * sizeof(double) <= kKsub * sizeof(float), "one subspace's table holds them");
  uint32_t* s_code = reinterpret_cast<uint32_t*>(s_ga + 4 * mr);   // [n_cand][mw] code words (code_lds)

  const float* lut = a.lut + static_cast<int64_t>(qi) * M * kKsub;
  for (int e = tid; e < M * kKsub; e += kTrainThreads) s_tab[e] = lut[e];
  if (a.code_lds)
    for (int e = tid; e < a.n_cand * a.mw; e += kTrainThreads) {
      const int64_t id = cand_id(a, qi, e / a.mw);
      const int64_t row = id < 0 ? 0 : (a.inv_perm ? a.inv_perm[id] : id);
      s_code[e] = a.codes_t[((row >> 6) * a.mw + e % a.mw) * 64 + (row & 63)];
    }
  __syncthreads();
  auto code_at = [&](int v, int64_t row, int mm) -> int {
    if (a.code_lds) return static_cast<int>((s_code[v * a.mw + (mm >> 2)] >> (8 * (mm & 3))) & 0xFFu);
    return code_of(a, row, mm);
  };

  // 1. Distances.
  for (int v = tid; v < a.n_cand; v += kTrainThreads) {
    const int64_t id = cand_id(a, qi, v);
    float dist = 0.0f;
    if (id >= 0) {
      const int64_t row = a.code_lds ? 0 : (a.inv_perm ? a.inv_perm[id] : id);
      for (int mm = 0; mm < M; ++mm) dist = __fadd_rn(dist, s_tab[mm * kKsub + code_at(v, row, mm)]);
    }
    s_v[v] = dist;
  }
  __syncthreads();

  // 2. Softmax statistics over the present candidates (fp64).
  const double inv_tau = 1.0 / static_cast<double>(a.tau);
  double mx = -INFINITY, pos_sum = 0.0, n_p = 0.0;
  for (int v = tid; v < a.n_cand; v += kTrainThreads) {
    if (cand_id(a, qi, v) < 0) continue;
    mx = fmax(mx, -static_cast<double>(s_v[v]) * inv_tau);
    if (v < a.n_pos) {
      pos_sum += static_cast<double>(s_v[v]);
      n_p += 1.0;
    }
  }
  mx = wave_max_d(mx);
  pos_sum = wave_sum_d(pos_sum);
  n_p = wave_sum_d(n_p);
  if (lane == 0) {
    s_red[wave] = mx;
    s_red[kTrainWaves + wave] = pos_sum;
    s_red[2 * kTrainWaves + wave] = n_p;
  }
  __syncthreads();
  mx = s_red[0];
  pos_sum = n_p = 0.0;
#pragma unroll
  for (int w = 0; w < kTrainWaves; ++w) {
    mx = fmax(mx, s_red[w]);
    pos_sum += s_red[kTrainWaves + w];
    n_p += s_red[2 * kTrainWaves + w];
  }
  __syncthreads();
  double z = 0.0;
  for (int v = tid; v < a.n_cand; v += kTrainThreads)
    if (cand_id(a, qi, v) >= 0) z += exp(-static_cast<double>(s_v[v]) * inv_tau - mx);
  z = wave_sum_d(z);
  if (lane == 0) s_red[wave] = z;
  __syncthreads();
  z = 0.0;
#pragma unroll
  for (int w = 0; w < kTrainWaves; ++w) z += s_red[w];
  const double lse = mx + log(z);
  const double ce = n_p > 0.0 ? lse + pos_sum * inv_tau / n_p : 0.0;
  // g_v = -(softmax_v - [v positive] / P) / tau / nq (0 without positives).
  for (int v = tid; v < a.n_cand; v += kTrainThreads) {
    float g = 0.0f;
    if (n_p > 0.0 && cand_id(a, qi, v) >= 0) {
      const double p = exp(-static_cast<double>(s_v[v]) * inv_tau - lse);
      const double share = v < a.n_pos ? 1.0 / n_p : 0.0;
      g = static_cast<float>(-(p - share) * inv_tau / a.nq);
    }
    s_v[v] = g;
  }
  __syncthreads();

  // 3. Table gradient: wavefront 0 adds the candidates in order, lane mm
  // updating subspace mm (one candidate touches one entry per subspace, and
  // a lane's updates to an entry are in program order).
  for (int e = tid; e < M * kKsub; e += kTrainThreads) s_tab[e] = 0.0f;
  __syncthreads();
  if (wave == 0) {
    for (int v = 0; v < a.n_cand; ++v) {
      const float g = s_v[v];
      const int64_t id = cand_id(a, qi, v);
      if (g == 0.0f || id < 0) continue;
      const int64_t row = a.code_lds ? 0 : (a.inv_perm ? a.inv_perm[id] : id);
      for (int mm = lane; mm < M; mm += 64) {
        const int at = mm * kKsub + code_at(v, row, mm);
        s_tab[at] = __fadd_rn(s_tab[at], g);
      }
    }
  }
  __syncthreads();

  // 4. Delta gradient (thread = codeword), alpha and w_f gradients.  Group
  // `grp` of 256 threads takes subspaces grp, grp + 4, ...; `part` is a
  // wavefront's place in its group.
  const int c = tid & (kKsub - 1), grp = tid / kKsub, part = wave & 3;
  const float anchor = static_cast<float>(2.0 * a.lam / (static_cast<double>(M) * kKsub * d) / a.nq);
  const float* qrow = a.q + static_cast<int64_t>(qi) * a.dim;
  const float* wrow = a.wf + static_cast<int64_t>(qi) * a.dim;
  const float* arow = a.alpha + static_cast<int64_t>(qi) * mr;
  float* gdq = a.gdelta + static_cast<int64_t>(qi) * M * kKsub * d;
  double reg = 0.0;
  for (int mm = grp; mm < M; mm += kTrainGroups) {
    const float gl = s_tab[mm * kKsub + c];
    const float* wm = a.W + (static_cast<int64_t>(mm) * r * kKsub + c) * d;       // + t * 256 d + j
    const float* cm = a.cpq + (static_cast<int64_t>(mm) * kKsub + c) * d;
    float* gm = gdq + (static_cast<int64_t>(mm) * kKsub + c) * d;
    if constexpr (D > 0) {
      float wv[R][D], gd[D], gw[D], ga[R];
#pragma unroll
      for (int t = 0; t < R; ++t)
#pragma unroll
        for (int j = 0; j < D; ++j) wv[t][j] = wm[t * kKsub * D + j];
#pragma unroll
      for (int j = 0; j < D; ++j) {
        float delta = 0.0f;
#pragma unroll
        for (int t = 0; t < R; ++t) delta = __fadd_rn(delta, __fmul_rn(arow[mm * R + t], wv[t][j]));
        const float e = __fsub_rn(qrow[mm * D + j], __fadd_rn(cm[j], delta));
        gd[j] = __fadd_rn(__fmul_rn(gl, __fmul_rn(-2.0f * wrow[mm * D + j], e)), __fmul_rn(anchor, delta));
        gm[j] = gd[j];
        reg += static_cast<double>(delta) * delta;
        gw[j] = __fmul_rn(gl, __fmul_rn(e, e));
      }
#pragma unroll
      for (int t = 0; t < R; ++t) {
        ga[t] = 0.0f;
#pragma unroll
        for (int j = 0; j < D; ++j) ga[t] = __fadd_rn(ga[t], __fmul_rn(gd[j], wv[t][j]));
      }
      // The D + R sums over the codewords side by side.
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
        for (int j = 0; j < D; ++j) gw[j] += __shfl_xor(gw[j], o, 64);
#pragma unroll
        for (int t = 0; t < R; ++t) ga[t] += __shfl_xor(ga[t], o, 64);
      }
      if (lane == 0) {
#pragma unroll
        for (int j = 0; j < D; ++j) s_gw[part * a.dim + mm * D + j] = gw[j];
#pragma unroll
        for (int t = 0; t < R; ++t) s_ga[part * mr + mm * R + t] = ga[t];
      }
    } else {
      for (int j = 0; j < d; ++j) {
        float delta = 0.0f;
        for (int t = 0; t < r; ++t) delta = __fadd_rn(delta, __fmul_rn(arow[mm * r + t], wm[t * kKsub * d + j]));
        const float e = __fsub_rn(qrow[mm * d + j], __fadd_rn(cm[j], delta));
        gm[j] = __fadd_rn(__fmul_rn(gl, __fmul_rn(-2.0f * wrow[mm * d + j], e)), __fmul_rn(anchor, delta));
        reg += static_cast<double>(delta) * delta;
        const float gw = wave_sum(__fmul_rn(gl, __fmul_rn(e, e)));
        if (lane == 0) s_gw[part * a.dim + mm * d + j] = gw;
      }
      for (int t = 0; t < r; ++t) {
        float ga = 0.0f;
        for (int j = 0; j < d; ++j) ga = __fadd_rn(ga, __fmul_rn(gm[j], wm[t * kKsub * d + j]));
        ga = wave_sum(ga);
        if (lane == 0) s_ga[part * mr + mm * r + t] = ga;
      }
    }
  }
  reg = wave_sum_d(reg);
  __syncthreads();
  if (lane == 0) s_red[wave] = reg;
  __syncthreads();
  if (tid == 0) {
    double rsum = 0.0;
    for (int w = 0; w < kTrainWaves; ++w) rsum += s_red[w];
    a.loss[qi] = static_cast<float>(ce + a.lam * rsum / (static_cast<double>(M) * kKsub * d));
  }
  float* garow = a.galpha + static_cast<int64_t>(qi) * mr;
  for (int e = tid; e < mr; e += kTrainThreads)
    garow[e] = __fadd_rn(__fadd_rn(__fadd_rn(s_ga[e], s_ga[mr + e]), s_ga[2 * mr + e]), s_ga[3 * mr + e]);
  if (a.dwz) {
    const float* zrow = a.w_z + static_cast<int64_t>(qi) * a.dim;
    float* drow = a.dwz + static_cast<int64_t>(qi) * a.dim;
    for (int e = tid; e < a.dim; e += kTrainThreads) {
      const double x = static_cast<double>(zrow[e]);
      const float gw = __fadd_rn(__fadd_rn(__fadd_rn(s_gw[e], s_gw[a.dim + e]), s_gw[2 * a.dim + e]),
                                 s_gw[3 * a.dim + e]);
      drow[e] = static_cast<float>(static_cast<double>(gw) / (1.0 + exp(-x)));
    }
  }
}

// grid = (64-entry runs of a subspace's (c, j) slab, subspaces): lane = entry,
// wavefront = quarter of the queries, RT directions at a time.
constexpr int kUpdateQuarters = 4;
template <int RT>
__global__ __launch_bounds__(64 * kUpdateQuarters) void train_update_w_kernel(
    float* __restrict__ W, const float* __restrict__ gdelta, const float* __restrict__ alpha, int nq, int m, int r,
    int dsub, float lr) {
  __shared__ float s_part[kUpdateQuarters][RT][64];
  const int lane = threadIdx.x & 63;
  const int part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int mm = blockIdx.y;
  const int64_t per_t = static_cast<int64_t>(kKsub) * dsub;
  const int64_t cj = static_cast<int64_t>(blockIdx.x) * 64 + lane;   // per_t is a multiple of 64
  const int q0 = static_cast<int>(static_cast<int64_t>(nq) * part / kUpdateQuarters);
  const int q1 = static_cast<int>(static_cast<int64_t>(nq) * (part + 1) / kUpdateQuarters);
  const float* gd = gdelta + static_cast<int64_t>(mm) * per_t + cj;
  const int64_t gstep = static_cast<int64_t>(m) * per_t;
  for (int t0 = 0; t0 < r; t0 += RT) {
    float g[RT] = {};
    const float* al = alpha + static_cast<int64_t>(mm) * r + t0;
    constexpr int kAhead = 8;
    for (int q = q0; q < q1; q += kAhead) {
      float v[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) v[u] = gd[(q + u < q1 ? q + u : q1 - 1) * gstep];
#pragma unroll
      for (int u = 0; u < kAhead; ++u)
        if (q + u < q1) {
#pragma unroll
          for (int t = 0; t < RT; ++t)
            if (t0 + t < r) g[t] = __fadd_rn(g[t], __fmul_rn(v[u], al[static_cast<int64_t>(q + u) * m * r + t]));
        }
    }
#pragma unroll
    for (int t = 0; t < RT; ++t) s_part[part][t][lane] = g[t];
    __syncthreads();
    for (int t = part; t < RT; t += kUpdateQuarters)
      if (t0 + t < r) {
        float sum = 0.0f;
#pragma unroll
        for (int p = 0; p < kUpdateQuarters; ++p) sum = __fadd_rn(sum, s_part[p][t][lane]);
        const int64_t at = (static_cast<int64_t>(mm) * r + t0 + t) * per_t + cj;
        W[at] = __fsub_rn(W[at], __fmul_rn(lr, sum));
      }
    __syncthreads();
  }
}

// One workgroup per (query, hash function) pair p; the first pair that hits
// a row sums the alpha gradients of all pairs hitting it, in pair order, and
// applies them (the other pairs of the row return).  256 pairs are compared
// at once, their matches taken from ballots in order (a thread walking all
// pairs took 50 us for 512 of them, this 6).
__global__ __launch_bounds__(256) void train_update_bank_kernel(float* __restrict__ bank, int mr,
                                                                const int32_t* __restrict__ rows, int h,
                                                                const float* __restrict__ galpha, int pairs,
                                                                float lr) {
  __shared__ uint64_t s_hit[4];
  const int p = blockIdx.x;
  const int wave = threadIdx.x >> 6;
  const int32_t row = rows[p];
  bool earlier = false;
  for (int p2 = threadIdx.x; p2 < p; p2 += 256) earlier = earlier || rows[p2] == row;
  if (__syncthreads_or(earlier ? 1 : 0)) return;
  for (int e0 = 0; e0 < mr; e0 += 256) {
    const int e = e0 + threadIdx.x;
    float g = 0.0f;
    for (int base = p; base < pairs; base += 256) {
      const int p2 = base + threadIdx.x;
      const uint64_t hit = __ballot(p2 < pairs && rows[p2 < pairs ? p2 : p] == row);
      __syncthreads();
      if ((threadIdx.x & 63) == 0) s_hit[wave] = hit;
      __syncthreads();
      for (int w = 0; w < 4; ++w)
        for (uint64_t x = s_hit[w]; x != 0; x &= x - 1) {
          const int at = base + 64 * w + __builtin_ctzll(x);
          if (e < mr) g = __fadd_rn(g, galpha[static_cast<int64_t>(at / h) * mr + e]);
        }
    }
    if (e < mr) {
      const int64_t at = static_cast<int64_t>(row) * mr + e;
      bank[at] = __fsub_rn(bank[at], __fmul_rn(lr, g));
    }
  }
}

__global__ void invert_perm_kernel(const int32_t* __restrict__ perm, int64_t n, int32_t* __restrict__ inv) {
  const int64_t r = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (r < n) inv[perm[r]] = static_cast<int32_t>(r);
}

}  // namespace

// LDS of train_query_kernel without the staged code words: its table, the
// candidates' values, the w_f and alpha gradients of four wavefronts.
size_t train_query_lds_bytes(int m, int dim, int n_cand, int mr) {
  const size_t floats = static_cast<size_t>(m) * kKsub + n_cand + 4 * static_cast<size_t>(dim) + 4 * static_cast<size_t>(mr);
  return floats * sizeof(float);
}

hipError_t launch_train_query(const TrainArgs& args, hipStream_t s) {
  TrainArgs a = args;
  size_t lds = train_query_lds_bytes(a.m, a.dim, a.n_cand, a.m * a.r);
  const size_t codes = static_cast<size_t>(a.n_cand) * a.mw * sizeof(uint32_t);
  a.code_lds = lds + codes <= static_cast<size_t>(kLdsBudget) ? 1 : 0;
  if (a.code_lds) lds += codes;
  const void* fn = a.r != 8     ? reinterpret_cast<const void*>(&train_query_kernel<0, 0>)
                   : a.dsub == 2 ? reinterpret_cast<const void*>(&train_query_kernel<2, 8>)
                   : a.dsub == 4 ? reinterpret_cast<const void*>(&train_query_kernel<4, 8>)
                   : a.dsub == 8 ? reinterpret_cast<const void*>(&train_query_kernel<8, 8>)
                                 : reinterpret_cast<const void*>(&train_query_kernel<0, 0>);
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  if (e != hipSuccess) return e;
  void* params[] = {&a};
  return hipLaunchKernel(fn, dim3(static_cast<unsigned>(a.nq)), dim3(kTrainThreads), params, lds, s);
}

hipError_t launch_train_update_w(float* W, const float* gdelta, const float* alpha, int nq, int m, int r,
                                 int dsub, float lr, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(kKsub * dsub / 64), static_cast<unsigned>(m));
  train_update_w_kernel<8><<<grid, dim3(64 * kUpdateQuarters), 0, s>>>(W, gdelta, alpha, nq, m, r, dsub, lr);
  return hipGetLastError();
}

hipError_t launch_train_update_bank(float* bank, int mr, const int32_t* rows, int h, const float* galpha,
                                    int nq, float lr, hipStream_t s) {
  if (nq * h <= 0) return hipSuccess;
  train_update_bank_kernel<<<dim3(nq * h), dim3(256), 0, s>>>(bank, mr, rows, h, galpha, nq * h, lr);
  return hipGetLastError();
}

hipError_t launch_invert_perm(const int32_t* perm, int64_t n, int32_t* inv, hipStream_t s) {
  invert_perm_kernel<<<dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, s>>>(perm, n, inv);
  return hipGetLastError();
}

}  // namespace ifvs
