// Stage 1 of Algorithm 1: router projection, softmax over all N experts (Eq. (1)), per-token
// top-k and mixing weights (Section 2.1).  Every decision in fp64.
//
// Up to 256 experts: the projection runs on the fp64 matrix cores (logits_mfma_kernel of prologue.hip) and
// gate_rows_kernel takes one wave per token.  More experts: logits_kernel, spread over (token, group of 4 experts)
// workgroups so that the whole chip takes part, and softmax_topk_kernel, one workgroup per token.
#include "common.h"

namespace moespec {

constexpr int kLogitThreads = 256;
constexpr int kRowsPerGroup = 4;                               // router rows per workgroup
constexpr int kSlices = kLogitThreads / kRowsPerGroup;         // threads that share one row (= 64)
constexpr int kSoftmaxThreads = 256;
constexpr int kGateThreads = 256;
constexpr int kSharedGateTokens = 512;

// logits[t, i] = w_i . h_t (+ b_i).  Thread (el, sl) takes the 16-byte pieces sl, sl+64, ... of row
// i = 4 blockIdx.x + el and of h_t; all loads of a batch are issued together (the router weights of a
// layer are cold in every cache).
template <typename T>
__global__ __launch_bounds__(kLogitThreads) void logits_kernel(const T *__restrict__ h, const T *__restrict__ w_r,
                                                               const float *__restrict__ b_r, int d, int N,
                                                               double *__restrict__ logits) {
  __shared__ double part[kLogitThreads];
  __shared__ double part2[kRowsPerGroup * 8];
  const int t = blockIdx.y, tid = threadIdx.x;
  const int el = tid / kSlices, sl = tid % kSlices;
  const int e = blockIdx.x * kRowsPerGroup + el;
  constexpr int VEC = 16 / sizeof(T);  // elements per 16-byte piece
  constexpr int PB = 4;                // pieces in flight per operand
  const int npieces = d / VEC;         // d is a multiple of VEC
  const T *wrow = w_r + (size_t)(e < N ? e : N - 1) * d;
  const T *hrow = h + (size_t)t * d;
  double acc = 0.0;
  for (int p0 = 0; p0 < npieces; p0 += PB * kSlices) {
    uint4 wr[PB], hr[PB];
#pragma unroll
    for (int q = 0; q < PB; ++q) {
      const int pc = p0 + sl + q * kSlices;
      const bool ok = pc < npieces;
      wr[q] = ok ? *reinterpret_cast<const uint4 *>(wrow + (size_t)pc * VEC) : uint4{0u, 0u, 0u, 0u};
      hr[q] = ok ? *reinterpret_cast<const uint4 *>(hrow + (size_t)pc * VEC) : uint4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int q = 0; q < PB; ++q)
#pragma unroll
      for (int v = 0; v < VEC; ++v)
        acc = fma((double)Elem<T>::load(reinterpret_cast<const T *>(&wr[q]) + v),
                  (double)Elem<T>::load(reinterpret_cast<const T *>(&hr[q]) + v), acc);
  }
  part[tid] = acc;
  __syncthreads();
  if (sl < 8) {
    double a = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) a += part[el * kSlices + sl * 8 + q];
    part2[el * 8 + sl] = a;
  }
  __syncthreads();
  if (sl == 0 && e < N) {
    double a = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) a += part2[el * 8 + q];
    logits[(size_t)t * N + e] = a + (b_r ? (double)b_r[e] : 0.0);
  }
}

// probs[t, :] = softmax(logits[t, :]) in place (max-subtracted) - or, with the sigmoid gate, 1 / (1 + exp(-logit))
// per expert - then the natural top-k and its mixing weights if asked for.  One workgroup per token.
__global__ __launch_bounds__(kSoftmaxThreads) void softmax_topk_kernel(double *__restrict__ probs, int N, int k,
                                                                       int renorm, int sigmoid_gate,
                                                                       int32_t *__restrict__ topk_ids,
                                                                       float *__restrict__ topk_w) {
  extern __shared__ __align__(16) unsigned char smem[];
  double *g = reinterpret_cast<double *>(smem);               // [N, even] logits, then probabilities
  double *part = g + ((N + 1) & ~1);                          // [32] partial reductions
  double *wsel = part + 32;                                   // [k, even] + 1 denominator (+1 pad)
  int32_t *sel = reinterpret_cast<int32_t *>(wsel + ((k + 1) & ~1) + 2);  // [k, multiple of 4]
  int32_t *rank = sel + ((k + 3) & ~3);                       // [N]
  const int t = blockIdx.x, tid = threadIdx.x;
  for (int i = tid; i < N; i += blockDim.x) g[i] = probs[(size_t)t * N + i];
  __syncthreads();
  if (sigmoid_gate) {  // uniform
    for (int i = tid; i < N; i += blockDim.x) {
      const double p = 1.0 / (1.0 + exp(-g[i]));
      g[i] = p;
      probs[(size_t)t * N + i] = p;
    }
    __syncthreads();
  } else {
    // 32 strided partial results, then every thread folds the 32 in index order
    if (tid < 32) {
      double m = -INFINITY;
      for (int i = tid; i < N; i += 32) m = fmax(m, g[i]);
      part[tid] = m;
    }
    __syncthreads();
    double m = part[0];
  #pragma unroll
    for (int j = 1; j < 32; ++j) m = fmax(m, part[j]);
    __syncthreads();
    for (int i = tid; i < N; i += blockDim.x) g[i] = exp(g[i] - m);
    __syncthreads();
    if (tid < 32) {
      double a = 0.0;
      for (int i = tid; i < N; i += 32) a += g[i];
      part[tid] = a;
    }
    __syncthreads();
    double denom = part[0];
  #pragma unroll
    for (int j = 1; j < 32; ++j) denom += part[j];
    for (int i = tid; i < N; i += blockDim.x) {
      const double p = g[i] / denom;
      g[i] = p;
      probs[(size_t)t * N + i] = p;
    }
    __syncthreads();
  }

  if (topk_ids == nullptr && topk_w == nullptr) return;
  select_topk(g, N, k, sel, rank);
  __syncthreads();
  mixing_weights(g, sel, k, renorm, wsel, wsel + ((k + 1) & ~1));
  __syncthreads();
  for (int s = tid; s < k; s += blockDim.x) {
    if (topk_ids) topk_ids[(size_t)t * k + s] = sel[s];
    if (topk_w) topk_w[(size_t)t * k + s] = (float)wsel[s];
  }
}

// Eq. (1) and, if wanted, the natural top-k of Section 2.1 row by row: probs[t, :] = gate(sum of the Q slices of the router
// projection + bias), top-k by rank counts over the row in LDS.  A lane holds up to NU experts; 16-lane DPP reductions, then
// two cross-row steps.  partial may be probs (a wave reads its whole row before anybody writes it).
// One wave per token, or (kShare) the 4 waves of a workgroup: all of them evaluate the row, each counts against a quarter of
// the rivals.  Bound by the launch and one round of cold loads, by the row's N / 4 LDS reads (or a quarter of them) where
// experts are many (4096 tokens x 64 experts with top-8 and weights: 8.2 us, against 15 us of softmax_topk_kernel).
template <int Q, int NU, bool kTopK, bool kShare>
__global__ __launch_bounds__(kGateThreads) void gate_rows_kernel(const double *partial, const float *__restrict__ bias,
                                                                 int M, int N, int sigmoid_gate, double *probs, int k,
                                                                 int renorm, int32_t *__restrict__ topk_ids,
                                                                 float *__restrict__ topk_w) {
  constexpr int kWaves = kGateThreads / kWave, kRows = kTopK ? (kShare ? 1 : kWaves) : 1;
  __shared__ double rows[kRows][kTopK ? NU * kWave : 1];
  __shared__ int32_t sels[kRows][kWave];
  __shared__ int32_t rank[kShare ? NU * kWave : 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, t = kShare ? blockIdx.x : blockIdx.x * kWaves + wave;
  if (t >= M) return;
  double val[NU];
  load_logits<Q, NU>(partial, bias, M, N, t, val);
  gate_of_row<NU>(val, sigmoid_gate);
  if constexpr (kShare) {
    for (int i = threadIdx.x; i < NU * kWave; i += kGateThreads) rank[i] = 0;
    if (wave == 0) {
#pragma unroll
      for (int u = 0; u < NU; ++u) rows[0][lane + kWave * u] = lane + kWave * u < N ? val[u] : kNoRival;
    }
    __syncthreads();  // also: every wave has read its row of partial
    int c[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) c[u] = 0;
    const int quads = (N + 3) / 4;
    rank_counts<NU>(rows[0], quads * wave / kWaves * 4, quads * (wave + 1) / kWaves * 4, lane, 0, val, c);
#pragma unroll
    for (int u = 0; u < NU; ++u)
      if (lane + kWave * u < N && c[u]) atomicAdd(&rank[lane + kWave * u], c[u]);
    __syncthreads();
    if (wave > 0) return;
  }
#pragma unroll
  for (int u = 0; u < NU; ++u)
    if (lane + kWave * u < N) probs[(size_t)t * N + lane + kWave * u] = val[u];
  if constexpr (kTopK) {
    double *row = rows[kShare ? 0 : wave];
    int32_t *sel = sels[kShare ? 0 : wave];
    int c[NU];
    sel[lane] = -1;  // stays -1 where NaN values leave a slot unclaimed
    bool real[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) real[u] = lane + kWave * u < N;
    if constexpr (kShare) {
#pragma unroll
      for (int u = 0; u < NU; ++u) c[u] = rank[lane + kWave * u];
      wave_lds_sync();
    } else {
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        c[u] = 0;
        row[lane + kWave * u] = lane + kWave * u < N ? val[u] : kNoRival;
      }
      wave_lds_sync();
      rank_counts<NU>(row, 0, N, lane, 0, val, c);
    }
#pragma unroll
    for (int u = 0; u < NU; ++u)
      if (real[u] & (c[u] < k) & (val[u] == val[u])) sel[c[u]] = lane + kWave * u;
    const int nan = nan_claim<NU>(val, real, nullptr);
    wave_lds_sync();
    const int e = lane == 0 && nan >= 0 ? nan : sel[lane];  // -1 behind the last slot
    const double ge = lane < k && e >= 0 ? row[e] : 0.0, denom = renorm ? slot_sum(ge, k) : 1.0;
    if (lane < k) {
      if (topk_ids) topk_ids[(size_t)t * k + lane] = e;
      if (topk_w) topk_w[(size_t)t * k + lane] = (float)(e < 0 ? 0.0 : (renorm ? ge / denom : ge));
    }
  }
}

// Eq. (1) as above and the sums of the probabilities over the tokens of a workgroup, one per wave (Eq. (5)), which spare the budget
// stage a pass over the table in a launch of its own (4.8 us; layer of 511 tokens x 64 experts, d = 2048, 155.0 -> 152.6 us, of 2048
// tokens 381.8 -> 379.6).  parts[b, i]: workgroup b, added in token order.
template <int Q, int NU>
__global__ __launch_bounds__(1024) void gate_parts_kernel(const double *partial, const float *__restrict__ bias, int M, int N,
                                                          int sigmoid_gate, double *probs, double *__restrict__ parts) {
  __shared__ double rows[16][NU * kWave];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n_waves = blockDim.x >> 6;
  const int t = blockIdx.x * n_waves + wave;
  double val[NU];
  if (t < M) {  // uniform in the wave; partial may be probs: a row belongs to one wave
    load_logits<Q, NU>(partial, bias, M, N, t, val);
    gate_of_row<NU>(val, sigmoid_gate);
  } else {
#pragma unroll
    for (int u = 0; u < NU; ++u) val[u] = 0.0;
  }
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int i = lane + kWave * u;
    rows[wave][i] = val[u];
    if (i < N && t < M) probs[(size_t)t * N + i] = val[u];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < N; i += blockDim.x) {
    double a = rows[0][i];
    for (int w = 1; w < n_waves; ++w) a += rows[w][i];
    parts[(size_t)blockIdx.x * N + i] = a;
  }
}
// Waves of such a workgroup: the budget stage adds up to 128 parts in one round of loads (256 up to 128 experts in two).  0: too many tokens.
static int gate_part_tokens(int M, int N) {
  if (M <= 8 * 128) return 8;
  return N <= 2 * kWave && M <= 16 * 256 ? 16 : M <= 16 * 128 ? 16 : 0;
}
int gate_parts(const moespec_desc &ds, int M) {
  const int w = mfma_route_ok(ds) ? gate_part_tokens(M, ds.n_experts) : 0;
  return w ? (M + w - 1) / w : 0;
}

hipError_t launch_gate_rows(const moespec_desc &ds, const moespec_weights &wt, int M, int slices, const double *partial,
                            double *probs, int32_t *topk_ids, float *topk_w, double *parts, hipStream_t st) {
  const int N = ds.n_experts, sig = ds.gate == MOESPEC_GATE_SIGMOID ? 1 : 0;
  if (parts) {
    const int waves = gate_part_tokens(M, N);
    auto run = [&](auto kern) -> hipError_t {
      kern<<<(M + waves - 1) / waves, waves * kWave, 0, st>>>(partial, wt.b_router, M, N, sig, probs, parts);
      return hipGetLastError();
    };
#define MOESPEC_PARTS(Q) \
  (N <= 64 ? run(gate_parts_kernel<Q, 1>) : N <= 128 ? run(gate_parts_kernel<Q, 2>) : run(gate_parts_kernel<Q, 4>))
    return slices == 1 ? MOESPEC_PARTS(1) : slices == 2 ? MOESPEC_PARTS(2) : slices == 4 ? MOESPEC_PARTS(4) : MOESPEC_PARTS(8);
#undef MOESPEC_PARTS
  }
  const bool topk = topk_ids || topk_w;
  // a workgroup per token where the counts take longer than the launch and the tokens leave compute units idle (projection
  // and gate, wave / workgroup per token, us: 7 tokens x 256 experts 20.8 / 11.6, x 128 11.5 / 8.6; 511 x 256 31 / 23)
  const bool share = topk && N > kWave && M <= kSharedGateTokens;
  const int per_wg = share ? 1 : kGateThreads / kWave;
  auto run = [&](auto kern) -> hipError_t {
    kern<<<(M + per_wg - 1) / per_wg, kGateThreads, 0, st>>>(partial, wt.b_router, M, N, sig, probs, ds.top_k, ds.renorm,
                                                             topk_ids, topk_w);
    return hipGetLastError();
  };
#define MOESPEC_GATE(Q, NU)                                              \
  (!topk ? run(gate_rows_kernel<Q, NU, false, false>)                    \
         : share ? run(gate_rows_kernel<Q, NU, true, (NU > 1)>) : run(gate_rows_kernel<Q, NU, true, false>))
#define MOESPEC_GATE_Q(Q) (N <= 64 ? MOESPEC_GATE(Q, 1) : N <= 128 ? MOESPEC_GATE(Q, 2) : MOESPEC_GATE(Q, 4))
  return slices == 1 ? MOESPEC_GATE_Q(1) : slices == 2 ? MOESPEC_GATE_Q(2) : slices == 4 ? MOESPEC_GATE_Q(4) : MOESPEC_GATE_Q(8);
#undef MOESPEC_GATE_Q
#undef MOESPEC_GATE
}

hipError_t launch_route(const moespec_desc &ds, const moespec_weights &wt, const void *h, int M, double *probs,
                        int32_t *topk_ids, float *topk_w, double *partial, int partial_slices, double *parts, hipStream_t st) {
  const int N = ds.n_experts, k = ds.top_k, d = ds.d;
  if (mfma_route_ok(ds)) {
    // one slice is accumulated in the caller's table (above kSelfMaxTokens a table of several has the place of y: 1025 tokens
    // x 8 experts of d = 4096 19.3 -> 11.2 us, where the output tiles do not fill the chip)
    const int slices = logit_slices(ds, M, partial_slices);
    double *logits = slices == 1 ? probs : partial;
    hipError_t e = launch_logits(ds, wt, h, M, slices, logits, st);
    return e != hipSuccess ? e : launch_gate_rows(ds, wt, M, slices, logits, probs, topk_ids, topk_w, parts, st);
  }
  dim3 grid((N + kRowsPerGroup - 1) / kRowsPerGroup, M);
  if (ds.dtype == MOESPEC_BF16) {
    logits_kernel<uint16_t><<<grid, kLogitThreads, 0, st>>>(static_cast<const uint16_t *>(h),
                                                            static_cast<const uint16_t *>(wt.w_router), wt.b_router, d,
                                                            N, probs);
  } else {
    logits_kernel<float><<<grid, kLogitThreads, 0, st>>>(static_cast<const float *>(h),
                                                         static_cast<const float *>(wt.w_router), wt.b_router, d, N,
                                                         probs);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const size_t smem = sizeof(double) * (((N + 1) & ~1) + 32 + ((k + 1) & ~1) + 2) +
                      sizeof(int32_t) * (((k + 3) & ~3) + N);
  softmax_topk_kernel<<<M, kSoftmaxThreads, smem, st>>>(probs, N, k, ds.renorm, ds.gate == MOESPEC_GATE_SIGMOID ? 1 : 0,
                                                        topk_ids, topk_w);
  return hipGetLastError();
}

}  // namespace moespec
