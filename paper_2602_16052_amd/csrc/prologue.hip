// Stages 1-3 of Algorithm 1 for the fused layer call on small trees, in two or three launches with no dependence
// between workgroups inside a launch:
//
//   logits_table_kernel   small tables: the router projection w_i . h_t of Eq. (1) for all tokens and experts on the fp64
//                         matrix cores, finished
//   route_budget_kernel   a workgroup per tree token and one per shortlist rank (on larger trees the same ones for both).
//                         EVERY workgroup rebuilds the whole M x N table of
//                         routing probabilities from the projection (softmax or sigmoid gate of
//                         Eq. (1)), the aggregate scores of Eq. (5) and the top-B shortlist (Section 3.2) in its
//                         LDS - a few thousand exponentials, cheaper than a second pass over global memory and a
//                         grid-wide wait - then restricts its own token's routing (Eq. (7) / Eq. (8)) or
//                         writes the pair lists of the shortlist ranks it is responsible for: for every loaded
//                         expert the (token, slot) pairs routed to it, tokens ascending, which is what the
//                         expert passes consume.
//
// and for tables too large to be rebuilt by everyone:
//
//   logits_mfma_kernel    the projection as partial sums over slices of the hidden dimension
//   rank_rows_kernel      Eq. (1) row by row, the ranks in every row and sums over a few tokens each
//   route_budget_kernel   as above from the ranks and those sums
//
// Every decision in fp64, ties to the lowest expert id, as in the staged kernels of route.hip / budget.hip, which remain
// the path of the stage calls, of larger trees (fused_prologue_ok) and of layers whose passes take the grouped form.  Their
// projection is here too: logits_mfma_kernel, or logits_block_kernel for many tokens.
#include "common.h"

namespace moespec {

typedef __attribute__((ext_vector_type(4))) double f64x4;

constexpr int kLogitWaves = 4;
constexpr int kPrologueThreads = 1024;
constexpr int kFusedMaxTokens = 256;  // see fused_prologue_ok
// Tables above this many entries get their softmax, and the ranks of their rows, in a launch of their own.  Whole bf16 layer of
// d = 2048, us, rebuilt in every workgroup / extra launch: 47 x 64 35.8 / 37.1, 63 x 64 37.9 / 39.0, 40 x 128 41.6 / 42.0, 79 x 64
// 44.3 / 43.8, 93 x 64 45.6 / 44.7, 127 x 64 49.3 / 47.5.
constexpr long long kSplitSoftmaxAbove = 5500;

// 8 consecutive elements of a row, widened one by one
template <typename T> struct LogitPiece;
template <> struct LogitPiece<uint16_t> {
  uint4 v;
  __device__ __forceinline__ void load(const uint16_t *p) { v = *reinterpret_cast<const uint4 *>(p); }
  // n elements of the row are left (a multiple of 8): zeros past its end
  __device__ __forceinline__ void load_part(const uint16_t *p, int n) {
    v = uint4{0, 0, 0, 0};
    if (n > 0) load(p);
  }
  __device__ __forceinline__ double get(int m) const {
    const uint32_t word = reinterpret_cast<const uint32_t *>(&v)[m >> 1];
    return (double)__uint_as_float(m & 1 ? (word & 0xffff0000u) : (word << 16));
  }
};
template <> struct LogitPiece<float> {
  float4 v[2];
  __device__ __forceinline__ void load(const float *p) {
    v[0] = reinterpret_cast<const float4 *>(p)[0];
    v[1] = reinterpret_cast<const float4 *>(p)[1];
  }
  __device__ __forceinline__ void load_part(const float *p, int n) {  // n: a multiple of 4
    v[0] = v[1] = float4{0.f, 0.f, 0.f, 0.f};
    if (n > 0) v[0] = reinterpret_cast<const float4 *>(p)[0];
    if (n > 4) v[1] = reinterpret_cast<const float4 *>(p)[1];
  }
  __device__ __forceinline__ double get(int m) const { return (double)reinterpret_cast<const float *>(v)[m]; }
};

// partial[q][t][e] = sum over the q-th slice of the hidden dimension of h[t][j] * w_r[e][j], in fp64.
// Workgroup (x, q): x = output tile (16 tokens x 16 experts), q = slice; its 4 waves cut the slice again into
// runs of 32-element blocks and add their results through LDS in wave order.  v_mfma_f64_16x16x4: lane (i, g)
// = (lane % 16, lane / 16) supplies A[i][g] and B[g][i] and receives D[g + 4 r][i] in accumulator r.  A lane
// loads 8 consecutive elements of its token row and of its expert row per block; which of the 32
// elements of a block meet in one instruction is immaterial, the sum over the block is complete after 8 of them.
// kAhead: the loads of the next blocks are in flight while the present ones are multiplied.
template <typename T, bool kAhead>
__global__ __launch_bounds__(kLogitWaves *kWave) void logits_mfma_kernel(const T *__restrict__ h, const T *__restrict__ w_r,
                                                                          int M, int N, int d, int n_slices,
                                                                          double *__restrict__ partial) {
  __shared__ double red[kLogitWaves][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int e_tiles = (N + 15) / 16;
  const int tt = blockIdx.x / e_tiles, et = blockIdx.x % e_tiles, q = blockIdx.y;
  const int i = lane & 15, g = lane >> 4;
  const int t = min(tt * 16 + i, M - 1), e = min(et * 16 + i, N - 1);  // pad rows repeat the last one, never stored
  const int n_blocks = d / 32, parts = n_slices * kLogitWaves, part = q * kLogitWaves + wave;
  const int b0 = (int)((long long)part * n_blocks / parts), b1 = (int)((long long)(part + 1) * n_blocks / parts);
  const T *ha = h + (size_t)t * d + g * 8, *wb = w_r + (size_t)e * d + g * 8;
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  constexpr int PB = sizeof(T) == 2 ? 4 : 2, kSets = kAhead ? 2 : 1;  // blocks per set of loads
  LogitPiece<T> A[kSets][PB], Bv[kSets][PB];
  auto load = [&](int set, int b) {
#pragma unroll
    for (int u = 0; u < PB; ++u) {
      const int bb = min(b + u, b1 - 1);  // past the end: the last block again, not multiplied
      A[set][u].load(ha + (size_t)bb * 32);
      Bv[set][u].load(wb + (size_t)bb * 32);
    }
  };
  auto multiply = [&](int set, int b) {
#pragma unroll
    for (int u = 0; u < PB; ++u) {
      if (b + u < b1) {  // uniform in the wave
#pragma unroll
        for (int m = 0; m < 8; ++m)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(A[set][u].get(m), Bv[set][u].get(m), acc, 0, 0, 0);
      }
    }
  };
  if constexpr (kAhead) {
    int b = b0;
    if (b < b1) load(0, b);
    for (; b + 2 * PB < b1; b += 2 * PB) {
      load(1, b + PB);
      multiply(0, b);
      load(0, b + 2 * PB);
      multiply(1, b + PB);
    }
    if (b + PB < b1) load(1, b + PB);
    multiply(0, b);
    multiply(1, b + PB);
  } else {
    for (int b = b0; b < b1; b += PB) {
      load(0, b);
      multiply(0, b);
    }
  }
  if (d % 32 != 0 && part == parts - 1) {  // fp32 layers: the last 4 to 28 elements, 4 at a time, one per lane group
    for (int j = n_blocks * 32; j < d; j += 4)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)Elem<T>::load(h + (size_t)t * d + j + g),
                                                 (double)Elem<T>::load(w_r + (size_t)e * d + j + g), acc, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) red[wave][(g + 4 * r) * 16 + i] = acc[r];
  __syncthreads();
  const int x = threadIdx.x, row = tt * 16 + x / 16, col = et * 16 + x % 16;
  if (row < M && col < N) {
    double a = red[0][x];
#pragma unroll
    for (int w = 1; w < kLogitWaves; ++w) a += red[w][x];
    partial[((size_t)q * M + row) * N + col] = a;
  }
}

// The same in tiles of 32 tokens x 16 TE experts: an operand is widened once for two (TE = 2) instructions of a wave.  What bounds
// the projection of many tokens is the fp64 unit, which widens as well as it multiplies.  8 waves share the slice, so that a
// workgroup per compute unit still makes two waves per SIMD (four were slower than the 16 x 16 tiles: no load latency is hidden).
// d = 2048, 64 experts, us, 16 x 16 tiles / these: 4096 tokens 26.6 / 24.2, 2048 tokens 17.3 / 16.1.  (Without the conversions the
// 16 x 16 tiles would take 24.8; widening with integer operations 32.2.)
constexpr int kBlockWaves = 8;
template <typename T, int TE>
__global__ __launch_bounds__(kBlockWaves *kWave, 2) void logits_block_kernel(const T *__restrict__ h, const T *__restrict__ w_r, int M,
                                                                             int N, int d, int n_slices, double *__restrict__ partial) {
  __shared__ double red[kBlockWaves][2 * TE][256];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int e_tiles = (N + 16 * TE - 1) / (16 * TE);
  const int tt = blockIdx.x / e_tiles, et = blockIdx.x % e_tiles, q = blockIdx.y;
  const int i = lane & 15, g = lane >> 4;
  const int n_blocks = d / 32, parts = n_slices * kBlockWaves, part = q * kBlockWaves + wave;
  const int b0 = (int)((long long)part * n_blocks / parts), b1 = (int)((long long)(part + 1) * n_blocks / parts);
  const T *rows[2 + TE];  // pad rows repeat the last one, never stored
#pragma unroll
  for (int x = 0; x < 2; ++x) rows[x] = h + (size_t)min(tt * 32 + 16 * x + i, M - 1) * d + g * 8;
#pragma unroll
  for (int x = 0; x < TE; ++x) rows[2 + x] = w_r + (size_t)min(et * 16 * TE + 16 * x + i, N - 1) * d + g * 8;
  f64x4 acc[2][TE];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < TE; ++y) acc[x][y] = f64x4{0.0, 0.0, 0.0, 0.0};
  constexpr int PB = 2;  // blocks per set of loads, two sets in turn
  LogitPiece<T> P[2][PB][2 + TE];
  auto load = [&](int set, int b) {
#pragma unroll
    for (int u = 0; u < PB; ++u)
#pragma unroll
      for (int x = 0; x < 2 + TE; ++x) P[set][u][x].load(rows[x] + (size_t)min(b + u, b1 - 1) * 32);  // past the end: the last one again
  };
  auto multiply = [&](int set, int b) {
#pragma unroll
    for (int u = 0; u < PB; ++u) {
      if (b + u < b1) {  // uniform in the wave
#pragma unroll
        for (int m = 0; m < 8; ++m) {
          double v[2 + TE];
#pragma unroll
          for (int x = 0; x < 2 + TE; ++x) v[x] = P[set][u][x].get(m);
#pragma unroll
          for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < TE; ++y) acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[x], v[2 + y], acc[x][y], 0, 0, 0);
        }
      }
    }
  };
  int b = b0;
  load(0, b);  // every wave has blocks (logits_in_blocks)
  for (; b + 2 * PB < b1; b += 2 * PB) {
    load(1, b + PB);
    multiply(0, b);
    load(0, b + 2 * PB);
    multiply(1, b + PB);
  }
  if (b + PB < b1) load(1, b + PB);
  multiply(0, b);
  multiply(1, b + PB);
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < TE; ++y)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][x * TE + y][(g + 4 * r) * 16 + i] = acc[x][y][r];
  __syncthreads();
  for (int o = threadIdx.x; o < 2 * TE * 256; o += kBlockWaves * kWave) {
    const int tile = o >> 8, at = o & 255;
    double a = red[0][tile][at];
#pragma unroll
    for (int w = 1; w < kBlockWaves; ++w) a += red[w][tile][at];
    const int row = tt * 32 + 16 * (tile / TE) + at / 16, col = et * 16 * TE + 16 * (tile % TE) + at % 16;
    if (row < M && col < N) partial[((size_t)q * M + row) * N + col] = a;
  }
}

// The same for small tables, finished in one launch: logits[t][e] = h[t] . w_r[e] + bias[e].  A workgroup owns 4 tokens x 4
// experts and the whole hidden dimension, which its 8 waves share in chunks of 128 elements.  v_mfma_f64_4x4x4 multiplies four
// independent blocks: lane (i, c) = (lane % 4, lane / 4) supplies A[i] and B[i] of its own piece c of the hidden dimension
// (block c % 4, element c / 4), and D[i][j] of block b arrives in lane 16 i + 4 b + j; the four blocks are added at the end.
// Sixteen times as many workgroups as 16 x 16 tiles, so that the hidden dimension need not be cut over workgroups and the consumer
// loads one table instead of up to eight; twice the widening per multiply-add, which matters only where tables are large.
constexpr int kTableWaves = 8, kTableChunk = 128;
template <typename T>
__global__ __launch_bounds__(kTableWaves *kWave) void logits_table_kernel(const T *__restrict__ h, const T *__restrict__ w_r,
                                                                          const float *__restrict__ bias, int M, int N, int d,
                                                                          double *__restrict__ logits) {
  __shared__ double red[kTableWaves][kWave];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int e_tiles = (N + 3) / 4;
  const int tt = blockIdx.x / e_tiles, et = blockIdx.x % e_tiles;
  const int i = lane & 3, at = (lane >> 2) * 8;
  const int t = min(tt * 4 + i, M - 1), e = min(et * 4 + i, N - 1);  // pad rows repeat the last one, never stored
  const T *ha = h + (size_t)t * d, *wb = w_r + (size_t)e * d;
  const int n_chunks = (d + kTableChunk - 1) / kTableChunk;
  double acc[2] = {0.0, 0.0};
  constexpr int PB = 4;  // chunks in flight
  for (int c0 = wave; c0 < n_chunks; c0 += PB * kTableWaves) {
    LogitPiece<T> A[PB], Bv[PB];
#pragma unroll
    for (int u = 0; u < PB; ++u) {
      if (c0 + u * kTableWaves < n_chunks) {  // uniform in the wave
        const int j = (c0 + u * kTableWaves) * kTableChunk + at;
        A[u].load_part(ha + j, d - j);
        Bv[u].load_part(wb + j, d - j);
      }
    }
#pragma unroll
    for (int u = 0; u < PB; ++u) {
      if (c0 + u * kTableWaves < n_chunks) {
#pragma unroll
        for (int m = 0; m < 8; ++m)
          acc[m & 1] = __builtin_amdgcn_mfma_f64_4x4x4f64(A[u].get(m), Bv[u].get(m), acc[m & 1], 0, 0, 0);
      }
    }
  }
  red[wave][lane] = acc[0] + acc[1];
  __syncthreads();
  if (wave == 0) {
    double v[kTableWaves];
#pragma unroll
    for (int w = 0; w < kTableWaves; ++w) v[w] = red[w][lane];
    double a = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    a += dpp_f64<kDppRor8>(a);
    a += dpp_f64<kDppRor4>(a);
    const int row = tt * 4 + (lane >> 4), col = et * 4 + (lane & 3);
    if ((lane & 12) == 0 && row < M && col < N) logits[(size_t)row * N + col] = a + (bias ? (double)bias[col] : 0.0);
  }
}

// Larger tables take a launch between the projection and the last one: Eq. (1) row by row, and what the last kernel needs of the
// table in place of its fp64 values.
//   ranks[t][i]  (16 bits) the natural rank of expert i for token t: how many experts go before it by (probability descending,
//                id ascending).  The restricted routings compare ranks only: a rank among the shortlisted experts is the number
//                of shortlisted experts with a smaller natural one.  kNaNRank where the probability is a NaN, which ranks nowhere.
//   parts[b][i]  the sum of the probabilities of expert i over the tokens kPartTokens b, ... (Eq. (5))
// Every workgroup of the last kernel loads a quarter of the bytes, and adds 32 rows at 127 tokens where it added 127.
// The first workgroups make a part each, a token per wave; the others a token's ranks each: all 4 waves evaluate its row and count
// against a quarter of the rivals.  That the rows are evaluated twice costs nothing, they lie side by side on compute units that
// would idle (4 tokens and their part in one workgroup of 16 waves: 6.6 us instead of 4.8 at 127 tokens x 128 experts).
constexpr int kPartTokens = 4, kRankThreads = 4 * kWave, kNaNRank = 0xffff;
// Elements from one row of ranks to the next, in memory and in the LDS: 16 bytes more than the row is long, so that the 4 tokens of a
// wave touch different banks.
__host__ __device__ inline int rank_row(int N) { return ((N + 7) & ~7) + 8; }
template <int Q, int NU>
__global__ __launch_bounds__(kRankThreads) void rank_rows_kernel(const double *__restrict__ partial, const float *__restrict__ bias,
                                                                 int M, int N, int n_parts, int sigmoid_gate,
                                                                 double *__restrict__ probs, double *__restrict__ parts,
                                                                 uint16_t *__restrict__ ranks) {
  __shared__ double rows[4][NU * kWave];
  __shared__ int32_t counts[4][NU * kWave];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool part = (int)blockIdx.x < n_parts;
  const int t = part ? (int)blockIdx.x * kPartTokens + wave : (int)blockIdx.x - n_parts;
  double val[NU];
  load_logits<Q, NU>(partial, bias, M, N, min(t, M - 1), val);
  gate_of_row<NU>(val, sigmoid_gate);
  if (part) {
#pragma unroll
    for (int u = 0; u < NU; ++u) rows[wave][lane + kWave * u] = t < M ? val[u] : 0.0;
    __syncthreads();
    for (int i = threadIdx.x; i < N; i += kRankThreads)
      parts[(size_t)blockIdx.x * N + i] = ((rows[0][i] + rows[1][i]) + rows[2][i]) + rows[3][i];
    return;
  }
  if (wave == 0) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int i = lane + kWave * u;
      rows[0][i] = i < N ? val[u] : kNoRival;
      if (i < N) probs[(size_t)t * N + i] = val[u];
    }
  }
  __syncthreads();
  int c[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) c[u] = 0;
  const int quads = (N + 3) / 4;
  rank_counts<NU>(rows[0], quads * wave / 4 * 4, quads * (wave + 1) / 4 * 4, lane, 0, val, c);
#pragma unroll
  for (int u = 0; u < NU; ++u) counts[wave][lane + kWave * u] = c[u];
  __syncthreads();
  for (int i = threadIdx.x; i < N; i += kRankThreads) {
    const double v = rows[0][i];
    const int r = (counts[0][i] + counts[1][i]) + (counts[2][i] + counts[3][i]);
    ranks[(size_t)t * rank_row(N) + i] = (uint16_t)(v == v ? r : kNaNRank);
  }
}

// LDS of route_budget_kernel.  Rows of the table are N + 1 doubles apart: lanes that walk down a column (one token per lane) then
// touch different banks.
struct PrologueLds {
  size_t g, s, red, count, S, cand, pos, sel, inS, total;
};
__host__ __device__ inline PrologueLds prologue_lds(int M, int N, int k, int B, bool ranked) {
  PrologueLds L;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off += (bytes + 15) & ~(size_t)15;
    return at;
  };
  L.g = take(ranked ? sizeof(uint16_t) * (size_t)M * rank_row(N) : sizeof(double) * (size_t)M * (N + 1));
  L.s = take(sizeof(double) * N);
  L.red = take(ranked ? sizeof(double) * kPrologueThreads : 0);
  L.count = take(sizeof(int32_t) * 2 * (kPrologueThreads / kWave));
  L.S = take(sizeof(int32_t) * (B + kWave));
  L.cand = take(sizeof(int32_t) * (B + kWave));
  L.pos = take(sizeof(int32_t) * N);
  L.sel = take(sizeof(int32_t) * (k + 1));
  L.inS = take((size_t)N);
  L.total = off;
  return L;
}

// list_count[r] = number of pairs routed to the expert at shortlist rank r after the restriction;
// lists[r * list_stride + p] = flat id t * k + slot of its p-th pair, tokens ascending.
// NE > 0: table = logits with their bias; NE = ceil(N / 16) = elements of a table row per lane in the softmax (compile-time so that
// the short loops unroll: a taken branch costs this hardware about as much as ten fp64 operations).  NE = 0: table = the ranks,
// beside them probs and parts, all from rank_rows_kernel.  16 consecutive lanes share a row, a column, a candidate or a token
// and reduce through DPP; the 64 groups of a round that have nothing to do are skipped wave by wave, because 16 waves share the
// issue slots of 4 SIMDs (the chain of fp64 operations of a 15 x 8 table took 1.0 us in 16 waves, of which 12 had no row).
// Comparisons are written without short-circuit evaluation and loops in fixed blocks of four, so that the code stays straight-line.
enum : int { kSigmoidGate = 1, kTruncate = 2, kRenorm = 4 };
template <int NE>
__global__ __launch_bounds__(kPrologueThreads) void route_budget_kernel(
    const void *__restrict__ table, int M, int N, int k, int B, int list_wgs, int flags, int list_stride,
    const int32_t *__restrict__ ext_shortlist, const double *__restrict__ parts, const double *__restrict__ probs,
    double *__restrict__ probs_out, double *__restrict__ scores_out, int32_t *__restrict__ budget_ids,
    int32_t *__restrict__ seg_expert, int32_t *__restrict__ tok_ids, float *__restrict__ tok_w,
    int32_t *__restrict__ list_count, int32_t *__restrict__ lists) {
  constexpr bool kRanked = NE == 0;
  extern __shared__ __align__(16) unsigned char smem[];
  const PrologueLds L = prologue_lds(M, N, k, B, kRanked);
  double *g = reinterpret_cast<double *>(smem + L.g);        // [M][N + 1] logits, then routing probabilities
  uint16_t *nr = reinterpret_cast<uint16_t *>(smem + L.g);   // kRanked: [M][rank_row(N)] natural ranks
  double *s = reinterpret_cast<double *>(smem + L.s);        // [N] aggregate scores, as they rank
  double *red = reinterpret_cast<double *>(smem + L.red);    // kRanked: [1024] sums of the parts by group
  int32_t *count = reinterpret_cast<int32_t *>(smem + L.count);  // [2][16] pairs per wave of a list (two lists in turn)
  int32_t *S = reinterpret_cast<int32_t *>(smem + L.S);      // [B] shortlist in rank order, -1 behind it
  int32_t *pos = reinterpret_cast<int32_t *>(smem + L.pos);  // [N] shortlist rank of every expert
  int32_t *sel = reinterpret_cast<int32_t *>(smem + L.sel);  // [k] this token's selection; [1] nan_key of the NaN that claims slot 0
  uint8_t *inS = smem + L.inS;
  constexpr int nt = kPrologueThreads, kGroups = nt / 16, kWaves = nt / kWave, kWaveGroups = kGroups / kWaves;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = tid >> 4, seg = tid & 15, group0 = wave * kWaveGroups;  // group0: the first of this wave
  const bool truncate = flags & kTruncate;
  // The first list_wgs workgroups build the pair lists and the others take a token each; list_wgs = 0: a workgroup does both.
  // own: this workgroup's token; below zero or past the end: it only builds pair lists
  const int own = (int)blockIdx.x - list_wgs;
  const int list_step = list_wgs ? list_wgs : max(M, B), last_wg = (list_wgs ? M + B : max(M, B)) - 1;
  const int NS = N + 1, NR = rank_row(N);

  const bool want_scores = ext_shortlist == nullptr || scores_out != nullptr;
  if constexpr (kRanked) {
    const int total = M * NR / 8;  // pieces of 16 bytes
    const uint4 *from = static_cast<const uint4 *>(table);
    uint4 *to = reinterpret_cast<uint4 *>(nr);
    uint4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = from[min(u * nt + tid, total - 1)];
    if (want_scores) {  // Eq. (5) from the parts, with the first ranks on their way: a group of threads adds every n_groups-th
      int cp2 = 64, cp2_log = 6;
      while (cp2 < N) cp2 <<= 1, ++cp2_log;
      const int col = tid & (cp2 - 1), n_rows = (M + kPartTokens - 1) / kPartTokens, n_groups = nt >> cp2_log;
      double a = 0.0;
      for (int r = tid >> cp2_log; r < n_rows; r += 4 * n_groups) {
        double x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = col < N && r + u * n_groups < n_rows ? parts[(size_t)(r + u * n_groups) * N + col] : 0.0;
#pragma unroll
        for (int u = 0; u < 4; ++u) a += x[u];
      }
      red[tid] = a;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (u * nt + tid < total) to[u * nt + tid] = v[u];
    for (int x0 = 4 * nt; x0 < total; x0 += 4 * nt) {
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = from[min(x0 + u * nt + tid, total - 1)];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (x0 + u * nt + tid < total) to[x0 + u * nt + tid] = v[u];
    }
  } else {
    const double *logits = static_cast<const double *>(table);
    const int MN = M * N, dt = nt / N, di = nt % N;
    int t = tid / N, i = tid % N;
    for (int x0 = 0; x0 < MN; x0 += 4 * nt) {
      double v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = x0 + u * nt + tid < MN ? logits[x0 + u * nt + tid] : 0.0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (x0 + u * nt + tid < MN) g[t * NS + i] = v[u];
        t += dt;
        i += di;
        if (i >= N) i -= N, ++t;
      }
    }
  }
  for (int i = tid; i < N; i += nt) {
    inS[i] = 0;
    pos[i] = 0x7fffffff;
  }
  for (int r = tid; r < B + kWave; r += nt) S[r] = -1;
  for (int j = tid; j <= k; j += nt) sel[j] = j < k ? -1 : kNoNaN;
  __syncthreads();

  // Eq. (1): 16 lanes per row, 64 rows per round; a lane holds its NE elements of the row in registers
  for (int t0 = 0; !kRanked && t0 + group0 < M; t0 += kGroups) {
    constexpr int NE_ = kRanked ? 1 : NE;
    const int t = t0 + group;
    double *row = g + (t < M ? t : M - 1) * NS;
    double val[NE_];
#pragma unroll
    for (int u = 0; u < NE_; ++u) val[u] = (t < M && seg + 16 * u < N) ? row[seg + 16 * u] : -INFINITY;
    if (flags & kSigmoidGate) {
#pragma unroll
      for (int u = 0; u < NE_; ++u)
        if (t < M && seg + 16 * u < N) row[seg + 16 * u] = 1.0 / (1.0 + exp(-val[u]));
    } else {
      double m = val[0];
#pragma unroll
      for (int u = 1; u < NE_; ++u) m = fmax(m, val[u]);
      m = row16_max(m);
      double a = 0.0;
#pragma unroll
      for (int u = 0; u < NE_; ++u) {
        val[u] = exp_nonpos(val[u] - m);  // elements past the row end are -inf: they come out as 0
        a += val[u];
      }
      const double inv = 1.0 / row16_sum(a);
#pragma unroll
      for (int u = 0; u < NE_; ++u)
        if (t < M && seg + 16 * u < N) row[seg + 16 * u] = val[u] * inv;
    }
  }
  if constexpr (!kRanked) __syncthreads();
  if (!kRanked && probs_out && own >= 0 && own < M)  // (rank_rows_kernel writes where the caller wants it)
    for (int i = tid; i < N; i += nt) probs_out[(size_t)own * N + i] = g[own * NS + i];

  // Eq. (5): s_i = sum_t g_i(h_t).  Lane p of a column adds tokens p, p + 16, ... in ascending order and the 16 sums are folded
  // through DPP; 64 columns per round.
  if (want_scores) {
    if constexpr (kRanked) {
      int cp2 = 64;
      while (cp2 < N) cp2 <<= 1;
      if (tid < N) {
        double a = red[tid];
        for (int r = cp2; r < nt; r += cp2) a += red[r + tid];
        s[tid] = ranking_score(a);
        if (scores_out && (int)blockIdx.x == last_wg) scores_out[tid] = a;
      }
    } else {
      for (int c0 = 0; c0 + group0 < N; c0 += kGroups) {
        const int col = min(c0 + group, N - 1);
        double a = 0.0;
        for (int t = seg; t < M; t += 64) {  // fixed blocks of 4 tokens: the loads go out together
          double v[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) v[u] = t + 16 * u < M ? g[(t + 16 * u) * NS + col] : 0.0;
#pragma unroll
          for (int u = 0; u < 4; ++u) a += v[u];  // rows past the end add +0.0, which leaves the sum unchanged
        }
        a = row16_sum(a);
        if (seg == 0 && c0 + group < N) {
          s[col] = ranking_score(a);
          if (scores_out && (int)blockIdx.x == last_wg) scores_out[col] = a;
        }
      }
    }
    __syncthreads();
  }
  // Section 3.2: the B highest aggregate scores, ties to the lowest id - or the caller's shortlist.  Every rank is claimed once, so that
  // inS and pos name the experts of S and no others.
  if (ext_shortlist == nullptr) {
    // 16 lanes share a candidate and split its rivals: lane p takes p, p + 16, ...; 64 candidates per round
    for (int c0 = 0; c0 + group0 < N; c0 += kGroups) {
      const int i = c0 + group;
      const double vi = s[min(i, N - 1)];
      int c = 0;
      for (int j = seg; j < N; j += 64) {
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = s[min(j + 16 * u, N - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          c += (int)((j + 16 * u < N) & ((v[u] > vi) | ((v[u] == vi) & (j + 16 * u < i))));
      }
      c = row16_sum(c);
      if (seg == 0 && i < N && c < B) {
        S[c] = i;
        pos[i] = c;
        inS[i] = 1;
      }
    }
  } else {
    for (int r = tid; r < B; r += nt) {
      const int e = ext_shortlist[r];
      S[r] = e;
      if ((uint32_t)e < (uint32_t)N) {  // ids outside [0, N) are ignored
        inS[e] = 1;
        atomicMin(&pos[e], r);  // an expert named twice counts at its first rank
      }
    }
  }
  __syncthreads();
  // a token's candidates: all experts under truncation (Eq. (7) restricts the natural top-k afterwards), the
  // shortlist in rank order under substitution (Eq. (8)); -1 marks an entry of an external shortlist that is out of
  // range or a repeat, and what lies behind the end
  const int32_t *cand = S;
  const int n_cand = truncate ? N : B;
  if (ext_shortlist != nullptr && !truncate) {
    int32_t *checked = reinterpret_cast<int32_t *>(smem + L.cand);  // [B + 64]
    for (int x = tid; x < B + kWave; x += nt) {
      const int j = S[x];
      checked[x] = (uint32_t)j < (uint32_t)N && pos[j] == x ? j : -1;
    }
    cand = checked;
    __syncthreads();
  }
  // copies for the caller and for the expert passes, written by the last workgroup: it has no pair list to build where the
  // lists have workgroups of their own or the tokens outnumber the shortlist
  if ((int)blockIdx.x == last_wg) {
    for (int i = tid; i < N; i += nt) {
      if (seg_expert && inS[i]) {  // position of expert i among the shortlisted experts in ascending id
        int at = 0;
        for (int j = 0; j < i; ++j) at += inS[j];
        seg_expert[at] = i;
      }
    }
    if (tid < B) {
      int n_member = 0;  // < B only if an external shortlist repeats or misnames an expert
      if (seg_expert)
        for (int j = 0; j < N; ++j) n_member += inS[j];
      for (int r = tid; r < B; r += nt) {
        if (seg_expert && r >= n_member) seg_expert[r] = -1;
        budget_ids[r] = S[r];
      }
    }
  }

  // "x goes before y" in a ranking by (probability descending, id ascending), without short-circuit evaluation
  // (which would turn into divergent control flow)
  auto before = [](double vx, int jx, double vy, int jy) { return (vx > vy) | ((vx == vy) & (jx < jy)); };
  // The number of token t's candidates that go before expert e, counted by 16 lanes; kNaNRank or more where its probability is a NaN.
  auto rank_among = [&](int t, int e) {
    int c = 0;
    if constexpr (kRanked) {
      const uint16_t *row = nr + t * NR;
      const int own_rank = row[e];
      if (truncate) return own_rank;
      for (int y = seg; y < B; y += 64) {
        int jy[4], ry[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) jy[u] = cand[min(y + 16 * u, B)];  // entry B: -1
#pragma unroll
        for (int u = 0; u < 4; ++u) ry[u] = row[max(jy[u], 0)];
#pragma unroll
        for (int u = 0; u < 4; ++u) c += (int)((jy[u] >= 0) & (ry[u] < own_rank));
      }
      return row16_sum(c) + (own_rank == kNaNRank ? kNaNRank : 0);
    } else {
      const double *row = g + t * NS;
      const double v = row[e];
      if (truncate) {
        for (int y = seg; y < N; y += 64) {
          double vy[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) vy[u] = row[min(y + 16 * u, N - 1)];
#pragma unroll
          for (int u = 0; u < 4; ++u) c += (int)((y + 16 * u < N) & before(vy[u], y + 16 * u, v, e));
        }
      } else {
        for (int y = seg; y < B; y += 64) {
          int jy[4];
          double vy[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) jy[u] = cand[min(y + 16 * u, B)];  // entry B: -1
#pragma unroll
          for (int u = 0; u < 4; ++u) vy[u] = row[max(jy[u], 0)];
#pragma unroll
          for (int u = 0; u < 4; ++u) c += (int)((jy[u] >= 0) & before(vy[u], jy[u], v, e));
        }
      }
      return row16_sum(c) + (v == v ? 0 : kNaNRank);
    }
  };

  // This token's restricted routing.  Eq. (7) keeps the natural top-k slots that fall inside S with their weights
  // unchanged; Eq. (8) takes the top-k inside S and weights over that selection.  A candidate's rank is the number
  // of candidates that go before it; rank r < k fills slot r.  A NaN claims slot 0 (nan_claim), decided when all candidates are through.
  if (own >= 0) {
    for (int x0 = 0; x0 + group0 < n_cand; x0 += kGroups) {
      const int x = x0 + group, j = x >= n_cand ? -1 : truncate ? x : cand[x];
      const int c = rank_among(min(own, M - 1), max(j, 0));
      if (seg == 0 && j >= 0) {
        if (c < k) sel[c] = j;
        else if (c >= kNaNRank) atomicMin(&sel[k], nan_key(j, inS[j] != 0));
      }
    }
  }
  auto token_write = [&]() {
    if (tid < k && own < M) {
      const int32_t nan = sel[k];
      const int e = tid == 0 && nan != kNoNaN ? nan_key_id(nan) : sel[tid];
      const bool keep = e >= 0 && inS[e] != 0;  // an unfilled slot is dropped
      const double ge = e >= 0 ? (kRanked ? probs[(size_t)own * N + e] : g[own * NS + e]) : 0.0;
      double denom = 0.0;  // over the selected set in slot order (before any slot is dropped: Eq. (7)); k <= 64: one wave
      for (int sl = 0; sl < k; ++sl)
        denom += __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(ge), sl),
                                  __builtin_amdgcn_readlane(__double2loint(ge), sl));
      const double w = keep ? (flags & kRenorm ? ge / denom : ge) : 0.0;
      tok_ids[(size_t)own * k + tid] = keep ? e : -1;
      tok_w[(size_t)own * k + tid] = (float)w;
    }
  };
  bool token_done = own < 0;

  // Pair lists of this workgroup's shortlist ranks: token t is routed to expert e = S[r] iff e ranks among the
  // first k of t's candidates; its rank is the slot.  A wave takes 4 tokens per round, one behind the other, and its
  // routed tokens are compacted with one ballot per round; the waves' counts are exchanged once per list.
  constexpr int kMaxRounds = (kFusedMaxTokens + kGroups - 1) / kGroups;
  const int rounds = (M + kGroups - 1) / kGroups;
  int parity = 0;
  for (int r = list_wgs && own >= 0 ? B : (int)blockIdx.x; r < B; r += list_step, parity ^= 1) {
    const int e = S[r];
    const bool real = (uint32_t)e < (uint32_t)N && pos[e] == r;  // not a repeat, not out of range
    const int wave_t0 = wave * kWaveGroups * rounds;
    int c[kMaxRounds], n_wave = 0;
    unsigned long long mask[kMaxRounds];
#pragma unroll
    for (int rd = 0; rd < kMaxRounds; ++rd) {
      mask[rd] = 0;
      c[rd] = 0;
      const int t0 = wave_t0 + rd * kWaveGroups;
      if (rd < rounds && t0 < M) {  // uniform in the wave
        const int t = t0 + (lane >> 4);
        c[rd] = rank_among(min(t, M - 1), real ? e : 0);
        mask[rd] = __ballot(real & (t < M) & (seg == 0) & (c[rd] < k));  // NaN ranks nowhere
        n_wave += __popcll(mask[rd]);
      }
    }
    if (lane == 0) count[parity * kWaves + wave] = n_wave;
    __syncthreads();  // the counts, and the selection of the token
    if (!token_done) token_write();
    token_done = true;
    int at = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const int cw = count[parity * kWaves + w];
      at += w < wave ? cw : 0;
      total += cw;
    }
#pragma unroll
    for (int rd = 0; rd < kMaxRounds; ++rd) {
      if ((mask[rd] >> lane) & 1)
        lists[(size_t)r * list_stride + at + __popcll(mask[rd] & ((1ull << lane) - 1ull))] =
            (wave_t0 + rd * kWaveGroups + (lane >> 4)) * k + c[rd];
      at += __popcll(mask[rd]);
    }
    if (tid == 0) list_count[r] = total;
  }
  if (!token_done) {  // a workgroup without a pair list
    __syncthreads();
    token_write();
  }
}

// seg_expert / seg_off / perm / n_loaded from the pair lists (only when a caller asks for those arrays):
// segments in ascending expert id, each list copied in order.  One workgroup; N <= 256.
__global__ __launch_bounds__(256) void lists_to_segments_kernel(const int32_t *__restrict__ budget_ids,
                                                                const int32_t *__restrict__ list_count,
                                                                const int32_t *__restrict__ lists, int list_stride,
                                                                int B, int N, int n_pairs,
                                                                int32_t *__restrict__ seg_off,
                                                                int32_t *__restrict__ perm,
                                                                int32_t *__restrict__ n_loaded) {
  __shared__ int32_t rank_of[kSelfMaxExperts];  // expert -> first shortlist rank, or -1
  __shared__ int32_t seg_rank[kSelfMaxExperts];  // segment (ascending expert id) -> shortlist rank
  __shared__ int32_t off[kSelfMaxExperts + 1];
  __shared__ int32_t n_member;
  const int tid = threadIdx.x;
  for (int i = tid; i < N; i += blockDim.x) rank_of[i] = 0x7fffffff;
  __syncthreads();
  for (int r = tid; r < B; r += blockDim.x)
    if ((uint32_t)budget_ids[r] < (uint32_t)N) atomicMin(&rank_of[budget_ids[r]], r);
  __syncthreads();
  for (int i = tid; i < N; i += blockDim.x)
    if (rank_of[i] != 0x7fffffff) {
      int at = 0;
      for (int j = 0; j < i; ++j) at += rank_of[j] != 0x7fffffff;
      seg_rank[at] = rank_of[i];
    }
  if (tid == 0) {
    int n = 0;
    for (int j = 0; j < N; ++j) n += rank_of[j] != 0x7fffffff;
    n_member = n;
  }
  __syncthreads();
  if (tid == 0) {
    int run = 0, loaded = 0;
    for (int sg = 0; sg < B; ++sg) {
      off[sg] = run;
      const int c = sg < n_member ? list_count[seg_rank[sg]] : 0;
      run += c;
      loaded += c > 0;
    }
    off[B] = run;
    if (n_loaded) *n_loaded = loaded;
  }
  __syncthreads();
  if (seg_off)
    for (int sg = tid; sg <= B; sg += blockDim.x) seg_off[sg] = off[sg];
  if (perm) {
    for (int sg = 0; sg < n_member; ++sg) {
      const int r = seg_rank[sg], c = off[sg + 1] - off[sg];
      for (int p = tid; p < c; p += blockDim.x) perm[off[sg] + p] = lists[(size_t)r * list_stride + p];
    }
    for (int p = off[B] + tid; p < n_pairs; p += blockDim.x) perm[p] = -1;
  }
}

// The fused prologue covers layers with at most kSelfMaxExperts experts (one thread per shortlist rank in the expert passes) and at
// most one token per compute unit.  With more tokens the workgroups, each of which loads the whole table and ranks its experts
// again, come in rounds, while the staged kernels grow with the tokens alone.  Whole fp32 layer of 4 experts, us, fused
// less staged: 128 tokens -4, 160 -2, 200 to 256 +1, 300 +2, 400 +5, 512 +16, 1024 +68; of 64 experts, top-8: 128 -5, 256 -5,
// 300 0; bf16 within 4 up to 256.
// Tables that as doubles would not leave the LDS room for other work (above 151 KB; the ranks do) have more than 18500 entries, and
// there the fused form pays only in part (90 x 208, d = 1120, 183 shortlisted 45.1 us staged, 47.7 fused).  Its prologue saves 4 to 8
// us up to 128 experts; with more the last kernel, where every workgroup loads all ranks and, under substitution, ranks an expert
// against the whole shortlist, takes that back: -4 us at 57000 entries.  And its expert passes look up their item in the lists: 1.15
// us per 1000 workgroups of bf16 passes (8192 x 32, 256 experts, 90 tokens, down pass 80 / 117 us).  Line by layers of 60 to 256 tokens
// and 80 to 256 experts, either policy, budgets of 1/16 to all: over 379 bf16 layers the side taken is 0.2 % slower than the better
// one on average, 5 % at most; staged alone is 3.1 % (24 %), fused alone 3.2 % (36 %).  fp32 segments of more than 128 tokens are cut
// in pieces by the staged kernels only, and where routing concentrates that decides: 5385 drawn layers of 129 to 256 tokens against
// the kernels before the fused form reached them, fused 1.141x (0.77x at worst, 127 slower by more than 5 %; top-1 1.09x), staged
// 1.147x (0.91x, 1; top-1 1.11x).
static bool fused_beyond_lds(const moespec_desc &ds, int M, int B, int policy) {
  const int N = ds.n_experts;
  if (ds.dtype == MOESPEC_F32 && M > kPiecePairs) return false;
  const long long pass_wgs = (long long)B * ((ds.d_ff + 63) / 64 + (ds.d + 127) / 128);
  if (N <= 128) return pass_wgs <= 4000;
  return pass_wgs <= 3000 && (policy == MOESPEC_TRUNCATE ? M * N <= 36000 : M * N <= 32000 && M * B <= 12000);
}
bool fused_prologue_ok(const moespec_desc &ds, int M, int B, int policy) {
  const int N = ds.n_experts;
  if (N > kSelfMaxExperts || M > kFusedMaxTokens) return false;
  const bool ranked = (long long)M * N > kSplitSoftmaxAbove;
  // the ranks lie in the place of y: [kMaxDownSplits][M k, d] floats
  if (ranked && sizeof(uint16_t) * rank_row(N) > sizeof(float) * kMaxDownSplits * ds.top_k * ds.d) return false;
  if (ranked && prologue_lds(M, N, ds.top_k, N, false).total > 151 * 1024 && !fused_beyond_lds(ds, M, B, policy)) return false;
  return prologue_lds(M, N, ds.top_k, N, ranked).total <= 160 * 1024;
}

// Tiles of 32 tokens x 32 experts (16 for up to 16 experts) where they and the slices make a workgroup per compute unit, leave every
// wave four blocks of the hidden dimension, and do not spend on padding what they save, which is 5 to 10 % (3000 tokens x 100 experts,
// 128 columns of tiles instead of 112: 0.93 of the speed).  One such workgroup is resident per compute unit, so that they come in whole
// rounds, in each of which a compute unit is through with 4 (2) of the 16 x 16 tiles: not where those alone would give none of the
// compute units as many (1165 tokens x 218 experts, d = 3296, 259 workgroups 62 us, 16 x 16 tiles 39), nor in several rounds of fewer
// than six blocks per wave, which start up each time.  3133 projections of 400 to 16384 tokens against 16 x 16 tiles alone: 1.03x, 6 of
// them slower by more than 3 % (0.94x); wherever they and the slices made 256 workgroups it was 0.96x (0.64x at least).  In two
// slices the others are the less even ones (0.75 and 0.87), but where one slice makes a workgroup per compute unit two were 0.92x.
static int block_experts(const moespec_desc &ds) { return ds.n_experts > 16 ? 2 : 1; }
static bool logits_in_blocks(const moespec_desc &ds, int M, int slices) {
  const int N = ds.n_experts, te = block_experts(ds), rows = 16 * te;
  const long long tiles = (long long)((M + 31) / 32) * ((N + rows - 1) / rows), plain = (long long)((M + 15) / 16) * ((N + 15) / 16);
  const long long rounds = (tiles * slices + 255) / 256, most_plain = (plain * slices + 255) / 256;  // per compute unit
  if (ds.dtype != MOESPEC_BF16 || tiles * slices < 256 || (slices > 1 && tiles >= 256)) return false;
  return ds.d / 32 >= (rounds > 1 ? 6 : 4) * kBlockWaves * slices &&
         tiles * 2 * te * 95 <= plain * 100 && rounds * 2 * te * (slices == 1 ? 95 : te == 1 ? 75 : 87) <= most_plain * 100;
}

// Slices of the hidden dimension (1, 2, 4 or 8, at most `most`): more slices spread the matrix work over more compute units
// (a wave issues one fp64 matrix instruction per 64 cycles), but the row-wise gate kernel re-reads its row once per slice.
// Picks the count with the smallest estimated sum of the two (rates measured on MI355X: 2.4 GHz, about 150 GB/s
// from L2 into one compute unit).
int logit_slices(const moespec_desc &ds, int M, int most) {
  const double tiles = ((M + 15) / 16) * ((ds.n_experts + 15) / 16), n_blocks = ds.d / 32;
  for (int q = 1; q <= 2 && q <= most; q *= 2)
    if (logits_in_blocks(ds, M, q)) return q;
  int best = 1;
  double best_us = 1e30;
  for (int q = 1; q <= kMaxLogitSlices && (q == 1 || q <= most); q *= 2) {
    if (q > 1 && n_blocks < 2.0 * q * kLogitWaves) break;  // at least two 32-element blocks per wave
    const double waves_per_simd = tiles * q * kLogitWaves / 1024.0;  // 256 compute units x 4 SIMDs
    const double mfma_us = (n_blocks / (q * kLogitWaves)) * 8 * 64 / 2400.0 * (waves_per_simd > 1 ? waves_per_simd : 1);
    const double read_us = q * 8.0 * ds.n_experts / 150e3;
    if (mfma_us + read_us < best_us) {
      best_us = mfma_us + read_us;
      best = q;
    }
  }
  return best;
}

// Whether Eq. (1) runs on the matrix cores and row by row (layers of up to kSelfMaxExperts experts, any tree).
bool mfma_route_ok(const moespec_desc &ds) { return ds.n_experts <= kSelfMaxExperts; }

hipError_t launch_logits(const moespec_desc &ds, const moespec_weights &wt, const void *h, int M, int slices,
                         double *partial, hipStream_t st) {
  if (logits_in_blocks(ds, M, slices)) {
    const int te = block_experts(ds);
    const dim3 bgrid(((M + 31) / 32) * ((ds.n_experts + 16 * te - 1) / (16 * te)), slices);
    auto kern = te == 2 ? logits_block_kernel<uint16_t, 2> : logits_block_kernel<uint16_t, 1>;
    kern<<<bgrid, kBlockWaves * kWave, 0, st>>>(static_cast<const uint16_t *>(h), static_cast<const uint16_t *>(wt.w_router), M,
                                                ds.n_experts, ds.d, slices, partial);
    return hipGetLastError();
  }
  dim3 grid(((M + 15) / 16) * ((ds.n_experts + 15) / 16), slices);
  // Loads ahead, except in bf16 (sets of four blocks) for five blocks per wave, where most of the second set repeats the last
  // block, and for up to eight in more workgroups than the registers of two sets leave resident.  Measured inside layers whose
  // weights pass through the caches in between (replayed by itself, with its operands in the L2, the kernel gains nothing at eight
  // blocks).  Without / with, bf16: 5 blocks 0.90 to 0.98; 6 to 8 1.02 to 1.13 at up to 456 workgroups (one 0.95), 0.98 to
  // 1.01 at 648, 0.97 to 0.98 above; 9 and more 1.03 to 1.18, also at 1024; up to 4 1.01 to 1.06 on average.  (511 tokens x 64 experts,
  // d = 2048: 7.1 -> 6.2 us; 1500 x 64, d = 640: 6.7 -> 7.5.)  fp32 (sets of two): 1.00 to 1.27, 0.96 to 0.98 at 7 and 8 blocks from 648
  // workgroups on.
  const int n_blocks = ds.d / 32, parts = kLogitWaves * slices;
  const bool plain = n_blocks > 4 * parts && (n_blocks <= 5 * parts || (n_blocks <= 8 * parts && (long long)grid.x * slices > 700));
  if (ds.dtype != MOESPEC_BF16)
    logits_mfma_kernel<float, true><<<grid, kLogitWaves * kWave, 0, st>>>(static_cast<const float *>(h), static_cast<const float *>(wt.w_router),
                                                                    M, ds.n_experts, ds.d, slices, partial);
  else
    (plain ? logits_mfma_kernel<uint16_t, false> : logits_mfma_kernel<uint16_t, true>)
        <<<grid, kLogitWaves * kWave, 0, st>>>(static_cast<const uint16_t *>(h), static_cast<const uint16_t *>(wt.w_router), M,
                                               ds.n_experts, ds.d, slices, partial);
  return hipGetLastError();
}

hipError_t launch_fused_prologue(const moespec_desc &ds, const moespec_weights &wt, const void *h, int M, int B,
                                 int policy, const int32_t *ext_shortlist, double *partial, double *parts, void *ranks_ws, double *probs_ws,
                                 double *probs_out, double *scores_out, int32_t *budget_ids, int32_t *seg_expert, int32_t *tok_ids,
                                 float *tok_w, int32_t *list_count, int32_t *lists, int list_stride,
                                 int32_t *seg_off, int32_t *perm, int32_t *n_loaded, hipStream_t st) {
  const int N = ds.n_experts, k = ds.top_k;
  // Large tables: the routing probabilities are finished row by row in a launch of their own and the last kernel
  // only loads them; small tables: every workgroup of the last kernel rebuilds the table itself.
  const bool split = (long long)M * N > kSplitSoftmaxAbove;
  const size_t smem = prologue_lds(M, N, k, B, split).total;
  const int flags = (ds.gate == MOESPEC_GATE_SIGMOID ? kSigmoidGate : 0) |
                    (policy == MOESPEC_TRUNCATE ? kTruncate : 0) | (ds.renorm ? kRenorm : 0);
  double *probs = nullptr;
  uint16_t *ranks = static_cast<uint16_t *>(ranks_ws);
  hipError_t e;
  if (split) {
    const int q = logit_slices(ds, M, kMaxLogitSlices);
    if ((e = launch_logits(ds, wt, h, M, q, partial, st)) != hipSuccess) return e;
    probs = probs_out ? probs_out : probs_ws;
    const int n_parts = (M + kPartTokens - 1) / kPartTokens;
    auto rank = [&](auto kern) {
      kern<<<M + n_parts, kRankThreads, 0, st>>>(partial, wt.b_router, M, N, n_parts, flags & kSigmoidGate, probs, parts, ranks);
      return hipGetLastError();
    };
#define MOESPEC_RANK(Q) \
  (N <= 64 ? rank(rank_rows_kernel<Q, 1>) : N <= 128 ? rank(rank_rows_kernel<Q, 2>) : rank(rank_rows_kernel<Q, 4>))
    e = q == 1 ? MOESPEC_RANK(1) : q == 2 ? MOESPEC_RANK(2) : q == 4 ? MOESPEC_RANK(4) : MOESPEC_RANK(8);
#undef MOESPEC_RANK
    if (e != hipSuccess) return e;
  } else {
    const int tiles = ((M + 3) / 4) * ((N + 3) / 4);
    if (ds.dtype == MOESPEC_BF16)
      logits_table_kernel<uint16_t><<<tiles, kTableWaves * kWave, 0, st>>>(
          static_cast<const uint16_t *>(h), static_cast<const uint16_t *>(wt.w_router), wt.b_router, M, N, ds.d, partial);
    else
      logits_table_kernel<float><<<tiles, kTableWaves * kWave, 0, st>>>(
          static_cast<const float *>(h), static_cast<const float *>(wt.w_router), wt.b_router, M, N, ds.d, partial);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  // instantiation for the elements of a table row per lane: ceil(N / 16) rounded up to a power of two
  auto run = [&](auto kern) -> hipError_t {
    if (smem > 64 * 1024) {  // beyond the default limit of a launch
      hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
      if (err != hipSuccess) return err;
    }
    // a workgroup per token, and at least one per shortlist rank: pair lists built one after the other by the same
    // workgroup cost 0.8 us each (7 tokens, 16 ranks: 11.9 -> 10.3 us).  Where the compute units suffice, the tokens and the
    // lists have workgroups of their own (15 tokens x 8 experts 6.8 -> 6.4 us, 7 x 64 10.3 -> 8.6, 63 x 64 10.5 -> 9.7, 127 x 128 12.3
    // -> 11.7); each loads the whole table, so not in a second round.
    const int list_wgs = M + B <= 256 ? B : 0;
    kern<<<list_wgs ? M + B : (M > B ? M : B), kPrologueThreads, smem, st>>>(
        split ? static_cast<const void *>(ranks) : partial, M, N, k, B, list_wgs, flags, list_stride, ext_shortlist, parts, probs,
        probs_out, scores_out, budget_ids, seg_expert, tok_ids, tok_w, list_count, lists);
    return hipGetLastError();
  };
  const int ne = (N + 15) / 16;
  e = split     ? run(route_budget_kernel<0>)
      : ne <= 1 ? run(route_budget_kernel<1>)
      : ne <= 2 ? run(route_budget_kernel<2>)
      : ne <= 4 ? run(route_budget_kernel<4>)
      : ne <= 8 ? run(route_budget_kernel<8>)
                : run(route_budget_kernel<16>);
  if (e != hipSuccess) return e;
  if (seg_off || perm || n_loaded) {
    lists_to_segments_kernel<<<1, 256, 0, st>>>(budget_ids, list_count, lists, list_stride, B, N, M * k, seg_off, perm,
                                                n_loaded);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace moespec
