// Stages 2-3 of Algorithm 1 without the expert maths: per-expert aggregation of routing
// probability over the tree (Eq. (5)), top-B shortlist (Section 3.2), restriction of every token's
// routing by truncation (Eq. (7)) or substitution (Eq. (8)), and the grouping of the surviving
// (token, slot) pairs into per-expert segments.  All decisions in fp64, ties to the lowest id.
//
// Three launches, none of which has a workgroup that does the whole tree's work by itself:
//   score_parts_kernel   column sums of blocks of rows (large trees, unless the gate kernel has made them; the others add the
//                        rows in the next launch)
//   budget_kernel        one WAVE per token: every workgroup adds the partial sums and ranks the experts itself
//                        (many experts: one WORKGROUP per token, budget_many_kernel)
//   group_pairs_kernel   one workgroup per shortlisted expert: its pairs, its offset, its work items
#include "common.h"

namespace moespec {

// Up to this many tokens every workgroup of the budget kernel adds the rows of the table itself: one round of loads at 128
// tokens and up to 256 experts, two at 256 tokens and up to 128 experts, where a second round still costs less than a launch
// (whole stage, us, rows / row blocks first: 256 tokens x 8 experts 9.8 / 12.3, x 64 13.9 / 14.8, x 128 19.0 / 18.8, but
// x 256 22.6 / 20.1, x 300 27.9 / 22.5).  Above, the row blocks are summed once by a launch of its own (4.8 us at 511 and at
// 2048 tokens).
inline int direct_score_rows(int N) { return N <= 2 * kWave ? 256 : 128; }
constexpr int kScoreLoads = 32;  // rows in flight per thread of those sums

// part[b, i] = sum of probs[t, i] over the rows t of block b, ascending.  Wave w of a workgroup adds the rows w, w + 16,
// ... of the block, and thread i the 16 results in wave order.  N <= 1024.
__global__ __launch_bounds__(kScoreThreads) void score_parts_kernel(const double *__restrict__ probs, int M, int N,
                                                                    int rows, double *__restrict__ part) {
  extern __shared__ __align__(16) unsigned char smem[];
  double *tab = reinterpret_cast<double *>(smem);  // [16][N]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t0 = blockIdx.x * rows, t1 = min(M, t0 + rows);
  for (int i = lane; i < N; i += kWave) {
    double a = 0.0;
    for (int t = t0 + wave; t < t1; t += 4 * kScoreWaves) {
      double v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = t + u * kScoreWaves < t1 ? probs[(size_t)(t + u * kScoreWaves) * N + i] : 0.0;
#pragma unroll
      for (int u = 0; u < 4; ++u) a += v[u];  // rows past the end add +0.0, which leaves the sum unchanged
    }
    tab[wave * N + i] = a;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < N; i += kScoreThreads) {
    double a = tab[i];
    for (int w = 1; w < kScoreWaves; ++w) a += tab[w * N + i];
    part[(size_t)blockIdx.x * N + i] = a;
  }
}

// Threads of a budget_kernel workgroup: four tokens at a time, and more where the scores and the ranking of more
// experts, which every workgroup repeats, need the threads (at most kScoreLoads rows per thread at 128 tokens and up to 256 experts).
inline int budget_threads(int N) { return N <= 64 ? 256 : N <= 128 ? 512 : 1024; }

constexpr int kMaxBudgetGroups = 512;

struct BudgetLds {
  size_t s, red, rows, row_stride, S, rank, sel, inS, total;
};
// tokens: how many the workgroup has at a time
__host__ __device__ inline BudgetLds budget_lds(int N, int B, int threads, int tokens) {
  BudgetLds L;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off += (bytes + 15) & ~(size_t)15;
    return at;
  };
  L.row_stride = (size_t)((N + 3) & ~3);
  L.s = take(sizeof(double) * L.row_stride);
  L.red = take(sizeof(double) * threads);
  L.rows = take(sizeof(double) * L.row_stride * tokens);
  L.S = take(sizeof(int32_t) * B);
  L.rank = take(sizeof(int32_t) * N);
  L.sel = take(sizeof(int32_t) * kWave * tokens);
  L.inS = take((size_t)N);
  L.total = off;
  return L;
}

// s[i] = sum of column i of src [n_src, N] as it ranks, i < N <= nt; kNoRival up to row_stride.  scores (may be NULL) receives the
// sums.  The threads with the same index modulo a power of two >= N share a column, each a contiguous run of rows.  Called by
// the whole workgroup (it synchronises once; the caller does before it reads s).
__device__ __forceinline__ void tree_scores(const double *__restrict__ src, int n_src, int N, int row_stride, double *red,
                                            double *s, double *__restrict__ scores) {
  const int nt = blockDim.x, tid = threadIdx.x;
  int np2 = 1, np2_log = 0;
  while (np2 < N) np2 <<= 1, ++np2_log;
  const int parts = nt >> np2_log > 0 ? nt >> np2_log : 1, per = (n_src + parts - 1) / parts;
  const int i = tid & (np2 - 1), p = tid >> np2_log;
  double a = 0.0;
  if (i < N) {
    const int r1 = min(n_src, (p + 1) * per);
    for (int r = p * per; r < r1; r += kScoreLoads) {  // the loads of a block go out together: one memory latency
      double x[kScoreLoads];
#pragma unroll
      for (int u = 0; u < kScoreLoads; ++u) x[u] = r + u < r1 ? src[(size_t)(r + u) * N + i] : 0.0;
#pragma unroll
      for (int u = 0; u < kScoreLoads; ++u) a += x[u];
    }
  }
  red[tid] = a;
  __syncthreads();
  if (tid < row_stride) {
    double sum = tid < N ? red[tid] : kNoRival;
    for (int q = 1; tid < N && q < parts; ++q) sum += red[q * np2 + tid];
    s[tid] = tid < N ? ranking_score(sum) : sum;
    if (scores && tid < N) scores[tid] = sum;
  }
}

// The copies of one workgroup for the caller: the shortlist in rank order and in ascending id.  Every wave builds
// the membership mask of all experts, 64 at a time; the position of an expert among the shortlisted ones is a population
// count.
__device__ __forceinline__ void publish_shortlist(int N, int B, const uint8_t *inS, const int32_t *S,
                                                  int32_t *__restrict__ seg_expert, int32_t *__restrict__ budget_ids) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int n_member = 0;  // in the end < B only if an external shortlist repeats or misnames an expert
  for (int i0 = 0; i0 < N; i0 += kWave) {
    const int i = i0 + lane;
    const bool in = i < N && inS[i] != 0;
    const unsigned long long mask = __ballot(in);
    if (wave == 0 && in) seg_expert[n_member + __popcll(mask & ((1ull << lane) - 1ull))] = i;
    n_member += __popcll(mask);
  }
  for (int r = tid; r < B; r += blockDim.x) {
    if (r >= n_member) seg_expert[r] = -1;
    budget_ids[r] = S[r];
  }
}

// One wave per tree token.  src holds n_src rows of N values whose column sums are the scores of Eq. (5): the
// probabilities themselves or the sums of row blocks.  Every workgroup recomputes the (tiny) scores and shortlist so
// that no grid-wide synchronisation is needed; workgroup 0 also writes them out.  NU = candidates per lane.
// A token's selection is a rank count: lane i compares its candidates with the whole row, read from LDS four values at
// a time (the same address in every lane: a broadcast).  k <= 64, N <= 64 NU, NU <= 4.
// What bounds it: the launch, two rounds of cold loads and the row's N / 4 LDS reads; the tokens are independent.
// The kernel it replaces had one workgroup per token, whose last one to finish grouped the pairs of the whole tree
// (MI355X: 973 us with the sum of the scores at 2048 tokens x 64 experts, 32 us at 127 x 128, 17 us at 63 x 64; the
// three kernels here take 22, 17 and 13 us).
template <int NU>
__global__ __launch_bounds__(1024) void budget_kernel(
    const double *__restrict__ probs, const double *__restrict__ src, int n_src, int M, int N, int k, int B, int policy,
    int renorm, const int32_t *__restrict__ ext_shortlist, double *__restrict__ scores,
    int32_t *__restrict__ budget_ids, int32_t *__restrict__ seg_expert, int32_t *__restrict__ tok_ids,
    float *__restrict__ tok_w) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int nt = blockDim.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const BudgetLds L = budget_lds(N, B, nt, nt / kWave);
  double *s = reinterpret_cast<double *>(smem + L.s);      // [N] aggregate scores
  double *red = reinterpret_cast<double *>(smem + L.red);  // [threads] partial column sums
  double *row = reinterpret_cast<double *>(smem + L.rows) + wave * L.row_stride;  // this wave's token
  int32_t *S = reinterpret_cast<int32_t *>(smem + L.S);    // [B] shortlist in rank order
  int32_t *rank = reinterpret_cast<int32_t *>(smem + L.rank);
  int32_t *sel = reinterpret_cast<int32_t *>(smem + L.sel) + wave * kWave;  // [k] this wave's selection
  uint8_t *inS = smem + L.inS;

  // the first token's row is requested before the shortlist is known
  const int n_waves = gridDim.x * (nt / kWave);
  int t = blockIdx.x * (nt / kWave) + wave;
  double v[NU];
  auto load_row = [&](int tok) {
#pragma unroll
    for (int u = 0; u < NU; ++u) v[u] = (tok < M && lane + kWave * u < N) ? probs[(size_t)tok * N + lane + kWave * u] : 0.0;
  };
  load_row(t);

  for (int i = tid; i < N; i += nt) inS[i] = 0;
  if (ext_shortlist == nullptr || scores != nullptr) {
    tree_scores(src, n_src, N, (int)L.row_stride, red, s, blockIdx.x == 0 ? scores : nullptr);
  }
  for (int i = tid; i < N; i += nt) rank[i] = 0;
  __syncthreads();
  if (ext_shortlist == nullptr) {
    // Section 3.2: the B highest aggregate scores, ties to the lowest id.  Each wave ranks all experts against its share
    // of the rivals; the shares add up through integer LDS atomics.
    double sv[NU];
    int c[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      c[u] = 0;
      sv[u] = lane + kWave * u < N ? s[lane + kWave * u] : 0.0;
    }
    const int quads = (int)L.row_stride / 4, n_w = nt / kWave;
    rank_counts<NU>(s, quads * wave / n_w * 4, quads * (wave + 1) / n_w * 4, lane, 0, sv, c);
#pragma unroll
    for (int u = 0; u < NU; ++u)
      if (lane + kWave * u < N && c[u]) atomicAdd(&rank[lane + kWave * u], c[u]);
    __syncthreads();
    for (int i = tid; i < N; i += nt)
      if (rank[i] < B) S[rank[i]] = i;
  } else {
    for (int r = tid; r < B; r += nt) S[r] = ext_shortlist[r];
  }
  __syncthreads();
  for (int r = tid; r < B; r += nt)
    if ((uint32_t)S[r] < (uint32_t)N) inS[S[r]] = 1;  // ids outside [0, N) in an external shortlist are ignored
  __syncthreads();

  if (blockIdx.x == 0) {
    publish_shortlist(N, B, inS, S, seg_expert, budget_ids);
  }

  const bool truncate = policy == MOESPEC_TRUNCATE;
  bool member[NU];  // candidates: every expert under truncation, the shortlist under substitution
#pragma unroll
  for (int u = 0; u < NU; ++u) member[u] = lane + kWave * u < N && (truncate || inS[lane + kWave * u] != 0);
  for (; t < M; t += n_waves) {
    wave_lds_sync();  // the previous token's reads are done
#pragma unroll
    for (int u = 0; u < NU; ++u)
      if (lane + kWave * u < (int)L.row_stride) row[lane + kWave * u] = member[u] ? v[u] : kNoRival;
    sel[lane] = -1;  // stays -1 where an external shortlist names fewer than k experts or NaN values leave a slot unclaimed
    wave_lds_sync();
    int c[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) c[u] = 0;
    rank_counts<NU>(row, 0, N, lane, 0, v, c);
#pragma unroll
    for (int u = 0; u < NU; ++u)
      if (member[u] & (c[u] < k) & (v[u] == v[u])) sel[c[u]] = lane + kWave * u;
    const int nan = nan_claim<NU>(v, member, inS);
    wave_lds_sync();
    // weights over the selected set in slot order, before any slot is dropped (Eq. (7)); truncation drops the slots outside S, kept
    // weights are unchanged
    const int e = lane == 0 && nan >= 0 ? nan : sel[lane];
    const double ge = lane < k && e >= 0 ? row[e] : 0.0, denom = renorm ? slot_sum(ge, k) : 1.0;
    if (lane < k) {
      const bool keep = e >= 0 && inS[e] != 0;
      tok_ids[(size_t)t * k + lane] = keep ? e : -1;
      tok_w[(size_t)t * k + lane] = (float)(keep ? (renorm ? ge / denom : ge) : 0.0);
    }
    load_row(t + n_waves);
  }
}

// Many experts (N <= 1024 = blockDim.x): one workgroup per token.  A wave counts one block of 64 candidates
// against its share of the rivals, and the shares add up through integer LDS atomics, for the shortlist as for a token.
// Bound by the N^2 / 1024 comparisons per thread, once for the shortlist and once per token.  One wave per token, as above,
// would hold 16 candidates per lane for 1024 experts: its registers spill, and the stage took 405 us for 63 tokens x 300
// experts (680 for 512) against 20 us (25) this way.
__device__ __forceinline__ void rank_in_workgroup(const double *row, int N, int32_t *rank) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int blocks = (N + kWave - 1) / kWave, parts = (int)(blockDim.x >> 6) / blocks;
  const int block = wave % blocks, part = wave / blocks, quads = (N + 3) / 4, i = block * kWave + lane;
  if (part >= parts) return;
  const double v[1] = {i < N ? row[i] : 0.0};
  int c[1] = {0};
  rank_counts<1>(row, quads * part / parts * 4, quads * (part + 1) / parts * 4, lane, block, v, c);
  if (i < N && c[0]) atomicAdd(&rank[i], c[0]);
}

__global__ __launch_bounds__(1024) void budget_many_kernel(
    const double *__restrict__ probs, const double *__restrict__ src, int n_src, int M, int N, int k, int B, int policy,
    int renorm, const int32_t *__restrict__ ext_shortlist, double *__restrict__ scores,
    int32_t *__restrict__ budget_ids, int32_t *__restrict__ seg_expert, int32_t *__restrict__ tok_ids,
    float *__restrict__ tok_w) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int32_t nan;  // nan_key of the NaN that claims slot 0
  const int nt = blockDim.x, tid = threadIdx.x;
  const BudgetLds L = budget_lds(N, B, nt, 1);
  double *s = reinterpret_cast<double *>(smem + L.s);
  double *red = reinterpret_cast<double *>(smem + L.red);
  double *row = reinterpret_cast<double *>(smem + L.rows);
  int32_t *S = reinterpret_cast<int32_t *>(smem + L.S);
  int32_t *rank = reinterpret_cast<int32_t *>(smem + L.rank);
  int32_t *sel = reinterpret_cast<int32_t *>(smem + L.sel);
  uint8_t *inS = smem + L.inS;

  int t = blockIdx.x;
  double v = tid < N ? probs[(size_t)t * N + tid] : 0.0;  // grid <= M; requested before the shortlist is known
  for (int i = tid; i < N; i += nt) {
    inS[i] = 0;
    rank[i] = 0;
  }
  if (ext_shortlist == nullptr || scores != nullptr)
    tree_scores(src, n_src, N, (int)L.row_stride, red, s, blockIdx.x == 0 ? scores : nullptr);
  __syncthreads();
  if (ext_shortlist == nullptr) {
    rank_in_workgroup(s, N, rank);
    __syncthreads();
    if (tid < N && rank[tid] < B) S[rank[tid]] = tid;
  } else {
    for (int r = tid; r < B; r += nt) S[r] = ext_shortlist[r];
  }
  __syncthreads();
  for (int r = tid; r < B; r += nt)
    if ((uint32_t)S[r] < (uint32_t)N) inS[S[r]] = 1;
  __syncthreads();
  if (blockIdx.x == 0) publish_shortlist(N, B, inS, S, seg_expert, budget_ids);

  const bool truncate = policy == MOESPEC_TRUNCATE, member = tid < N && (truncate || inS[tid] != 0);
  for (; t < M; t += gridDim.x) {
    if (tid < (int)L.row_stride) row[tid] = member ? v : kNoRival;
    if (tid < N) rank[tid] = 0;
    if (tid < kWave) sel[tid] = -1;
    if (tid == 0) nan = kNoNaN;
    __syncthreads();
    rank_in_workgroup(row, N, rank);
    __syncthreads();
    if (member) {
      if (v != v) atomicMin(&nan, nan_key(tid, inS[tid] != 0));
      else if (rank[tid] < k) sel[rank[tid]] = tid;
    }
    __syncthreads();
    if (tid < kWave) {
      const int e = tid == 0 && nan != kNoNaN ? nan_key_id(nan) : sel[tid];
      const double ge = tid < k && e >= 0 ? row[e] : 0.0, denom = renorm ? slot_sum(ge, k) : 1.0;  // as in budget_kernel
      if (tid < k) {
        const bool keep = e >= 0 && inS[e] != 0;
        tok_ids[(size_t)t * k + tid] = keep ? e : -1;
        tok_w[(size_t)t * k + tid] = (float)(keep ? (renorm ? ge / denom : ge) : 0.0);
      }
    }
    if (tid < N && t + (int)gridDim.x < M) v = probs[(size_t)(t + gridDim.x) * N + tid];
    __syncthreads();  // the row and the selection have been read
  }
}

// Groups the surviving (token, slot) pairs by expert: segment i = blockIdx.x holds the pairs routed to seg_expert[i],
// tokens ascending.  Every workgroup counts the pairs of ALL experts itself (integer LDS atomics: order-independent),
// which gives it its own offset and rank without any exchange, then collects its own pairs 64 tokens per ballot.
// items receives the work items of the expert passes: the non-empty segments ordered by size, largest first (ties:
// lower segment first), each cut into piece_count(size) pieces of (almost) equal size; items[0].x = number of pieces,
// items[1 + r] = (segment, expert, offset, size) of piece r - the order in which the expert passes hand them out.
// kHeld: a thread holds the ids of its token (at most kHeldSlots, one token per thread) from the count to the collection, which
// otherwise loads them again: 63 tokens, top-8 of 64 experts 4.7 -> 3.9 us.  Not in workgroups of 1024 threads, whose registers
// it takes (511 tokens 5.4 us, held 7.0).
constexpr int kHeldSlots = 8;
template <bool kHeld>
__global__ __launch_bounds__(1024) void group_pairs_kernel(const int32_t *__restrict__ tok_ids, int M, int N, int k,
                                                           int B, const int32_t *__restrict__ seg_expert,
                                                           int32_t *__restrict__ seg_off, int32_t *__restrict__ perm,
                                                           int32_t *__restrict__ n_loaded, int4 *__restrict__ items) {
  __shared__ int32_t cnt[1024];        // pairs per expert (N <= 1024)
  __shared__ int32_t tot[5];           // offset of this segment, its first item; all pairs, segments, pieces
  __shared__ int32_t wave_cnt[2][16];  // routed tokens per wave, two rounds
  const int nt = blockDim.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n_waves = nt >> 6, i = blockIdx.x;
  const int n_pairs = M * k;
  int32_t held[kHeld ? kHeldSlots : 1];
  if constexpr (kHeld) {
#pragma unroll
    for (int j = 0; j < kHeldSlots; ++j) held[j] = j < k && tid < M ? tok_ids[(size_t)tid * k + j] : -1;
  }
  const int e = seg_expert[i];
  for (int x = tid; x < N; x += nt) cnt[x] = 0;
  if (tid < 5) tot[tid] = 0;
  __syncthreads();
  if constexpr (kHeld) {
#pragma unroll
    for (int j = 0; j < kHeldSlots; ++j)
      if (held[j] >= 0) atomicAdd(&cnt[held[j]], 1);
  } else {
    for (int p0 = 0; p0 < n_pairs; p0 += 4 * nt) {
      int id[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) id[u] = p0 + u * nt + tid < n_pairs ? tok_ids[p0 + u * nt + tid] : -1;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (id[u] >= 0) atomicAdd(&cnt[id[u]], 1);
    }
  }
  __syncthreads();
  const int c = e >= 0 ? cnt[e] : 0;
  for (int j0 = 0; j0 + (tid & ~63) < B; j0 += nt) {  // uniform in the wave
    const int j = j0 + tid, ej = j < B ? seg_expert[j] : -1, cj = ej >= 0 ? cnt[ej] : 0, q = piece_count(cj);
    const int sum[5] = {j < i ? cj : 0, (cj > c || (cj == c && j < i)) ? q : 0, cj, cj > 0 ? 1 : 0, q};
#pragma unroll
    for (int x = 0; x < 5; ++x) {
      const int s = row16_sum(sum[x]);  // through DPP: six shuffles per sum took 1 us
      if ((lane & 15) == 0 && s) atomicAdd(&tot[x], s);
    }
  }
  __syncthreads();
  const int off = tot[0], total = tot[2];
  if (tid == 0) {
    seg_off[i] = off;
    if (i == B - 1) {
      seg_off[B] = total;
      items[0] = int4{tot[4], 0, 0, 0};
      if (n_loaded) *n_loaded = tot[3];
    }
  }
  for (int p = total + i * nt + tid; p < n_pairs; p += B * nt) perm[p] = -1;
  if (c == 0) return;
  const int q = piece_count(c), len = (c + q - 1) / q;
  for (int p = tid; p < q; p += nt) items[1 + tot[1] + p] = int4{i, e, off + p * len, min(len, c - p * len)};
  int base = 0;
  for (int t0 = 0, round = 0; base < c && t0 < M; t0 += nt, round ^= 1) {
    const int t = t0 + tid;
    int slot = -1;
    if constexpr (kHeld) {
#pragma unroll
      for (int j = 0; j < kHeldSlots; ++j)
        if (held[j] == e) slot = j;
    } else if (t < M) {
#pragma unroll 8
      for (int j = 0; j < k; ++j)
        if (tok_ids[(size_t)t * k + j] == e) slot = j;
    }
    const unsigned long long mask = __ballot(slot >= 0);
    if (lane == 0) wave_cnt[round][wave] = __popcll(mask);
    __syncthreads();  // the two sets of counts alternate: one barrier a round
    int at = base;
    for (int w = 0; w < n_waves; ++w) {
      const int cw = wave_cnt[round][w];
      at += w < wave ? cw : 0;
      base += cw;
    }
    if (slot >= 0) perm[off + at + __popcll(mask & ((1ull << lane) - 1ull))] = t * k + slot;
  }
}

hipError_t launch_score_parts(const double *probs, int M, int N, double *part, int *n_parts, hipStream_t st) {
  const int rows = score_block_rows(M);
  *n_parts = (M + rows - 1) / rows;
  const size_t smem = sizeof(double) * kScoreWaves * N;
  if (smem > 64 * 1024) {  // beyond the default limit of a launch
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(score_parts_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
  }
  score_parts_kernel<<<*n_parts, kScoreThreads, smem, st>>>(probs, M, N, rows, part);
  return hipGetLastError();
}

hipError_t launch_budget(const moespec_desc &ds, const double *probs, int M, int B, int policy,
                         const int32_t *ext_shortlist, double *scores, int32_t *budget_ids, int32_t *tok_ids,
                         float *tok_w, int32_t *seg_expert, int32_t *seg_off, int32_t *perm, int32_t *n_loaded,
                         int4 *items, double *score_parts, const double *parts, int n_parts, hipStream_t st) {
  const int N = ds.n_experts, k = ds.top_k;
  const double *src = probs;
  int n_src = M;
  hipError_t e;
  if (n_parts > 0) {
    src = parts;
    n_src = n_parts;
  } else if (M > direct_score_rows(N) && (ext_shortlist == nullptr || scores != nullptr)) {
    if ((e = launch_score_parts(probs, M, N, score_parts, &n_src, st)) != hipSuccess) return e;
    src = score_parts;
  }
  // Every workgroup ranks the experts again: no more of them than two per compute unit.  One wave per token leaves most
  // compute units idle on small trees, one workgroup per token repeats the barriers of a token on large ones.  Whole stage,
  // us, wave / workgroup per token: 256 experts, 63 tokens 37 / 17, 511 tokens 40 / 30, 2048 tokens 43 / 57; 130 experts
  // 26 / 14, 29 / 25, 32 / 42 (1024 tokens: 41 / 40 and 30 / 31).  Up to 128 experts a row takes two candidates per lane,
  // and the wave is within 3 us at any size.
  const bool many = N > 4 * kWave || (N > 2 * kWave && M <= kMaxBudgetGroups);
  const int nt = budget_threads(N), tokens = many ? 1 : nt / kWave;
  const int want = (M + tokens - 1) / tokens, grid = want < kMaxBudgetGroups ? want : kMaxBudgetGroups;
  const size_t smem = budget_lds(N, B, nt, tokens).total;
  auto run = [&](auto kern) -> hipError_t {
    kern<<<grid, nt, smem, st>>>(probs, src, n_src, M, N, k, B, policy, ds.renorm, ext_shortlist, scores, budget_ids,
                                 seg_expert, tok_ids, tok_w);
    return hipGetLastError();
  };
  e = N <= 64 ? run(budget_kernel<1>) : N <= 128 ? run(budget_kernel<2>) : !many ? run(budget_kernel<4>)
                                                                                 : run(budget_many_kernel);
  if (e != hipSuccess) return e;
  const int gt = (int64_t)M * k <= 2048 ? 256 : 1024;
  (gt == 256 && k <= kHeldSlots && M <= gt ? group_pairs_kernel<true> : group_pairs_kernel<false>)<<<B, gt, 0, st>>>(
      tok_ids, M, N, k, B, seg_expert, seg_off, perm, n_loaded, items);
  return hipGetLastError();
}

}  // namespace moespec
