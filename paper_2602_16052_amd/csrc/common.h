// Shared device/host helpers of the moespec kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "moespec.h"

namespace moespec {

constexpr int kWave = 64;

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// bfloat16 bit pattern <-> float.  Storage tensors hold raw uint16 patterns.
__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}
// Round-to-nearest-even; NaN stays NaN.
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return static_cast<uint16_t>((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return static_cast<uint16_t>(u >> 16);
}

// A division, not the reciprocal instruction: that one gives 0 where 1 + exp(-z) exceeds 2^126 (gates of -87.3 and below).
__device__ __forceinline__ float silu_f(float z) { return z / (1.0f + __expf(-z)); }
// Four floats to bf16 (round-to-nearest-even), stored as 8 bytes.
__device__ __forceinline__ void store_bf16x4(uint16_t *p, f32x4 v) {
  typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
  *reinterpret_cast<bf16x4 *>(p) = __builtin_convertvector(v, bf16x4);
}

template <typename T> struct Elem;
template <> struct Elem<float> {
  static __device__ __forceinline__ float load(const float *p) { return *p; }
  static __device__ __forceinline__ void store(float *p, float v) { *p = v; }
  static __device__ __forceinline__ float stored(float v) { return v; }  // the value a store of v leaves behind
  // four in a row, the address aligned to their size
  static __device__ __forceinline__ f32x4 load4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }
  static __device__ __forceinline__ void store4(float *p, f32x4 v) { *reinterpret_cast<f32x4 *>(p) = v; }
};
template <> struct Elem<uint16_t> {
  static __device__ __forceinline__ float load(const uint16_t *p) { return bf16_bits_to_float(*p); }
  static __device__ __forceinline__ void store(uint16_t *p, float v) { *p = float_to_bf16_bits(v); }
  static __device__ __forceinline__ float stored(float v) { return bf16_bits_to_float(float_to_bf16_bits(v)); }
  static __device__ __forceinline__ f32x4 load4(const uint16_t *p) {
    const uint2 b = *reinterpret_cast<const uint2 *>(p);
    return f32x4{__uint_as_float(b.x << 16), __uint_as_float(b.x & 0xffff0000u), __uint_as_float(b.y << 16),
                 __uint_as_float(b.y & 0xffff0000u)};
  }
  static __device__ __forceinline__ void store4(uint16_t *p, f32x4 v) { store_bf16x4(p, v); }
};

// Ranking order used by every selection: larger value first, then lower index.
__device__ __forceinline__ bool ranks_before(double vj, int j, double vi, int i) {
  return vj > vi || (vj == vi && j < i);
}

// What an aggregate score ranks by (Section 3.2): a NaN, which no comparison would order, goes behind every number, by id.  So B experts
// claim the B places of the shortlist, one each, whatever the scores: one NaN hidden row makes all of them NaN.
__device__ __forceinline__ double ranking_score(double s) { return s == s ? s : -INFINITY; }

// ---- 16-lane all-reductions through DPP (no LDS, no barrier).  Every lane of a row of 16 ends with the same
// bits: each step combines a value with its partner's, and the operations used are commutative.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140, kDppRor4 = 0x124, kDppRor8 = 0x128;
__device__ __forceinline__ double row16_max(double v) {
  v = fmax(v, dpp_f64<kDppXor1>(v));
  v = fmax(v, dpp_f64<kDppXor2>(v));
  v = fmax(v, dpp_f64<kDppHalfMirror>(v));
  return fmax(v, dpp_f64<kDppMirror>(v));
}
__device__ __forceinline__ double row16_sum(double v) {
  v += dpp_f64<kDppXor1>(v);
  v += dpp_f64<kDppXor2>(v);
  v += dpp_f64<kDppHalfMirror>(v);
  return v + dpp_f64<kDppMirror>(v);
}
__device__ __forceinline__ float row16_sum(float v) {
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kDppXor1, 0xf, 0xf, false));
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kDppXor2, 0xf, 0xf, false));
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kDppHalfMirror, 0xf, 0xf, false));
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kDppMirror, 0xf, 0xf, false));
}
__device__ __forceinline__ int row16_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, kDppXor1, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, kDppXor2, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, kDppHalfMirror, 0xf, 0xf, false);
  return v + __builtin_amdgcn_update_dpp(0, v, kDppMirror, 0xf, 0xf, false);
}

// exp(x) for x <= 0 (the max-subtracted argument of a softmax): x = n ln 2 + r with |r| <= ln 2 / 2, the Taylor
// polynomial of degree 12 in r (truncation error below 2.4e-16 relative) and a scaling by 2^n.  Every workgroup of
// route_budget_kernel evaluates the whole table, so the two dozen instructions of this form matter.  Arguments below -800
// give 0; a NaN stays NaN and so makes its whole row NaN through the normalisation.
__device__ __forceinline__ double exp_nonpos(double x) {
  const double c = fmax(x, -800.0);  // drops a NaN: put back at the end
  const double n = rint(c * 1.4426950408889634);
  double r = fma(n, -6.93147180369123816490e-01, c);
  r = fma(n, -1.90821492927058770002e-10, r);
  double p = 1.0 / 479001600.0;
  p = fma(p, r, 1.0 / 39916800.0);
  p = fma(p, r, 1.0 / 3628800.0);
  p = fma(p, r, 1.0 / 362880.0);
  p = fma(p, r, 1.0 / 40320.0);
  p = fma(p, r, 1.0 / 5040.0);
  p = fma(p, r, 1.0 / 720.0);
  p = fma(p, r, 1.0 / 120.0);
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  p = fma(p, r, 1.0);
  p = fma(p, r, 1.0);
  return x != x ? x : ldexp(p, (int)n);
}

// x = row / sqrt(mean of squares) in fp32 for one row held by a workgroup of kRmsThreads threads: thread i holds the
// elements (c * kRmsThreads + i) * 4 .. + 3 of chunk c = 0 .. kRmsChunks-1 in v[c][0..3] (zeros past the row end;
// the hidden size is at most 8192).  Squares are
// added chunk by chunk and element by element per thread, the per-thread sums pairwise through LDS (a fixed tree):
// the result depends on the values alone.  Used by rms_scale_kernel and by the combine that also writes the next
// layer's input, which therefore agree bit for bit.  part: kRmsThreads floats of LDS.  Synchronises.
constexpr int kRmsThreads = 1024, kRmsChunks = 2;
__device__ inline float rms_scale_of_row(const float (&v)[kRmsChunks][4], int d, float *part) {
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < kRmsChunks; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i) ss = fmaf(v[c][i], v[c][i], ss);
  part[threadIdx.x] = ss;
  __syncthreads();
  for (int s = kRmsThreads / 2; s >= 1; s >>= 1) {
    if ((int)threadIdx.x < s) part[threadIdx.x] += part[threadIdx.x + s];
    __syncthreads();
  }
  return 1.0f / sqrtf(part[0] / (float)d);
}

// Orders the LDS accesses of one wave: they execute in program order, so only the compiler has to keep it.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Ranks before nothing: every comparison with it is false, whatever the other value (also an infinity or a log-probability).
constexpr double kNoRival = __builtin_nan("");

// c[u] += number of the values row[j0 .. j1) that go before candidate lane + 64 (first + u) with value v[u] in a ranking by
// (value descending, index ascending).  j0 is a multiple of 4; row is padded to a multiple of 4 with kNoRival, which also
// stands for the entries that are no rivals.  first is uniform in the wave.
// Four values per step, the same address in every lane (an LDS broadcast).  Against a rival of another block of 64
// experts the tie rule is the same for all lanes (>= or >): one comparison and one add with carry per rival.
template <int NU>
__device__ __forceinline__ void rank_counts(const double *row, int j0, int j1, int lane, int first, const double (&v)[NU],
                                            int (&c)[NU]) {
  // rivals in front of all candidates' blocks (b = -1), in block first + b, behind all (b = NU)
#pragma unroll
  for (int b = -1; b <= NU; ++b) {
    const int lo = b < 0 ? j0 : max(j0, kWave * (first + b)), hi = b == NU ? j1 : min(j1, kWave * (first + b + 1));
#pragma unroll 2
    for (int j = lo; j < hi; j += 4) {
      double r[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) r[q] = row[j + q];
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int u = 0; u < NU; ++u)
          c[u] += u > b ? (int)(r[q] >= v[u]) : u < b ? (int)(r[q] > v[u])
                        : (int)((r[q] > v[u]) | ((r[q] == v[u]) & (j + q < lane + kWave * (first + u))));
    }
  }
}

// val[u] = logit of expert lane + 64 u of token t (-inf past the row end): its Q slices in order, plus the router bias.
template <int Q, int NU>
__device__ __forceinline__ void load_logits(const double *partial, const float *bias, int M, int N, int t, double (&val)[NU]) {
  const size_t MN = (size_t)M * N, at = (size_t)t * N;
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int i = (threadIdx.x & 63) + kWave * u;
    val[u] = -INFINITY;
    if (i < N) {
      double v[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) v[q] = partial[q * MN + at + i];
      val[u] = v[0];
#pragma unroll
      for (int q = 1; q < Q; ++q) val[u] += v[q];
      val[u] += bias ? (double)bias[i] : 0.0;
    }
  }
}

// Eq. (1) for a row held by a wave: val[u] = logit of expert lane + 64 u (-inf past the row end), replaced by its probability.
template <int NU>
__device__ __forceinline__ void gate_of_row(double (&val)[NU], int sigmoid_gate) {
  if (sigmoid_gate) {
#pragma unroll
    for (int u = 0; u < NU; ++u) val[u] = 1.0 / (1.0 + exp(-val[u]));
    return;
  }
  auto all_lanes = [](double v, auto op) {  // the 16-lane result of every row of lanes combined across the 4 rows
    v = op(v, __shfl_xor(v, 16, kWave));
    return op(v, __shfl_xor(v, 32, kWave));
  };
  double m = val[0];
#pragma unroll
  for (int u = 1; u < NU; ++u) m = fmax(m, val[u]);
  m = all_lanes(row16_max(m), [](double a, double b) { return fmax(a, b); });
  double a = 0.0;
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    val[u] = exp_nonpos(val[u] - m);  // lanes past the row end come out as 0
    a += val[u];
  }
  const double inv = 1.0 / all_lanes(row16_sum(a), [](double x, double y) { return x + y; });
#pragma unroll
  for (int u = 0; u < NU; ++u) val[u] *= inv;
}

// v of lane 0 + v of lane 1 + ... + v of lane k - 1, in that order (k <= 64 and uniform; every lane gets the sum): without the LDS
// reads, one behind the other, of a loop over slots.
__device__ __forceinline__ double slot_sum(double v, int k) {
  double a = 0.0;
  for (int j = 0; j < k; ++j)
    a += __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), j), __builtin_amdgcn_readlane(__double2loint(v), j));
  return a;
}

// A token's probabilities that are NaN rank nowhere and nothing ranks behind them, but the token must not come out finite by that: the NaN
// with the lowest id among the shortlisted experts claims slot 0, or the lowest of all where none is shortlisted.  Its weight makes
// the token's output NaN, unless the slot is dropped (Eq. (7)).  nan_claim: that id, -1 without a NaN, for a row held by a wave (v[u] =
// candidate lane + 64 u, or none where member[u] is false).  The loops in LDS use an integer minimum over nan_key(id, listed).
constexpr int32_t kNaNUnlisted = 1 << 16, kNoNaN = 0x7fffffff;
__device__ __forceinline__ int32_t nan_key(int id, bool listed) { return listed ? id : id + kNaNUnlisted; }
__device__ __forceinline__ int nan_key_id(int32_t key) { return key & (kNaNUnlisted - 1); }
template <int NU>
__device__ __forceinline__ int nan_claim(const double (&v)[NU], const bool (&member)[NU], const uint8_t *listed) {
  const int lane = threadIdx.x & 63;
  int32_t key = kNoNaN;
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const bool nan = member[u] & (v[u] != v[u]);
    if (__ballot(nan) != 0) {  // uniform
      const unsigned long long in = __ballot(nan && (listed == nullptr || listed[lane + kWave * u] != 0)), all = __ballot(nan);
      key = min(key, nan_key(kWave * u + __ffsll((long long)(in ? in : all)) - 1, in != 0));
    }
  }
  return key == kNoNaN ? -1 : nan_key_id(key);
}

// Rank-count selection of the k best of v[0..n).  sel[r] receives the index with rank r < k.  Equivalent to sorting by
// (value descending, index ascending) and keeping the first k.  v, sel and the scratch rank[n] live in LDS.  Called by
// every thread of the workgroup (it synchronises); the caller synchronises again before reading sel.  The n x n
// comparisons are spread over the whole workgroup: thread (i, part) counts the rivals of candidate i inside its part of
// the index range and adds its count to rank[i] with an integer LDS atomic (order-independent, hence deterministic).
// Every slot of sel is first set to -1: NaN values rank nowhere, so that slots may stay unfilled.  The lowest NaN claims slot 0: until
// every value has been looked at the slot holds kNaNMark less its index.
constexpr int32_t kNaNMark = 1 << 30;
__device__ inline void select_topk(const double *v, int n, int k, int32_t *sel, int32_t *rank) {
  const int nt = blockDim.x, tid = threadIdx.x;
  int np2 = 1;
  while (np2 < n) np2 <<= 1;
  for (int x = tid; x < n; x += nt) rank[x] = 0;
  for (int x = tid; x < k; x += nt) sel[x] = -1;
  __syncthreads();
  const int parts = np2 <= nt ? nt / np2 : 1;
  const int chunk = (n + parts - 1) / parts;
  for (int i = np2 <= nt ? (tid & (np2 - 1)) : tid; i < n; i += np2 <= nt ? n : nt) {
    const int part = np2 <= nt ? tid / np2 : 0;
    const int j0 = part * chunk, j1 = min(n, j0 + chunk);
    const double vi = v[i];
    if (vi != vi) {
      atomicMax(&sel[0], kNaNMark - i);
      continue;
    }
    int cnt = 0;
#pragma unroll 4
    for (int j = j0; j < j1; ++j) cnt += ranks_before(v[j], j, vi, i) ? 1 : 0;
    if (cnt) atomicAdd(&rank[i], cnt);
  }
  __syncthreads();
  for (int x = tid; x < n; x += nt) {
    if (v[x] != v[x]) {
      if (sel[0] == kNaNMark - x) sel[0] = x;
    } else if (rank[x] < k && (rank[x] > 0 || sel[0] < 0)) {  // slot 0 is claimed by one value of either kind
      sel[rank[x]] = x;
    }
  }
}

// Mixing weights of the slots sel[0..k): raw g or g / sum over the slots (summed in slot order).
// An unfilled slot (sel < 0) gets weight 0.  Called by every thread (it synchronises); denom is one
// LDS double of scratch.
__device__ inline void mixing_weights(const double *g, const int32_t *sel, int k, int renorm, double *w,
                                      double *denom) {
  if (threadIdx.x == 0 && renorm) {
    double acc = 0.0;
    for (int s = 0; s < k; ++s)
      if (sel[s] >= 0) acc += g[sel[s]];
    *denom = acc;
  }
  __syncthreads();
  for (int s = threadIdx.x; s < k; s += blockDim.x)
    w[s] = sel[s] < 0 ? 0.0 : (renorm ? g[sel[s]] / *denom : g[sel[s]]);
}

constexpr int kMaxDownSplits = 4;  // K-split copies of the per-pair outputs y

// The LDS-tiled expert passes take up to 128 pairs (8 token tiles of 16) per walk over an expert's weights.
// A longer segment is cut into ceil(c / 128) pieces of (almost) equal size, each a work item of its own, so
// that its walks run side by side on different compute units instead of one after the other.
constexpr int kPiecePairs = 128;
__host__ __device__ inline int piece_count(int c) { return (c + kPiecePairs - 1) / kPiecePairs; }
// Upper bound on the pieces of n_seg well-formed segments (disjoint, at most one pair per token each).
inline int items_capacity(int n_seg, int64_t M, int64_t k) {
  const int64_t a = (int64_t)n_seg * ((M + kPiecePairs - 1) / kPiecePairs), b = n_seg + M * k / kPiecePairs;
  return (int)(a < b ? a : b);
}
constexpr int kMaxLogitSlices = 8;    // slices of the hidden dimension in the fused prologue's router projection
constexpr int kSelfMaxTokens = 1024;  // largest tree with a place of its own for partial projections and pair lists
constexpr int kSelfMaxExperts = 256;  // ... and the most experts; also the limit of the matrix-core router projection

// Row blocks whose column sums are the first half of Eq. (5) on large trees: at most kScoreMaxParts of them, one
// workgroup each, a multiple of its waves.
constexpr int kScoreThreads = 1024, kScoreWaves = kScoreThreads / kWave, kScoreMaxParts = 64;
inline int score_block_rows(int64_t M) {
  return kScoreWaves * (int)((M + kScoreMaxParts * kScoreWaves - 1) / (kScoreMaxParts * kScoreWaves));
}

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Workspace carve-up shared by all entry points (host).
struct Workspace {
  double *probs;      // [M, N]
  int32_t *budget_ids;  // [N]
  int32_t *tok_ids;   // [M, k]
  float *tok_w;       // [M, k]
  int32_t *seg_expert;  // [N]
  int32_t *seg_off;   // [N + 1]
  int32_t *perm;      // [M * k]
  int4 *items;        // [items_capacity(N, M, k) + 1] count, then (segment, expert, offset, size) of every piece
  void *act;          // [M * k, F] dtype
  float *y;           // [kMaxDownSplits][M * k, d]
  double *gram;       // [N, N + 3] scratch of the oracle ranking
  double *score_parts;  // [kScoreMaxParts, N] column sums of row blocks (budget stage; shares the place of gram)
  double *partial;    // [partial_slices, M, N] partial router projections
  int partial_slices;  // kMaxLogitSlices, or what fits the place of y, which later stages fill
  int32_t *list_count;  // [N] pairs per shortlist rank (fused prologue)
  int32_t *lists;     // [N, M] their pair lists (only for shapes the fused prologue covers)
  void *xnorm;        // [M, d] dtype: the scaled layer input of the layer stack
  size_t bytes;
};

inline Workspace carve_workspace(const moespec_desc &ds, int64_t M, void *base) {
  Workspace w;
  size_t off = 0;
  char *b = static_cast<char *>(base);
  auto take = [&](size_t n) {
    void *p = b ? b + off : nullptr;
    off += align_up(n, 256);
    return p;
  };
  const int64_t N = ds.n_experts, k = ds.top_k, F = ds.d_ff, d = ds.d;
  const size_t es = ds.dtype == MOESPEC_BF16 ? 2 : 4;
  w.probs = static_cast<double *>(take(sizeof(double) * M * N));
  w.budget_ids = static_cast<int32_t *>(take(sizeof(int32_t) * N));
  w.tok_ids = static_cast<int32_t *>(take(sizeof(int32_t) * M * k));
  w.tok_w = static_cast<float *>(take(sizeof(float) * M * k));
  w.seg_expert = static_cast<int32_t *>(take(sizeof(int32_t) * N));
  w.seg_off = static_cast<int32_t *>(take(sizeof(int32_t) * (N + 1)));
  w.perm = static_cast<int32_t *>(take(sizeof(int32_t) * M * k));
  w.items = static_cast<int4 *>(take(sizeof(int4) * (items_capacity((int)N, M, k) + 1)));
  w.act = take(es * M * k * F);
  w.y = static_cast<float *>(take(sizeof(float) * kMaxDownSplits * M * k * d));
  w.gram = static_cast<double *>(take(sizeof(double) * N * (N + 3 > kScoreMaxParts ? N + 3 : kScoreMaxParts)));
  w.score_parts = w.gram;
  const bool small = N <= kSelfMaxExperts && M <= kSelfMaxTokens;
  if (small) {
    w.partial = static_cast<double *>(take(sizeof(double) * kMaxLogitSlices * M * N));
    w.partial_slices = kMaxLogitSlices;
  } else {
    w.partial = reinterpret_cast<double *>(w.y);
    w.partial_slices = (int)(sizeof(float) * kMaxDownSplits * k * d / (sizeof(double) * N));
  }
  w.list_count = static_cast<int32_t *>(take(sizeof(int32_t) * N));
  w.lists = static_cast<int32_t *>(take(small ? sizeof(int32_t) * N * M : 0));
  w.xnorm = take(es * M * d);
  w.bytes = off;
  return w;
}

// Launchers (defined in the .hip files).  Each returns hipGetLastError() after its launches.
// topk_ids / topk_w may be NULL.  partial: [partial_slices, M, N] doubles of scratch (partial_slices may be 0).
// parts (may be NULL; no top-k then): [gate_parts(), N] doubles, the sums of the probabilities over blocks of tokens.
hipError_t launch_route(const moespec_desc &ds, const moespec_weights &wt, const void *h, int M, double *probs,
                        int32_t *topk_ids, float *topk_w, double *partial, int partial_slices, double *parts, hipStream_t st);
int gate_parts(const moespec_desc &ds, int M);  // 0: this shape has none
// score_parts: [kScoreMaxParts, N] doubles of scratch.  scores and n_loaded may be NULL.
// n_parts > 0: parts [n_parts, N] holds the sums of the probabilities over blocks of tokens already.
hipError_t launch_budget(const moespec_desc &ds, const double *probs, int M, int B, int policy,
                         const int32_t *ext_shortlist, double *scores, int32_t *budget_ids, int32_t *tok_ids,
                         float *tok_w, int32_t *seg_expert, int32_t *seg_off, int32_t *perm, int32_t *n_loaded,
                         int4 *items, double *score_parts, const double *parts, int n_parts, hipStream_t st);
// items: table of the work items ([items_capacity(n_seg, M, k) + 1] int4 of scratch: the non-empty segments,
// those above kPiecePairs pairs cut into pieces); items_ready says that the budget stage has already filled
// it from the same segment arrays, otherwise it is built first.
// rank_count, shortlist, lists (NULL, or all three from the fused prologue): the shortlist in rank order ([n_seg]), the
// surviving pairs of each of its experts and their lists (rank r at lists + r * list_stride); every workgroup then
// finds its work item in them (needs expert_ffn_self_segmenting) and seg_expert / seg_off / perm / items are not read.
// trace (may be NULL): 3 events recorded after the gate/up pass, the down pass and the combine.
// x_next (may be NULL): [M, d] dtype; the combine then also writes out scaled row by row to unit root-mean-square,
// the next layer's input in a stack (d <= 8192).
hipError_t launch_expert_ffn(const moespec_desc &ds, const moespec_weights &wt, const void *h, int M, int n_seg,
                             const int32_t *seg_expert, const int32_t *seg_off, const int32_t *perm,
                             const int32_t *tok_ids, const float *tok_w, const void *residual, void *out, void *act,
                             float *y, int4 *items, bool items_ready, const int32_t *rank_count,
                             const int32_t *shortlist, const int32_t *lists, int list_stride, hipStream_t st,
                             void *const *trace = nullptr, void *x_next = nullptr);
// The fused prologue of the layer call (prologue.hip): router projection on the fp64 matrix cores, then one
// launch that leaves the shortlist (budget_ids), the restricted routing (tok_ids, tok_w) and, for every shortlist
// rank r, the pairs routed to its expert (list_count[r]; lists[r * list_stride ..], flat ids t * k + slot, tokens
// ascending).  partial: [logit_slices, M, N] doubles of scratch, parts: [64, N], ranks_ws: what fused_prologue_ok asks of y.  probs_out, scores_out, seg_expert, seg_off,
// perm, n_loaded are optional copies for the caller (the last three cost one more small launch).
bool fused_prologue_ok(const moespec_desc &ds, int M, int B, int policy);
// The two halves of stage 1 for layers of up to kSelfMaxExperts experts (mfma_route_ok): the router projection on
// the fp64 matrix cores (partial [slices, M, N] out), then bias, gate and - if wanted - the natural top-k, one wave per
// token (partial may be probs itself when there is one slice).
bool mfma_route_ok(const moespec_desc &ds);
hipError_t launch_logits(const moespec_desc &ds, const moespec_weights &wt, const void *h, int M, int slices,
                         double *partial, hipStream_t st);
hipError_t launch_gate_rows(const moespec_desc &ds, const moespec_weights &wt, int M, int slices, const double *partial,
                            double *probs, int32_t *topk_ids, float *topk_w, double *parts, hipStream_t st);
int logit_slices(const moespec_desc &ds, int M, int most);
hipError_t launch_fused_prologue(const moespec_desc &ds, const moespec_weights &wt, const void *h, int M, int B,
                                 int policy, const int32_t *ext_shortlist, double *partial, double *parts, void *ranks_ws, double *probs_ws,
                                 double *probs_out, double *scores_out, int32_t *budget_ids, int32_t *seg_expert, int32_t *tok_ids,
                                 float *tok_w, int32_t *list_count, int32_t *lists, int list_stride,
                                 int32_t *seg_off, int32_t *perm, int32_t *n_loaded, hipStream_t st);
bool expert_ffn_self_segmenting(const moespec_desc &ds, int M);
// Number of K-split copies of y that launch_expert_ffn writes for n_seg segments; out == NULL there skips
// the combine and leaves the per-pair expert outputs in y.
int down_splits(const moespec_desc &ds, int M, int n_seg);
int streaming_down_splits(const moespec_desc &ds, int n_seg);  // what the streaming form of the down pass takes
// The passes as a grouped GEMM (expert_wide.hip): whether the gate/up pass runs in that form (the layer call then takes the
// staged prologue), whether the down pass does too, and one of them.
bool expert_ffn_wide(const moespec_desc &ds, int M, int n_seg);
bool expert_down_wide(const moespec_desc &ds, int M, int n_seg);
hipError_t launch_wide_pass(const moespec_desc &ds, const moespec_weights &wt, bool gate_up, const void *x, int M,
                            const int4 *items, const int32_t *perm, int cap, void *out, hipStream_t st);
// Analysis kernels (analysis.hip).  part: 2 M doubles of scratch.
hipError_t launch_calibration_count(const int32_t *topk_ids, int M, int k, int N, int64_t *counts, hipStream_t st);
hipError_t launch_static_shortlist(const int64_t *counts, int N, int B, int32_t *shortlist, hipStream_t st);
hipError_t launch_coverage_curve(const double *scores, int N, double *curve, hipStream_t st);
// Greedy oracle ranking on the per-pair outputs y (splits copies, split_stride floats apart) of a run with
// natural routing (tok_ids / tok_w = natural top-k).  pair_gram: M k k doubles, gram: N N + 3 N doubles of scratch.
hipError_t launch_oracle_ranking(const moespec_desc &ds, const float *y, int splits, size_t split_stride,
                                 const int32_t *tok_ids, const float *tok_w, int M, int B, double *pair_gram,
                                 double *gram, int32_t *ranking, double *err, hipStream_t st);
// x[t] = h[t] / rms(h[t]) (stack.hip); x may alias h.
hipError_t launch_rms_scale(const moespec_desc &ds, const void *h, int M, void *x, hipStream_t st);
hipError_t launch_stream_read(const void *buf, size_t bytes, uint32_t *checksum, hipStream_t st);
hipError_t launch_reconstruction_error(const moespec_desc &ds, const void *out_budgeted, const void *out_full, int M,
                                       double *part, double *err, hipStream_t st);

}  // namespace moespec
