// The expert passes (Eq. (2)/(7)/(8)) on trees and prompt chunks whose experts serve so many pairs that the passes are
// no longer bound by the weight stream alone: a grouped GEMM over the work items of the budget stage.
//
// What bounds it: the traffic between the L2s and memory, then the LDS port and the matrix cores.  A workgroup of 8 waves
// owns a compute unit and a tile of 256 weight rows (gate/up: 128 gate + the same 128 up rows) x up to 128 pairs, a wave
// 64 x 64 of it (4 x 2 waves): 8 KB of LDS operands per 16 matrix instructions instead of the 10 KB of the streaming form,
// and a weight byte that is fetched once serves 128 pairs.  Both operands go from memory straight into LDS
// (global_load_lds_dwordx4: no registers, no LDS stores), 64 elements (one cache line of every row) per stage in a ring
// of three 48 KB stages, of which two are in flight.  While one half of a stage is multiplied the operands of the next
// half are read from LDS into the other register set; one barrier per stage, where the stage just read is refilled.
// Gate/up + down pass, 2048 tokens x top-8 of 64 experts of 2048 x 1024: 218 + 138 us against 287 + 166 us of the streaming
// form (511 tokens over 32 experts: 79 + 50 against 99 + 60).  The loads alone take 197 us of the 218 (0.75 GB from memory,
// 2.1 GB into LDS), the LDS reads and matrix instructions alone 122.  With the operands read right before their matrix
// instructions the gate/up pass took 244 us, with 32 elements (half a line) per stage 255 us.
// A row of a stage is 128 bytes = 8 pieces of 16; piece c of row r sits in slot c ^ (r & 7), so that 8 lanes that read
// the same piece of 8 consecutive rows touch all 32 banks.  The lane that fetches a slot applies the permutation to its
// global address (the DMA writes lane after lane).
#include <math.h>

#include <type_traits>

#include "common.h"

namespace moespec {

constexpr int kWideThreads = 512, kWideRows = 256, kWideK = 64, kWideStages = 3;
constexpr int kWideRowBytes = 2 * kWideK;
constexpr int kWideA = kWideRows * kWideRowBytes, kWideB = kPiecePairs * kWideRowBytes, kWideStage = kWideA + kWideB;
constexpr int kWideLds = kWideStages * kWideStage;
constexpr int kWideGrid = 256;  // one workgroup per compute unit
constexpr int kWideXcds = 8, kWideBlock = 4;  // consecutive work items that run side by side on one XCD

// 64 lanes x 16 bytes from base + voff (per lane) to LDS bytes [lds, lds + 1024), lane after lane.  Completion is
// counted by vmcnt in issue order; the compiler does not see the load, so the waits are written by hand.  m0 is a register
// that the compiler reserves for sequences of its own, and warns about in a clobber list; named there, it keeps a value of
// its own in m0 from being carried across.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma_to_lds(uint32_t lds, const void *base, uint32_t voff) {
  const uint64_t b = reinterpret_cast<uint64_t>(base);  // uniform, and the compiler is told so
  const uint64_t ub = (uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)) << 32 |
                      (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(
                   __builtin_amdgcn_readfirstlane(lds)),
               "v"(voff), "s"(ub)
               : "m0", "memory");
}
#pragma clang diagnostic pop
template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"i"(N) : "memory");
}
__device__ __forceinline__ void wide_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// One work item: acc[i][j] += rows of weight tile i x pairs of token tile 2 j + wc over K.  wa: first weight row of the
// half that this wave fetches, aoff / boff: this lane's byte offsets of its rows (piece included) from wa / xb.  The walk
// starts at stage c0 and wraps; a last stage of 32 elements (K % 64 != 0, then c0 = 0) overlaps the one before, and only
// its second half is multiplied.
template <bool kGateUp, int NB>
__device__ __forceinline__ void wide_walk(const uint16_t *wa, const uint32_t (&aoff)[4], const uint16_t *xb,
                                          const uint32_t (&boff)[2], int K, int c0, unsigned char *lds,
                                          f32x4 (&acc)[4][NB]) {
  constexpr int NBL = (NB + 1) / 2, LD = 4 + NBL;  // loads per wave and stage: weights, tokens
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wr = wave >> 1, wc = wave & 1;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)lds);
  const int nst = (K + kWideK - 1) / kWideK;
  int kf = c0 * kWideK, at = 0;  // element and ring offset of the next stage to fetch
  auto issue = [&]() {
    const uint32_t dst = lds0 + at;
    const int k = min(kf, K - kWideK);
#pragma unroll
    for (int q = 0; q < 4; ++q) dma_to_lds(dst + (wave * 4 + q) * 1024, wa + k, aoff[q]);
#pragma unroll
    for (int q = 0; q < NBL; ++q) dma_to_lds(dst + kWideA + (wave * NBL + q) * 1024, xb + k, boff[q]);
    kf = kf + kWideK >= K ? 0 : kf + kWideK;
    at = at + kWideStage == kWideLds ? 0 : at + kWideStage;
  };
  const int r = lane & 15, kg = lane >> 4;
  const unsigned char *pa = lds + ((kGateUp ? 32 : 64) * wr + r) * kWideRowBytes;
  const unsigned char *pb = lds + kWideA + (16 * wc + r) * kWideRowBytes;
  const int slot[2] = {(kg ^ (r & 7)) << 4, ((4 + kg) ^ (r & 7)) << 4};  // this lane's piece in each half of a stage
  bf16x8 fa[2][4], fb[2][NB];
  auto fetch = [&](int rd, int half) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      fa[half][i] = *reinterpret_cast<const bf16x8 *>(
          pa + rd + slot[half] + (kGateUp ? (i >> 1) * 128 + 16 * (i & 1) : 16 * i) * kWideRowBytes);
#pragma unroll
    for (int j = 0; j < NB; ++j)
      fb[half][j] = *reinterpret_cast<const bf16x8 *>(pb + rd + slot[half] + 32 * j * kWideRowBytes);
  };
  auto multiply = [&](int half) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[half][i], fb[half][j], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  int rd = 0;
  // One stage with LEFT stages behind it (3: three or more).  At the barrier this wave has read all of the stage and its
  // share of the next one has arrived, then everybody's: the stage's place takes the stage three ahead.  Straight-line
  // code: behind a branch the compiler would wait for the operands it has just requested before the multiplications.
  auto stage = [&](auto left_) {
    constexpr int LEFT = decltype(left_)::value;
    fetch(rd, 1);
    if (LEFT > 0 || K % kWideK == 0) multiply(0);
    if constexpr (LEFT > 0) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      wait_vm<(LEFT > 1 ? LD : 0)>();
      wide_barrier();
      if constexpr (LEFT > 2) issue();
      rd = rd + kWideStage == kWideLds ? 0 : rd + kWideStage;
      fetch(rd, 0);
    }
    multiply(1);
  };
#pragma unroll
  for (int s = 0; s < kWideStages; ++s)
    if (s < nst) issue();
  if (nst >= kWideStages) wait_vm<2 * LD>();
  else wait_vm<0>();
  wide_barrier();
  fetch(0, 0);
  for (int left = nst - 1; left > 2; --left) stage(std::integral_constant<int, 3>{});
  if (nst >= 3) stage(std::integral_constant<int, 2>{});
  if (nst >= 2) stage(std::integral_constant<int, 1>{});
  stage(std::integral_constant<int, 0>{});
}

// kGateUp: x = hidden rows [M, K], R = F, out = act [M k, F] bf16; otherwise x = act [M k, K], R = d, out = y [M k, d] fp32.
// Persistent: workgroup b runs on XCD b mod 8 and takes every (grid / 8)-th unit (work item, row tile) of that XCD's list.
// The items come sorted by size, the pieces of an expert side by side; whole rounds of 8 x 4 items give every XCD four
// neighbours, which it walks row tile by row tile: pieces that share weight rows, and row tiles that share token rows,
// run at the same time and meet in one L2.  The units of the items left over are dealt one by one.
template <bool kGateUp>
__global__ __launch_bounds__(kWideThreads, 2) void ffn_wide_kernel(
    const uint16_t *__restrict__ x, const uint16_t *__restrict__ w0, const uint16_t *__restrict__ w1,
    const int4 *__restrict__ items, const int32_t *__restrict__ perm, int cap, int M, int N, int k, int K, int R,
    void *__restrict__ out) {
  extern __shared__ __align__(16) unsigned char lds[];
  constexpr int kTileRows = kGateUp ? kWideRows / 2 : kWideRows;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wr = wave >> 1, wc = wave & 1;
  const int tiles = (R + kTileRows - 1) / kTileRows, n_pairs = M * k;
  int L = items[0].x;
  L = L < 0 ? 0 : (L > cap ? cap : L);
  const int xcd = blockIdx.x % kWideXcds, slots = gridDim.x / kWideXcds;
  const int full = L / (kWideXcds * kWideBlock), rest = L - full * kWideXcds * kWideBlock;
  const int n_full = full * kWideBlock * tiles, n_units = n_full + (rest * tiles - xcd + kWideXcds - 1) / kWideXcds;
  const int lrow = lane >> 3, piece = ((lane & 7) ^ lrow) * 16;  // row and piece (bytes) that this lane fetches
  for (int u = blockIdx.x / kWideXcds; u < n_units; u += slots) {
    int item, tile;
    // every other XCD walks its list backwards: the large items are bound by the matrix cores and the LDS, the small
    // ones, which share no weights, by memory, and so both kinds run at any time
    const int ord = (xcd & 1) ? n_units - 1 - u : u;
    if (ord < n_full) {
      const int v = ord % (kWideBlock * tiles);
      item = (ord / (kWideBlock * tiles) * kWideXcds + xcd) * kWideBlock + v % kWideBlock;
      tile = v / kWideBlock;
    } else {
      const int v = xcd + kWideXcds * (ord - n_full);
      item = full * kWideXcds * kWideBlock + v / tiles;
      tile = v % tiles;
    }
    const int4 it = items[1 + item];
    const int e = it.y, beg = it.z, m = it.w;
    if (it.x < 0 || e < 0 || e >= N || m <= 0 || m > kPiecePairs || beg < 0 || (long long)beg + m > n_pairs) continue;
    const int f0 = tile * kTileRows;
    // weight rows: waves 0-3 fetch the first 128 rows of the tile, waves 4-7 the others (gate/up: the up rows)
    const uint16_t *wa = (kGateUp && wave >= 4 ? w1 : w0) + ((size_t)e * R + f0) * K;
    uint32_t aoff[4], boff[2];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = (kGateUp ? (wave & 3) : wave) * 32 + q * 8 + lrow;
      aoff[q] = 2u * (uint32_t)min(row, R - 1 - f0) * (uint32_t)K + piece;  // rows past the end repeat the last one
    }
    const int nbl = m > 64 ? 2 : 1;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      int px = perm[beg + min((wave * nbl + q) * 8 + lrow, m - 1)];  // so do the pairs; their columns are never stored
      px = px < 0 ? 0 : (px >= n_pairs ? n_pairs - 1 : px);
      boff[q] = 2u * (uint32_t)(kGateUp ? px / k : px) * (uint32_t)K + piece;
    }
    // experts start their walk 256 bytes apart, row tiles 512 (see k_stagger)
    const int c0 = K % kWideK == 0 ? (2 * e + 4 * tile) % (K / kWideK) : 0;
    auto run = [&](auto nb) {
      constexpr int NB = decltype(nb)::value;
      f32x4 acc[4][NB];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      wide_walk<kGateUp, NB>(wa, aoff, x, boff, K, c0, lds, acc);
      const int col = lane & 15, kg = lane >> 4;
      int pr[NB];  // one round of loads, not one per token tile
#pragma unroll
      for (int j = 0; j < NB; ++j) pr[j] = perm[beg + min((2 * j + wc) * 16 + col, m - 1)];
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        pr[j] = pr[j] < 0 ? 0 : (pr[j] >= n_pairs ? n_pairs - 1 : pr[j]);
        if ((2 * j + wc) * 16 + col < m) {
          if constexpr (kGateUp) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
              const int f = f0 + 32 * wr + 16 * i + 4 * kg;
              f32x4 o;
#pragma unroll
              for (int c = 0; c < 4; ++c) o[c] = silu_f(acc[i][j][c]) * acc[i + 2][j][c];
              if (f < R) store_bf16x4(static_cast<uint16_t *>(out) + (size_t)pr[j] * R + f, o);
            }
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int f = f0 + 64 * wr + 16 * i + 4 * kg;
              if (f < R) *reinterpret_cast<f32x4 *>(static_cast<float *>(out) + (size_t)pr[j] * R + f) = acc[i][j];
            }
          }
        }
      }
    };
    if (m <= 32) run(std::integral_constant<int, 1>{});
    else if (m <= 64) run(std::integral_constant<int, 2>{});
    else if (m <= 96) run(std::integral_constant<int, 3>{});
    else run(std::integral_constant<int, 4>{});
    wide_barrier();  // everybody has read the last stages before the next unit's loads overwrite them
  }
}

// Where the grouped form is the faster one.  A segment of more than 128 pairs makes the streaming form read its expert
// once per piece; with up to 256 tokens that is at most twice, and only segments that are large on average (96 pairs)
// pay for 256 workgroups whose last round is partly empty.  Measured per layer, streaming / grouped, us (64 experts of
// 2048 x 1024, top-8): 127 tokens over 16 segments 85 / 92; 255 over 32 124 / 139, over 16 114 / 98; 383 over 64
// 168 / 154; 511 over 64 198 / 190, over 32 190 / 163; 2048 over 64 511 / 425.
//
// How many pairs a segment really has is known on the device only: between pairs / n_seg (substitution keeps them all) and
// pairs / N (truncation of a flat routing).  segment_mean is the geometric mean of the two; with the segments that large:
//   - up to 256 tokens, a layer of a few units keeps the streaming form and the fused prologue in front of it (8 experts of
//     512 x 128, 2 to 4 shortlisted, 160 to 200 tokens: 34 to 38 / 39 to 43 us);
//   - weight rows of more than 4 KB: a unit is one walk over a long row at one workgroup per compute unit, and the weights
//     stream slower than to two.  Where they are many (more than 8e7 elements a matrix) the segments have to be larger to
//     make up for it (16 of 4096 x 2048, top-2: 300 tokens 202 / 240 us, 2048 tokens 487 / 378; 32 of 4096 x 1024, top-4,
//     383 tokens 200 / 245); most of all where the streaming form would cut F in four (2 of 8 experts of 4096 x 14336, 160
//     tokens: 147 / 191 under truncation, 320 / 343 under substitution; 511 tokens 651 / 525).
static double segment_mean(const moespec_desc &ds, int M, int n_seg) {
  return (double)M * ds.top_k / sqrt((double)n_seg * ds.n_experts);
}
static long long expected_pieces(const moespec_desc &ds, int M, int n_seg) {
  const double mean = segment_mean(ds, M, n_seg);
  return (long long)n_seg * piece_count((int)ceil(mean < M ? mean : M));
}
bool expert_ffn_wide(const moespec_desc &ds, int M, int n_seg) {
  if (ds.dtype != MOESPEC_BF16 || ds.d < kWideK || ds.d_ff < kWideK) return false;
  const long long pairs = (long long)M * ds.top_k;
  if (!((M > 2 * kPiecePairs && pairs >= 32ll * n_seg) || (M > kPiecePairs && pairs >= 96ll * n_seg))) return false;
  const int tiles = (ds.d_ff + kWideRows / 2 - 1) / (kWideRows / 2) + (ds.d + kWideRows - 1) / kWideRows;  // both passes
  if (M <= 2 * kPiecePairs && expected_pieces(ds, M, n_seg) * tiles < 48) return false;
  if (ds.d > 2048) {
    const double mean = segment_mean(ds, M, n_seg);
    if (streaming_down_splits(ds, n_seg) == kMaxDownSplits ? mean < 160.0
                                                           : mean < 80.0 && (long long)n_seg * ds.d * ds.d_ff > 80000000ll)
      return false;
  }
  return true;
}

// Whether the down pass takes the grouped form as well.  It has no split of K, so where the streaming form cuts F in two or
// four (long rows, few row tiles) the grouped pass lasts as long as one walk over F, 0.85 us per stage of 64, unless its
// units fill a good part of the 256 workgroups.  Down pass alone, streaming with splits / grouped, us: one of 4 experts of
// 1024 x 8192, 300 tokens 40 less; 2 of 8 of 4096 x 14336, 160 tokens 130 less; but 2 of 8 of 4096 x 4096, 1023 tokens (256
// units) 67 more, 3 of 6 of 3072 x 8192 (216 units) 104 more.
bool expert_down_wide(const moespec_desc &ds, int M, int n_seg) {
  return expert_ffn_wide(ds, M, n_seg) &&
         (streaming_down_splits(ds, n_seg) == 1 ||
          expected_pieces(ds, M, n_seg) * ((ds.d + kWideRows - 1) / kWideRows) >= 96);
}

hipError_t launch_wide_pass(const moespec_desc &ds, const moespec_weights &wt, bool gate_up, const void *x, int M,
                            const int4 *items, const int32_t *perm, int cap, void *out, hipStream_t st) {
  auto run = [&](auto kern, const void *w0, const void *w1, int K, int R) -> hipError_t {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       kWideLds);
    if (e != hipSuccess) return e;
    kern<<<kWideGrid, kWideThreads, kWideLds, st>>>(static_cast<const uint16_t *>(x), static_cast<const uint16_t *>(w0),
                                                    static_cast<const uint16_t *>(w1), items, perm, cap, M, ds.n_experts,
                                                    ds.top_k, K, R, out);
    return hipGetLastError();
  };
  return gate_up ? run(ffn_wide_kernel<true>, wt.w_gate, wt.w_up, ds.d, ds.d_ff)
                 : run(ffn_wide_kernel<false>, wt.w_down, nullptr, ds.d_ff, ds.d);
}

}  // namespace moespec
