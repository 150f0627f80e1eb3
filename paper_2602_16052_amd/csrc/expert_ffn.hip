// The expert networks over the loaded experts (Eq. (2)/(7)/(8)) and the weighted combine.
//
// E_i(x) = W_down,i ( silu(W_gate,i x) * (W_up,i x) ) is evaluated per segment (one expert, the
// hidden rows of its (token, slot) pairs) in two passes over that expert's weights:
//   pass 1  act[p, :] = silu(W_gate x_p) * (W_up x_p)        streams W_gate,i and W_up,i once
//   pass 2  y[pair, :] = W_down act[p, :]                    streams W_down,i once
// and a final combine adds the k weighted rows of every token in slot order (deterministic).
//
// bf16 path.  Weight rows are the MFMA "A" side (v_mfma_f32_16x16x32_bf16), tokens the "B" side
// (16 per tile, up to 8 tiles per pass, so a segment of up to 128 pairs reads its expert once).
// Work is cut into equal-byte items: a workgroup of 4 waves takes 128 weight rows (32 per wave)
// of one expert and walks K in chunks; however uneven the segment sizes, every compute unit
// streams the same number of weight bytes.  Per chunk each wave loads its rows with fully
// coalesced 16-byte loads, parks them in a wave-private, XOR-swizzled LDS tile and reads them
// back in MFMA operand layout; the token chunk is loaded once per workgroup into a shared LDS
// tile (double-buffered up to 4 token tiles; one 32 KB buffer and a second barrier for 8).  (Loading
// operands from global memory directly in MFMA layout costs a cache-line lookup per lane and saturates
// the texture-address path long before HBM.)  A segment of more than 128 pairs is cut into pieces that
// are work items of their own: its walks over the expert run side by side, not one after the other.
// Workgroups start their K walk at staggered offsets: weight rows are a power-of-two stride
// apart, and equal offsets would pile the concurrent reads onto the same memory channels.
// Where K is not a multiple of the 128-element chunk (kTail), the pieces of the last chunk past the row end are not
// loaded and count as zeros.
// The intermediate act and the per-pair outputs y are indexed by the flat pair id t * k + slot.
//
// Where its segment comes from: either from the work items that the budget stage has built beside the segment
// arrays (seg_expert, seg_off, perm; any caller), or - inside the fused layer, for small trees - from the pair lists
// of the fused prologue.
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace moespec {

constexpr int kFfnThreads = 256;
static_assert(kSelfMaxExperts <= kFfnThreads, "one thread per shortlist rank");
constexpr int kFfnWaves = kFfnThreads / kWave;
static_assert(kPiecePairs == 128, "8 token tiles of 16 per pass over the weights");

// A segment is processed only if it names a real expert and lies inside the pair table; the passes clamp
// pair indices into [0, M*k) so that malformed tables cannot address outside the buffers.
__device__ __forceinline__ bool segment_ok(int e, int beg, int m, long long list_len, int N) {
  return e >= 0 && e < N && m > 0 && beg >= 0 && (long long)beg + m <= list_len;
}
// base + a 32-bit byte offset: with a uniform base the load needs one offset register, not a 64-bit address
__device__ __forceinline__ const uint16_t *at_bytes(const uint16_t *base, uint32_t bytes) {
  return reinterpret_cast<const uint16_t *>(reinterpret_cast<const char *>(base) + bytes);
}
__device__ __forceinline__ bf16x8 ld_frag(const uint16_t *p) { return *reinterpret_cast<const bf16x8 *>(p); }
// Weight bytes are read exactly once: load them with the non-temporal hint so that the stream does
// not push the (re-read) token rows out of the caches.
__device__ __forceinline__ bf16x8 ld_stream(const uint16_t *p) {
  return __builtin_nontemporal_load(reinterpret_cast<const bf16x8 *>(p));
}

// Workgroup -> (segment, row tile) for the LDS-tiled passes.  Workgroups are handed to the 8 XCDs
// round-robin by linear id, and each XCD has an L2 of its own and a share of the chip's streaming
// bandwidth.  The work items are the non-empty segments, largest first (a segment of more than 128 pairs
// counts as several, one per piece; "segment" below means work item).  Whole rounds of 8 segments are dealt
// one segment per XCD (all row tiles of a segment get ids that are equal modulo 8, so that its token
// rows are fetched into one L2); the L mod 8 segments left over (all of them when L < 8) have their
// row tiles cut into 8 equal contiguous ranges, one per XCD, so that every XCD streams the same
// number of bytes.  Measured on an idle chip, an XCD places its workgroups on its 32 compute units
// round-robin in id order, two per unit, and a workgroup with many token tiles runs slower than one
// with few (more LDS and matrix work per weight byte); in this order the heavy workgroups of the
// first rounds share their compute unit with the light ones of the later rounds, or with nothing.
// Returns false if the workgroup has no work.  L = number of work items.
constexpr int kXcds = 8;
__device__ __forceinline__ bool xcd_map(int tiles, int L, int &rank, int &tile) {
  const int x = blockIdx.x % kXcds, j = blockIdx.x / kXcds;
  const int full = L / kXcds, rest = L % kXcds;
  if (j < full * tiles) {
    rank = x + kXcds * (j / tiles);
    tile = j % tiles;
    return true;
  }
  const int wr = rest * tiles, lo = wr * x / kXcds, hi = wr * (x + 1) / kXcds;
  const int w = lo + (j - full * tiles);
  rank = full * kXcds + w / tiles;
  tile = w % tiles;
  return w < hi;
}
// items[0].x = number of work items L; items[1 + r] = (segment index, expert, offset, size) of item r: the
// non-empty segments, largest first, each cut into piece_count(size) pieces.  The table has cap + 1 entries.
// tiles_of(L, large): the row tiles of an item when there are L of them and large says that the largest has more than 64 pairs.
template <class TF>
__device__ __forceinline__ int4 xcd_item(TF tiles_of, int cap, const int4 *__restrict__ items, int &tile, int &rank) {
  int L = items[0].x;
  L = L < 0 ? 0 : (L > cap ? cap : L);
  return xcd_map(tiles_of(L, L > 0 && items[1].w > 64), L, rank, tile) ? items[1 + rank] : int4{-1, -1, 0, 0};
}
// The table above built from segment arrays that did not come from the budget stage.  One workgroup.
// Only well-formed segments take part (inside the pair table, at most one pair per token), and only as
// long as their pieces fit the table (they always do when the segments are disjoint).
__global__ __launch_bounds__(256) void segment_items_kernel(const int32_t *__restrict__ seg_expert,
                                                            const int32_t *__restrict__ seg_off, int n_seg, int M,
                                                            int k, int cap, int4 *__restrict__ items) {
  __shared__ int n_items, sizes[1024];  // n_seg <= n_experts <= 1024
  if (threadIdx.x == 0) n_items = 0;
  for (int j = threadIdx.x; j < n_seg; j += blockDim.x) {
    const int lo = seg_off[j], c = seg_off[j + 1] - lo;
    sizes[j] = (lo >= 0 && c > 0 && c <= M && (long long)lo + c <= (long long)M * k) ? c : 0;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < n_seg; i += blockDim.x) {
    const int c = sizes[i];
    if (c > 0) {
      int first = 0;  // pieces of the segments that rank before this one
      for (int j = 0; j < n_seg; ++j) {
        const int cj = sizes[j];
        first += (cj > c || (cj == c && j < i)) ? piece_count(cj) : 0;
      }
      const int q = piece_count(c), len = (c + q - 1) / q, lo = seg_off[i];
      if (first + q <= cap) {
        for (int p = 0; p < q; ++p)
          items[1 + first + p] = int4{i, seg_expert[i], lo + p * len, min(len, c - p * len)};
        atomicAdd(&n_items, q);
      }
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) items[0] = int4{n_items, 0, 0, 0};
}
// Workgroups of a pass: room for whole rounds of 8 work items.
inline int xcd_grid(int tiles, int n_items) { return kXcds * tiles * ((n_items + kXcds - 1) / kXcds); }

// Start offset (elements) of a walk over K: 128 elements (256 bytes) apart for consecutive ids.  The ids are made of the
// expert and the row tile, not of the order of the work items: every route to the passes adds in the same order.  (By
// rank, by expert alone and by 5 e + 3 tile: 582 / 587 / 582 us for four layers of two 4096 x 14336 experts, the others
// within 0.7 %; by e + tile 627.)
__device__ __forceinline__ int k_stagger(int id, int K) { return (int)(((long long)id * 128) % K); }

// ---- LDS-tiled bf16 passes  --------------------------------------------------------
// Geometry of one K chunk: U MFMA K-steps of 32 elements; a row of the chunk is RB = 64 U bytes =
// CPR = 4 U pieces of 16 bytes.  Piece c of row r sits at LDS offset r*RB + ((c ^ (r & (CPR-1))) * 16):
// 8 consecutive lanes then touch 8 different 16-byte bank groups both when a row is written
// (lanes along the row) and when it is read in operand layout (lanes across rows).
template <int U>
struct Chunk {
  static constexpr int KC = 32 * U;        // elements per chunk
  static constexpr int CPR = 4 * U;        // 16-byte pieces per row
  static constexpr int RB = 64 * U;        // bytes per row
  static constexpr int RPI = 64 / CPR;     // rows covered by one wave-wide load
  static constexpr int TILE = 16 * RB;     // bytes of a 16-row tile
  static __device__ __forceinline__ int swz(int row, int piece) { return row * RB + ((piece ^ (row & (CPR - 1))) << 4); }
};

// The wave index is taken through readfirstlane in these kernels: it is uniform within a wave, and the
// compiler then keeps everything derived from it (row offsets, tile bases) in scalar registers.
constexpr int kPrefetchTiles = 4;  // walks of up to this many token tiles read their LDS operands one K-step ahead
constexpr int kLdsBytes = 65536;  // 32 KB of wave-private weight tiles + token tile: 2 x (4..16) KB or 1 x 32 KB

// One workgroup pass over K for NT token tiles.  wt0 / wt1: first row of this wave's two 16-row weight
// tiles (row stride K elements).  xbase + xsrc[q] bytes: this lane's source row (already at its 16-byte piece)
// for its q-th share of the token tile.  Accumulates acc0[j] (tile 0) and acc1[j] (tile 1) over the K range
// [kb, kb + kl) of the rows (row stride K).
// make_xsrc(xsrc) fills the token-row offsets from the pair ids the caller has ALREADY loaded into registers; it is
// called after the weight loads of the first chunk have been issued.  Loads complete in issue order, so the wait for
// the (earlier issued) pair ids leaves those weight loads in flight: the expert's first bytes are on their way while
// the token rows are still being looked up.
template <int NT, int U, bool kTail, class XF>
__device__ __forceinline__ void lds_pass(const uint16_t *wt0, const uint16_t *wt1, int K, int kb, int kl, int ks,
                                         const uint16_t *xbase, XF make_xsrc, unsigned char *lds,
                                         f32x4 (&acc0)[NT], f32x4 (&acc1)[NT]) {
  using C = Chunk<U>;
  constexpr int IPW = NT * U / 4;  // token-tile loads per wave per chunk (4 waves share the tile)
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  unsigned char *a_lds = lds + wave * 2 * C::TILE;                 // wave-private: two weight tiles
  constexpr int XBUF = NT * 16 * C::RB;
  unsigned char *x_lds = lds + kFfnWaves * 2 * C::TILE;  // shared: 2 buffers of NT*16 rows
  // two token-tile buffers if they fit beside the weight tiles, else one (and a second barrier per chunk)
  constexpr bool kDoubleX = kFfnWaves * 2 * C::TILE + 2 * XBUF <= kLdsBytes;

  // global -> register staging
  // uniform base + 32-bit byte offset per lane (a tile is 16 rows of at most 2^20 elements): the loads need
  // one offset register each instead of a 64-bit address
  const int lrow = lane / C::CPR, lpc = lane % C::CPR;
  const uint32_t lane_off = 2u * ((uint32_t)lrow * (uint32_t)K + (uint32_t)lpc * 8u);
  bf16x8 GA[2][U], GX[IPW];
  uint32_t xsrc[IPW];
  // kTail: whether this lane's piece of the chunk at element k lies inside the row (the same piece for weights and
  // tokens); a lane past the end loads the first piece of its group of rows again and parks zeros
  auto inside = [&](int k) { return !kTail || k + lpc * 8 < kb + kl; };
  auto issue_w = [&](int k) {
    const uint32_t back = inside(k) ? 0u : (uint32_t)lpc * 16u;
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const uint32_t off = lane_off + 2u * ((uint32_t)(q * C::RPI) * (uint32_t)K + (uint32_t)k) - back;
      GA[0][q] = ld_stream(at_bytes(wt0, off));
      GA[1][q] = ld_stream(at_bytes(wt1, off));
    }
  };
  auto issue_x = [&](int k) {
    const uint32_t back = inside(k) ? 0u : (uint32_t)lpc * 16u;
#pragma unroll
    for (int q = 0; q < IPW; ++q) GX[q] = ld_frag(at_bytes(xbase, xsrc[q] + 2u * (uint32_t)k - back));
  };
  auto issue = [&](int k) {
    issue_w(k);
    issue_x(k);
  };
  auto park = [&](int buf, int k) {
    if (kTail && !inside(k)) {
#pragma unroll
      for (int q = 0; q < U; ++q) GA[0][q] = GA[1][q] = bf16x8{};
#pragma unroll
      for (int q = 0; q < IPW; ++q) GX[q] = bf16x8{};
    }
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int row = q * C::RPI + lrow;
      *reinterpret_cast<bf16x8 *>(a_lds + C::swz(row, lpc)) = GA[0][q];
      *reinterpret_cast<bf16x8 *>(a_lds + C::TILE + C::swz(row, lpc)) = GA[1][q];
    }
#pragma unroll
    for (int q = 0; q < IPW; ++q) {
      const int g = (wave * IPW + q) * 64 + lane;
      *reinterpret_cast<bf16x8 *>(x_lds + buf * XBUF + C::swz(g / C::CPR, g % C::CPR)) = GX[q];
    }
  };
  const int r = lane & 15, kg = lane >> 4;
  // Up to kPrefetchTiles token tiles: the operands of K-step u + 1 are read from LDS into a second register set
  // before the matrix instructions of step u are issued, so that the LDS latency of a step is covered by the
  // previous step's MFMAs (the scheduling barriers keep the compiler from sinking the reads back to their uses).
  // With 8 token tiles the registers do not hold a second set and the reads stay next to their uses (measured:
  // issuing all reads of a step first is 2-4 % slower there).
  auto compute = [&](int buf) {
    if constexpr (NT <= kPrefetchTiles) {
      bf16x8 fa0[2], fa1[2], fb[2][NT];
      auto fetch = [&](int u) {
        const int pc = 4 * u + kg, st = u & 1;
        fa0[st] = *reinterpret_cast<const bf16x8 *>(a_lds + C::swz(r, pc));
        fa1[st] = *reinterpret_cast<const bf16x8 *>(a_lds + C::TILE + C::swz(r, pc));
#pragma unroll
        for (int j = 0; j < NT; ++j)
          fb[st][j] = *reinterpret_cast<const bf16x8 *>(x_lds + buf * XBUF + C::swz(16 * j + r, pc));
      };
      fetch(0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (u + 1 < U) fetch(u + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          acc0[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa0[u & 1], fb[u & 1][j], acc0[j], 0, 0, 0);
          acc1[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa1[u & 1], fb[u & 1][j], acc1[j], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int pc = 4 * u + kg;
        const bf16x8 a0 = *reinterpret_cast<const bf16x8 *>(a_lds + C::swz(r, pc));
        const bf16x8 a1 = *reinterpret_cast<const bf16x8 *>(a_lds + C::TILE + C::swz(r, pc));
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          const bf16x8 b = *reinterpret_cast<const bf16x8 *>(x_lds + buf * XBUF + C::swz(16 * j + r, pc));
          acc0[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b, acc0[j], 0, 0, 0);
          acc1[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b, acc1[j], 0, 0, 0);
        }
      }
    }
  };

  // the walk covers the elements [kb, kb + kl) of every row in chunks (kl a multiple of the chunk unless kTail), starting
  // ks elements into that range and wrapping inside it
  const int nst = kTail ? (kl + C::KC - 1) / C::KC : kl / C::KC;
  int k = ((ks % kl) / C::KC) * C::KC;
  issue_w(kb + k);
  __builtin_amdgcn_sched_barrier(0);  // keep the weight loads ahead of the wait for the pair ids
  make_xsrc(xsrc);
  issue_x(kb + k);
  for (int i = 0; i < nst; ++i) {
    park(kDoubleX ? (i & 1) : 0, kb + k);
    k += C::KC;
    k = k >= nst * C::KC ? 0 : k;
    if (i + 1 < nst) issue(kb + k);
    __syncthreads();  // token tile i complete; also orders this wave's tile writes before its reads
    compute(kDoubleX ? (i & 1) : 0);
    if (!kDoubleX) __syncthreads();  // everybody has read the single token tile before it is overwritten
  }
  __syncthreads();  // the LDS tiles may be reused by the caller's next pass
}

// The walk of a wave that has a part [kb, kb + kl) of K to itself: it shares nothing with the other waves and waits for none
// of them (the caller adds up their sums).  Two token tiles at a time go through the LDS, against the chunk of weights parked
// there, so that a chunk is read from memory once for all NT tiles.  Loads return in the order of their issue: the next
// chunk of weights is requested after the last tokens of the present one.  make_off(xsrc) is called with the first weights on
// their way.  Up to two token tiles: it fills xsrc with the byte offsets from xbase of the rows that this lane loads.  More: it fills
// xoff[0 .. 16 NT), in the LDS, with those of all pairs, and synchronises.
template <int NT, bool kTail, class XF>
__device__ __forceinline__ void cut_pass(const uint16_t *wt0, const uint16_t *wt1, int K, int kb, int kl, int ks,
                                         const uint16_t *xbase, const uint32_t *xoff, XF make_off, unsigned char *lds,
                                         f32x4 (&acc0)[NT], f32x4 (&acc1)[NT]) {
  constexpr int U = 4;
  using C = Chunk<U>;
  constexpr int G = NT < 2 ? 1 : 2, NG = NT / G, IPW = G * U;  // tiles and loads of a group of tokens
  static_assert(kFfnWaves * (2 + G) * C::TILE <= kLdsBytes, "private tiles fit the LDS");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  unsigned char *a_lds = lds + wave * (2 + G) * C::TILE, *x_lds = a_lds + 2 * C::TILE;
  const int lrow = lane / C::CPR, lpc = lane % C::CPR;
  const uint32_t lane_off = 2u * ((uint32_t)lrow * (uint32_t)K + (uint32_t)lpc * 8u);
  bf16x8 GA[2][U], GX[IPW];
  uint32_t xsrc[IPW];
  auto inside = [&](int k) { return !kTail || k + lpc * 8 < kb + kl; };  // see lds_pass
  auto issue_w = [&](int k) {
    const uint32_t back = inside(k) ? 0u : (uint32_t)lpc * 16u;
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const uint32_t off = lane_off + 2u * ((uint32_t)(q * C::RPI) * (uint32_t)K + (uint32_t)k) - back;
      GA[0][q] = ld_stream(at_bytes(wt0, off));
      GA[1][q] = ld_stream(at_bytes(wt1, off));
    }
  };
  auto issue_x = [&](int g, int k) {
    const uint32_t at = 2u * (uint32_t)k + (inside(k) ? (uint32_t)lpc * 16u : 0u);
#pragma unroll
    for (int q = 0; q < IPW; ++q)
      GX[q] = ld_frag(at_bytes(xbase, (NG == 1 ? xsrc[q] : xoff[g * 16 * G + q * C::RPI + lrow]) + at));
  };
  auto park_w = [&](int k) {
    const bool in = inside(k);
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int row = q * C::RPI + lrow;
      *reinterpret_cast<bf16x8 *>(a_lds + C::swz(row, lpc)) = in ? GA[0][q] : bf16x8{};
      *reinterpret_cast<bf16x8 *>(a_lds + C::TILE + C::swz(row, lpc)) = in ? GA[1][q] : bf16x8{};
    }
  };
  auto park_x = [&](int k) {
    const bool in = inside(k);
#pragma unroll
    for (int q = 0; q < IPW; ++q)
      *reinterpret_cast<bf16x8 *>(x_lds + C::swz(q * C::RPI + lrow, lpc)) = in ? GX[q] : bf16x8{};
  };
  const int r = lane & 15, kg = lane >> 4;
  auto compute = [&](int g) {
    bf16x8 fa0[2], fa1[2], fb[2][G];  // the operands of step u + 1 are read before the matrix instructions of step u
    auto fetch = [&](int u) {
      const int pc = 4 * u + kg, st = u & 1;
      fa0[st] = *reinterpret_cast<const bf16x8 *>(a_lds + C::swz(r, pc));
      fa1[st] = *reinterpret_cast<const bf16x8 *>(a_lds + C::TILE + C::swz(r, pc));
#pragma unroll
      for (int j = 0; j < G; ++j) fb[st][j] = *reinterpret_cast<const bf16x8 *>(x_lds + C::swz(16 * j + r, pc));
    };
    fetch(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u + 1 < U) fetch(u + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < G; ++j) {
        acc0[g * G + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa0[u & 1], fb[u & 1][j], acc0[g * G + j], 0, 0, 0);
        acc1[g * G + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa1[u & 1], fb[u & 1][j], acc1[g * G + j], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  const int nst = kTail ? (kl + C::KC - 1) / C::KC : kl / C::KC;
  int k = ((ks % kl) / C::KC) * C::KC;
  issue_w(kb + k);
  __builtin_amdgcn_sched_barrier(0);  // keep the weight loads ahead of the wait for the pair ids
  make_off(xsrc);
  issue_x(0, kb + k);
  // one chunk; last: none behind it.  Without a branch around the loads, so that the waits can be counted.
  auto chunk = [&](auto last_) {
    constexpr bool last = decltype(last_)::value;
    int kn = k + C::KC;
    kn = kn >= nst * C::KC ? 0 : kn;
    park_w(kb + k);
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      park_x(kb + k);
      if (g + 1 < NG) issue_x(g + 1, kb + k);
      if (!last && g + 2 >= NG && (NG == 1 || g + 2 == NG)) issue_w(kb + kn);
      if (!last && g + 1 == NG) issue_x(0, kb + kn);
      wave_lds_sync();
      compute(g);
      wave_lds_sync();
    }
    k = kn;
  };
  for (int i = 0; i + 1 < nst; ++i) chunk(std::false_type{});
  chunk(std::true_type{});
  __syncthreads();  // the caller reuses the LDS
}

// The workgroup's work item found in the fused prologue's lists: shortlist[r] = expert with rank r in the shortlist
// (descending aggregate score, which is also roughly descending segment size), rank_count[r] = number of its surviving
// pairs, listed at lists + r * list_stride.  The work items are the pieces (piece_count per expert) of the shortlisted
// experts in rank order; the workgroup takes the one that xcd_map assigns to it.  Requires B <= kFfnThreads.
// Every wave looks for itself, a lane per rank, with counts of ballots instead of a scan through LDS and two barriers: nothing of
// the pass is requested before the item is known.  The results are uniform, so that the addresses made of them stay in scalar
// registers.  Returns the expert (-1: no work item), its piece of m pairs (list) and the work item's number.
template <class TF>
__device__ __forceinline__ int listed_segment(const int32_t *__restrict__ rank_count,
                                              const int32_t *__restrict__ shortlist, int B, TF tiles_of,
                                              int &m, int &item, int &tile, const int32_t *__restrict__ lists,
                                              int list_stride, const int32_t *&list) {
  constexpr int kGroups = kFfnThreads / kWave;  // of 64 ranks
  const int lane = threadIdx.x & 63;
  const unsigned long long below = (1ull << lane) - 1ull;
  int c[kGroups], ex[kGroups], first[kGroups], n_items = 0;
  bool large = false;
#pragma unroll
  for (int i = 0; i < kGroups; ++i) {
    const int r = i * kWave + lane;
    c[i] = r < B ? rank_count[r] : 0;
    ex[i] = r < B ? shortlist[r] : -1;
  }
#pragma unroll
  for (int i = 0; i < kGroups; ++i) {
    first[i] = n_items;
    if (i * kWave < B) {  // uniform
      const int q = piece_count(max(c[i], 0));
      large |= __ballot(c[i] > 64) != 0;
      for (int bit = 0; __ballot((q >> bit) != 0) != 0; ++bit) {
        const unsigned long long set = __ballot((q >> bit) & 1);
        first[i] += __popcll(set & below) << bit;
        n_items += __popcll(set) << bit;
      }
    }
  }
  m = 0;
  list = lists;
  int e = -1;
  if (!xcd_map(tiles_of(n_items, large), n_items, item, tile)) return e;
#pragma unroll
  for (int i = 0; i < kGroups; ++i) {
    if (i * kWave < B) {
      const int q = piece_count(max(c[i], 0));
      const unsigned long long hit = __ballot(item >= first[i] && item < first[i] + q);
      if (hit) {  // one lane
        const int src = __ffsll((long long)hit) - 1, size = __builtin_amdgcn_readlane(c[i], src);
        const int pieces = piece_count(size), len = (size + pieces - 1) / pieces;
        const int lo = (item - __builtin_amdgcn_readlane(first[i], src)) * len;
        e = __builtin_amdgcn_readlane(ex[i], src);
        m = min(len, size - lo);
        list = lists + (size_t)(i * kWave + src) * list_stride + lo;
      }
    }
  }
  return e;
}

// Whether the 4 waves of a workgroup take a quarter of K each (cut_pass) instead of a quarter of its rows (lds_pass): the same
// bytes are in flight per workgroup, but there are four times as many of them and a walk is a quarter as long; in exchange
// every 32 weight rows load the tokens for themselves.  That pays until the workgroups of the other form, `units`, would
// occupy every second compute unit, and a little longer where a walk by rows is slowed down by more than 64 pairs.  489
// passes measured (512 to 4096 x 128 to 2048, 1 to 250 tokens, 1 to 85 loaded experts), time by rows / by K: 1.0 to 2.2,
// mostly 1.5, at up to 120 units; then up to 64 pairs 1.1 to 1.35 at 128 to 135, 0.85 to 0.95 at 140 to 200; more
// pairs 1.0 to 1.7 at 130 to 160, 0.75 to 1.7 at 160 to 190, 0.8 to 1.0 above 200 (gate/up of 42 experts of 2048 x 192 with up
// to 126 pairs, 126 units: 37.7 / 20.5 us; of 27 of 2048 x 1024, 432 units: 40 / 52).  How many experts are loaded is known
// here only: the host's bound, the shortlist, is up to ten times that.
constexpr int kCutUnits = 132, kCutUnitsLarge = 176;
__device__ __forceinline__ bool walk_is_cut(int units, bool large, int K, int splits) {
  return splits == 1 && K >= 4 * 128 && units <= (large ? kCutUnitsLarge : kCutUnits);
}

// plist: the segment's pairs (flat ids t * k + slot, tokens ascending), in global memory or LDS; n_pairs = M * k.
__device__ __forceinline__ int pair_at(const int32_t *plist, int p, int n_pairs) {
  const int q = plist[p];
  return q < 0 ? 0 : (q >= n_pairs ? n_pairs - 1 : q);
}

// The sums of the 4 waves added in wave order; wave w gets the totals of the token tiles w, w + 4.  Synchronises; the caller may use the
// LDS again afterwards.
template <int NT>
__device__ __forceinline__ void add_waves(unsigned char *lds, f32x4 (&a0)[NT], f32x4 (&a1)[NT]) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  static_assert(kFfnWaves * NT * 2 * 64 * sizeof(f32x4) <= kLdsBytes, "the sums fit the LDS");
  f32x4 *part = reinterpret_cast<f32x4 *>(lds);  // [wave][tile][2][lane]
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    part[((wave * NT + j) * 2 + 0) * 64 + lane] = a0[j];
    part[((wave * NT + j) * 2 + 1) * 64 + lane] = a1[j];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < NT; ++j)
    if (j % kFfnWaves == wave) {
      a0[j] = part[(j * 2 + 0) * 64 + lane];
      a1[j] = part[(j * 2 + 1) * 64 + lane];
#pragma unroll
      for (int w = 1; w < kFfnWaves; ++w) {
        a0[j] += part[((w * NT + j) * 2 + 0) * 64 + lane];
        a1[j] += part[((w * NT + j) * 2 + 1) * 64 + lane];
      }
    }
  __syncthreads();
}

// Whether token tile j is this wave's to store (kCut: the waves have shared the tiles out, see add_waves).
template <bool kCut>
__device__ __forceinline__ bool own_tile(int j, int wave) { return !kCut || j % kFfnWaves == wave; }

// kCut: cut_pass instead of lds_pass, the waves' sums added up; xoff: 128 words of LDS for it.
template <int NT, bool kTail, bool kCut>
__device__ __forceinline__ void gateup_lds(const uint16_t *wt0, const uint16_t *wt1, const uint16_t *__restrict__ h,
                                           const int32_t *plist, int n_pairs, int k, int d, int F, int kb, int kl, int m,
                                           int f0, int ks, unsigned char *lds, uint32_t *xoff, uint16_t *__restrict__ act) {
  using C = Chunk<4>;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // 32-bit byte offsets: M * d < 2^31 elements (checked on the host)
  auto row_off = [&](int pr) {
    pr = pr < 0 ? 0 : (pr >= n_pairs ? n_pairs - 1 : pr);
    return 2u * ((uint32_t)(pr / k) * (uint32_t)d);
  };
  f32x4 accg[NT], accu[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) accg[j] = accu[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  if constexpr (kCut) {
    constexpr bool kFew = NT <= 2;  // see cut_pass; pad rows repeat the last pair, and their columns are never stored
    constexpr int kPairs = kFew ? 4 * NT : 1;
    int pair[kPairs];
#pragma unroll
    for (int q = 0; q < kPairs; ++q) pair[q] = plist[min(kFew ? q * C::RPI + lane / C::CPR : (int)threadIdx.x, m - 1)];
    auto make_off = [&](auto &xsrc) {
      if constexpr (kFew) {
#pragma unroll
        for (int q = 0; q < kPairs; ++q) xsrc[q] = row_off(pair[q]);
      } else {
        if (threadIdx.x < 16 * NT) xoff[threadIdx.x] = row_off(pair[0]);
        __syncthreads();
      }
    };
    cut_pass<NT, kTail>(wt0, wt1, d, kb, kl, ks, h, xoff, make_off, lds, accg, accu);
    add_waves<NT>(lds, accg, accu);
  } else {
    int pair[NT];  // this lane's pair ids, loaded now and turned into row offsets inside lds_pass
#pragma unroll
    for (int q = 0; q < NT; ++q) pair[q] = plist[min(((wave * NT + q) * 64 + lane) / C::CPR, m - 1)];
    auto make_xsrc = [&](uint32_t (&xsrc)[NT]) {
#pragma unroll
      for (int q = 0; q < NT; ++q) xsrc[q] = row_off(pair[q]) + (uint32_t)(lane % C::CPR) * 16u;
    };
    lds_pass<NT, 4, kTail>(wt0, wt1, d, kb, kl, ks, h, make_xsrc, lds, accg, accu);
  }
  const int col = lane & 15, kg = lane >> 4;
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int p = j * 16 + col;
    if (p < m && own_tile<kCut>(j, wave)) {
      f32x4 o;
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = silu_f(accg[j][i]) * accu[j][i];
      store_bf16x4(act + (size_t)pair_at(plist, p, n_pairs) * F + f0 + 4 * kg, o);
    }
  }
}

// rank_count != NULL: work items from the prologue's lists (items / perm unused; n_seg = B); otherwise items + perm.
// A workgroup takes 64 gate and the same 64 up rows of an item, or, with its walk cut, 16 and 16.
template <bool kTail>
__global__ __launch_bounds__(kFfnThreads, 2) void ffn_gateup_lds_kernel(
    const int32_t *__restrict__ rank_count, const int32_t *__restrict__ shortlist, const int32_t *__restrict__ lists,
    int list_stride, int n_seg, int cap, int M, int N, int k, int d, int F, const int4 *__restrict__ items,
    const int32_t *__restrict__ perm, const uint16_t *__restrict__ h, const uint16_t *__restrict__ w_gate,
    const uint16_t *__restrict__ w_up, uint16_t *__restrict__ act) {
  __shared__ __align__(16) unsigned char lds[kLdsBytes];
  __shared__ uint32_t xoff[kPiecePairs];
  const int row_tiles = (F / 16 + kFfnWaves - 1) / kFfnWaves;
  bool cut = false;
  auto tiles_of = [&](int n_items, bool large) {
    cut = walk_is_cut(n_items * row_tiles, large, d, 1);
    return cut ? F / 16 : row_tiles;
  };
  int tile, rank, e, m;
  const int32_t *plist;
  if (rank_count) {
    e = listed_segment(rank_count, shortlist, n_seg, tiles_of, m, rank, tile, lists, list_stride, plist);
    if (e < 0 || e >= N || m <= 0 || m > kPiecePairs) return;
  } else {
    const int4 it = xcd_item(tiles_of, cap, items, tile, rank);
    e = it.y;
    m = it.w;
    if (it.x < 0 || m > kPiecePairs || !segment_ok(e, it.z, m, (long long)M * k, N)) return;
    plist = perm + it.z;
  }
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // F is a multiple of 32 but a workgroup covers 64 gate rows: the waves of a last, partial workgroup
  // redo rows of the previous tile (same values, same destination) so that every wave reaches the barriers.
  int f0 = cut ? tile * 16 : (tile * kFfnWaves + wave) * 16;
  f0 = f0 < F ? f0 : F - 16;
  const uint16_t *wt0 = w_gate + ((size_t)e * F + f0) * d;
  const uint16_t *wt1 = w_up + ((size_t)e * F + f0) * d;
  const int n_pairs = M * k;
  if (cut) {
    const int nch = (d + 127) / 128, kb = wave * nch / kFfnWaves * 128, kl = min((wave + 1) * nch / kFfnWaves * 128, d) - kb;
    const int ks = k_stagger(5 * e + 3 * tile, kl);
    if (m <= 16) gateup_lds<1, kTail, true>(wt0, wt1, h, plist, n_pairs, k, d, F, kb, kl, m, f0, ks, lds, xoff, act);
    else if (m <= 32) gateup_lds<2, kTail, true>(wt0, wt1, h, plist, n_pairs, k, d, F, kb, kl, m, f0, ks, lds, xoff, act);
    else if (m <= 64) gateup_lds<4, kTail, true>(wt0, wt1, h, plist, n_pairs, k, d, F, kb, kl, m, f0, ks, lds, xoff, act);
    else gateup_lds<8, kTail, true>(wt0, wt1, h, plist, n_pairs, k, d, F, kb, kl, m, f0, ks, lds, xoff, act);
  } else {
    const int ks = k_stagger(5 * e + 3 * tile, d);
    if (m <= 16) gateup_lds<1, kTail, false>(wt0, wt1, h, plist, n_pairs, k, d, F, 0, d, m, f0, ks, lds, xoff, act);
    else if (m <= 32) gateup_lds<2, kTail, false>(wt0, wt1, h, plist, n_pairs, k, d, F, 0, d, m, f0, ks, lds, xoff, act);
    else if (m <= 64) gateup_lds<4, kTail, false>(wt0, wt1, h, plist, n_pairs, k, d, F, 0, d, m, f0, ks, lds, xoff, act);
    else gateup_lds<8, kTail, false>(wt0, wt1, h, plist, n_pairs, k, d, F, 0, d, m, f0, ks, lds, xoff, act);
  }
}

template <int NT, bool kTail, bool kCut>
__device__ __forceinline__ void down_lds(const uint16_t *wt0, const uint16_t *wt1, const uint16_t *__restrict__ act,
                                         const int32_t *plist, int n_pairs, int d, int F, int kb, int kl, int m, int j0,
                                         int ks, unsigned char *lds, uint32_t *xoff, float *__restrict__ y) {
  using C = Chunk<4>;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // 32-bit byte offsets: M * k * F < 2^31 elements (checked on the host)
  auto row_off = [&](int pr) {
    pr = pr < 0 ? 0 : (pr >= n_pairs ? n_pairs - 1 : pr);
    return 2u * ((uint32_t)pr * (uint32_t)F);
  };
  f32x4 acc0[NT], acc1[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) acc0[j] = acc1[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  if constexpr (kCut) {
    constexpr bool kFew = NT <= 2;
    constexpr int kPairs = kFew ? 4 * NT : 1;
    int pair[kPairs];
#pragma unroll
    for (int q = 0; q < kPairs; ++q) pair[q] = plist[min(kFew ? q * C::RPI + lane / C::CPR : (int)threadIdx.x, m - 1)];
    auto make_off = [&](auto &xsrc) {
      if constexpr (kFew) {
#pragma unroll
        for (int q = 0; q < kPairs; ++q) xsrc[q] = row_off(pair[q]);
      } else {
        if (threadIdx.x < 16 * NT) xoff[threadIdx.x] = row_off(pair[0]);
        __syncthreads();
      }
    };
    cut_pass<NT, kTail>(wt0, wt1, F, kb, kl, ks, act, xoff, make_off, lds, acc0, acc1);
    add_waves<NT>(lds, acc0, acc1);
  } else {
    int pair[NT];  // this lane's pair ids, loaded now and turned into row offsets inside lds_pass
#pragma unroll
    for (int q = 0; q < NT; ++q) pair[q] = plist[min(((wave * NT + q) * 64 + lane) / C::CPR, m - 1)];
    auto make_xsrc = [&](uint32_t (&xsrc)[NT]) {
#pragma unroll
      for (int q = 0; q < NT; ++q) xsrc[q] = row_off(pair[q]) + (uint32_t)(lane % C::CPR) * 16u;
    };
    lds_pass<NT, 4, kTail>(wt0, wt1, F, kb, kl, ks, act, make_xsrc, lds, acc0, acc1);
  }
  const int col = lane & 15, kg = lane >> 4;
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int p = j * 16 + col;
    if (p < m && own_tile<kCut>(j, wave)) {
      float *dst = y + (size_t)pair_at(plist, p, n_pairs) * d + j0 + 4 * kg;
      *reinterpret_cast<f32x4 *>(dst) = acc0[j];
      *reinterpret_cast<f32x4 *>(dst + 16) = acc1[j];
    }
  }
}

template <bool kTail>
__global__ __launch_bounds__(kFfnThreads, 2) void ffn_down_lds_kernel(
    const int32_t *__restrict__ rank_count, const int32_t *__restrict__ shortlist, const int32_t *__restrict__ lists,
    int list_stride, int n_seg, int cap, int M, int N, int k, int d, int F, int splits, const int4 *__restrict__ items,
    const int32_t *__restrict__ perm, const uint16_t *__restrict__ act, const uint16_t *__restrict__ w_down,
    float *__restrict__ y) {
  __shared__ __align__(16) unsigned char lds[kLdsBytes];
  __shared__ uint32_t xoff[kPiecePairs];
  // a work item is (row tile, K split): split sp sums the 128-element chunks [sp n / splits, (sp + 1) n / splits)
  // of F into its own copy of y, which the combine adds up in split order
  const int row_tiles = ((d / 32 + kFfnWaves - 1) / kFfnWaves) * splits;
  bool cut = false;
  auto tiles_of = [&](int n_items, bool large) {
    cut = walk_is_cut(n_items * row_tiles, large, F, splits);
    return cut ? d / 32 : row_tiles;
  };
  int tile, rank, e, m;
  const int32_t *plist;
  if (rank_count) {
    e = listed_segment(rank_count, shortlist, n_seg, tiles_of, m, rank, tile, lists, list_stride, plist);
    if (e < 0 || e >= N || m <= 0 || m > kPiecePairs) return;
  } else {
    const int4 it = xcd_item(tiles_of, cap, items, tile, rank);
    e = it.y;
    m = it.w;
    if (it.x < 0 || m > kPiecePairs || !segment_ok(e, it.z, m, (long long)M * k, N)) return;
    plist = perm + it.z;
  }
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sp = cut ? 0 : tile % splits;
  if (!cut) tile /= splits;
  int j0 = cut ? tile * 32 : (tile * kFfnWaves + wave) * 32;
  j0 = j0 < d ? j0 : d - 32;  // see ffn_gateup_lds_kernel
  const uint16_t *wt0 = w_down + ((size_t)e * d + j0) * F;
  const uint16_t *wt1 = wt0 + (size_t)16 * F;
  const int part = cut ? wave : sp, parts = cut ? kFfnWaves : splits;
  const int nch = (F + 127) / 128, kb = (int)((long long)part * nch / parts) * 128;
  const int kl = min((int)((long long)(part + 1) * nch / parts) * 128, F) - kb;
  const int ks = k_stagger(5 * e + sp + 3 * tile, kl);
  const int n_pairs = M * k;
  y += (size_t)sp * n_pairs * d;
  if (cut) {
    if (m <= 16) down_lds<1, kTail, true>(wt0, wt1, act, plist, n_pairs, d, F, kb, kl, m, j0, ks, lds, xoff, y);
    else if (m <= 32) down_lds<2, kTail, true>(wt0, wt1, act, plist, n_pairs, d, F, kb, kl, m, j0, ks, lds, xoff, y);
    else if (m <= 64) down_lds<4, kTail, true>(wt0, wt1, act, plist, n_pairs, d, F, kb, kl, m, j0, ks, lds, xoff, y);
    else down_lds<8, kTail, true>(wt0, wt1, act, plist, n_pairs, d, F, kb, kl, m, j0, ks, lds, xoff, y);
  } else {
    if (m <= 16) down_lds<1, kTail, false>(wt0, wt1, act, plist, n_pairs, d, F, kb, kl, m, j0, ks, lds, xoff, y);
    else if (m <= 32) down_lds<2, kTail, false>(wt0, wt1, act, plist, n_pairs, d, F, kb, kl, m, j0, ks, lds, xoff, y);
    else if (m <= 64) down_lds<4, kTail, false>(wt0, wt1, act, plist, n_pairs, d, F, kb, kl, m, j0, ks, lds, xoff, y);
    else down_lds<8, kTail, false>(wt0, wt1, act, plist, n_pairs, d, F, kb, kl, m, j0, ks, lds, xoff, y);
  }
}

// ---- fp32 path ------------------------------------------------------------------------------------------------
// Vector form, for trees of one or two tokens, of up to 8 over large weights, and for the gate/up pass over short rows by the ten
// thousand with few pairs each: a stream of weights.
// A wave owns 8 weight rows (gate/up: 4 gate rows and the same 4 up rows) and P pairs at a time: lane l adds the
// products of the elements l, l + 64, ... of K in ascending order, 8 P sums side by side, and the 64 lanes of a sum are
// folded in the order 32, 16, 8, 4, 2, 1.  The sums are folded together: in each step a lane keeps one half of them and
// hands the other half over, so that 8 P sums cost 8 P - 1 exchanges in all and every lane ends with one of them.
// What bounds it: reading the weights; with many pairs the fp32 multiply-adds (packed fp32 is not used) and their loads, 16 per 64 of
// them, which is why those go to the matrix cores (below).
constexpr int kF32Rows = 8, kF32Pairs = 8;

// v[0 .. n/2) = the sums of the half of v[0 .. n) that this lane keeps: lanes with bit MASK set keep the upper half
template <int MASK, int N_>
__device__ __forceinline__ void fold_half(float *v) {
#pragma unroll
  for (int a = 0; a < N_ / 2; ++a) {
    if constexpr (MASK >= 16) {
      // swaps the odd rows of 32 (16) lanes of one register with the even rows of the other
      const auto r = MASK == 32 ? __builtin_amdgcn_permlane32_swap(__float_as_uint(v[a]), __float_as_uint(v[a + N_ / 2]), false, false)
                                : __builtin_amdgcn_permlane16_swap(__float_as_uint(v[a]), __float_as_uint(v[a + N_ / 2]), false, false);
      v[a] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    } else {
      const bool up = (threadIdx.x & MASK) != 0;
      const float keep = up ? v[a + N_ / 2] : v[a], give = up ? v[a] : v[a + N_ / 2];
      v[a] = keep + __shfl_xor(give, MASK, kWave);
    }
  }
}
// After it, lane l holds the complete sum number l / (64 / N_) in v[0].
template <int N_>
__device__ __forceinline__ float fold_sums(float (&v)[N_]) {
  static_assert(N_ == 8 || N_ == 16 || N_ == 32 || N_ == 64, "one to eight lanes per sum");
  fold_half<32, N_>(v);
  fold_half<16, N_ / 2>(v);
  fold_half<8, N_ / 4>(v);
  if constexpr (N_ >= 16) fold_half<4, N_ / 8>(v);
  else v[0] += __shfl_xor(v[0], 4, kWave);
  if constexpr (N_ >= 32) fold_half<2, N_ / 16>(v);
  else v[0] += __shfl_xor(v[0], 2, kWave);
  if constexpr (N_ == 64) fold_half<1, 2>(v);
  else v[0] += __shfl_xor(v[0], 1, kWave);
  return v[0];
}

// sums[r * P + p] = this lane's part of row[r] . x[p] over K
template <int P>
__device__ __forceinline__ void f32_dots(const float *const (&row)[kF32Rows], const float *const (&x)[P], int K,
                                         float (&sums)[kF32Rows * P]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < kF32Rows * P; ++i) sums[i] = 0.f;
  constexpr int kUnroll = P <= 2 ? 8 : 2;  // few pairs leave the registers for more loads in flight (8 against 4: 2 to 5 %)
#pragma unroll kUnroll
  for (int j0 = 0; j0 < K; j0 += kWave) {
    const int j = j0 + lane;
    const bool in = j < K;  // lanes past the end add +0 * +0
    float w[kF32Rows], xv[P];
#pragma unroll
    for (int r = 0; r < kF32Rows; ++r) w[r] = in ? row[r][j] : 0.f;
#pragma unroll
    for (int p = 0; p < P; ++p) xv[p] = in ? x[p][j] : 0.f;
#pragma unroll
    for (int r = 0; r < kF32Rows; ++r)
#pragma unroll
      for (int p = 0; p < P; ++p) sums[r * P + p] = fmaf(w[r], xv[p], sums[r * P + p]);
  }
}

// The work of grid row `seg`: a shortlist rank of the prologue's lists, a work item of the budget stage or a segment of the
// caller's arrays.  Ranks and work items come largest first, so that the last round of workgroups is a short one, and work
// items end at 128 pairs, so that more of them run side by side.  Whole layer of 300 tokens, us, by rank / by ascending
// segment / by work item: 40 experts of 1024 x 512, top-6, 329 / 349 / 289; 8 of 256 x 1024, top-2, 159 / 155 / 91.
// kItems: the kernels for work items are their own; as one more choice at run time it cost the others 3 %.
template <bool kItems>
__device__ __forceinline__ bool f32_segment(int seg, const int32_t *seg_expert, const int32_t *seg_off, const int4 *items,
                                            const int32_t *perm, const int32_t *rank_count, const int32_t *shortlist,
                                            const int32_t *lists, int list_stride, int M, int N, int k, int &e, int &m,
                                            const int32_t *&plist) {
  if constexpr (kItems) {
    if (seg >= items[0].x) return false;
    const int4 it = items[1 + seg];  // gridDim.y does not exceed the table
    e = it.y;
    m = it.w;
    plist = perm + it.z;
    return segment_ok(e, it.z, m, (long long)M * k, N);
  }
  if (rank_count) {
    e = shortlist[seg];
    m = rank_count[seg];
    plist = lists + (size_t)seg * list_stride;
    return e >= 0 && e < N && m > 0 && m <= M;
  }
  e = seg_expert[seg];
  const int beg = seg_off[seg];
  m = seg_off[seg + 1] - beg;
  plist = perm + beg;
  return segment_ok(e, beg, m, (long long)M * k, N);
}

template <int P>
__device__ __forceinline__ void gateup_f32_tile(const float *__restrict__ h, const float *wg, const float *wu,
                                                const int32_t *plist, int p0, int m, int n_pairs, int k, int d, int F,
                                                int f0, float *__restrict__ act) {
  const int lane = threadIdx.x & 63;
  const float *row[kF32Rows], *x[P];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int f = min(f0 + r, F - 1);
    row[r] = wg + (size_t)f * d;
    row[4 + r] = wu + (size_t)f * d;
  }
#pragma unroll
  for (int p = 0; p < P; ++p) x[p] = h + (size_t)(pair_at(plist, min(p0 + p, m - 1), n_pairs) / k) * d;
  float sums[kF32Rows * P];
  f32_dots<P>(row, x, d, sums);
  const float g = fold_sums(sums), u = __shfl_xor(g, 32, kWave);
  constexpr int LPS = 64 / (kF32Rows * P);  // lanes per sum
  const int idx = lane / LPS, f = f0 + idx / P, p = p0 + idx % P;
  if (lane < 32 && lane % LPS == 0 && f < F && p < m) act[(size_t)pair_at(plist, p, n_pairs) * F + f] = g / (1.0f + expf(-g)) * u;
}

// kFew: every segment has at most two pairs (trees of one or two tokens), so that the passes are a stream of weights: 8 rows
// against a tile of 4 pairs spent a third of the loads and three quarters of the sums on pairs that are not there (one token,
// 2 experts of 4096 x 14336: 340 us per layer against 290; 8 of 1024 x 2048: 69 / 62).  A kernel of its own, because in one
// kernel with the larger tiles each costs the other its registers (154 VGPRs against 168 to 170).
template <bool kFew, bool kItems>
__global__ __launch_bounds__(kFfnThreads) void ffn_gateup_f32_kernel(
    const int32_t *__restrict__ rank_count, const int32_t *__restrict__ shortlist, const int32_t *__restrict__ lists,
    int list_stride, int M, int N, int k, int d, int F, const float *__restrict__ w_gate, const float *__restrict__ w_up,
    const float *__restrict__ h, const int32_t *__restrict__ seg_expert, const int32_t *__restrict__ seg_off,
    const int4 *__restrict__ items, const int32_t *__restrict__ perm, float *__restrict__ act) {
  int e, m;
  const int32_t *plist;
  if (!f32_segment<kItems>(blockIdx.y, seg_expert, seg_off, items, perm, rank_count, shortlist, lists, list_stride, M, N, k, e, m,
                   plist))
    return;
  const int f0 = (blockIdx.x * kFfnWaves + (int)(threadIdx.x >> 6)) * 4;
  if (f0 >= F) return;
  const float *wg = w_gate + (size_t)e * F * d, *wu = w_up + (size_t)e * F * d;
  constexpr int kPairs = kFew ? 2 : kF32Pairs;
  for (int p0 = blockIdx.z * kPairs; p0 < m; p0 += gridDim.z * kPairs) {
    if constexpr (kFew) {
      if (m - p0 == 1) gateup_f32_tile<1>(h, wg, wu, plist, p0, m, M * k, k, d, F, f0, act);
      else gateup_f32_tile<2>(h, wg, wu, plist, p0, m, M * k, k, d, F, f0, act);
    } else {
      if (m - p0 <= kF32Pairs / 2) gateup_f32_tile<kF32Pairs / 2>(h, wg, wu, plist, p0, m, M * k, k, d, F, f0, act);
      else gateup_f32_tile<kF32Pairs>(h, wg, wu, plist, p0, m, M * k, k, d, F, f0, act);
    }
  }
}

template <int P>
__device__ __forceinline__ void down_f32_tile(const float *__restrict__ act, const float *wd, const int32_t *plist, int p0,
                                              int m, int n_pairs, int d, int F, int j0, float *__restrict__ y) {
  const int lane = threadIdx.x & 63;
  const float *row[kF32Rows], *x[P];
#pragma unroll
  for (int r = 0; r < kF32Rows; ++r) row[r] = wd + (size_t)min(j0 + r, d - 1) * F;
#pragma unroll
  for (int p = 0; p < P; ++p) x[p] = act + (size_t)pair_at(plist, min(p0 + p, m - 1), n_pairs) * F;
  float sums[kF32Rows * P];
  f32_dots<P>(row, x, F, sums);
  const float v = fold_sums(sums);
  constexpr int LPS = 64 / (kF32Rows * P);
  const int idx = lane / LPS, j = j0 + idx / P, p = p0 + idx % P;
  if (lane % LPS == 0 && j < d && p < m) y[(size_t)pair_at(plist, p, n_pairs) * d + j] = v;
}

template <bool kFew, bool kItems>
__global__ __launch_bounds__(kFfnThreads) void ffn_down_f32_kernel(
    const int32_t *__restrict__ rank_count, const int32_t *__restrict__ shortlist, const int32_t *__restrict__ lists,
    int list_stride, int M, int N, int k, int d, int F, const float *__restrict__ w_down, const float *__restrict__ act,
    const int32_t *__restrict__ seg_expert, const int32_t *__restrict__ seg_off, const int4 *__restrict__ items,
    const int32_t *__restrict__ perm, float *__restrict__ y) {
  int e, m;
  const int32_t *plist;
  if (!f32_segment<kItems>(blockIdx.y, seg_expert, seg_off, items, perm, rank_count, shortlist, lists, list_stride, M, N, k, e, m,
                   plist))
    return;
  const int j0 = (blockIdx.x * kFfnWaves + (int)(threadIdx.x >> 6)) * kF32Rows;
  if (j0 >= d) return;
  const float *wd = w_down + (size_t)e * d * F;
  constexpr int kPairs = kFew ? 2 : kF32Pairs;
  for (int p0 = blockIdx.z * kPairs; p0 < m; p0 += gridDim.z * kPairs) {
    if constexpr (kFew) {
      if (m - p0 == 1) down_f32_tile<1>(act, wd, plist, p0, m, M * k, d, F, j0, y);
      else down_f32_tile<2>(act, wd, plist, p0, m, M * k, d, F, j0, y);
    } else {
      if (m - p0 <= kF32Pairs / 2) down_f32_tile<kF32Pairs / 2>(act, wd, plist, p0, m, M * k, d, F, j0, y);
      else down_f32_tile<kF32Pairs>(act, wd, plist, p0, m, M * k, d, F, j0, y);
    }
  }
}

// ---- fp32 passes on the matrix cores ----------------------------------------------------------------------------
// A workgroup owns two tiles of 16 weight rows (gate/up: 16 gate rows and the same 16 up rows) and NP tiles of 16 pairs; its
// 8 waves take two of every 16 steps of 16 elements of K each.  A lane loads 4 consecutive elements of its row and of its
// pair per step, which feed 4 v_mfma_f32_16x16x4 (lane (i, g) supplies A[i][g], B[g][i] and receives D[4 g + r][i]); which
// elements meet in one instruction is immaterial.  Every wave keeps kF32Chains sums side by side that are added pairwise, then
// the waves' in the order of a tree: 64 short chains from K = 256 on (below, 8 per 32 elements: a wave without a step
// adds zeros), like the 64 lanes of the vector form above, so that the rounding error of a sum is the same (against 64 bits
// 1.4e-7 and 5.1e-8 before and after, 15 tokens of 128 x 256 and 63 of 512 x 1024 with a residual).
// What bounds it: the chain of a workgroup, which is about 5 us long (tables, pair ids, loads, sums), times the rounds of
// workgroups.  One token tile leaves room for two workgroups per compute unit, two tiles for one.  63 tokens over 8 experts of
// 512 x 1024, top-4, us, vector form / one / two tiles: gate/up 29.9 / 21.1 / 20.7, down 22.6 / 14.5 / 12.5.  A second set
// of loads in flight changed nothing (its registers cost the second workgroup where one tile is taken).
constexpr int kMfWaves = 8, kMfThreads = kMfWaves * kWave, kF32Chains = 8, kMfStep = 16;

// v[2][NP] of this wave += its share of K of (rows w[0], w[1]) x (pairs x[0 .. NP)): pointers to this lane's row / pair
template <int NP>
__device__ __forceinline__ void f32_mfma_walk(const float *const (&w)[2], const float *const (&x)[NP], int K,
                                              f32x4 (&v)[2][NP]) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4;
  const int steps = (K + kMfStep - 1) / kMfStep;
  f32x4 acc[kF32Chains][2][NP];
#pragma unroll
  for (int c = 0; c < kF32Chains; ++c)
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int p = 0; p < NP; ++p) acc[c][a][p] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr int kAhead = 2;  // steps per round, next to each other: whole cache lines
  for (int s0 = kAhead * wave; s0 < steps; s0 += kAhead * kMfWaves) {
    f32x4 A[kAhead][2], B[kAhead][NP];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int k = (s0 + u) * kMfStep + 4 * g;
      const bool in = k < K;  // K is a multiple of 4; lanes past the end multiply zeros
#pragma unroll
      for (int a = 0; a < 2; ++a) A[u][a] = in ? *reinterpret_cast<const f32x4 *>(w[a] + k) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int p = 0; p < NP; ++p) B[u][p] = in ? *reinterpret_cast<const f32x4 *>(x[p] + k) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int p = 0; p < NP; ++p)
            acc[4 * u + m][a][p] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[u][a][m], B[u][p][m], acc[4 * u + m][a][p], 0, 0, 0);
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int p = 0; p < NP; ++p)
      v[a][p] = ((acc[0][a][p] + acc[1][a][p]) + (acc[2][a][p] + acc[3][a][p])) +
                ((acc[4][a][p] + acc[5][a][p]) + (acc[6][a][p] + acc[7][a][p]));
}

// part: [kMfWaves][2][NP][kMfPart] floats of LDS.  Calls out(row, pair, sum of the first tile's row, of the second's) for the rows
// 0 .. 15 and pairs 0 .. 16 NP - 1; 16 consecutive threads have 16 consecutive rows of one pair.
constexpr int kMfPart = 4 * 68;  // 4 registers of 64 lanes, 68 apart: the threads that read 16 rows of 4 pairs touch all banks
template <int NP, class F>
__device__ __forceinline__ void f32_mfma_tile(const float *const (&w)[2], const float *const (&x)[NP], int K, float *part, F out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  f32x4 v[2][NP];
  f32_mfma_walk<NP>(w, x, K, v);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int r = 0; r < 4; ++r) part[((wave * 2 + a) * NP + p) * kMfPart + 68 * r + lane] = v[a][p][r];
  __syncthreads();
  if (threadIdx.x < 256 * NP) {
    const int row = threadIdx.x & 15, pair = (threadIdx.x >> 4) & 15, p = threadIdx.x >> 8;
    float s[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      float q[kMfWaves];
#pragma unroll
      for (int i = 0; i < kMfWaves; ++i) q[i] = part[((i * 2 + a) * NP + p) * kMfPart + 68 * (row & 3) + 16 * (row >> 2) + pair];
      s[a] = ((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7]));
    }
    out(row, 16 * p + pair, s[0], s[1]);
  }
  __syncthreads();  // the sums have been read
}

// A segment of one or two pairs: the tile of the matrix instructions would be nearly empty, and the weights are a stream.  Every
// wave takes 4 of the workgroup's 32 rows, 16 lanes per row and 4 elements per lane, so that a load covers 64 elements of all 4
// rows, with 8 steps in flight and nobody to wait for.  s[p] = row . x[p] in every lane of the row; w and x point to this lane's
// first elements.  64 sums side by side per row here too.  How many pairs a segment has is known on the device only: 64 experts of
// 1400 x 1400 with one pair each, us, vector kernels / matrix tile / this form: 277 / 304 / 252, with two 280 / 308 / 255.  (With
// three and four pairs 282 / 315 / 316: the pairs are loaded again for every 4 rows.  Eight rows per wave and K in two
// halves took 272 for three, but 1 to 8 % longer than the matrix tile in calls of a few workgroups.)
constexpr int kF32Few = 2;
__device__ __forceinline__ void f32_few_dots(const float *w, const float *const (&x)[kF32Few], int K, float (&s)[kF32Few]) {
  const int c = 4 * (threadIdx.x & 15);
  constexpr int U = 8;  // steps of 64 elements in flight
  f32x4 acc[kF32Few];
#pragma unroll
  for (int p = 0; p < kF32Few; ++p) acc[p] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < K; k0 += 64 * U) {
    f32x4 wv[U], xv[U][kF32Few];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + 64 * u;
      const bool in = k + c < K;  // K is a multiple of 4; lanes past the end multiply zeros
      wv[u] = in ? __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(w + k)) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int p = 0; p < kF32Few; ++p) xv[u][p] = in ? *reinterpret_cast<const f32x4 *>(x[p] + k) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int p = 0; p < kF32Few; ++p)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[p][i] = fmaf(wv[u][i], xv[u][p][i], acc[p][i]);
  }
#pragma unroll
  for (int p = 0; p < kF32Few; ++p) s[p] = row16_sum((acc[p][0] + acc[p][1]) + (acc[p][2] + acc[p][3]));
}
// Whether a segment (or piece) takes that form; the pieces of a segment that was cut take one form, whatever the last one's size.
template <bool kItems>
__device__ __forceinline__ bool f32_few(int m, int item, const int4 *items) {
  if (m > kF32Few) return false;
  return !kItems || item == 0 || items[item].x != items[1 + item].x;
}

__device__ __forceinline__ void gateup_f32_few(const float *__restrict__ h, const float *wg, const float *wu, const int32_t *plist,
                                               int m, int n_pairs, int k, int d, int F, int f0, float *__restrict__ act) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = lane & 15;
  const int f = f0 + 2 * wave + ((lane >> 4) & 1);
  const float *w = (lane < 32 ? wg : wu) + (size_t)min(f, F - 1) * d + 4 * c, *x[kF32Few];
#pragma unroll
  for (int p = 0; p < kF32Few; ++p) x[p] = h + (size_t)(pair_at(plist, min(p, m - 1), n_pairs) / k) * d + 4 * c;
  float s[kF32Few];
  f32_few_dots(w, x, d, s);
#pragma unroll
  for (int p = 0; p < kF32Few; ++p) {
    const float u = __shfl_xor(s[p], 32, kWave);
    if (lane < 32 && c == p && f < F && p < m) act[(size_t)pair_at(plist, p, n_pairs) * F + f] = s[p] / (1.0f + expf(-s[p])) * u;
  }
}

__device__ __forceinline__ void down_f32_few(const float *__restrict__ act, const float *wd, const int32_t *plist, int m, int n_pairs,
                                             int d, int F, int j0, float *__restrict__ y) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = lane & 15, j = j0 + 4 * wave + (lane >> 4);
  const float *w = wd + (size_t)min(j, d - 1) * F + 4 * c, *x[kF32Few];
#pragma unroll
  for (int p = 0; p < kF32Few; ++p) x[p] = act + (size_t)pair_at(plist, min(p, m - 1), n_pairs) * F + 4 * c;
  float s[kF32Few];
  f32_few_dots(w, x, F, s);
#pragma unroll
  for (int p = 0; p < kF32Few; ++p)
    if (c == p && j < d && p < m) y[(size_t)pair_at(plist, p, n_pairs) * d + j] = s[p];
}

template <int NP, bool kItems>
__global__ __launch_bounds__(kMfThreads, NP == 1 ? 4 : 2) void ffn_gateup_f32_mfma_kernel(
    const int32_t *__restrict__ rank_count, const int32_t *__restrict__ shortlist, const int32_t *__restrict__ lists,
    int list_stride, int M, int N, int k, int d, int F, const float *__restrict__ w_gate, const float *__restrict__ w_up,
    const float *__restrict__ h, const int32_t *__restrict__ seg_expert, const int32_t *__restrict__ seg_off,
    const int4 *__restrict__ items, const int32_t *__restrict__ perm, float *__restrict__ act) {
  __shared__ float part[kMfWaves * 2 * NP * kMfPart];
  int e, m;
  const int32_t *plist;
  if (!f32_segment<kItems>(blockIdx.y, seg_expert, seg_off, items, perm, rank_count, shortlist, lists, list_stride, M, N, k, e, m,
                   plist))
    return;
  const int f0 = blockIdx.x * 16, i = threadIdx.x & 15, n_pairs = M * k;
  if (__builtin_expect(f32_few<kItems>(m, blockIdx.y, items), 0)) {  // its code behind the tiles': 0.3 us of a small call
    if (blockIdx.z != 0) return;
    const float *wg = w_gate + (size_t)e * F * d, *wu = w_up + (size_t)e * F * d;
    gateup_f32_few(h, wg, wu, plist, m, n_pairs, k, d, F, f0, act);
    return;
  }
  const size_t row = ((size_t)e * F + min(f0 + i, F - 1)) * d;  // rows and pairs past the end repeat the last one, never stored
  const float *const w[2] = {w_gate + row, w_up + row};
  for (int p0 = blockIdx.z * 16 * NP; p0 < m; p0 += gridDim.z * 16 * NP) {
    auto run = [&](auto np) {
      constexpr int T = decltype(np)::value;
      const float *x[T];
#pragma unroll
      for (int p = 0; p < T; ++p) x[p] = h + (size_t)(pair_at(plist, min(p0 + 16 * p + i, m - 1), n_pairs) / k) * d;
      const float *const(&xc)[T] = x;
      f32_mfma_tile<T>(w, xc, d, part, [&](int r, int pair, float g, float u) {
        if (f0 + r < F && p0 + pair < m)
          act[(size_t)pair_at(plist, p0 + pair, n_pairs) * F + f0 + r] = g / (1.0f + expf(-g)) * u;
      });
    };
    if (NP == 1 || m - p0 <= 16) run(std::integral_constant<int, 1>{});
    else run(std::integral_constant<int, NP>{});
  }
}

template <int NP, bool kItems>
__global__ __launch_bounds__(kMfThreads, NP == 1 ? 4 : 2) void ffn_down_f32_mfma_kernel(
    const int32_t *__restrict__ rank_count, const int32_t *__restrict__ shortlist, const int32_t *__restrict__ lists,
    int list_stride, int M, int N, int k, int d, int F, const float *__restrict__ w_down, const float *__restrict__ act,
    const int32_t *__restrict__ seg_expert, const int32_t *__restrict__ seg_off, const int4 *__restrict__ items,
    const int32_t *__restrict__ perm, float *__restrict__ y) {
  __shared__ float part[kMfWaves * 2 * NP * kMfPart];
  int e, m;
  const int32_t *plist;
  if (!f32_segment<kItems>(blockIdx.y, seg_expert, seg_off, items, perm, rank_count, shortlist, lists, list_stride, M, N, k, e, m,
                   plist))
    return;
  const int j0 = blockIdx.x * 32, i = threadIdx.x & 15, n_pairs = M * k;
  if (__builtin_expect(f32_few<kItems>(m, blockIdx.y, items), 0)) {
    if (blockIdx.z != 0) return;
    const float *wd = w_down + (size_t)e * d * F;
    down_f32_few(act, wd, plist, m, n_pairs, d, F, j0, y);
    return;
  }
  const float *const w[2] = {w_down + ((size_t)e * d + min(j0 + i, d - 1)) * F, w_down + ((size_t)e * d + min(j0 + 16 + i, d - 1)) * F};
  for (int p0 = blockIdx.z * 16 * NP; p0 < m; p0 += gridDim.z * 16 * NP) {
    auto run = [&](auto np) {
      constexpr int T = decltype(np)::value;
      const float *x[T];
#pragma unroll
      for (int p = 0; p < T; ++p) x[p] = act + (size_t)pair_at(plist, min(p0 + 16 * p + i, m - 1), n_pairs) * F;
      const float *const(&xc)[T] = x;
      f32_mfma_tile<T>(w, xc, F, part, [&](int r, int pair, float a, float b) {
        if (p0 + pair >= m) return;
        float *dst = y + (size_t)pair_at(plist, p0 + pair, n_pairs) * d + j0 + r;
        if (j0 + r < d) dst[0] = a;
        if (j0 + 16 + r < d) dst[16] = b;
      });
    };
    if (NP == 1 || m - p0 <= 16) run(std::integral_constant<int, 1>{});
    else run(std::integral_constant<int, NP>{});
  }
}

// The same sums for K up to 768 with the weights held in registers: a workgroup owns NA tiles of 16 rows and passes the segment's
// pairs by them in tiles of 16, so that the weights are read once per workgroup, all its loads of a tile are in flight together and
// those of the next tile go out before the sums of the present one are folded.  KA = rounds of 2 steps per wave (K <= 256 KA).
// The chains are worked off one after the other and added as they end, in the order of f32_mfma_walk (bit-identical): one
// chain and its partial sums live instead of 8, which leaves the registers for two workgroups per compute unit.
// Elements past the end of K come from a line of zeros: no branch around a load, so that the waits can be counted.
// What bounds it: a tile of pairs is a chain of LDS sums and a barrier behind 8 KA matrix instructions per tile of rows; two workgroups
// take turns.  63 tokens over 8 experts of 512 x 1024: gate/up pass 20.2 -> 16.0 us, layer 42.7 -> 37.9; 57 drawn layers of 64 to
// 1024 elements and up to 127 tokens 1.03x, up to 1.24x, 0.97x at least.  Up to 768 elements: held for four rounds the weights of two
// tiles leave one workgroup per compute unit, and those of one tile read the pairs twice as often (down pass above, K = 1024,
// 12.4 -> 15.3 us either way; 628 x 872, 11 segments of 2 pairs, layer 25.3 -> 28.2).  But where row tiles and segments make at most 112
// workgroups, up to four of which share a segment's pairs, the down pass holds one tile of up to 1024 elements: what bounds it there is
// the time of a workgroup.  Layers, us, streamed / held: 24 workgroups of 64 x 972, 7 pairs per segment 20.2 / 18.2; 35 of 72 x 1004, 21 pairs 28.9 /
// 24.0; 102 of 260 x 964, 27 pairs 41.4 / 32.9; 32 such layers 1.01 to 1.25x.  124 to 180 workgroups 0.95 to 1.27x, 300 and more 0.92 to
// 1.06x.  The gate/up pass, which has two tiles at least, gained nothing there (21 layers 0.98 to 1.06x, half of them slower).
// x_row(id): row of a pair; out(row, pair, its id, sums of the NA tiles' rows).  part: 2 [kMfWaves][NA][kMfPart] floats of LDS.
constexpr int kF32HeldK = 768, kF32HeldKFew = 1024;
constexpr long long kF32HeldFew = 112;
__device__ const f32x4 kF32Zeros = {0.f, 0.f, 0.f, 0.f};
template <int NA, int KA, class X, class F>
__device__ __forceinline__ void f32_held_tiles(const float *const (&w)[NA], const int32_t *plist, int n_pairs, X x_row, int K, int p0,
                                               int step, int m, float *part, F out) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = lane & 15;
  const int k0 = wave * 2 * kMfStep + 4 * (lane >> 4);
  const bool whole = ((KA - 1) * kMfWaves + wave) * 2 * kMfStep < K;
  f32x4 A[KA][2][NA], B[KA][2];
  auto id_of = [&](int p) { return plist[min(p + i, m - 1)]; };  // pairs past the end repeat the last one, never stored
  auto load = [&](const float *row, int r, int u) {
    const int k = k0 + r * (kMfWaves * 2 * kMfStep) + u * kMfStep;
    const float *p = k < K ? row + k : reinterpret_cast<const float *>(&kF32Zeros);
    return *(const __attribute__((address_space(1))) f32x4 *)(p);  // both are global memory: no flat load
  };
  auto load_pairs = [&](int id) {
    const float *x = x_row(min(max(id, 0), n_pairs - 1));
#pragma unroll
    for (int r = 0; r < KA; ++r)
#pragma unroll
      for (int u = 0; u < 2; ++u) B[r][u] = load(x, r, u);
  };
  int id = id_of(p0);
  __builtin_amdgcn_sched_barrier(0);  // loads return in the order of their issue
#pragma unroll
  for (int r = 0; r < KA; ++r)
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int a = 0; a < NA; ++a) A[r][u][a] = load(w[a], r, u);
  int next = id_of(p0 + step);
  __builtin_amdgcn_sched_barrier(0);  // the weights are on their way before the pair ids are waited for
  load_pairs(id);
  int parity = 0;
  for (int p = p0; p < m; p += step, parity ^= 1) {
    f32x4 sum[NA];
    auto chains = [&](auto rounds_) {
      constexpr int R = decltype(rounds_)::value;
      f32x4 one[NA], two[NA], four[NA];  // sums of 1, 2 and 4 chains that wait for their neighbours
#pragma unroll
      for (int c = 0; c < kF32Chains; ++c) {
        f32x4 v[NA];
#pragma unroll
        for (int a = 0; a < NA; ++a) v[a] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int a = 0; a < NA; ++a)
            v[a] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[r][c >> 2][a][c & 3], B[r][c >> 2][c & 3], v[a], 0, 0, 0);
#pragma unroll
        for (int a = 0; a < NA; ++a) {
          if ((c & 1) == 0) {
            one[a] = v[a];
          } else if ((c & 2) == 0) {
            two[a] = one[a] + v[a];
          } else if ((c & 4) == 0) {
            four[a] = two[a] + (one[a] + v[a]);
          } else {
            sum[a] = four[a] + (two[a] + (one[a] + v[a]));
          }
        }
        if (c & 1) {  // two chains at a time, added here: eight side by side would cost the second workgroup its registers
#pragma unroll
          for (int a = 0; a < NA; ++a) {
            if (c == 7) asm volatile("" : "+v"(sum[a]));
            else if (c == 3) asm volatile("" : "+v"(four[a]));
            else asm volatile("" : "+v"(two[a]));
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    if (whole) chains(std::integral_constant<int, KA>{});
    else chains(std::integral_constant<int, KA - 1>{});  // this wave has no step in the last round
    const int present = id;
    if (p + step < m) {
      id = next;
      load_pairs(id);
      next = id_of(p + 2 * step);
    }
    float *mine = part + parity * (kMfWaves * NA * kMfPart);  // two buffers in turn: one barrier per tile
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r) mine[(wave * NA + a) * kMfPart + 68 * r + lane] = sum[a][r];
    __syncthreads();
    if ((wave >> 2) == parity) {  // the two halves of the workgroup take the tiles in turn
      const int row = threadIdx.x & 15, pair = (threadIdx.x >> 4) & 15;
      float s[NA];
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        float q[kMfWaves];
#pragma unroll
        for (int v = 0; v < kMfWaves; ++v) q[v] = mine[(v * NA + a) * kMfPart + 68 * (row & 3) + 16 * (row >> 2) + pair];
        s[a] = ((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7]));
      }
      out(row, p + pair, min(max(__shfl(present, pair, kWave), 0), n_pairs - 1), s);
    }
  }
}

// How many of the up to four workgroups along z share the pairs of a segment: one per `walk` of them.  The kernels find walk above the
// 8 bits of top_k, in an argument that is preloaded: nothing else is waited for before the first weights are requested.
__device__ __forceinline__ int f32_parts(int m, int k_walk) {
  const int walk = k_walk >> 8;
  return min(1 + (m > walk) + (m > 2 * walk) + (m > 3 * walk), (int)gridDim.z);
}

template <int KA, bool kItems>
__global__ __launch_bounds__(kMfThreads, 4) void ffn_gateup_f32_held_kernel(
    const int32_t *__restrict__ rank_count, const int32_t *__restrict__ shortlist, const int32_t *__restrict__ lists,
    int list_stride, int M, int N, int k_walk, int d, int F, const float *__restrict__ w_gate, const float *__restrict__ w_up,
    const float *__restrict__ h, const int32_t *__restrict__ seg_expert, const int32_t *__restrict__ seg_off,
    const int4 *__restrict__ items, const int32_t *__restrict__ perm, float *__restrict__ act) {
  __shared__ float part[2 * kMfWaves * 2 * kMfPart];
  const int k = k_walk & 0xff;
  int e, m;
  const int32_t *plist;
  if (!f32_segment<kItems>(blockIdx.y, seg_expert, seg_off, items, perm, rank_count, shortlist, lists, list_stride, M, N, k, e, m,
                   plist))
    return;
  const int f0 = blockIdx.x * 16, i = threadIdx.x & 15, n_pairs = M * k;
  if (__builtin_expect(f32_few<kItems>(m, blockIdx.y, items), 0)) {  // its code behind the tiles': 0.3 us of a small call
    if (blockIdx.z != 0) return;
    const float *wg = w_gate + (size_t)e * F * d, *wu = w_up + (size_t)e * F * d;
    gateup_f32_few(h, wg, wu, plist, m, n_pairs, k, d, F, f0, act);
    return;
  }
  const int parts = f32_parts(m, k_walk);
  if ((int)blockIdx.z >= parts) return;
  const size_t row = ((size_t)e * F + min(f0 + i, F - 1)) * d;  // rows past the end repeat the last one, never stored
  const float *const w[2] = {w_gate + row, w_up + row};
  f32_held_tiles<2, KA>(
      w, plist, n_pairs, [&](int id) { return h + (size_t)(id / k) * d; }, d, blockIdx.z * 16, parts * 16, m, part,
      [&](int r, int pair, int id, const float (&s)[2]) {
        if (f0 + r < F && pair < m) act[(size_t)id * F + f0 + r] = s[0] / (1.0f + expf(-s[0])) * s[1];
      });
}

template <int NA, int KA, bool kItems>
__global__ __launch_bounds__(kMfThreads, 4) void ffn_down_f32_held_kernel(
    const int32_t *__restrict__ rank_count, const int32_t *__restrict__ shortlist, const int32_t *__restrict__ lists,
    int list_stride, int M, int N, int k_walk, int d, int F, const float *__restrict__ w_down, const float *__restrict__ act,
    const int32_t *__restrict__ seg_expert, const int32_t *__restrict__ seg_off, const int4 *__restrict__ items,
    const int32_t *__restrict__ perm, float *__restrict__ y) {
  __shared__ float part[2 * kMfWaves * NA * kMfPart];
  const int k = k_walk & 0xff;
  int e, m;
  const int32_t *plist;
  if (!f32_segment<kItems>(blockIdx.y, seg_expert, seg_off, items, perm, rank_count, shortlist, lists, list_stride, M, N, k, e, m,
                   plist))
    return;
  const int j0 = blockIdx.x * 16 * NA, i = threadIdx.x & 15, n_pairs = M * k;
  if (__builtin_expect(f32_few<kItems>(m, blockIdx.y, items), 0)) {
    if (blockIdx.z != 0 || (NA == 1 && (blockIdx.x & 1))) return;  // that form takes 32 rows
    const float *wd = w_down + (size_t)e * d * F;
    down_f32_few(act, wd, plist, m, n_pairs, d, F, j0, y);
    return;
  }
  const int parts = f32_parts(m, k_walk);
  if ((int)blockIdx.z >= parts) return;
  const float *w[NA];
#pragma unroll
  for (int a = 0; a < NA; ++a) w[a] = w_down + ((size_t)e * d + min(j0 + 16 * a + i, d - 1)) * F;
  const float *const(&wc)[NA] = w;
  f32_held_tiles<NA, KA>(
      wc, plist, n_pairs, [&](int id) { return act + (size_t)id * F; }, F, blockIdx.z * 16, parts * 16, m, part,
      [&](int r, int pair, int id, const float (&s)[NA]) {
        if (pair >= m) return;
        float *dst = y + (size_t)id * d + j0 + r;
#pragma unroll
        for (int a = 0; a < NA; ++a)
          if (j0 + 16 * a + r < d) dst[16 * a] = s[a];
      });
}

// ---- combine: out[t] = residual[t] + sum over surviving slots (slot order) of w * y[t*k+slot] ---
// y holds SP partial copies split_stride floats apart (K-split down pass), added in split order.  The rows of dropped slots
// hold stale scratch: they are loaded (valid memory) but never enter the sum.
// The four outputs j .. j+3 of token t (before storage rounding).  What bounds it is one round of cold loads: those of U slots go
// out together, up to 8 rows (with 4 rows at a time and one by one for the remainder of k it was up to k / 4 + k % 4 rounds).
// Whole layer of 7 tokens, top-8 of 64 experts of 2048 x 1024: 49.1 -> 47.6 us, with the workgroups of one wave below and
// kernel arguments preloaded into registers.
template <typename T, int SP, int U>
__device__ __forceinline__ f32x4 combine_four(const float *__restrict__ y, const int32_t *__restrict__ tok_ids,
                                              const float *__restrict__ tok_w, const T *__restrict__ residual, int t,
                                              int j, int k, int d, size_t split_stride) {
  const float *yt = y + (size_t)t * k * d + j;
  const int32_t *ids = tok_ids + (size_t)t * k;
  const float *wt = tok_w + (size_t)t * k;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (residual) acc = Elem<T>::load4(residual + (size_t)t * d + j);
  for (int s0 = 0; s0 < k; s0 += U) {
    f32x4 v[U][SP];
    float w[U];
    int id[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int s = min(s0 + u, k - 1);  // past the last slot: its row again, not added
#pragma unroll
      for (int sp = 0; sp < SP; ++sp) v[u][sp] = *reinterpret_cast<const f32x4 *>(yt + (size_t)s * d + sp * split_stride);
      id[u] = ids[s];
      w[u] = wt[s];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u < k && id[u] >= 0) {
        f32x4 r = v[u][0];
#pragma unroll
        for (int sp = 1; sp < SP; ++sp) r += v[u][sp];
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = fmaf(w[u], r[i], acc[i]);
      }
    }
  }
  return acc;
}

// Workgroups of one wave: the rows of a token are spread over as many compute units as there are.
constexpr int kCombineThreads = 64;
template <typename T, int SP, int U>
__global__ __launch_bounds__(kCombineThreads) void combine_kernel(const float *__restrict__ y, const int32_t *__restrict__ tok_ids,
                                                                  const float *__restrict__ tok_w, const T *__restrict__ residual,
                                                                  T *__restrict__ out, int M, int k, int d) {
  const int t = blockIdx.y;
  const int j = (blockIdx.x * kCombineThreads + threadIdx.x) * 4;
  if (j >= d) return;
  Elem<T>::store4(out + (size_t)t * d + j, combine_four<T, SP, U>(y, tok_ids, tok_w, residual, t, j, k, d, (size_t)M * k * d));
}

// The combine of a layer inside a stack that scales its layer inputs: one workgroup per token writes the row of the
// new hidden state and, from the STORED (rounded) values, the next layer's input x = row / rms(row) - with the
// element-to-thread mapping and summation order of rms_scale_row, so that the result equals, bit for bit, what
// rms_scale_kernel makes of the stored row.  d <= 8192: a thread holds up to 8 outputs.
template <typename T, int SP, int U>
__global__ __launch_bounds__(kRmsThreads) void combine_scale_kernel(const float *__restrict__ y,
                                                                    const int32_t *__restrict__ tok_ids,
                                                                    const float *__restrict__ tok_w,
                                                                    const T *__restrict__ residual,
                                                                    T *__restrict__ out, T *__restrict__ x_next, int M, int k,
                                                                    int d) {
  __shared__ float part[kRmsThreads];
  const int t = blockIdx.x, tid = threadIdx.x;
  float v[kRmsChunks][4];
#pragma unroll
  for (int c = 0; c < kRmsChunks; ++c) {
    const int j = (c * kRmsThreads + tid) * 4;
    if (j < d) {
      const f32x4 acc = combine_four<T, SP, U>(y, tok_ids, tok_w, residual, t, j, k, d, (size_t)M * k * d);
      Elem<T>::store4(out + (size_t)t * d + j, acc);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[c][i] = Elem<T>::stored(acc[i]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[c][i] = 0.f;
    }
  }
  const float scale = rms_scale_of_row(v, d, part);
#pragma unroll
  for (int c = 0; c < kRmsChunks; ++c) {
    const int j = (c * kRmsThreads + tid) * 4;
    if (j < d) Elem<T>::store4(x_next + (size_t)t * d + j, f32x4{v[c][0] * scale, v[c][1] * scale, v[c][2] * scale, v[c][3] * scale});
  }
}

template <typename T>
static hipError_t launch_combine(const moespec_desc &ds, const float *y, const int32_t *tok_ids, const float *tok_w,
                                 const void *residual, void *out, void *x_next, int M, int splits, hipStream_t st) {
  const int k = ds.top_k, d = ds.d;
  auto run = [&](auto sp, auto slots) {
    constexpr int SP = decltype(sp)::value, U = decltype(slots)::value;
    if (x_next)
      combine_scale_kernel<T, SP, U><<<M, kRmsThreads, 0, st>>>(y, tok_ids, tok_w, static_cast<const T *>(residual),
                                                                static_cast<T *>(out), static_cast<T *>(x_next), M, k, d);
    else
      combine_kernel<T, SP, U><<<dim3((d / 4 + kCombineThreads - 1) / kCombineThreads, M), kCombineThreads, 0, st>>>(
          y, tok_ids, tok_w, static_cast<const T *>(residual), static_cast<T *>(out), M, k, d);
    return hipGetLastError();
  };
  using std::integral_constant;
  const integral_constant<int, 2> two;
  const integral_constant<int, 4> four;
  if constexpr (sizeof(T) == 2) {  // fp32 layers are not split
    if (splits == kMaxDownSplits) return run(four, two);
    if (splits == 2) return k <= 2 ? run(two, two) : run(two, four);
  }
  const integral_constant<int, 1> one;
  return k <= 2 ? run(one, two) : k <= 4 ? run(one, four) : run(one, integral_constant<int, 8>{});
}

// Whether the passes can take their pairs from the prologue's lists.
bool expert_ffn_self_segmenting(const moespec_desc &ds, int M) {
  return ds.n_experts <= kSelfMaxExperts && M <= kSelfMaxTokens;
}

// K-split of the LDS-tiled down pass: when its (segment, row tile) items alone cannot give every compute
// unit two workgroups, each item is cut along F into up to kMaxDownSplits parts with their own copy of y,
// as long as a part keeps at least 16 chunks (shorter walks are dominated by their start-up: measured
// slower at F = 1024, 1.6x to 2.7x faster at F = 14336 with 4 or 2 loaded experts).
int streaming_down_splits(const moespec_desc &ds, int n_seg) {
  int splits = 1;
  if (ds.dtype == MOESPEC_BF16) {
    const int tiles = (ds.d / 32 + kFfnWaves - 1) / kFfnWaves;
    while (splits < kMaxDownSplits && (long long)n_seg * tiles * splits * 2 <= 512 && ds.d_ff / 128 >= 32 * splits)
      splits *= 2;
  }
  return splits;
}
int down_splits(const moespec_desc &ds, int M, int n_seg) {
  return expert_down_wide(ds, M, n_seg) ? 1 : streaming_down_splits(ds, n_seg);
}

// Workgroups of a streaming pass.  The device picks the form of the walk: room for whole rounds of 8 of n_items items in
// row tiles, and for kCutUnitsLarge units of which each is up to four (and a last round that is dealt to 8 XCDs).
static int pass_grid(int row_tiles, int cut_tiles, int n_items, int K, int splits) {
  const int by_rows = xcd_grid(row_tiles, n_items);
  if (splits != 1 || K < 4 * 128) return by_rows;
  const long long by_k = std::min<long long>((long long)xcd_grid(cut_tiles, n_items), 4 * kCutUnitsLarge + kXcds);
  return std::max<long long>(by_rows, by_k);
}

hipError_t launch_expert_ffn(const moespec_desc &ds, const moespec_weights &wt, const void *h, int M, int n_seg,
                             const int32_t *seg_expert, const int32_t *seg_off, const int32_t *perm,
                             const int32_t *tok_ids, const float *tok_w, const void *residual, void *out, void *act,
                             float *y, int4 *items, bool items_ready, const int32_t *rank_count,
                             const int32_t *shortlist, const int32_t *lists, int list_stride, hipStream_t st,
                             void *const *trace, void *x_next) {
  const int d = ds.d, F = ds.d_ff, k = ds.top_k;
  hipError_t e;
  if (rank_count && !(shortlist && lists && expert_ffn_self_segmenting(ds, M) && n_seg <= kFfnThreads))
    return hipErrorInvalidValue;
  if (!rank_count && !items_ready && !items) return hipErrorInvalidValue;
  const bool wide_gate_up = !rank_count && expert_ffn_wide(ds, M, n_seg);
  const bool wide_down = !rank_count && expert_down_wide(ds, M, n_seg);
  const int cap = items_capacity(n_seg, M, k);  // work items of the LDS-tiled passes
  // ... and how many there can be: the prologue's and the budget stage's segments hold every pair once at most
  const int most = rank_count || items_ready ? (int)std::min<long long>(cap, (long long)M * k) : cap;
  if (ds.dtype == MOESPEC_BF16 && !rank_count && !items_ready) {
    segment_items_kernel<<<1, 256, 0, st>>>(seg_expert, seg_off, n_seg, M, k, cap, items);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  auto mark = [&](int i) {
    if (trace && trace[i]) (void)hipEventRecord(static_cast<hipEvent_t>(trace[i]), st);
  };
  const int splits = down_splits(ds, M, n_seg);
  if (ds.dtype == MOESPEC_BF16) {
    for (int pass = 1; pass <= 2; ++pass) {
      if (pass == 1 ? wide_gate_up : wide_down) {
        e = launch_wide_pass(ds, wt, pass == 1, pass == 1 ? h : act, M, items, perm, cap,
                             pass == 1 ? act : static_cast<void *>(y), st);
        if (e != hipSuccess) return e;
        mark(pass - 1);
        continue;
      }
      const int K = pass == 1 ? d : F, row_tiles = pass == 1 ? (F / 16 + kFfnWaves - 1) / kFfnWaves
                                                             : (d / 32 + kFfnWaves - 1) / kFfnWaves * splits;
      const bool tail = K % 128 != 0;
      const int grid = pass_grid(row_tiles, pass == 1 ? F / 16 : d / 32, most, K, pass == 1 ? 1 : splits);
      if (pass == 1) {
        auto kern = tail ? ffn_gateup_lds_kernel<true> : ffn_gateup_lds_kernel<false>;
        kern<<<grid, kFfnThreads, 0, st>>>(rank_count, shortlist, lists, list_stride, n_seg, cap, M, ds.n_experts, k, d, F,
                                           items, perm, static_cast<const uint16_t *>(h),
                                           static_cast<const uint16_t *>(wt.w_gate),
                                           static_cast<const uint16_t *>(wt.w_up), static_cast<uint16_t *>(act));
      } else {
        auto kern = tail ? ffn_down_lds_kernel<true> : ffn_down_lds_kernel<false>;
        kern<<<grid, kFfnThreads, 0, st>>>(rank_count, shortlist, lists, list_stride, n_seg, cap, M, ds.n_experts, k, d, F,
                                           splits, items, perm, static_cast<const uint16_t *>(act),
                                           static_cast<const uint16_t *>(wt.w_down), y);
      }
      if ((e = hipGetLastError()) != hipSuccess) return e;
      mark(pass - 1);
    }
    if (!out) return hipSuccess;  // the caller only wants the per-pair outputs y
    e = launch_combine<uint16_t>(ds, y, tok_ids, tok_w, residual, out, x_next, M, splits, st);
    mark(2);
    return e;
  }
  const bool few = M <= 2;
  const int4 *work = !rank_count && items_ready ? items : nullptr;
  const int rows = work ? cap : n_seg;
  // The matrix cores from three tokens on, unless the weights are so large and the pairs so few that reading them is all there
  // is (vector / matrix form, us per layer: 64 experts of 1024 x 2048, top-8 of 16, 8 tokens 98 / 104; 8 of 4096 x 4096, 3
  // tokens 164 / 170, 16 tokens 288 / 191; with less than 2^21 elements per matrix 1.0 to 1.17 times as fast from 3 to 8 tokens).
  const bool matrix = !few && !(M <= 8 && (long long)d * F >= 1 << 21);
  // Two token tiles per workgroup read the weights half as often; one tile makes twice as many workgroups, two per compute
  // unit.  Two tiles where even they come to two workgroups per compute unit (layers of 300 tokens 1.01 to 1.13 times as
  // fast, 63 tokens over 8 experts of 512 x 1024 1.05; but 58 tokens over 13 experts of 832 x 84 0.89, 21 over 7 of 252 x 256 0.91).
  // The gate/up pass decides for both: counted by its own 32-row tiles the down pass takes one tile too early (1 expert of 2532 x 3920,
  // 93 tokens, 117 -> 143 us; 2 of 364 x 2688, 264 tokens, 109 -> 125; 320 drawn layers 0.996, 25 of them 4 to 18 % slower).
  const long long mean = (long long)M * k / n_seg;
  const bool two = matrix && mean > 16 && (long long)((F + 15) / 16) * n_seg * ((mean + 31) / 32) >= 512;
  for (int pass = 1; pass <= 2; ++pass) {
    const int R = pass == 1 ? F : d, K = pass == 1 ? d : F;
    // up to 4 workgroups share the pairs of a segment: enough waves to hide the loads where rows are few
    auto groups = [&](int tile) { return std::min((M + tile - 1) / tile, 4); };
    const int mf_tile = two ? 32 : 16, mf_rows = 16 * pass, mf_row_tiles = (R + mf_rows - 1) / mf_rows;
    // Short rows leave half of the 8 waves without a step, and with few pairs per segment the 5 us of a workgroup are all there is:
    // where workgroups come by the ten thousand the gate/up pass keeps the vector form (layers, us, vector / matrix: 141 of
    // 200 experts of 88 x 3324, 324 tokens, 247 / 304; 190 of 200 of 72 x 2204, 768 pairs, 222 / 248; 53 of 100 of 76 x 1228, 77
    // tokens, 59 / 69; but few large segments 94 / 81: 12 of 256 experts of 132 x 624, 177 tokens).  Not the down pass, whose
    // workgroups have twice the rows (32 of 256 experts of 2900 x 152, 128 tokens 204 / 179).
    const bool mf = matrix && !(pass == 1 && K <= 160 && mean <= 6 && (long long)mf_row_tiles * n_seg * groups(mf_tile) >= 24576);
    const bool few_rows = pass == 2 && (long long)((R + 15) / 16) * n_seg <= kF32HeldFew;
    const int ka = (K + 255) / 256, pair_tiles = (int)std::min<long long>(std::max<long long>((mean + 15) / 16, 1), 4);
    // The down pass takes 32 rows, which reads the pairs half as often, where there is still a workgroup for every second compute unit
    // (layers, us, 32 / 16 rows: 352 x 268 over 17 segments of 2 pairs 19.2 / 19.9, 884 x 88 over 9 of 4 19.5 / 20.3; 84 x 604 over 8
    // of 35 21.6 / 20.5).
    const int na = pass == 2 && (ka == 4 || (long long)((R + 31) / 32) * n_seg * pair_tiles < 128) ? 1 : 2;
    // Up to 16 tokens make one tile of pairs, for which nothing is held: the streaming form then, except where the down pass gains
    // workgroups by its 16 rows (held / streaming, 122 gate/up passes 1.01x, 78 down passes of 32 rows 1.03x, of 8192 x 64 over 128
    // segments 51.7 / 44.8 us; 58 of 16 rows 0.87x).  Segments of less than four pairs make little more than a tile each, and with one
    // workgroup per segment in one or two rounds (512 to 1023) the longest of them decide, which the streaming form shares out: held
    // / streaming, layers, 280 such gate/up passes 1.02x (0.93 to 1.11x); in more workgroups what each costs decides, from 2048 on 0.91x.
    // 244 such down passes 1.01x (0.91 to 1.12x): held.
    const int tiles = pass == 1 ? (R + 15) / 16 : (R + 16 * na - 1) / (16 * na);
    const long long held_wgs = (long long)tiles * n_seg;
    const bool reused = M > 16 && !(pass == 1 && mean < 4 && held_wgs >= 512 && held_wgs < 1024);
    if (mf && K <= (few_rows ? kF32HeldKFew : kF32HeldK) && (reused || na == 1)) {
      // workgroups share the pairs of a segment until there are two per compute unit
      int z = 1;
      while (z < 4 && 16 * z < M && held_wgs * z < 512) ++z;
      // Routing concentrates, and a segment (or a piece of one) is then far longer than the mean, the only length known here: where one
      // could have five tiles of pairs or more and six times the mean, more workgroups stand by for it, and segments of the mean length
      // keep to one.  Layers, us, without / with them: 464 x 192, 50 of 100 experts, 249 tokens, top-2 69.9 / 44.1; 196 x 256, 64 of
      // 256, 218 tokens 58.8 / 47.2; 592 x 464, 50 of 200, 253 tokens 93.5 / 77.8.  56 drawn passes of this kind 1.15x, with a bias that
      // concentrates the routing 1.3x; evenly spread 0.92x, because a workgroup that finds nothing costs 1 ns (at most 4096 in all).
      // In 156 passes where no segment can be that much longer the same was 0.98x.
      const int longest = (int)(std::min<long long>(M, work ? kPiecePairs : M) + 15) / 16;
      const int usual = (int)std::min<long long>((std::max<long long>(mean, 1) + 15) / 16, longest);
      int parts = z;
      if (longest >= 5 && longest >= 6 * usual)
        while (parts < groups(16) && held_wgs * (parts + 1) <= 4096) ++parts;
      const int k_walk = k | (parts > z ? 16 * usual : 16) << 8;
      const dim3 hgrid(tiles, rows, parts);
      auto pick = [&](auto ka_) {
        constexpr int KA = decltype(ka_)::value;
        auto down = [&](auto kern) {
          kern<<<hgrid, kMfThreads, 0, st>>>(rank_count, shortlist, lists, list_stride, M, ds.n_experts, k_walk, d, F,
                                             static_cast<const float *>(wt.w_down), static_cast<const float *>(act), seg_expert,
                                             seg_off, work, perm, y);
        };
        if constexpr (KA == 4) {
          down(work ? ffn_down_f32_held_kernel<1, KA, true> : ffn_down_f32_held_kernel<1, KA, false>);
        } else if (pass == 1) {
          auto kern = work ? ffn_gateup_f32_held_kernel<KA, true> : ffn_gateup_f32_held_kernel<KA, false>;
          kern<<<hgrid, kMfThreads, 0, st>>>(rank_count, shortlist, lists, list_stride, M, ds.n_experts, k_walk, d, F,
                                             static_cast<const float *>(wt.w_gate), static_cast<const float *>(wt.w_up),
                                             static_cast<const float *>(h), seg_expert, seg_off, work, perm, static_cast<float *>(act));
        } else {
          down(na == 1 ? (work ? ffn_down_f32_held_kernel<1, KA, true> : ffn_down_f32_held_kernel<1, KA, false>)
                       : (work ? ffn_down_f32_held_kernel<2, KA, true> : ffn_down_f32_held_kernel<2, KA, false>));
        }
      };
      if (ka == 1) pick(std::integral_constant<int, 1>{});
      else if (ka == 2) pick(std::integral_constant<int, 2>{});
      else if (ka == 3) pick(std::integral_constant<int, 3>{});
      else pick(std::integral_constant<int, 4>{});
      if ((e = hipGetLastError()) != hipSuccess) return e;
      mark(pass - 1);
      continue;
    }
    const int wg_rows = mf ? mf_rows : pass == 1 ? 4 * kFfnWaves : kF32Rows * kFfnWaves;
    const dim3 grid((R + wg_rows - 1) / wg_rows, rows, groups(mf ? mf_tile : kF32Pairs));
    if (pass == 1) {
      auto kern = mf ? (two ? (work ? ffn_gateup_f32_mfma_kernel<2, true> : ffn_gateup_f32_mfma_kernel<2, false>)
                            : (work ? ffn_gateup_f32_mfma_kernel<1, true> : ffn_gateup_f32_mfma_kernel<1, false>))
                  : work ? (few ? ffn_gateup_f32_kernel<true, true> : ffn_gateup_f32_kernel<false, true>)
                         : (few ? ffn_gateup_f32_kernel<true, false> : ffn_gateup_f32_kernel<false, false>);
      kern<<<grid, mf ? kMfThreads : kFfnThreads, 0, st>>>(
          rank_count, shortlist, lists, list_stride, M, ds.n_experts, k, d, F, static_cast<const float *>(wt.w_gate),
          static_cast<const float *>(wt.w_up), static_cast<const float *>(h), seg_expert, seg_off, work, perm,
          static_cast<float *>(act));
    } else {
      auto kern = mf ? (two ? (work ? ffn_down_f32_mfma_kernel<2, true> : ffn_down_f32_mfma_kernel<2, false>)
                            : (work ? ffn_down_f32_mfma_kernel<1, true> : ffn_down_f32_mfma_kernel<1, false>))
                  : work ? (few ? ffn_down_f32_kernel<true, true> : ffn_down_f32_kernel<false, true>)
                         : (few ? ffn_down_f32_kernel<true, false> : ffn_down_f32_kernel<false, false>);
      kern<<<grid, mf ? kMfThreads : kFfnThreads, 0, st>>>(
          rank_count, shortlist, lists, list_stride, M, ds.n_experts, k, d, F, static_cast<const float *>(wt.w_down),
          static_cast<const float *>(act), seg_expert, seg_off, work, perm, y);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    mark(pass - 1);
  }
  if (!out) return hipSuccess;
  e = launch_combine<float>(ds, y, tok_ids, tok_w, residual, out, x_next, M, 1, st);
  mark(2);
  return e;
}

}  // namespace moespec
