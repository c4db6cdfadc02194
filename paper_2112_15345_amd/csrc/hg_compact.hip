// Per-hop compaction on gfx950 (DistDGLv2, arXiv 2112.15345, Sec. 4.2.2: the
// frontier of the next hop is the unique set of this hop's vertices, and
// compaction relabels vertices and edges).
//
// The newly reached vertices of a node type are deduplicated and put in
// ascending ID order with one mark per vertex: the sampler marks every kept
// source v reached (a byte, or a bit laid out as the frontier bits), and the
// new vertices are the reached vertices whose frontier bit is clear; a prefix
// count of those (per node type) then gives each one its rank, which is its
// position among the new vertices.
// The count is a reduce-then-scan over kTile-word tiles in three launches
// (count per tile; scan of the tile counts; rank and assign), which needs no
// inter-block waiting.  A dense int32 map (vertex -> local ID, meaningful while
// the vertex's frontier bit is set) holds the local IDs of the frontier and of
// the new vertices for the relabel.
#include "hg_device.hpp"
#include "hg_internal.hpp"

namespace hg {

namespace {

unsigned grid_for(int64_t n, int threads, int64_t cap = 1 << 20) {
  int64_t b = (n + threads - 1) / threads;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return unsigned(b);
}

struct CompactArgs {
  HopView hv;
  const TypeStatic *ts;
  int32_t n_types;
  uint8_t *reached;  // reached this hop (one byte per vertex)
  uint32_t *fbits;   // in the frontier (one bit per vertex)
  uint32_t *rbits;   // non-NULL: the hop marked reached bits (laid out as fbits) instead
  const int64_t *tile_base;
  int64_t n_tiles;
  int64_t copy_total;
  int64_t *tile_pre;  // [n_tiles + 1] set bits in earlier tiles, of any type (or look-back words)
  int32_t *tile_cnt;  // per tile: set bits
  int64_t *small;
  bool collect;       // only list the vertices (no map, no frontier bits)
};

// Four flag bytes (each 0 or 1) as four bits: byte k of x lands on bit 24 + k
// of x * 0x01020408, with no carries from the other partial products.
__device__ __forceinline__ uint32_t pack4(uint32_t x) {
  return ((x & 0x01010101u) * 0x01020408u) >> 24;
}
__device__ __forceinline__ uint32_t pack16(uint4 v) {
  return pack4(v.x) | (pack4(v.y) << 4) | (pack4(v.z) << 8) | (pack4(v.w) << 12);
}

// A thread's share of a tile (kTileItems * 32 vertices): their reached flags
// as bits, and their frontier words.
struct TileWords {
  uint2 reached, front;
  __device__ uint2 fresh() const {  // reached, not yet in the frontier
    return uint2{reached.x & ~front.x, reached.y & ~front.y};
  }
};
static_assert(kTileItems == 2, "a thread covers 64 vertices");
__device__ __forceinline__ const uint4 *reached_of(const CompactArgs &A, int64_t tile) {
  return reinterpret_cast<const uint4 *>(A.reached + (tile * kTile + threadIdx.x * kTileItems) * 32);
}
__device__ __forceinline__ TileWords tile_words(const CompactArgs &A, int64_t tile) {
  const int64_t w = tile * kTile + threadIdx.x * kTileItems;
  const uint2 front = *reinterpret_cast<const uint2 *>(A.fbits + w);
  if (A.rbits) return TileWords{*reinterpret_cast<const uint2 *>(A.rbits + w), front};
  const uint4 *r = reached_of(A, tile);
  const uint4 r0 = r[0], r1 = r[1], r2 = r[2], r3 = r[3];
  return TileWords{uint2{pack16(r0) | (pack16(r1) << 16), pack16(r2) | (pack16(r3) << 16)},
                   front};
}
// A lane's value on every lane, in scalar registers.
__device__ __forceinline__ int64_t uniform_from(int64_t x, int lane) {
  const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(uint64_t(x)), lane));
  const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int(uint64_t(x) >> 32), lane));
  return int64_t((uint64_t(hi) << 32) | lo);
}

// Clears the thread's reached bytes or bits (when any is set).
__device__ __forceinline__ void clear_reached(const CompactArgs &A, int64_t tile,
                                              const TileWords &tw) {
  if (A.rbits) {
    if ((tw.reached.x | tw.reached.y) != 0)
      *reinterpret_cast<uint2 *>(A.rbits + tile * kTile + threadIdx.x * kTileItems) =
          uint2{0, 0};
    return;
  }
  if ((tw.reached.x | tw.reached.y) != 0) {
    uint4 *r = const_cast<uint4 *>(reached_of(A, tile));
    const uint4 z{0, 0, 0, 0};
    r[0] = z;
    r[1] = z;
    r[2] = z;
    r[3] = z;
  }
}

// Copies kTile frontier entries into the head of the source lists.
__device__ void copy_tile(const CompactArgs &A, int64_t ct) {
  for (int k = 0; k < kTileItems; ++k) {
    const int64_t x = ct * kTile + k * kTileThreads + threadIdx.x;
    if (x >= A.copy_total) return;
    int64_t acc = 0;
    int t = 0;
    for (; t < A.n_types - 1; ++t) {
      if (x < acc + A.hv.nF[t]) break;
      acc += A.hv.nF[t];
    }
    A.hv.src_out[t][x - acc] = A.hv.frontier[t][x - acc];
  }
}

// 1. Set bits per tile; the blocks past the tiles copy the frontier.
__global__ __launch_bounds__(kTileThreads) void k_bits_count(CompactArgs A) {
  __shared__ int64_t lds[8];
  const int64_t tile = blockIdx.x;
  if (tile >= A.n_tiles) {
    copy_tile(A, tile - A.n_tiles);
    return;
  }
  static_assert(kTileItems == 2, "one 8-byte load per thread");
  const TileWords tw = tile_words(A, tile);
  const uint2 w = tw.fresh();
  int64_t total;
  block_excl_scan_256(__popc(w.x) + __popc(w.y), lds, &total);
  if (threadIdx.x == 0) A.tile_cnt[tile] = int32_t(total);
  // a tile without new vertices is done: the assign pass skips it
  if (total == 0) clear_reached(A, tile, tw);
}

// 2. Exclusive scan of the tile counts over all tiles, in one block: tile_pre
// gets the set bits of every earlier tile (of any type), and tile_pre[n_tiles]
// the total.  A tile's prefix within its type is then tile_pre[tile] -
// tile_pre[first tile of the type]; each type's count of new vertices is the
// difference at its bounds.
constexpr int kScanThreads = 1024;
// Tile counts per thread and pass: all of a pass's loads are issued before
// the block scan, so a pass costs one memory round trip (11k tiles of the
// billion-edge share in one pass instead of eleven).
constexpr int kScanItems = 16;
__global__ __launch_bounds__(kScanThreads) void k_bits_scan(CompactArgs A) {
  constexpr int kWaves = kScanThreads / kWave;
  __shared__ int64_t s_wave[kWaves];
  const int wave = threadIdx.x / kWave;
  const int lane = lane_id();
  int64_t carry = 0;
  for (int64_t c0 = 0; c0 < A.n_tiles; c0 += int64_t(kScanThreads) * kScanItems) {
    const int64_t base = c0 + int64_t(threadIdx.x) * kScanItems;
    int32_t x[kScanItems];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) x[k] = base + k < A.n_tiles ? A.tile_cnt[base + k] : 0;
    int64_t mine = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) mine += x[k];
    const int64_t inc = wave_incl_scan_i64(mine);
    if (lane == kWave - 1) s_wave[wave] = inc;
    __syncthreads();
    int64_t before = 0, sum = 0;
    for (int v = 0; v < kWaves; ++v) {
      const int64_t y = s_wave[v];
      if (v < wave) before += y;
      sum += y;
    }
    int64_t run = carry + before + inc - mine;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      if (base + k < A.n_tiles) A.tile_pre[base + k] = run;
      run += x[k];
    }
    carry += sum;
    __syncthreads();
  }
  if (threadIdx.x == 0) A.tile_pre[A.n_tiles] = carry;
  __syncthreads();
  // new vertices of each type (the block's own stores are visible to it)
  for (int t = threadIdx.x; t < A.n_types; t += kScanThreads)
    A.small[kSlotNew + t] = A.tile_pre[A.tile_base[t + 1]] - A.tile_pre[A.tile_base[t]];
}

// Gives the new vertices of the thread's share of a tile (the first has local
// ID `local`) their local IDs, adds them to the frontier bits and clears the
// reached bits.  All threads of a wavefront call it.  Where many of its vertices
// are new, the wavefront takes its 64 shares of 64 vertices one after the other, a
// lane per vertex, so that the map entries and the listed IDs of a share are
// written together: lanes that each write their own share's vertices make every
// store touch up to 64 lines.  Where few are, those lanes are done in a few
// stores.  A share taken together costs about 35 cycles, a round of stores of n
// lanes about 2 n and not less than those: together it is when some share has more
// new vertices than there are shares with any, or than 17.  (Academic graph, second
// hop, 16 mini-batches, 3.7M new vertices of 31M: 72 us by lanes, 48 together;
// first hop, 0.25M: 13 by lanes, 19 together.)
constexpr int kTogetherFrom = 17;
__device__ __forceinline__ void assign_bits(const CompactArgs &A, int t, int64_t first,
                                            int64_t tile, const TileWords &tw, int64_t local) {
  clear_reached(A, tile, tw);
  const uint2 ab = tw.fresh();
  const uint64_t shares = __ballot((ab.x | ab.y) != 0);
  if (shares == 0) return;
  if ((ab.x | ab.y) != 0 && !A.collect)
    *reinterpret_cast<uint2 *>(A.fbits + tile * kTile + threadIdx.x * kTileItems) =
        uint2{tw.front.x | ab.x, tw.front.y | ab.y};
  int32_t *map = A.ts[t].map;
  int64_t *out = A.hv.src_out[t];
  const int64_t v0 = ((tile - first) * kTile + threadIdx.x * kTileItems) * 32;
  const int many = min(kTogetherFrom, __popcll(shares));
  if (__ballot(__popc(ab.x) + __popc(ab.y) > many) == 0) {
    uint64_t m = uint64_t(ab.x) | (uint64_t(ab.y) << 32);
    for (; m; m &= m - 1) {
      const int64_t v = v0 + (__ffsll((unsigned long long)m) - 1);
      if (!A.collect) map[v] = int32_t(local);
      out[local] = v;
      ++local;
    }
    return;
  }
  const int lane = lane_id();
  const uint64_t below = lanes_below();
  const int64_t w0 = v0 - lane * (kTileItems * 32);  // the wavefront's first vertex
  for (uint64_t m = shares; m; m &= m - 1) {
    const int from = __ffsll((unsigned long long)m) - 1;
    const uint64_t w = uint64_t(uint32_t(__builtin_amdgcn_readlane(int(ab.x), from))) |
                       (uint64_t(uint32_t(__builtin_amdgcn_readlane(int(ab.y), from))) << 32);
    const int64_t at = uniform_from(local, from) + __popcll(w & below);
    const int64_t v = w0 + from * (kTileItems * 32) + lane;
    if ((w >> lane) & 1) {
      if (!A.collect) map[v] = int32_t(at);
      out[at] = v;
    }
  }
}

// 3. Ranks the set bits of a tile within its node type, gives each new vertex
// its local ID and clears the tile's words.
__global__ __launch_bounds__(kTileThreads) void k_bits_assign(CompactArgs A) {
  __shared__ int64_t lds[8];
  const int64_t tile = blockIdx.x;
  if (A.tile_cnt[tile] == 0) return;
  const int t = find_segment(A.tile_base, A.n_types, tile);
  const TileWords tw = tile_words(A, tile);
  const uint2 ab = tw.fresh();
  int64_t total;
  const int64_t pre = block_excl_scan_256(__popc(ab.x) + __popc(ab.y), lds, &total);
  const int64_t first = A.tile_base[t];
  assign_bits(A, t, first, tile, tw,
              A.hv.nF[t] + (A.tile_pre[tile] - A.tile_pre[first]) + pre);
}

// The three steps in one launch for a few tiles: tiles in ticket order, each
// tile's prefix within its type by decoupled look-back (words in tile_pre);
// the last tile of a type writes the type's count.  Tickets past the tiles
// copy the frontier.
__global__ __launch_bounds__(kTileThreads) void k_bits_single(CompactArgs A, uint32_t epoch,
                                                              uint64_t ticket_base) {
  __shared__ int64_t lds[8];
  const int64_t tile = take_ticket(A.small, ticket_base, lds);
  if (tile >= A.n_tiles) {
    copy_tile(A, tile - A.n_tiles);
    return;
  }
  const int t = find_segment(A.tile_base, A.n_types, tile);
  const int64_t first = A.tile_base[t];
  const TileWords tw = tile_words(A, tile);
  const uint2 ab = tw.fresh();
  int64_t agg[1];
  const int64_t pre = block_excl_scan_256(__popc(ab.x) + __popc(ab.y), lds, &agg[0]);
  int64_t ex[1];
  tile_lookback<1>(Lookback{reinterpret_cast<uint64_t *>(A.tile_pre)}, tile, first, epoch, agg,
                   ex, A.small);
  if (tile == A.tile_base[t + 1] - 1 && threadIdx.x == 0)
    A.small[kSlotNew + t] = ex[0] + agg[0];  // new vertices of type t
  assign_bits(A, t, first, tile, tw, A.hv.nF[t] + ex[0] + pre);
}

// Edges per thread of the relabel: four once that leaves eight blocks a CU, else
// one, since the map's random reads are spread over the CUs by the blocks (25k
// edges: 3.9 us with one, 6.0 with four; 7M: 64 and 59).
constexpr int64_t kRelabelLargeFrom = int64_t(2048) * 1024;

// src_local[j] = map of edge j's source type at src_gid[j].  A block takes
// kRelabelTile consecutive edges; the edge types of its first and last edge are
// found by all its threads at once (one round of loads and a barrier), and in a
// block of one edge type, as most are, no edge looks for its own.  Bound by
// the map entries' random reads: a block of 256 edges that staged every edge start
// in LDS and searched them for each edge waited on its steps for 80% of its time
// (75 us in the academic graph's second hop in bundles of 16, 7M edges, against
// 59).
template <int kRelabelItems>
__global__ __launch_bounds__(256) void k_relabel(HopView hv, HopView next, const EtypeStatic *es,
                                                 const int64_t *tile_base, const int64_t *small,
                                                 int32_t n_types, int32_t n_etypes,
                                                 int64_t n_edges, const int64_t *src_gid,
                                                 int32_t *src_local, bool xcd,
                                                 int64_t n_blocks, uint4 *clear,
                                                 int64_t clear_vecs) {
  constexpr int64_t kRelabelTile = 256 * kRelabelItems;
  if (int64_t(blockIdx.x) >= n_blocks) {  // the blocks past the edges' clear
    const int64_t threads = (int64_t(gridDim.x) - n_blocks) * blockDim.x;
    for (int64_t i = (int64_t(blockIdx.x) - n_blocks) * blockDim.x + threadIdx.x; i < clear_vecs;
         i += threads)
      clear[i] = uint4{0, 0, 0, 0};
    return;
  }
  if (blockIdx.x == 0)
    plan_next_hop(hv, next, es, tile_base, small, n_types, n_etypes);
  const int64_t *ebase = small + kSlotNew + n_types;
  // n_blocks is a multiple of kXcds, so that the blocks can be ordered
  // per XCD (xcd_block): a mini-batch's map lines then stay in one L2
  for (int64_t blk = xcd_block(blockIdx.x, n_blocks, xcd); blk * kRelabelTile < n_edges;
       blk += n_blocks) {
    const int64_t j0 = blk * kRelabelTile;
    const int64_t j1 = j0 + kRelabelTile < n_edges ? j0 + kRelabelTile : n_edges;
    int64_t g[kRelabelItems];
#pragma unroll
    for (int u = 0; u < kRelabelItems; ++u) {
      const int64_t j = j0 + u * 256 + threadIdx.x;
      g[u] = j < j1 ? load_global(src_gid + j) : 0;
    }
    // the thread whose edge type holds the first (last) edge says so
    __shared__ int s_e0, s_e1;
    __shared__ const int32_t *s_map;
    for (int e = threadIdx.x; e < n_etypes; e += 256) {
      const int64_t start = ebase[e], end = ebase[e + 1];
      const int32_t *map = es[e].src_map;
      if (start <= j0 && j0 < end) {
        s_e0 = e;
        s_map = map;
      }
      if (start < j1 && j1 <= end) s_e1 = e;
    }
    __syncthreads();
    const int e0 = s_e0, e1 = s_e1;
    const int32_t *map = s_map;
    __syncthreads();  // they are written again for the next tile
    int32_t l[kRelabelItems];
    if (e0 == e1) {
#pragma unroll
      for (int u = 0; u < kRelabelItems; ++u)
        l[u] = j0 + u * 256 + threadIdx.x < j1 ? load_global(map + g[u]) : 0;
    } else {
#pragma unroll
      for (int u = 0; u < kRelabelItems; ++u) {
        const int64_t j = j0 + u * 256 + threadIdx.x;
        l[u] = 0;
        if (j < j1) {
          // ebase[e0] <= j0 <= j < ebase[e1 + 1]
          const int e = e0 + find_segment(ebase + e0, e1 + 1 - e0, j);
          l[u] = load_global(es[e].src_map + g[u]);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < kRelabelItems; ++u) {
      const int64_t j = j0 + u * 256 + threadIdx.x;
      if (j < j1) src_local[j] = l[u];
    }
  }
}

}  // namespace

hipError_t launch_compact(HopView hv, const TypeStatic *ts, int32_t n_types,
                          uint8_t *reached, uint32_t *fbits, const int64_t *tile_base,
                          int64_t n_tiles, int64_t copy_total, int64_t *tile_sums,
                          uint32_t epoch, uint64_t ticket_base, int64_t *small,
                          int64_t *ticketed, hipStream_t stream, bool collect, StageEv ev,
                          uint32_t *rbits) {
  CompactArgs A{hv, ts, n_types, reached, fbits, rbits, tile_base, n_tiles, copy_total, tile_sums,
                reinterpret_cast<int32_t *>(tile_sums + n_tiles + 1), small, collect};
  const int64_t copy_blocks = (copy_total + kTile - 1) / kTile;
  *ticketed = 0;
  if (n_tiles <= kSinglePassTiles) {
    const int64_t blocks = n_tiles + copy_blocks;
    if (blocks > 0) {
      launch_k(k_bits_single, dim3(unsigned(blocks)), dim3(kTileThreads), 0, stream, ev.start,
               ev.stop, A, epoch, ticket_base);
      *ticketed = blocks;
    } else if (ev.any()) {
      hipError_t e = record_empty_stage(ev, stream);
      if (e != hipSuccess) return e;
    }
    return hipGetLastError();
  }
  // n_tiles > kSinglePassTiles here, so every launch has blocks
  launch_k(k_bits_count, dim3(unsigned(n_tiles + copy_blocks)), dim3(kTileThreads), 0, stream,
           ev.start, nullptr, A);
  hipLaunchKernelGGL(k_bits_scan, dim3(1), dim3(kScanThreads), 0, stream, A);
  launch_k(k_bits_assign, dim3(unsigned(n_tiles)), dim3(kTileThreads), 0, stream, nullptr,
           ev.stop, A);
  return hipGetLastError();
}

hipError_t launch_relabel(HopView hv, HopView next, const EtypeStatic *es,
                          const int64_t *tile_base, const int64_t *small,
                          int32_t n_types, int32_t n_etypes, int64_t n_edges,
                          const int64_t *src_gid, int32_t *src_local,
                          hipStream_t stream, StageEv ev, bool xcd_order, uint32_t *clear,
                          int64_t clear_words) {
  // at least one block: block 0 plans the next hop
  const bool large = n_edges >= kRelabelLargeFrom;
  const int64_t blocks = xcd_round(grid_for(n_edges, large ? 1024 : 256));
  const int64_t vecs = clear_words / 4;
  const unsigned grid = unsigned(blocks + (vecs > 0 ? grid_for(vecs, 1024, 2048) : 0));
  launch_k(large ? k_relabel<4> : k_relabel<1>, dim3(grid), dim3(256), 0, stream, ev.start, ev.stop,
           hv, next, es, tile_base, small, n_types, n_etypes, n_edges, src_gid, src_local,
           xcd_order, blocks, reinterpret_cast<uint4 *>(clear), vecs);
  return hipGetLastError();
}

}  // namespace hg
