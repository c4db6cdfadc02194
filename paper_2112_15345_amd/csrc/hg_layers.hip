// Layer-wise (LADIES) sampling on gfx950.  DistDGLv2 (arXiv 2112.15345, Sec.
// 4.2.2) names layer-wise sampling as fitting the same decomposition of
// sampling, compaction and feature copy; the algorithm is LADIES (Zou et al.,
// NeurIPS 2019, Algorithm 1).  Each hop draws a fixed number of vertices per
// node type for the whole layer, with probability proportional to their
// importance, and keeps every in-edge of the frontier from the next frontier.
//
// One hop, after the counting pass has numbered every in-edge of the frontier
// (fanout -1: pair p's in-edges are positions off[p] .. off[p+1]-1); no
// sampler runs, and the edges are read from the CSC where needed:
//  1-4. k_lw_tile_pairs, k_lw_bin_* : the first pair of every 2048-position tile;
//                    then the in-edges grouped into bins of 8192 sources, each
//                    bin's importance summed in LDS (a large bin's by several
//                    blocks) and its candidates listed with its prefix;
//                    k_lw_bin_draw draws among them.  Hops of fewer than
//                    kBinsFromEdges in-edges, and calls whose vertices make more
//                    than kMaxBins bins, instead:
//  1. k_lw_tile_pairs, k_lw_weights : the first pair of every 2048-position
//                    tile; then the importance of every candidate (a source
//                    not in the frontier, which is marked reached): sum of
//                    floor(2^32 / deg(v)^2) over its edges into the frontier,
//                    64-bit atomics (exact in any order), a block per tile of
//                    positions whose etypes, and each position's pair, are in
//                    LDS (as in the kept-edge passes);
//  2. compaction   : (collect mode) the candidates of each type, ascending;
//  3. k_lw_scan_*  : exclusive prefix of their importance per type
//                    (reduce-then-scan over 512-candidate tiles);
//  4. k_lw_draw    : draw k takes r = floor(x * total / 2^64), x from
//                    Philox4x32-10 at (k, 2^30 | hop, type), and marks the
//                    candidate whose interval [prefix, prefix + weight) holds
//                    r (binary search);
//  5. compaction   : the drawn vertices join the frontier (ascending);
//  6. k_lw_keep_*  : the kept in-edges (source in the next frontier): one bit
//                    per in-edge, a scan of the tiles' counts, and the kept
//                    ones emitted in order;
//  7. k_lw_indptr  : the block CSC, the kept edge starts per etype, and the
//                    next hop's plan.
#include <algorithm>

#include "hg_device.hpp"
#include "hg_internal.hpp"

namespace hg {

namespace {

constexpr int kLwThreads = 256;
constexpr int kLwItems = 2;
constexpr int64_t kLwTile = int64_t(kLwThreads) * kLwItems;
static_assert(kLwTile == kLayerTile, "the runtime sizes the scans in these tiles");

__device__ __forceinline__ int64_t gs_start() {
  return int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
}
__device__ __forceinline__ int64_t gs_step() {
  return int64_t(gridDim.x) * blockDim.x;
}

unsigned grid_for(int64_t n, int threads, int64_t cap = 1 << 16) {
  int64_t b = (n + threads - 1) / threads;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return unsigned(b);
}

// floor(2^32 / d^2) for d >= 1 (zero once d^2 > 2^32).  The correctly
// rounded double quotient lies between the two integers around the exact one,
// so its floor is the exact floor or one above; integer checks settle it.
__device__ __forceinline__ uint64_t layer_weight(int64_t d) {
  const uint64_t d2 = uint64_t(d) * uint64_t(d);
  constexpr uint64_t kOne = uint64_t(1) << 32;
  if (d2 > kOne) return 0;
  uint64_t q = uint64_t(4294967296.0 / double(d2));
  if (q * d2 > kOne) --q;
  else if ((q + 1) * d2 <= kOne) ++q;
  return q;
}

// A record of an in-edge: its source's place in the bin (13 bits) and the code of
// the destination's in-degree d (17 bits): d, or 0 past 65536, where the
// importance floor(2^32 / d^2) is 0.
__device__ __forceinline__ uint32_t degree_code(int64_t d) {
  return d <= 65536 ? uint32_t(d) : 0u;
}
constexpr int kBinBits = 13, kDegreeBits = 17;
static_assert(kBinVerts == int64_t(1) << kBinBits, "a place in a bin takes 13 bits");
__device__ __forceinline__ uint64_t code_weight(uint32_t d) {
  return d ? layer_weight(int64_t(d)) : 0;
}

__device__ __forceinline__ const int64_t *ebase_of(const LayerArgs &A) {
  return A.small + kSlotNew + A.n_types;  // starts of each etype's emitted edges
}
__device__ __forceinline__ int64_t *kept_base_of(const LayerArgs &A) {
  return A.small + kSlotNew + A.n_types + A.n_etypes + 1;
}

// The in-edges of the frontier are never written out.  The counting pass
// numbers them: pair p's in-edges are positions off[p] .. off[p+1]-1, at CSC
// slots plo[p] + (i - off[p]); position i lies in the last pair with
// off[p] <= i (empty pairs share the offset of the pair after them).  The
// kernels below read the source of position i from the CSC where they need it.

// The etypes that a block's contiguous range [j0, j1) of positions spans,
// resolved once per block: their starts and what the per-edge work reads of
// them.  A range over more than kTileSegs etypes leaves n = 0 and its edges
// search the etype starts one by one.
constexpr int kTileSegs = 32;
struct TileSegs {
  int64_t start[kTileSegs + 1];
  const uint32_t *fbits[kTileSegs];  // frontier bits of the source type
  void *per_seg[kTileSegs];          // importance array of the source type, or source map
  const int64_t *indices[kTileSegs];
  uint8_t *reached[kTileSegs];       // reached flags of the source type
  int64_t pair_base[kTileSegs];
  int32_t bin0[kTileSegs];           // first bin of the source type
  int e0, n;
};

// kKind 0: per_seg = importance array of the source type; 1: source map; 2: bins.
// pa, pb: the pair of the range's first position and a pair not before that of
// its last one (whose etypes bound the range's; two loads instead of two
// searches over the etype starts).
template <int kKind>
__device__ void tile_segs_load(const LayerArgs &A, int64_t pa, int64_t pb, TileSegs &T) {
  const int64_t *ebase = ebase_of(A);
  const int a = A.pa.pet[pa], b = A.pa.pet[pb];
  const int n = b - a + 1 <= kTileSegs ? b - a + 1 : 0;
  if (threadIdx.x == 0) {
    T.e0 = a;
    T.n = n;
  }
  if (int(threadIdx.x) <= n && n > 0) {
    const int e = a + int(threadIdx.x);
    T.start[threadIdx.x] = ebase[e];
    if (int(threadIdx.x) < n) {
      const EtypeStatic &E = A.es[e];
      T.fbits[threadIdx.x] = A.ts[E.src_type].fbits;
      if (kKind == 0)
        T.per_seg[threadIdx.x] = A.wt[E.src_type];
      else if (kKind == 1)
        T.per_seg[threadIdx.x] = E.src_map;
      T.indices[threadIdx.x] = E.indices;
      T.reached[threadIdx.x] = E.src_reached;
      T.pair_base[threadIdx.x] = A.hv.pair_base[e];
      if (kKind == 2)
        T.bin0[threadIdx.x] = int32_t(kBinsPerTile * A.tile_base[E.src_type]);
    }
  }
}

// Segment of position j in the block's table, from a hint not above it (the
// positions of one thread come in ascending order).
__device__ __forceinline__ int tile_seg(const TileSegs &T, int s, int64_t j) {
  while (s + 1 < T.n && T.start[s + 1] <= j) ++s;
  return s;
}

// What a position needs of its etype.
struct SegView {
  void *per_seg;
  const int64_t *indices;
  uint8_t *reached;
  int64_t pair_base;
};
// The etype of position j: its segment of the block's table, or without a
// table the etype itself.
__device__ __forceinline__ int seg_index(const LayerArgs &A, const TileSegs &T, int &s,
                                         int64_t j) {
  if (T.n > 0) return s = tile_seg(T, s, j);
  return find_segment(ebase_of(A), A.n_etypes, j);
}
template <int kKind>
__device__ __forceinline__ SegView seg_view(const LayerArgs &A, const TileSegs &T, int x) {
  if (T.n > 0)
    return SegView{T.per_seg[x], T.indices[x], T.reached[x], T.pair_base[x]};
  const EtypeStatic &E = A.es[x];
  return SegView{kKind == 0 ? static_cast<void *>(A.wt[E.src_type]) : static_cast<void *>(E.src_map),
                 E.indices, E.src_reached, A.hv.pair_base[x]};
}

// tile_pair[t] = the pair of position t * kEdgeTile, for every tile t of
// positions; tile_pair[n_tiles] = the last pair.  Each non-empty pair writes
// the tiles that start inside it.
__global__ __launch_bounds__(256) void k_lw_tile_pairs(LayerArgs A) {
  for (int64_t p = gs_start(); p < A.n_pairs; p += gs_step()) {
    const int64_t lo = A.pa.off[p], hi = A.pa.off[p + 1];
    for (int64_t t = (lo + kEdgeTile - 1) / kEdgeTile; t * kEdgeTile < hi; ++t)
      A.tile_pair[t] = p;
  }
  if (gs_start() == 0) A.tile_pair[A.n_edge_tiles] = A.n_pairs - 1;
}

// The pair of every position of a tile, in LDS: the tile's position at which the
// pair starts (0 for the first pair, which may start before the tile).  Each
// non-empty pair marks its start, and a running maximum over the positions spreads
// the marks.  `slot[start]` is the CSC slot that the tile's position 0 would have in
// the pair (modulo 2^32, as in-edges of a type are fewer), or for kPairs the pair
// itself, counted from the tile's first.  The marks are taken from the pairs between
// tile_pair of the tile and of the next one; of more than kTilePairs of them (long
// runs of empty pairs) no table is made, and each position searches the pair
// offsets.  A binary search of a table of pairs, for each position, was a chain of
// LDS reads eight times as long as this scan, and a table of 512 or 1024 pairs did
// not hold most tiles of sparse types (2^18 in-edges, two a pair: keep flags 28 us
// and weights 37, now 13 and 23).
constexpr int kPlaceBits = 11;
static_assert(kEdgeTile == int64_t(1) << kPlaceBits, "a place in a tile takes 11 bits");
static_assert(kPlaceBits + kDegreeBits <= 32, "a place and a degree's code share a word");
struct TilePairs {
  // per position its pair's start; at the start, above it, the pair's degree code
  uint32_t at[kEdgeTile];
  uint32_t slot[kEdgeTile];
};
struct PairRange {
  int64_t p0, p1;
  int n;  // 0: no table
};
template <int kKind, bool kPairs = false>
__device__ void tile_tables(const LayerArgs &A, int64_t tile, TileSegs &T, TilePairs &Q,
                            PairRange &R) {
  __shared__ uint32_t s_max[256 / kWave];
  const int64_t pa = A.tile_pair[tile], pb = A.tile_pair[tile + 1];
  const int64_t j0 = tile * kEdgeTile;
  R = PairRange{pa, pb, pb - pa + 1 <= kTilePairs ? int(pb - pa + 1) : 0};
  tile_segs_load<kKind>(A, pa, pb, T);
  if (R.n > 0) {
    uint4 *at = reinterpret_cast<uint4 *>(Q.at);
    at[threadIdx.x] = at[threadIdx.x + 256] = uint4{0, 0, 0, 0};
    __syncthreads();
#pragma unroll 2
    for (int64_t p = pa + threadIdx.x; p <= pb; p += 256) {
      const int64_t lo = A.pa.off[p], hi = A.pa.off[p + 1];
      // (the last of them may start with the next tile)
      if (hi <= lo || hi <= j0 || lo >= j0 + kEdgeTile) continue;
      const uint32_t x = lo > j0 ? uint32_t(lo - j0) : 0u;
      Q.at[x] = x | (kKind == 1 ? 0u : degree_code(A.pa.pdeg[p]) << kPlaceBits);
      Q.slot[x] = kPairs ? uint32_t(p - pa) : uint32_t(A.pa.plo[p] - (lo - j0));
    }
    __syncthreads();
    constexpr uint32_t kPlace = uint32_t(kEdgeTile) - 1;
    uint4 a = at[2 * threadIdx.x], b = at[2 * threadIdx.x + 1];
    uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    uint32_t m = 0;  // places ascend: the last start of the thread's positions
#pragma unroll
    for (int k = 0; k < 8; ++k) m = max(m, w[k] & kPlace);
    uint32_t inc = m;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const uint32_t o = __shfl_up(inc, d, kWave);
      if (lane_id() >= d) inc = max(inc, o);
    }
    const int wave = int(threadIdx.x) / kWave;
    if (lane_id() == kWave - 1) s_max[wave] = inc;
    uint32_t run = __shfl_up(inc, 1, kWave);
    if (lane_id() == 0) run = 0;
    __syncthreads();
    for (int x = 0; x < wave; ++x) run = max(run, s_max[x]);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      run = max(run, w[k] & kPlace);
      w[k] = (w[k] & ~kPlace) | run;
    }
    at[2 * threadIdx.x] = uint4{w[0], w[1], w[2], w[3]};
    at[2 * threadIdx.x + 1] = uint4{w[4], w[5], w[6], w[7]};
  }
  __syncthreads();
}

// The pair of a position j, as what its tile's table or the pair arrays say of it.
struct PairAt {
  int64_t start;  // its place in the tile, or (no table) the pair
};
__device__ __forceinline__ PairAt pair_at(const LayerArgs &A, const TilePairs &Q,
                                          const PairRange &R, int64_t j) {
  if (R.n > 0) return PairAt{int64_t(Q.at[j & (kEdgeTile - 1)] & uint32_t(kEdgeTile - 1))};
  int64_t lo = R.p0, hi = R.p1 + 1;
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (A.pa.off[mid] <= j)
      lo = mid;
    else
      hi = mid;
  }
  return PairAt{lo};
}
// Its CSC slot (of a table without kPairs), and its degree's code.
__device__ __forceinline__ int64_t slot_at(const LayerArgs &A, const TilePairs &Q,
                                           const PairRange &R, PairAt p, int64_t j) {
  return R.n > 0 ? int64_t(uint32_t(Q.slot[p.start] + uint32_t(j & (kEdgeTile - 1))))
                 : A.pa.plo[p.start] + (j - A.pa.off[p.start]);
}
__device__ __forceinline__ uint32_t code_at(const LayerArgs &A, const TilePairs &Q,
                                            const PairRange &R, PairAt p) {
  return R.n > 0 ? Q.at[p.start] >> kPlaceBits : degree_code(A.pa.pdeg[p.start]);
}

// Blocks of 256 threads take tiles of kEdgeTile positions, each thread every
// 256th position of the tile; the sources of all its positions are loaded
// before any is used, then their frontier words.
constexpr int kEdgeItems = int(kEdgeTile / 256);

// The source of each of a thread's positions (-1 past the end), and what the
// position needs of its etype and pair.
struct EdgeItems {
  int seg[kEdgeItems];
  PairAt pair[kEdgeItems];
  int64_t u[kEdgeItems];
};
__device__ __forceinline__ void edge_items(const LayerArgs &A, const TileSegs &T,
                                           const TilePairs &Q, const PairRange &R, int64_t tile,
                                           EdgeItems &I) {
  int s = 0;
#pragma unroll
  for (int k = 0; k < kEdgeItems; ++k) {
    const int64_t j = tile * kEdgeTile + k * 256 + threadIdx.x;
    I.u[k] = -1;
    I.seg[k] = 0;
    I.pair[k] = PairAt{0};
    if (j < A.n_all) {
      I.seg[k] = seg_index(A, T, s, j);
      I.pair[k] = pair_at(A, Q, R, j);
      const int64_t *ix = T.n > 0 ? T.indices[I.seg[k]] : A.es[I.seg[k]].indices;
      I.u[k] = load_global(ix + slot_at(A, Q, R, I.pair[k], j));
    }
  }
}

__global__ __launch_bounds__(256) void k_lw_weights(LayerArgs A) {
  __shared__ TileSegs T;
  __shared__ __align__(16) TilePairs Q;
  const int64_t tile = blockIdx.x;
  PairRange R;
  tile_tables<0>(A, tile, T, Q, R);
  EdgeItems I;
  edge_items(A, T, Q, R, tile, I);
  uint32_t f[kEdgeItems];
#pragma unroll
  for (int k = 0; k < kEdgeItems; ++k) {
    const uint32_t *fb = T.n > 0 ? T.fbits[I.seg[k]] : A.ts[A.es[I.seg[k]].src_type].fbits;
    f[k] = I.u[k] >= 0 ? load_global(fb + (I.u[k] >> 5)) : ~0u;
  }
#pragma unroll
  for (int k = 0; k < kEdgeItems; ++k) {
    const int64_t u = I.u[k];
    if (u < 0 || ((f[k] >> (u & 31)) & 1u)) continue;
    const SegView v = seg_view<0>(A, T, I.seg[k]);
    v.reached[u] = 1;  // a candidate
    const uint64_t w = code_weight(code_at(A, Q, R, I.pair[k]));
    if (w)
      atomicAdd(reinterpret_cast<unsigned long long *>(static_cast<uint64_t *>(v.per_seg) + u),
                (unsigned long long)w);
  }
}

// ---- importance by bins -------------------------------------------------------
// Global atomics run at 24e9 per second on this GPU wherever their targets lie (8
// MiB or 256 MiB, on one XCD or all), so adding every in-edge's importance to a
// global array takes 1.2 ms for the academic graph's second hop in bundles of 16
// (44M in-edges), and the candidates then have to be listed and scanned (0.27 ms).
// Grouped by bin first (count, scan, scatter: 4 bytes an in-edge), a bin's sums
// live in LDS, its candidates come out in ascending ID with their prefix, and only
// the bins are scanned: 183 us counting, 302 scattering, 199 summing and 30 for the
// scans in place of 1.5 ms.  Two kinds of hops keep the atomics: those of fewer than
// kBinsFromEdges in-edges, where the launches cost more than the atomics, and those of
// a call whose vertices make more than kMaxBins bins (67M vertices), whose in-edges
// are few next to its vertices and whose counts of the bins would no longer fit in a
// block's LDS beside its tables.

// Blocks of 256 threads take kBinTiles tiles of positions.
constexpr int kBinTiles = 2;

// The bin and record of each of a thread's positions in a tile (bin -1: past the
// end).
__device__ __forceinline__ void bin_items(const LayerArgs &A, const TileSegs &T,
                                          const TilePairs &Q, const PairRange &R, int64_t tile,
                                          int32_t (&bin)[kEdgeItems], uint32_t (&rec)[kEdgeItems]) {
  EdgeItems I;
  edge_items(A, T, Q, R, tile, I);
#pragma unroll
  for (int k = 0; k < kEdgeItems; ++k) {
    bin[k] = -1;
    rec[k] = 0;
    if (I.u[k] < 0) continue;
    const int32_t b0 = T.n > 0 ? T.bin0[I.seg[k]]
                               : int32_t(kBinsPerTile * A.tile_base[A.es[I.seg[k]].src_type]);
    const uint32_t d = code_at(A, Q, R, I.pair[k]);
    bin[k] = b0 + int32_t(I.u[k] >> kBinBits);
    rec[k] = uint32_t(I.u[k] & (kBinVerts - 1)) | (d << kBinBits);
  }
}

// In-edges per bin.
__global__ __launch_bounds__(256) void k_lw_bin_count(LayerArgs A) {
  __shared__ TileSegs T;
  __shared__ __align__(16) TilePairs Q;
  extern __shared__ __align__(16) char bin_lds[];
  uint32_t *cnt = reinterpret_cast<uint32_t *>(bin_lds);
  for (int b = threadIdx.x; b < A.n_bins; b += 256) cnt[b] = 0;
  for (int x = 0; x < kBinTiles; ++x) {
    const int64_t tile = int64_t(blockIdx.x) * kBinTiles + x;
    if (tile >= A.n_edge_tiles) break;
    __syncthreads();  // the counts are clear, and the tables free again
    PairRange R;
    tile_tables<2>(A, tile, T, Q, R);
    int32_t bin[kEdgeItems];
    uint32_t rec[kEdgeItems];
    bin_items(A, T, Q, R, tile, bin, rec);
#pragma unroll
    for (int k = 0; k < kEdgeItems; ++k)
      if (bin[k] >= 0) atomicAdd(cnt + bin[k], 1u);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < A.n_bins; b += 256)
    if (cnt[b]) atomicAdd(A.bin_edges + b, cnt[b]);
}

// Two exclusive scans over n values each in one block of 1024 threads: pa[i] of
// a(i), pb[i] of b(i), and their totals at n.
template <typename FA, typename FB>
__device__ void scan_two(int64_t n, FA a, FB b, int64_t *pa, int64_t *pb) {
  constexpr int kWaves = 1024 / kWave;
  constexpr int kPer = 8;
  __shared__ int64_t s_a[kWaves], s_b[kWaves];
  const int wave = int(threadIdx.x) / kWave, lane = lane_id();
  int64_t ca = 0, cb = 0;
  for (int64_t c0 = 0; c0 < n; c0 += 1024 * kPer) {
    const int64_t i0 = c0 + int64_t(threadIdx.x) * kPer;
    int64_t xa[kPer], xb[kPer], ma = 0, mb = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      xa[k] = i0 + k < n ? a(i0 + k) : 0;
      xb[k] = i0 + k < n ? b(i0 + k) : 0;
      ma += xa[k];
      mb += xb[k];
    }
    const int64_t ia = wave_incl_scan_i64(ma), ib = wave_incl_scan_i64(mb);
    if (lane == kWave - 1) {
      s_a[wave] = ia;
      s_b[wave] = ib;
    }
    __syncthreads();
    int64_t ra = ca + ia - ma, rb = cb + ib - mb;
    for (int w = 0; w < kWaves; ++w) {
      if (w < wave) {
        ra += s_a[w];
        rb += s_b[w];
      }
      ca += s_a[w];
      cb += s_b[w];
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      if (i0 + k < n) {
        pa[i0 + k] = ra;
        pb[i0 + k] = rb;
      }
      ra += xa[k];
      rb += xb[k];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    pa[n] = ca;
    pb[n] = cb;
  }
}

// Where each bin's records start, and the room for its candidates; the parts of the
// large bins, and their places among the large ones.
__global__ __launch_bounds__(1024) void k_lw_bin_starts(LayerArgs A) {
  scan_two(
      A.n_bins, [&](int64_t b) { return int64_t(A.bin_edges[b]); },
      [&](int64_t b) { return min(int64_t(A.bin_edges[b]), kBinVerts); }, A.bin_rec, A.bin_cap);
  scan_two(
      A.n_bins, [&](int64_t b) { return bin_parts(int64_t(A.bin_edges[b])); },
      [&](int64_t b) { return bin_parts(int64_t(A.bin_edges[b])) > 0 ? 1 : 0; }, A.bin_part,
      A.bin_big);
  __syncthreads();
  for (int64_t b = threadIdx.x; b < A.n_bins; b += 1024) A.bin_at[b] = uint32_t(A.bin_rec[b]);
}

// The records, grouped by bin (in any order within one): a block counts its
// in-edges per bin in LDS, takes room for them in each bin with one global atomic
// and writes them.
__global__ __launch_bounds__(256) void k_lw_bin_scatter(LayerArgs A) {
  __shared__ TileSegs T;
  __shared__ __align__(16) TilePairs Q;
  extern __shared__ __align__(16) char bin_lds[];
  uint32_t *cnt = reinterpret_cast<uint32_t *>(bin_lds);
  for (int b = threadIdx.x; b < A.n_bins; b += 256) cnt[b] = 0;
  int32_t bin[kBinTiles][kEdgeItems];
  uint32_t rec[kBinTiles][kEdgeItems], rank[kBinTiles][kEdgeItems];
#pragma unroll
  for (int x = 0; x < kBinTiles; ++x) {
    const int64_t tile = int64_t(blockIdx.x) * kBinTiles + x;
    __syncthreads();  // the counts are clear, and the tables free again
    if (tile < A.n_edge_tiles) {
      PairRange R;
      tile_tables<2>(A, tile, T, Q, R);
      bin_items(A, T, Q, R, tile, bin[x], rec[x]);
#pragma unroll
      for (int k = 0; k < kEdgeItems; ++k)
        rank[x][k] = bin[x][k] >= 0 ? atomicAdd(cnt + bin[x][k], 1u) : 0;
    } else {
#pragma unroll
      for (int k = 0; k < kEdgeItems; ++k) {
        bin[x][k] = -1;
        rec[x][k] = rank[x][k] = 0;
      }
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < A.n_bins; b += 256)
    if (cnt[b]) cnt[b] = atomicAdd(A.bin_at + b, cnt[b]);
  __syncthreads();
#pragma unroll
  for (int x = 0; x < kBinTiles; ++x)
#pragma unroll
    for (int k = 0; k < kEdgeItems; ++k)
      if (bin[x][k] >= 0) A.rec[cnt[bin[x][k]] + rank[x][k]] = rec[x][k];
}

// A block per bin, and before it a block per part of the bins of more than kBinPart
// records: a block adds a record in about 0.5 ns, so that one with a whole large
// bin works on while the chip is idle.  (A call of
// 4M in-edges from a type of 100k vertices, 12 bins: 425 us with a block per bin, 263
// with parts, 296 by atomics; 90% of them from one of 8000 vertices: 2326, 257 and
// 348, or 5040 by atomics where popular sources make those queue.)
// The importance of the bin's vertices is summed in LDS, then its
// candidates (sources of in-edges that are not in the frontier) in ascending ID
// with the importance before them.  An in-edge of no importance sets its source's
// top bit instead (the sums stay below 2^63: fewer than 2^31 in-edges of at most
// 2^32).  A thread lists 16 consecutive vertices; the place of a vertex in its
// group of 16 is turned by the group's number, so that the threads' reads spread
// over the LDS banks.
constexpr int kBinThreads = 512;
constexpr int kBinPer = int(kBinVerts) / kBinThreads;
static_assert(kBinPer == 16, "a thread lists half a frontier word");
constexpr int kBinLoads = 8;
__device__ __forceinline__ int bin_place(int v) { return v ^ ((v / kBinPer) & (kBinPer - 1)); }
constexpr unsigned long long kBinMark = 1ull << 63;

// Records [r0, r1) added to the cleared sums of their bin.  All threads of the block
// call it; it ends with a barrier.
__device__ void sum_records(const LayerArgs &A, int64_t r0, int64_t r1, unsigned long long *acc) {
  for (int i = threadIdx.x; i < int(kBinVerts); i += kBinThreads) acc[i] = 0;
  __syncthreads();
  // (records loaded kBinLoads at a time: one by one, the block would wait on
  // each load in turn)
  for (int64_t r = r0 + threadIdx.x; r < r1; r += kBinLoads * kBinThreads) {
    uint32_t x[kBinLoads];
#pragma unroll
    for (int k = 0; k < kBinLoads; ++k)
      x[k] = r + k * kBinThreads < r1 ? load_global(A.rec + r + k * kBinThreads) : ~0u;
#pragma unroll
    for (int k = 0; k < kBinLoads; ++k) {
      if (x[k] == ~0u) continue;  // (a record takes 30 bits)
      const int at = bin_place(int(x[k] & uint32_t(kBinVerts - 1)));
      const uint64_t w = code_weight(x[k] >> kBinBits);
      if (w)
        atomicAdd(acc + at, (unsigned long long)w);
      else
        atomicOr(acc + at, kBinMark);
    }
  }
  __syncthreads();
}

// A block per part of the large bins: the part's sums are added to the bin's in
// memory, which its block of k_lw_bin_sum then takes.
__global__ __launch_bounds__(kBinThreads) void k_lw_bin_parts(LayerArgs A) {
  __shared__ unsigned long long acc[kBinVerts];
  __shared__ int s_bin;
  const int64_t x = blockIdx.x;
  if (x >= A.bin_part[A.n_bins]) return;
  for (int b = threadIdx.x; b < A.n_bins; b += kBinThreads)
    if (A.bin_part[b] <= x && x < A.bin_part[b + 1]) s_bin = b;
  __syncthreads();
  const int b = s_bin;
  const int64_t r0 = A.bin_rec[b], n = A.bin_rec[b + 1] - r0;
  const int64_t parts = A.bin_part[b + 1] - A.bin_part[b], i = x - A.bin_part[b];
  sum_records(A, r0 + n * i / parts, r0 + n * (i + 1) / parts, acc);
  unsigned long long *sums = A.big_sums + A.bin_big[b] * kBinVerts;
  for (int v = threadIdx.x; v < int(kBinVerts); v += kBinThreads) {
    const unsigned long long w = acc[v];
    if (w & ~kBinMark)
      atomicAdd(sums + v, w & ~kBinMark);
    else if (w)
      atomicOr(sums + v, kBinMark);
  }
}

__global__ __launch_bounds__(kBinThreads) void k_lw_bin_sum(LayerArgs A) {
  __shared__ unsigned long long acc[kBinVerts];
  constexpr int kWaves = kBinThreads / kWave;
  const int64_t b = blockIdx.x;
  const int64_t r0 = A.bin_rec[b], r1 = A.bin_rec[b + 1];
  if (r0 == r1) {
    if (threadIdx.x == 0) A.bin_n[b] = A.bin_w[b] = 0;
    return;
  }
  if (bin_parts(r1 - r0) > 0) {  // summed by parts; the sums are zero between hops
    unsigned long long *sums = A.big_sums + A.bin_big[b] * kBinVerts;
    for (int v = threadIdx.x; v < int(kBinVerts); v += kBinThreads) {
      acc[v] = sums[v];
      sums[v] = 0;
    }
    __syncthreads();
  } else {
    sum_records(A, r0, r1, acc);
  }
  const int v0 = int(threadIdx.x) * kBinPer;
  const uint32_t front = A.fbits[b * (kBinVerts / 32) + v0 / 32] >> (v0 & 31);
  int64_t n = 0, w = 0;
  uint32_t cand = 0;
  int64_t a[kBinPer];
#pragma unroll
  for (int k = 0; k < kBinPer; ++k) {
    const unsigned long long x = acc[bin_place(v0 + k)];
    a[k] = int64_t(x & ~kBinMark);
    if (x != 0 && !((front >> k) & 1u)) {
      cand |= 1u << k;
      ++n;
      w += a[k];
    }
  }
  __syncthreads();  // the sums are read: their place holds the block scan
  int64_t *s_n = reinterpret_cast<int64_t *>(acc), *s_w = s_n + kWaves;
  const int wave = int(threadIdx.x) / kWave;
  const int64_t in = wave_incl_scan_i64(n), iw = wave_incl_scan_i64(w);
  if (lane_id() == kWave - 1) {
    s_n[wave] = in;
    s_w[wave] = iw;
  }
  __syncthreads();
  int64_t at = A.bin_cap[b] + in - n, pre = iw - w;
  int64_t tn = 0, tw = 0;
  for (int x = 0; x < kWaves; ++x) {
    if (x < wave) {
      at += s_n[x];
      pre += s_w[x];
    }
    tn += s_n[x];
    tw += s_w[x];
  }
#pragma unroll
  for (int k = 0; k < kBinPer; ++k) {
    if (!((cand >> k) & 1u)) continue;
    A.bin_cand_off[at] = v0 + k;
    A.bin_cand_pre[at] = uint64_t(pre);
    pre += a[k];
    ++at;
  }
  if (threadIdx.x == 0) {
    A.bin_n[b] = tn;
    A.bin_w[b] = tw;
  }
}

// Candidates and importance before each bin; the bins' in-edge counts are clear
// for the next hop.
__global__ __launch_bounds__(1024) void k_lw_bin_totals(LayerArgs A) {
  scan_two(
      A.n_bins, [&](int64_t b) { return A.bin_n[b]; }, [&](int64_t b) { return A.bin_w[b]; },
      A.bin_n_pre, A.bin_w_pre);
  for (int64_t b = threadIdx.x; b < A.n_bins; b += 1024) A.bin_edges[b] = 0;
}

// The last i in [lo, hi) with pre[i] <= x (pre non-decreasing, pre[lo] <= x).
template <typename V>
__device__ __forceinline__ int64_t last_not_above(const V *pre, int64_t lo, int64_t hi, V x) {
  while (hi - lo > 1) {
    const int64_t m = lo + (hi - lo) / 2;
    if (pre[m] <= x)
      lo = m;
    else
      hi = m;
  }
  return lo;
}

// k_lw_draw over the bins' candidates: a bin by its prefix, then a candidate in
// it.  As in k_lw_draw, a candidate (or bin) of no importance shares the prefix of
// the next one, and is never the last with a prefix not above r.
__global__ __launch_bounds__(256) void k_lw_bin_draw(LayerArgs A) {
  const int64_t n = A.draw_base[A.n_types];
  for (int64_t x = gs_start(); x < n; x += gs_step()) {
    const int t = find_segment(A.draw_base, A.n_types, x);
    const int64_t k = x - A.draw_base[t];
    const int64_t b0 = kBinsPerTile * A.tile_base[t], b1 = kBinsPerTile * A.tile_base[t + 1];
    if (b0 == b1) continue;
    int64_t b, c;
    if (A.draws[t] < 0) {
      if (k >= A.bin_n_pre[b1] - A.bin_n_pre[b0]) continue;
      const int64_t y = A.bin_n_pre[b0] + k;
      b = last_not_above(A.bin_n_pre, b0, b1, y);
      c = A.bin_cap[b] + (y - A.bin_n_pre[b]);
    } else {
      const int copy = t / A.key_T;
      const uint64_t sigma = A.sigmas[copy];
      const int64_t w0 = A.bin_w_pre[b0];
      const uint64_t total = uint64_t(A.bin_w_pre[b1] - w0);
      if (total == 0) continue;
      const U32x4 r4 = philox4x32_10(U32x4{uint32_t(k), uint32_t(uint64_t(k) >> 32),
                                           0x40000000u | uint32_t(A.hop),
                                           uint32_t(t - copy * A.key_T)},
                                     uint32_t(sigma), uint32_t(sigma >> 32));
      const uint64_t r = __umul64hi(uint64_t(r4.x) | (uint64_t(r4.y) << 32), total);
      b = last_not_above(A.bin_w_pre, b0, b1, w0 + int64_t(r));
      const uint64_t in = r - uint64_t(A.bin_w_pre[b] - w0);
      c = last_not_above(A.bin_cand_pre, A.bin_cap[b], A.bin_cap[b] + A.bin_n[b], in);
    }
    A.ts[t].reached[(b - b0) * kBinVerts + A.bin_cand_off[c]] = 1;
  }
}

// ---- the kept in-edges -------------------------------------------------------
// A kept in-edge has its source in the next frontier.  Few are (a hop keeps
// some thousands of millions of in-edges), so a first pass leaves one bit per
// position (keep_bits, a word per 64 positions), each word's kept edges before
// it within its tile (keep_pre) and the tile's count; after a scan of the tile
// counts only the set bits are looked at again, and the kept edges before any
// position are tile_pre + keep_pre + a population count.  The flags pass is
// bound by its reads (8 B a position and a frontier word); the academic graph's
// second hop in bundles of 16 (44M in-edges, 0.3M kept) takes 215 us for the
// flags, 18 for the scan and 61 for the kept edges, where a reduce and an apply
// pass that both read every source and wrote a prefix for every position took
// 690 with their scan.  Ordering the blocks per XCD changed none of them.
constexpr int kKeepWords = int(kEdgeTile / 64);  // words per tile

__global__ __launch_bounds__(256) void k_lw_keep_flags(LayerArgs A) {
  __shared__ TileSegs T;
  __shared__ __align__(16) TilePairs Q;
  __shared__ int32_t s_cnt[kKeepWords];
  const int64_t tile = blockIdx.x;
  PairRange R;
  tile_tables<1>(A, tile, T, Q, R);
  EdgeItems I;
  edge_items(A, T, Q, R, tile, I);
  const int wave = int(threadIdx.x) / kWave;
#pragma unroll
  for (int k = 0; k < kEdgeItems; ++k) {
    const uint32_t *fb = T.n > 0 ? T.fbits[I.seg[k]] : A.ts[A.es[I.seg[k]].src_type].fbits;
    const uint32_t f = I.u[k] >= 0 ? load_global(fb + (I.u[k] >> 5)) : 0u;
    const uint64_t bal = __ballot((f >> (I.u[k] & 31)) & 1u);
    if (lane_id() == 0) {
      const int w = k * 4 + wave;
      s_cnt[w] = __popcll(bal);
      A.keep_bits[tile * kKeepWords + w] = bal;
    }
  }
  __syncthreads();
  if (threadIdx.x < kKeepWords) {
    int inc = s_cnt[threadIdx.x];
#pragma unroll
    for (int d = 1; d < kKeepWords; d <<= 1) {
      const int o = __shfl_up(inc, d, kKeepWords);
      if (int(threadIdx.x) >= d) inc += o;
    }
    A.keep_pre[tile * kKeepWords + threadIdx.x] = inc - s_cnt[threadIdx.x];
    if (threadIdx.x == kKeepWords - 1) A.tile_sum[tile] = inc;
  }
}

// Kept edges before position i (i <= n_all).
__device__ __forceinline__ int64_t kept_before(const LayerArgs &A, int64_t i) {
  if (A.n_all <= 0) return 0;
  if (i >= A.n_all) return A.tile_pre[A.n_edge_tiles];
  const int64_t w = i >> 6;
  return A.tile_pre[i / kEdgeTile] + A.keep_pre[w] +
         __popcll(A.keep_bits[w] & ((uint64_t(1) << (i & 63)) - 1));
}

// Bit position of the k-th (from 0) set bit of m, which has more than k.
__device__ __forceinline__ int select_bit(uint64_t m, int k) {
  int pos = 0;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const int c = __popcll((m >> pos) & ((uint64_t(1) << d) - 1));
    if (c <= k) {
      k -= c;
      pos += d;
    }
  }
  return pos;
}

// A block per tile with kept edges: thread x writes the tile's kept edges x,
// x + 256, ...
__global__ __launch_bounds__(256) void k_lw_keep_emit(LayerArgs A) {
  __shared__ TileSegs T;
  __shared__ __align__(16) TilePairs Q;
  __shared__ int32_t s_pre[kKeepWords];
  __shared__ uint64_t s_bits[kKeepWords];
  const int64_t tile = blockIdx.x;
  const int64_t first = A.tile_pre[tile];
  const int n = int(A.tile_pre[tile + 1] - first);
  if (n == 0) return;
  if (threadIdx.x < kKeepWords) {
    s_pre[threadIdx.x] = A.keep_pre[tile * kKeepWords + threadIdx.x];
    s_bits[threadIdx.x] = A.keep_bits[tile * kKeepWords + threadIdx.x];
  }
  PairRange R;
  tile_tables<1, true>(A, tile, T, Q, R);  // also the barrier
  int s = 0;
  for (int x = threadIdx.x; x < n; x += 256) {
    int w = 0;  // the last word with s_pre <= x
#pragma unroll
    for (int d = kKeepWords / 2; d >= 1; d >>= 1)
      if (s_pre[w + d] <= x) w += d;
    const int64_t j = tile * kEdgeTile + w * 64 + select_bit(s_bits[w], x - s_pre[w]);
    const int sg = seg_index(A, T, s, j);
    const PairAt at = pair_at(A, Q, R, j);
    const int64_t p = R.n > 0 ? R.p0 + Q.slot[at.start] : at.start;
    const int64_t slot = A.pa.plo[p] + (j - A.pa.off[p]);
    const SegView v = seg_view<1>(A, T, sg);
    A.out_eid[first + x] = slot;
    A.out_dst_local[first + x] =
        int32_t(A.pa.pair_of(p) - v.pair_base);
    A.out_src_local[first + x] = static_cast<const int32_t *>(v.per_seg)[v.indices[slot]];
  }
}

// ---- reduce-then-scan over tiles of kLwTile candidates -----------------------
// The candidates' importance, one segment per node type (tiles cand_tile[t] ..
// cand_tile[t+1]; the type's candidates are counted in small[kSlotNew + t] by
// the collect compaction).
struct ScanSeg {
  int seg;
  int64_t first_tile, n;
};

__device__ __forceinline__ ScanSeg seg_of(const LayerArgs &A, int64_t tile) {
  const int t = find_segment(A.cand_tile, A.n_types, tile);
  return ScanSeg{t, A.cand_tile[t], A.small[kSlotNew + t]};
}

__global__ __launch_bounds__(kLwThreads) void k_lw_scan_reduce(LayerArgs A) {
  __shared__ int64_t lds[8];
  const int64_t tile = blockIdx.x;
  const ScanSeg S = seg_of(A, tile);
  const int64_t i0 = (tile - S.first_tile) * kLwTile + threadIdx.x * kLwItems;
  int64_t v = 0;
#pragma unroll
  for (int k = 0; k < kLwItems; ++k)
    if (i0 + k < S.n) v += int64_t(A.wt[S.seg][A.cand[S.seg][i0 + k]]);
  int64_t total;
  block_excl_scan_256(v, lds, &total);
  if (threadIdx.x == 0) A.tile_sum[tile] = total;
}

// One block: tile_pre = exclusive scan of tile_sum over all n_tiles tiles,
// tile_pre[n_tiles] = the grand total.  Each thread takes kLwScanPer
// consecutive tiles of a chunk.
constexpr int kLwScanThreads = 1024;
constexpr int kLwScanPer = 8;
__global__ __launch_bounds__(kLwScanThreads) void k_lw_scan_tiles(int64_t *tile_sum,
                                                                  int64_t *tile_pre,
                                                                  int64_t n_tiles) {
  constexpr int kWaves = kLwScanThreads / kWave;
  constexpr int64_t kChunk = int64_t(kLwScanThreads) * kLwScanPer;
  __shared__ int64_t s_wave[kWaves];
  const int wave = threadIdx.x / kWave;
  const int lane = lane_id();
  int64_t carry = 0;
  for (int64_t c0 = 0; c0 < n_tiles; c0 += kChunk) {
    const int64_t i0 = c0 + int64_t(threadIdx.x) * kLwScanPer;
    int64_t x[kLwScanPer];
    int64_t mine = 0;
#pragma unroll
    for (int k = 0; k < kLwScanPer; ++k) {
      x[k] = i0 + k < n_tiles ? tile_sum[i0 + k] : 0;
      mine += x[k];
    }
    const int64_t inc = wave_incl_scan_i64(mine);
    if (lane == kWave - 1) s_wave[wave] = inc;
    __syncthreads();
    int64_t before = 0, sum = 0;
    for (int w = 0; w < kWaves; ++w) {
      const int64_t y = s_wave[w];
      if (w < wave) before += y;
      sum += y;
    }
    int64_t run = carry + before + inc - mine;
#pragma unroll
    for (int k = 0; k < kLwScanPer; ++k) {
      if (i0 + k < n_tiles) tile_pre[i0 + k] = run;
      run += x[k];
    }
    carry += sum;
    __syncthreads();
  }
  if (threadIdx.x == 0) tile_pre[n_tiles] = carry;
}

// Each candidate gets the exclusive prefix of its importance within its type.
__global__ __launch_bounds__(kLwThreads) void k_lw_scan_apply(LayerArgs A) {
  __shared__ int64_t lds[8];
  const int64_t tile = blockIdx.x;
  const ScanSeg S = seg_of(A, tile);
  const int64_t i0 = (tile - S.first_tile) * kLwTile + threadIdx.x * kLwItems;
  int64_t c[kLwItems], v[kLwItems];
  int64_t sum = 0;
#pragma unroll
  for (int k = 0; k < kLwItems; ++k) {
    c[k] = i0 + k < S.n ? A.cand[S.seg][i0 + k] : -1;
    v[k] = c[k] >= 0 ? int64_t(A.wt[S.seg][c[k]]) : 0;
    sum += v[k];
  }
  int64_t total;
  int64_t pre = block_excl_scan_256(sum, lds, &total) +
                (A.tile_pre[tile] - A.tile_pre[S.first_tile]);
#pragma unroll
  for (int k = 0; k < kLwItems; ++k) {
    if (c[k] >= 0) {
      A.prefix[S.seg][i0 + k] = uint64_t(pre);
      A.wt[S.seg][c[k]] = 0;  // clean for the next hop and call
    }
    pre += v[k];
  }
}

// Draws: thread x of type t's range draw_base[t] .. draw_base[t+1] makes draw
// x - draw_base[t] (or, for a type that takes every candidate, marks
// candidate x - draw_base[t]).
__global__ __launch_bounds__(256) void k_lw_draw(LayerArgs A) {
  const int64_t n = A.draw_base[A.n_types];
  for (int64_t x = gs_start(); x < n; x += gs_step()) {
    const int t = find_segment(A.draw_base, A.n_types, x);
    const int64_t k = x - A.draw_base[t];
    const int copy = t / A.key_T;
    const uint64_t sigma = A.sigmas[copy];
    const int64_t nc = A.small[kSlotNew + t];
    const int64_t *cand = A.cand[t];
    uint8_t *reached = A.ts[t].reached;
    if (A.draws[t] < 0) {
      if (k < nc) reached[cand[k]] = 1;
      continue;
    }
    const uint64_t total = uint64_t(A.tile_pre[A.cand_tile[t + 1]] - A.tile_pre[A.cand_tile[t]]);
    if (total == 0 || nc == 0) continue;
    const U32x4 r4 = philox4x32_10(U32x4{uint32_t(k), uint32_t(uint64_t(k) >> 32),
                                         0x40000000u | uint32_t(A.hop),
                                         uint32_t(t - copy * A.key_T)},
                                   uint32_t(sigma), uint32_t(sigma >> 32));
    const uint64_t r = __umul64hi(uint64_t(r4.x) | (uint64_t(r4.y) << 32), total);
    // the last candidate whose prefix is not above r (zero-weight candidates
    // share the prefix of the next one and are never the last)
    const uint64_t *pre = A.prefix[t];
    int64_t a = 0, b = nc - 1;
    while (a < b) {
      const int64_t m = a + (b - a + 1) / 2;
      if (pre[m] <= r)
        a = m;
      else
        b = m - 1;
    }
    reached[cand[a]] = 1;
  }
}

// Per pair its block-CSC entry from the kept positions; the closing entry and
// the kept edge start of every etype; block 0 plans the next hop.
__global__ __launch_bounds__(256) void k_lw_indptr(LayerArgs A) {
  const int64_t *ebase = ebase_of(A);
  const int64_t *pb = A.hv.pair_base;
  auto pos = [&](int64_t i) { return kept_before(A, i); };
  if (blockIdx.x == 0) {
    int64_t *kept = kept_base_of(A);
    for (int e = threadIdx.x; e <= A.n_etypes; e += blockDim.x) {
      kept[e] = pos(ebase[e]);
      if (e < A.n_etypes) A.out_indptr[pb[e + 1] + e] = pos(ebase[e + 1]) - pos(ebase[e]);
    }
    plan_next_hop(A.hv, A.next, A.es, A.tile_base, A.small, A.n_types, A.n_etypes);
  }
  if (A.n_words == 0) {
    for (int64_t p = gs_start(); p < A.n_pairs; p += gs_step()) {
      const int e = A.pa.pet[p];
      A.out_indptr[pb[e] + e + (p - pb[e])] = pos(A.pa.off[p]) - pos(ebase[e]);
    }
    return;
  }
  // active pairs: lane i of a wavefront takes pair i of a word, whose entry is
  // that of the first active pair not before it
  for (int64_t y = gs_start(); y < A.n_words * kWave; y += gs_step()) {
    const int64_t x = y / kWave;
    const int e = A.pa.word_et[x];
    const int64_t i = ((x - pair_word(pb[e], e, 0)) << 6) + lane_id();
    const int64_t a = A.pa.act_pre[x] + __popcll(A.pa.bits[x] & lanes_below());
    if (i < pb[e + 1] - pb[e]) A.out_indptr[pb[e] + e + i] = pos(A.pa.off[a]) - pos(ebase[e]);
  }
}

}  // namespace

hipError_t launch_lw_weights(const LayerArgs &A, hipStream_t stream) {
  if (A.n_all <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_lw_tile_pairs, dim3(grid_for(A.n_pairs, 256)), dim3(256), 0, stream, A);
  hipLaunchKernelGGL(k_lw_weights, dim3(unsigned(A.n_edge_tiles)), dim3(256), 0,
                     stream, A);
  return hipGetLastError();
}

hipError_t launch_lw_bins(const LayerArgs &A, hipStream_t stream) {
  const size_t lds = sizeof(uint32_t) * size_t(A.n_bins);
  const unsigned grid = unsigned((A.n_edge_tiles + kBinTiles - 1) / kBinTiles);
  hipLaunchKernelGGL(k_lw_tile_pairs, dim3(grid_for(A.n_pairs, 256)), dim3(256), 0, stream, A);
  hipLaunchKernelGGL(k_lw_bin_count, dim3(grid), dim3(256), lds, stream, A);
  hipLaunchKernelGGL(k_lw_bin_starts, dim3(1), dim3(1024), 0, stream, A);
  hipLaunchKernelGGL(k_lw_bin_scatter, dim3(grid), dim3(256), lds, stream, A);
  hipLaunchKernelGGL(k_lw_bin_parts, dim3(unsigned(most_bin_parts(A.n_all))), dim3(kBinThreads), 0,
                     stream, A);
  hipLaunchKernelGGL(k_lw_bin_sum, dim3(unsigned(A.n_bins)), dim3(kBinThreads), 0, stream, A);
  hipLaunchKernelGGL(k_lw_bin_totals, dim3(1), dim3(1024), 0, stream, A);
  return hipGetLastError();
}

hipError_t launch_lw_prefix(const LayerArgs &A, hipStream_t stream) {
  const int64_t tiles = A.cand_tiles;
  if (tiles <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_lw_scan_reduce, dim3(unsigned(tiles)), dim3(kLwThreads), 0, stream, A);
  hipLaunchKernelGGL(k_lw_scan_tiles, dim3(1), dim3(kLwScanThreads), 0, stream, A.tile_sum,
                     A.tile_pre, tiles);
  hipLaunchKernelGGL(k_lw_scan_apply, dim3(unsigned(tiles)), dim3(kLwThreads), 0, stream, A);
  return hipGetLastError();
}

hipError_t launch_lw_draw(const LayerArgs &A, hipStream_t stream) {
  const int64_t n = A.draw_threads;
  if (n <= 0) return hipSuccess;
  if (A.n_bins > 0) {
    hipLaunchKernelGGL(k_lw_bin_draw, dim3(grid_for(n, 256)), dim3(256), 0, stream, A);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_lw_draw, dim3(grid_for(n, 256)), dim3(256), 0, stream, A);
  return hipGetLastError();
}

hipError_t launch_lw_keep(const LayerArgs &A, hipStream_t stream) {
  if (A.n_all > 0) {
    const unsigned grid = unsigned(A.n_edge_tiles);
    hipLaunchKernelGGL(k_lw_keep_flags, dim3(grid), dim3(256), 0, stream, A);
    hipLaunchKernelGGL(k_lw_scan_tiles, dim3(1), dim3(kLwScanThreads), 0, stream, A.tile_sum,
                       A.tile_pre, A.n_edge_tiles);
    hipLaunchKernelGGL(k_lw_keep_emit, dim3(grid), dim3(256), 0, stream, A);
  }
  // at least one block: block 0 writes the etype entries and plans the next hop
  hipLaunchKernelGGL(k_lw_indptr, dim3(grid_for(std::max(A.n_pairs, A.n_words * kWave), 256)), dim3(256),
                     0, stream, A);
  return hipGetLastError();
}

}  // namespace hg
