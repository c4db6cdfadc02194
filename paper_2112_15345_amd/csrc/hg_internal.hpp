// Internal interface between the host runtime (hg_runtime.cpp) and the gfx950
// kernels (hg_sample.hip, hg_compact.hip, hg_gather.hip).  Not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>

#include "hg.h"

#include <cstddef>
#include <cstdint>

namespace hg {

// Bitmap tiles: 256 threads x 2 words.
constexpr int kTileThreads = 256;
constexpr int kTileItems = 2;
constexpr int64_t kTile = int64_t(kTileThreads) * kTileItems;  // 512 words

// Pair tiles of the counting pass: 256 threads x 2 pairs.
// Pairs per thread of the counting pass: few for small hops (more blocks in
// flight), more for large ones (fewer tiles, whose tickets serialize).
constexpr int kPairItemsSmall = 2;
constexpr int kPairItemsLarge = 8;
constexpr int64_t kPairLargeFrom = int64_t(kTileThreads) * kPairItemsSmall * 512;
// Items per thread of a counting pass over active pairs, whose number the host
// only bounds, so that one size has to do.  Single calls with 2, 4 and 8 of them:
// 2^24 pairs, 25% active 1059, 859 and 769 us, 3% active 279, 262 and 249; 2^20
// pairs, 3% 144, 146 and 142 (runs differ by 4%).
constexpr int kPairItemsActive = 8;

// Candidate capacity of one bottom-K selection (LDS entries per wavefront,
// and per hub in the global candidate lists).
constexpr int kCandCap = 512;

// Node types whose per-hop table entries travel inside a launch's arguments.
constexpr int kInlineTypes = 8;
// Node types whose source-list pointers the sampler launch stores into the
// hop's table itself (a bundle of 32 mini-batches of 4 node types is 128).
constexpr int kInlineSrcOut = 128;

// Pairs whose in-edges are all kept and number at most this many are copied
// 64 pairs per wavefront; larger ones by a wavefront each.
constexpr int64_t kThreadTakeAll = 32;

// Pairs that keep K < deg edges with deg > kHubChunk ("hubs") are sampled in
// chunks of kHubChunk edges, handed to wavefronts in runs of chunks.
constexpr int64_t kHubChunk = 2048;

// Pairs that keep K < deg edges with deg <= kLaneSelect (and nothing
// excluded) are sampled by one lane each, among the pairs of the take-all
// groups: all their keys fit in registers.
constexpr int64_t kLaneSelect = 16;

// Readback slots of the small device buffer (int64 each).
constexpr int kSlotErr = 0;     // error bits in the low int32
constexpr int kSlotTicket = 1;  // tile tickets of the single-pass scans
constexpr int kSlotKeys = 2;    // random keys the sampler evaluates, summed over the hops so far
constexpr int kSlotPairs = 3;   // pairs of the hop
constexpr int kSlotEdges = 4;   // kept edges of the hop
constexpr int kSlotHubs = 5;    // hub pairs
constexpr int kSlotChunks = 6;  // hub chunks
constexpr int kSlotWaves = 7;   // pairs sampled by one wavefront each
constexpr int kSlotActive = 8;  // pairs that may have in-edges (hops with pair bits)
constexpr int kSlotActTicket = 9;  // tile tickets of their counting pass
constexpr int kSlotNew = 10;    // n_new[T], then ebase[R+1], then kept ebase[R+1]

constexpr int32_t kErrSeedRange = 1;   // a frontier vertex out of range
constexpr int32_t kErrSeedRepeat = 2;  // a vertex twice in a frontier
constexpr int32_t kErrLookback = 4;    // a scan wait exceeded its bound
constexpr int32_t kErrBound = 8;       // more pairs or chunks than buffers were sized for
constexpr int32_t kErrTarget = 16;     // a target edge out of range, or a bad reverse edge

// The dense vertex -> local-ID map of a workspace holds one int32 per vertex.
// An entry is meaningful only while the vertex's frontier bit is set (see
// TypeStatic); the frontier bitmap is cleared after every call, so stale
// entries are never read and the map itself is never cleared.

// Static per edge type (per workspace).
struct EtypeStatic {
  const int64_t *indptr;
  const int64_t *indices;
  int32_t *src_map;       // vertex -> local-ID map of the source type
  uint8_t *src_reached;   // reached flags of the source type
  uint32_t *src_rbits;    // reached bits of the source type (hops in bit mode)
  int64_t n_dst_nodes;
  int32_t src_type;
  int32_t dst_type;
};

// Node types with at least this many incoming edge types get a non-empty mask:
// per vertex a row of `words` 32-bit words whose bit s says whether the type's
// s-th incoming edge type has an in-edge there.
constexpr int32_t kNzMaskMinEtypes = 16;
// A node type with edges into it (per workspace, a bundle's copies each; only
// for graphs with a mask): its incoming edge types, in the order of the mask's
// bits, are nz_et[first] .. nz_et[first + n_in - 1].  mask: NULL for a type
// without one, whose pairs all count as non-empty.
struct NzType {
  const uint32_t *mask;
  int64_t num_nodes;
  int32_t type, words, n_in, first;
};
// Large hops of a graph with such a type work on the active pairs, those whose bit is
// set (every pair of the other types): of the pairs of a 200-relation graph 3%
// are.  The bit of pair (etype e, destination local ID i) is bit i & 63 of word
// pair_word(pair_base[e], e, i): the words of an etype are followed by at most
// one zero word before the next etype's, so the words in order hold the pairs
// in order, and there are pair_words(P, R) of them.
__host__ __device__ inline int64_t pair_word(int64_t pair_base, int e, int64_t i) {
  return (pair_base >> 6) + e + (i >> 6);
}
__host__ __device__ inline int64_t pair_words(int64_t n_pairs, int32_t n_etypes) {
  return (n_pairs >> 6) + n_etypes;
}
// Whether a hop of n_pairs pairs, n_active of them active, works on the active ones.
// Listing them is two launches and a walk over the mask's words (15 us with 64 edge
// types into the type, 25 with 200), and an active pair then costs about 190 ps,
// where going through every pair costs 50 ps a pair and 60 more an active one: the
// list pays from about kActiveFromPairs + 9/4 n_active pairs (and never past 4/9 of
// them active).  Single calls of one hop, us by the list and by every pair (64 edge
// types, fanout 5): 3% active, 2^18, 2^19 and 2^20 pairs 104 / 98, 110 / 116, 114 /
// 147; 20%, 2^19 and 2^20: 127 / 124, 145 / 161; 30%, 2^20 and 2^21: 166 / 165, 225 /
// 254; 50%, 2^18, 2^20 and 2^22: 151 / 109, 209 / 178, 493 / 436.  200 edge types, 3%,
// 2^19 and 2^20: 135 / 130, 135 / 163.
constexpr int64_t kActiveFromPairs = int64_t(320) << 10;
constexpr int64_t kActivePerWord = int64_t(1) << 15;  // per 32 edge types into the type
inline bool active_pairs_pay(int64_t n_pairs, int64_t n_active, int32_t mask_words) {
  return n_pairs > kActiveFromPairs + kActivePerWord * mask_words + n_active / 4 * 9;
}
constexpr int kPairListItems = 4;  // words per thread of the pass that lists the active pairs
// The blocks of the pass that makes their bits: x over the largest frontier, y over the
// node types of all copies; at most 2^16 in all (each strides over what is left), as a
// bundle of a graph of 2048 types has more of them than a grid's y takes, and most of
// those have few vertices or none in the frontier.
struct PairBitsGrid {
  unsigned x, y;
};
inline PairBitsGrid pair_bits_grid(int64_t max_front, int32_t n_nz) {
  constexpr int64_t kPerBlock = 256;  // frontier vertices, a wavefront for each 64
  const int64_t y = n_nz < 1024 ? (n_nz < 1 ? 1 : n_nz) : 1024;
  int64_t x = (max_front + 64 + kPerBlock - 1) / kPerBlock;
  x = x < 4096 ? x : 4096;
  x = x < (int64_t(1) << 16) / y ? x : (int64_t(1) << 16) / y;
  return PairBitsGrid{unsigned(x), unsigned(y)};
}

// Static per node type (per workspace).
// Per node type one flag byte and one frontier bit per vertex: the sampler
// stores 1 into the `reached` byte of every kept edge's source (a plain store,
// so that popular sources cost no atomics), and `fbits` holds the frontier.  A
// hop's new vertices are the reached vertices whose frontier bit is clear; the
// compaction adds them to fbits and clears the reached bytes.  Both are zero
// between calls.  The layouts follow the bitmap tiles: type t starts at tile
// tile_base[t], a tile covering kTile * 32 vertices.
struct TypeStatic {
  int32_t *map;
  uint8_t *reached;
  uint32_t *fbits;
  int64_t num_nodes;
  uint32_t *rbits;  // reached bits (hops in bit mode), laid out as fbits
};

// A hop marks its kept sources either with the byte flags above (plain
// stores: no atomics on popular sources) or, when the call's vertices far
// outnumber the hop's kept edges, with one reached bit per vertex (atomicOr
// without return), so that the compaction reads an eighth of the bytes.
// Bit mode is chosen when vertices > kBitModeRatio x kept edges.
constexpr int64_t kBitModeRatio = 16;
// The chip's XCDs, each with its own L2; workgroups are handed to them in turn.
// A call of at least kXcds mini-batches orders its sampler, hub selection and relabel blocks
// per XCD, so that each XCD runs whole mini-batches.
constexpr int kXcds = 8;

// One hop, as device arrays.  Host-written: frontier, src_out, fanout.
// nF and pair_base are written by the host for hop 0 and by the previous
// hop's relabel pass afterwards.
struct HopView {
  int64_t *nF;                  // [T] frontier sizes
  int64_t *pair_base;           // [R+1] pairs of etype e: [pair_base[e], pair_base[e+1])
  const int64_t *const *frontier;  // [T]
  int64_t *const *src_out;      // [T] source lists of this hop (frontier ++ new)
  const int32_t *fanout;        // [R]
};

// Words of a single-pass (decoupled look-back) scan of NV values: per tile
// NV 64-bit words, each epoch (20 bits) | state (2 bits) | value (42 bits);
// state 1 = aggregate, overwritten by state 2 = inclusive prefix.  Epochs run 1 .. 2^20-1;
// the words are zeroed before an epoch is reused.
struct Lookback {
  uint64_t *word;
};
constexpr uint32_t kEpochLimit = 1u << 20;

// Edges that no hop may sample (an edge-seeded mini-batch with exclusion), as
// two open-addressing hash tables with linear probing: the excluded edges,
// keyed (etype << 32 | eid), and per pair with excluded in-edges its count,
// keyed (etype << 32 | destination local ID).  Every excluded edge ends at a
// seed, and the seeds are the first local IDs of every hop's frontier, so
// only pairs whose destination local ID is below n_seed[etype] are looked up.
// edge_keys == nullptr: nothing is excluded.
constexpr uint64_t kHashEmpty = ~uint64_t(0);
struct ExclView {
  const uint64_t *edge_keys;  // [edge_mask + 1]
  const uint64_t *pair_keys;  // [pair_mask + 1]
  const int32_t *pair_cnt;    // [pair_mask + 1]
  const int64_t *n_seed;      // [R] seeds of each etype's destination type
  uint32_t edge_mask, pair_mask;
};

__host__ __device__ inline uint32_t hash_slot(uint64_t key, uint32_t mask) {
  return uint32_t((key * 0x9E3779B97F4A7C15ull) >> 32) & mask;
}

// Per-pair arrays of one hop (device), n_items entries each.  Items are the
// hop's pairs, or (act_pair not NULL) its active pairs in pair order.
struct PairArrays {
  int64_t *plo;      // first in-edge slot
  int64_t *pdeg;     // in-degree
  int64_t *off;      // exclusive scan of kept edges
  int32_t *pet;      // edge type of the item
  int64_t *wlist;    // the item of each wavefront pair, in pair order
  int32_t *hub_cnt;  // per hub: candidates appended
  int64_t *hub_pair; // per hub: its item
  int64_t *hub_choff; // per hub: its first chunk (strictly increasing)
  int64_t *act_pair; // per item: its pair
  uint64_t *bits;    // per word: its pairs' non-empty bits
  int64_t *act_pre;  // per word: active pairs before it
  int32_t *word_et;  // per word: its edge type
  __device__ int64_t pair_of(int64_t item) const { return act_pair ? act_pair[item] : item; }
};

// ---- runtime hooks (hg_runtime.cpp) for the pipeline ------------------------

// Sets this thread's hg_last_error text; returns st.
hg_status set_error(hg_status st, const char *msg);
// Later frees of the handle's arrays are ordered on the null stream (its own
// stream is going away; its work has completed).
void blocks_detach_stream(hg_blocks *b);
int graph_device(const hg_graph *g);

// ---- launchers (all asynchronous on `stream`) -------------------------------

// Device timestamps of one stage: `start` is carried by the stage's first
// kernel launch and `stop` by its last; a stage that launches nothing records
// both with hipEventRecord.  Null events: plain launches.
struct StageEv {
  hipEvent_t start = nullptr, stop = nullptr;
  bool any() const { return start || stop; }
};
// Records an empty stage's events (no kernel to carry them).
hipError_t record_empty_stage(const StageEv &ev, hipStream_t stream);

// The hop-0 frontier: the seed's frontier bit, map[seed] = position; flags
// range errors and repeats (a frontier bit already set).
hipError_t launch_insert_frontier(HopView hv, const TypeStatic *ts,
                                  int32_t n_types, int64_t total, int64_t *small,
                                  hipStream_t stream);

// The active pairs of a hop of a graph with masked types (nz, n_nz of them, every
// node type with edges into it among them): the words of their bits, then the
// list of the active pairs and their edge types in pair order.  max_front: at
// least the largest frontier; n_items: at least P + 1.
int64_t pair_list_tiles(int64_t n_items, int32_t n_etypes);
hipError_t launch_pair_list(HopView hv, const NzType *nz, const int32_t *nz_et, int32_t n_nz,
                            int32_t n_etypes, int64_t max_front, int64_t n_items, PairArrays pa,
                            Lookback lb, uint32_t epoch, uint64_t ticket_base, int64_t *small,
                            hipStream_t stream, StageEv ev);

// A counting pass of one tile that publishes (host not NULL): its block ends with
// what launch_publish does, copying the n readback slots to pinned host memory and
// then writing seq to host[n].  A pass of several tiles leaves that to
// launch_publish: its blocks would have to make their writes visible to the last
// of them, and that (an L2 write-back each) cost more than the launch, at 9 tiles
// (14.6 us against 11.1 + 4) as at 391 (63 against 25 + 4).
struct Publish {
  int64_t *host = nullptr;
  int32_t n = 0;
  uint64_t seq = 0;
};

// Counting pass over n_items >= P + 1 pair slots (P = pair_base[R]): per pair
// its in-edge range; exclusive scans of kept edges, hub chunks, wavefront
// pairs and hub flags; per-etype edge starts (ebase) and the hop totals into
// `small`.  Single pass, tiles taken by ticket.
int64_t count_tiles(int64_t n_items, bool active);
hipError_t launch_count_scan(HopView hv, const EtypeStatic *es, int32_t n_etypes,
                             int32_t n_types, int64_t n_items, PairArrays pa,
                             Lookback lb, uint32_t epoch, uint64_t ticket_base,
                             ExclView X, Publish pub, int64_t *small, hipStream_t stream,
                             StageEv ev = {});

// The sampler, two launches.  First: block CSC entries and small take-all
// pairs (a wavefront per 64 pairs), wavefront pairs (one wavefront each) and
// hub chunks (one wavefront each, appending candidates to the hub's list).
// Then one wavefront per hub selects from its list.  Writes each pair's kept
// edges at off[p], grouped by pair, ascending edge ID: source vertex, edge
// ID, destination local ID.
// The sampler launches.  With n_src_out <= kInlineSrcOut the first one also
// stores src_out[0..n_src_out) into src_out_slot (the hop's table entries).
// Edge type e is keyed as type e % key_R with seed sigmas[e / key_R] (device).
hipError_t launch_sample(HopView hv, const EtypeStatic *es, int32_t n_etypes,
                         int32_t n_types, int64_t n_items, int64_t n_words, int64_t n_wave,
                         int64_t n_chunks, int64_t n_hubs, PairArrays pa,
                         uint64_t *cand, const int64_t *small, const uint64_t *sigmas,
                         int32_t key_R, int32_t hop, int32_t key_bits, int64_t *src_gid,
                         int64_t *eid, int32_t *dst_local, int64_t *indptr_all,
                         int64_t **src_out_slot, int64_t *const *src_out, int32_t n_src_out,
                         ExclView X, hipStream_t stream, StageEv ev_sample = {},
                         StageEv ev_select = {}, bool bit_mode = false, bool xcd_order = false);


// Compaction pass: per bitmap tile, ranks of the set bits within the node
// type -> local IDs n_frontier + rank, written to the map and the source
// list, bits cleared; each type's new-vertex count goes to small[kSlotNew + t];
// extra blocks copy the frontier into the head of the source lists.  Up to
// kSinglePassTiles tiles: one launch, a single-pass scan whose look-back words
// are tile_sums (ticketed blocks: *ticketed is their number).  Beyond: three
// launches (reduce, scan, rank) with no inter-block waits; *ticketed = 0.
// tile_sums: device scratch of 2 * n_tiles + 2 64-bit words.  With `collect`
// the ranked vertices are only listed (in the source lists of hv, from local
// 0) and their reached flags cleared: the map and the frontier bits are left
// as they are.
constexpr int64_t kSinglePassTiles = 256;
hipError_t launch_compact(HopView hv, const TypeStatic *ts, int32_t n_types,
                          uint8_t *reached, uint32_t *fbits, const int64_t *tile_base,
                          int64_t n_tiles, int64_t copy_total, int64_t *tile_sums,
                          uint32_t epoch, uint64_t ticket_base, int64_t *small,
                          int64_t *ticketed, hipStream_t stream, bool collect = false,
                          StageEv ev = {}, uint32_t *rbits = nullptr);

// ---- layer-wise (LADIES) sampling (hg_layers.hip) ----------------------------

// One hop of a layer-wise call.  The sampler has emitted every in-edge of the
// frontier (all_src / all_eid / all_dst_local, grouped by pair at pa.off);
// per node type t (at most kInlineTypes), wt[t] holds the importance of every
// vertex (zero between uses), cand[t] and prefix[t] the candidates and the
// exclusive prefix of their importance, scan tiles cand_tile[t] ..
// cand_tile[t+1] of the candidate scan, and draws[t] the draws of the hop.
// Candidates per tile of the layer-wise scans (256 threads, two values each).
constexpr int64_t kLayerTile = 512;
// In-edges per tile of the layer-wise edge passes (256 threads, eight each).
constexpr int64_t kEdgeTile = 2048;
// Pairs of such a tile, empty ones included, that its block goes through to find
// each position's pair; of more, each position searches for its own (32 rounds of
// loads against 8 chains of 13).
constexpr int kTilePairs = 8192;

// The candidates' importance is summed in LDS, a bin of kBinVerts vertices (half a
// bitmap tile: bin b of all types has frontier words b * kBinVerts / 32 ...) to a
// block, when the call's vertices make at most kMaxBins bins (each block of the
// binning passes counts every bin in LDS); else by global atomics into an array of
// every vertex's importance.
constexpr int64_t kBinVerts = 8192;
constexpr int64_t kBinsPerTile = kTile * 32 / kBinVerts;
constexpr int64_t kMaxBins = 8192;
// Bins of more records than this are summed in parts of about as many, each by a
// block, through sums in memory; a call of n in-edges has fewer than n / kBinPart of
// them.
constexpr int64_t kBinPart = 32768;
__host__ __device__ inline int64_t bin_parts(int64_t records) {  // 0: not in parts
  return records > kBinPart ? (records + kBinPart - 1) / kBinPart : 0;
}
inline int64_t most_large_bins(int64_t n, int64_t n_bins) {
  return n / kBinPart + 1 < n_bins ? n / kBinPart + 1 : n_bins;
}
inline int64_t most_bin_parts(int64_t n) { return 2 * (n / kBinPart) + 1; }
// Hops of fewer in-edges use the atomics: a hop's binning is four launches more.
// Single calls of one hop, us by bins and by atomics, from a type of 100k, 2M and 20M
// vertices (12, 245 and 2442 bins): 2^19 in-edges 204 / 178, 190 / 196, 236 / 234;
// 2^20 215 / 206, 208 / 230, 251 / 288; 2^21 233 / 260, 240 / 288, 294 / 382.
constexpr int64_t kBinsFromEdges = int64_t(1) << 20;

struct LayerArgs {
  HopView hv, next;
  const EtypeStatic *es;
  const TypeStatic *ts;
  const int64_t *tile_base;  // bitmap tiles per type (plans the next hop)
  int32_t n_types, n_etypes;
  PairArrays pa;
  int64_t n_pairs, n_words;  // items, and words of active pairs' bits (0: items are pairs)
  // n_all in-edges of the frontier, numbered by the counting pass (pair p's
  // in-edges are positions off[p] .. off[p+1]-1, CSC slots plo[p] ..); they
  // are read from the CSC where they are needed, never written out
  int64_t n_all;
  int64_t n_edge_tiles;
  int64_t *tile_pair;  // [n_edge_tiles + 1]: the pair of position tile * kEdgeTile
  // per node type, in a device table of the hop (see LayerTable)
  uint64_t *const *wt;        // [T] importance of every vertex of the type
  int64_t *const *cand;       // [T] the type's candidates, ascending
  uint64_t *const *prefix;    // [T] their importance prefix
  const int64_t *cand_tile;   // [T+1] first scan tile of each type's candidates
  const int64_t *draw_base;   // [T+1] threads of the draw launch per type
  const int32_t *draws;       // [T] draws (-1: every candidate)
  int64_t cand_tiles, draw_threads;  // cand_tile[T], draw_base[T] (host copies)
  int64_t *tile_sum;   // per scan tile
  int64_t *tile_pre;   // per scan tile: exclusive scan over all tiles, then the grand total
  // binned importance (n_bins > 0): per bin its in-edges, their first record and
  // the room for its candidates (exclusive scans), its candidates and their
  // importance, and those of the bins before it
  int64_t n_bins;
  const uint32_t *fbits;   // frontier bits of all types
  uint32_t *bin_edges, *bin_at;
  int64_t *bin_rec, *bin_cap;  // [n_bins + 1]
  int64_t *bin_part, *bin_big;  // [n_bins + 1] parts of, and number of, the large bins before it
  unsigned long long *big_sums;  // [large bins * kBinVerts], zero between hops
  uint32_t *rec;           // [n_all] (edge_record)
  int32_t *bin_cand_off;   // per candidate: its vertex's place in the bin
  uint64_t *bin_cand_pre;  // per candidate: importance before it in the bin
  int64_t *bin_n, *bin_n_pre;  // [n_bins], [n_bins + 1]
  int64_t *bin_w, *bin_w_pre;  // [n_bins], [n_bins + 1]
  uint64_t *keep_bits;  // [n_edge_tiles * kEdgeTile / 64] kept flags
  int32_t *keep_pre;    // per word: kept edges before it within its tile
  int64_t *out_eid;
  int32_t *out_src_local, *out_dst_local;
  int64_t *out_indptr;  // [P + R]
  // node type t is keyed as type t % key_T with seed sigmas[t / key_T] (a
  // bundle's copy; a single batch: key_T = n_types)
  const uint64_t *sigmas;
  int32_t key_T;
  int32_t hop;
  int64_t *small;
};

// The per-type arrays of one layer-wise hop, as laid out in the call's
// tables (8-byte words): wt [T], cand [T], prefix [T], cand_tile [T+1],
// draw_base [T+1], draws [T] (int32, rounded up to words).
inline size_t layer_table_bytes(int32_t T) {
  return sizeof(int64_t) * (3 * size_t(T) + 2 * (size_t(T) + 1) + (size_t(T) + 1) / 2);
}

// The first pair of every kEdgeTile-position tile of the in-edges (tile_pair),
// then the importance of every candidate: for each in-edge u -> v of the
// frontier whose source is not in the frontier, u is marked reached and
// wt[type(u)][u] += floor(2^32 / deg(v)^2).
hipError_t launch_lw_weights(const LayerArgs &A, hipStream_t stream);
// The same by bins: records of the in-edges grouped by bin, then each bin's
// candidates with their importance prefix, and the scans over the bins.  Touches
// neither the reached flags nor an importance array.
hipError_t launch_lw_bins(const LayerArgs &A, hipStream_t stream);
// Exclusive prefix of the candidates' importance per node type (three
// launches: tile sums, one scan of the tile sums, apply); zeroes the
// candidates' importance entries.
hipError_t launch_lw_prefix(const LayerArgs &A, hipStream_t stream);
// The draws of every node type (among the bins' candidates with n_bins > 0):
// marks the drawn candidates reached.
hipError_t launch_lw_draw(const LayerArgs &A, hipStream_t stream);
// The kept in-edges (source in the next frontier): their flags, a scan of the
// tiles' counts, the kept ones emitted in order; then the block CSC, the kept edge starts per etype
// (small slots after ebase) and the next hop's plan.
hipError_t launch_lw_keep(const LayerArgs &A, hipStream_t stream);

// src_local[j] = map_{src_type(e)}[src_gid[j]] for the edges of etype e,
// which are [ebase[e], ebase[e+1]), ebase = small + kSlotNew + n_types.
// Block 0 also writes the next hop's frontier sizes (this hop's plus its new
// vertices) and pair layout into `next`.  With clear_words, further blocks zero
// that many words at `clear` (16-byte aligned, a multiple of four).
hipError_t launch_relabel(HopView hv, HopView next, const EtypeStatic *es,
                          const int64_t *tile_base, const int64_t *small,
                          int32_t n_types, int32_t n_etypes, int64_t n_edges,
                          const int64_t *src_gid, int32_t *src_local,
                          hipStream_t stream, StageEv ev = {}, bool xcd_order = false,
                          uint32_t *clear = nullptr, int64_t clear_words = 0);

// Fill helpers (kernels, so that they are safe under graph capture).
// One block copies small[0..n) to pinned host memory host[0..n) and then
// writes `seq` to host[n] (system scope, after the slots).  With `clear` it
// then zeroes small[0..n), ready for the next call.
hipError_t launch_publish(int64_t *small, int64_t *host, int32_t n, uint64_t seq, bool clear,
                          hipStream_t stream);
// dst[i] = vals[i] for i < n (device pointer table), stream-ordered, with the
// values passed in the launches.
hipError_t launch_store_ptrs(void **dst, void *const *vals, int32_t n, hipStream_t stream);
hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t stream);
hipError_t launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t stream);
// dst[0..n) = src[0..n) by a kernel that reads src, pinned host memory, over
// the host link (no DMA copy on the stream); dst and src 8-byte aligned, else
// hipErrorInvalidValue.  The host must not rewrite src until the kernel ran.
hipError_t launch_upload(void *dst, const void *src, int64_t n, hipStream_t stream);

// launch_upload of n bytes and then launch_insert_frontier over hv, whose tables
// are among them: one launch of one block for small calls (at most kStartBytes and
// kStartSeeds: with 4096 seeds the block takes 24 us, and the two launches 7), else
// both.
constexpr int64_t kStartBytes = 16384;
constexpr int64_t kStartSeeds = 1024;
hipError_t launch_start(void *dst, const void *src, int64_t n, HopView hv, const TypeStatic *ts,
                        int32_t n_types, int64_t total, int64_t *small, hipStream_t stream);

// The non-empty mask of one destination type: for v < n, bit k of row v
// (words per row) is set when indptrs[k][v + 1] > indptrs[k][v]; indptrs is a
// device array of n_etypes pointers.
// *n_set (device) gets the number of set bits added.
hipError_t launch_nonempty_mask(const int64_t *const *indptrs, int32_t n_etypes, int32_t words,
                                int64_t n, uint32_t *mask, unsigned long long *n_set,
                                hipStream_t stream);

// Graph check of one edge type: indptr[0] == 0, non-decreasing,
// indptr[n_dst] == nnz, indices in [0, n_src).  Sets *err on a violation.
hipError_t launch_check_etype(const int64_t *indptr, int64_t n_dst,
                              const int64_t *indices, int64_t nnz,
                              int64_t n_src, int32_t *err, hipStream_t stream);

// Row gather: out[i] = table[ids[i]] (row_bytes bytes); a zero row when the
// ID is out of range, which also adds 1 to *bad (when bad is not NULL).  Picks the widest vector width that divides row_bytes and the
// alignment of both pointers.
// With n_dev, the rows are min(*n_dev, n) (read on the device; n bounds them
// and sizes the grid).
hipError_t launch_gather(const void *table, int64_t n_rows, int64_t row_bytes,
                         const int64_t *ids, int64_t n, void *out,
                         hipStream_t stream, const int64_t *n_dev = nullptr,
                         unsigned long long *bad = nullptr);

// The allocation-free row pull keeps its counters in a static device array
// of this many bytes per GPU.  noalloc_scratch_init (with `device` current)
// looks up that GPU's address of the array once; noalloc_scratch returns it
// (NULL before the lookup).
constexpr size_t kNoAllocScratchBytes = HG_NOALLOC_SCRATCH_BYTES;
hipError_t noalloc_scratch_init(int device);
unsigned long long *noalloc_scratch(int device);

// One row gather of launch_gather_multi.
struct GatherJob {
  const void *table;
  int64_t n_rows;
  int64_t row_bytes;
  const int64_t *ids;
  int64_t n;             // rows (or, with n_dev, their bound)
  void *out;
  const int64_t *n_dev;  // device row count, or nullptr
};
// Several row gathers, as few launches as possible.  `start` / `stop` (may be
// NULL) are recorded by the batched launches themselves.
hipError_t launch_gather_multi(const GatherJob *jobs, int32_t n_jobs, hipStream_t stream,
                               hipEvent_t start, hipEvent_t stop);

// ---- edge-seeded mini-batches (hg_edges.hip) --------------------------------

// Per edge type of an edge-seeded call (device table).
struct EdgeEtype {
  const int64_t *eids;     // target edge IDs
  const int64_t *rev_eid;  // reverse edge ID of every edge (exclusion 2), or NULL
  int64_t nnz;
  int32_t rev;             // reverse edge type, or -1
};

struct EdgeBatchArgs {
  const EtypeStatic *es;
  const TypeStatic *ts;
  const EdgeEtype *et;     // [n_etypes]
  const int64_t *tbase;    // [n_etypes + 1] prefix of target counts
  int32_t n_etypes, n_types;
  int64_t n_targets;
  int32_t n_neg, exclude;
  // edge type e belongs to copy e / key_R of a bundle (a single batch: key_R
  // = n_etypes), keyed as type e % key_R with seed sigmas[e / key_R] (device)
  const uint64_t *sigmas;
  int32_t key_R;
  int64_t *tsrc, *tdst;    // [n_targets] endpoints (-1 for an invalid target)
  int64_t *tneg;           // [n_targets * n_neg]
  int64_t *trev;           // [n_targets] reverse edge ID (exclusion 2), -1 when none
  int32_t *pos_src, *pos_dst, *neg_dst;  // pair graphs, target order
  uint64_t *edge_keys, *pair_keys;
  int32_t *pair_cnt;
  int64_t *n_seed;         // [n_etypes]
  uint32_t edge_mask, pair_mask;
  int64_t *small;
};

// Endpoints and negatives of every target; sets their bitmap bits (the seeds,
// ranked by the compaction pass); flags bad targets and reverse edges.
hipError_t launch_edge_targets(const EdgeBatchArgs &A, hipStream_t stream);
// After the compaction of the seeds: the pair graphs' local IDs, the
// exclusion tables, and hop 0's frontier sizes and pair layout (`first`).
hipError_t launch_edge_relabel(const EdgeBatchArgs &A, HopView first,
                               const int64_t *tile_base, hipStream_t stream);

// Philox4x32-10 on n counters.
hipError_t launch_philox(const uint32_t *ctr, uint64_t key, int64_t n,
                         uint32_t *out, hipStream_t stream);

// The sampler's key loop alone over key groups 0 .. n_groups-1 (a multiple of
// 64) of (key, hop, etype): adds the number of keys <= lim to *count (device
// uint64).  start / stop (may be NULL) are carried by the launch.
hipError_t launch_philox_rate(uint64_t key, int32_t hop, int32_t etype, int64_t n_groups,
                              uint32_t lim, uint64_t *count, hipEvent_t start,
                              hipEvent_t stop, hipStream_t stream);

}  // namespace hg
