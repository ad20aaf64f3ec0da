// Per-level kernels of the breadth-first composition: shared arguments and
// launchers (expand.hip: join count, match emission, arc-pair write;
// merge.hip: segmented sort + reduce, visited-table insert, id assignment,
// result append).
#pragma once

#include "internal.hpp"

namespace fstc {

// Read-only view of a Csr on the device.
struct CsrView {
  const u32 *row, *seg_sym, *seg_off;
  const uint2 *arcs;
  const u32 *part_base;
  const uint2 *parts;
  u64 num_arcs;
  const u32 *cell_flag;  // [num_states] build_cell_flags; kCellBad: no product merge
};

inline CsrView view(const Csr &c) {
  return CsrView{c.row, c.seg_sym, c.seg_off, c.arcs, c.part_base, c.parts, c.num_arcs,
                 c.cell_flag};
}

// Host-visible per-level counters (one D2H copy per synchronisation).
struct Status {
  u64 R;        // unmerged composed arcs of the level
  u64 M;        // matched (source, inner symbol) segment pairs of the level
  u64 merged;   // merged arcs of the level
  u64 RB;       // records of the nbig sources merged by the multi-block path
  u32 nwide, nheavy, nbig, nnew;
  u32 err;      // kErr* bits, sticky for the whole call
  u32 max_small;  // largest record count of a source merged by the tiles
  u64 dense_records;  // records of the tiles merged through a dense table
  u64 dense_runs;     // merged arcs those tiles produced
  u64 sort_runs;      // merged arcs of the tiles merged by sorting
  u32 nsort;          // tiles k_merge_dense left to the sort kernel
  u32 scan_ctr;       // tile counter of the single-pass scans (0 between scans)
  u32 seq;            // host copy only: number of the last publication, written last
  u32 unfit;          // sources of the level of a shape the one-workgroup
                      // small-level kernel declines (kSmallShape)
  u32 nprod;          // sources of the product merge       } one u64, the total of
  u32 nprod_mfma;     // of those, summed on the matrix cores } the level's flag words
  u64 prod_records;   // their joined arc pairs (not written as records)
  u64 prod_entries;   // their (p1, p2) table entries: temp slots after the records
  u32 ngen;           // product-merge sources listed for the one-per-wave kernel
  u32 ngrp;           // sources listed for the 16-lane joins
  u32 declined;       // nonzero: the one-workgroup product level did not take the level
  u32 new_count;      // new pairs of the last merged level (kept when the counters clear)
  u64 general;        // nonzero: the level has sources the chunk merge left to the
                      // other kernels (product, long or large joins)
  u64 chunk_pairs;    // joined arc pairs of the sources it merged
  u32 nmid, pad;      // sources merged by a workgroup each
};
static_assert(offsetof(Status, nprod) % 8 == 0 &&
                  offsetof(Status, nprod_mfma) == offsetof(Status, nprod) + 4,
              "the flag total is stored as one u64 over nprod, nprod_mfma");

// Product merge (merge.hip, k_prod_sources).  A source (q1, q2) is merged
// by one wavefront from its staged arc matrices instead of through records
// when its states have P1 + P2 <= kProdRowSum parts in all, the shorter of
// its two inner-symbol lists has kProdMinSymbols to 64 symbols, and neither
// state has two arcs in one (part, inner symbol) cell.  The count kernel
// selects it from the list lengths and part counts alone; the product
// kernel counts its joined pairs.
constexpr u32 kProdRowSum = 16;
static_assert(kProdParts == kProdRowSum - 1, "a state of more parts is never selected");
constexpr u32 kProdMinSymbols = 8;
// Sources whose states have at most kProdMfmaParts parts each and whose
// weight products are normal float32 numbers (expand.hip, products_normal)
// are summed on the matrix cores (merge.hip).
constexpr u32 kProdMfmaParts = 4;

// Joins: a source whose serial join takes at most kThreadSteps binary-search
// steps (shorter length x bits of the longer length) is joined by one
// thread; one whose shorter list has at most kGroupMax symbols and whose
// longer one at most kGroupLong, by a group of kGroupLanes lanes; one whose
// shorter list is longer than kHeavyMin, by several workgroups; the others by
// a workgroup or, when they are many, a wavefront.
constexpr u32 kThreadSteps = 12;
constexpr u32 kGroupLanes = 16;
constexpr u32 kGroupMax = 32;
constexpr u32 kGroupLong = 512;
constexpr u32 kHeavyMin = 2048;
// The first kHeavySplit heavy sources of a level are joined by up to
// kHeavyChunks workgroups each (expand.hip, heavy_chunk).
constexpr u32 kHeavySplit = 256;
constexpr u32 kHeavyChunks = 64;
struct HeavyChunk {
  u64 cnt, mc;  // joined pairs and matched symbols of one chunk
};

// Merge tiles: 512 threads x 8 items = 4096 records of LDS capacity.  Sources
// of more than kMergeSmall records take a workgroup of 1,024 threads each
// (up to kMergeMid records, as many as its LDS sorts: k_merge_mid) or the
// multi-block path.  A tile takes
// the sources whose first record falls in a window of W records; with m the
// largest small-source count, every such source ends within the tile's
// capacity when W <= kMergeCap - m + 1 (and, when multi-block sources exist,
// W <= kMergeSmall keeps them last in their window).
constexpr int kMergeNT = 512;
constexpr int kMergeIT = 8;
constexpr int kMergeCap = kMergeNT * kMergeIT;
constexpr u64 kMergeSmall = kMergeCap / 2;
constexpr int kMidNT = 1024;
constexpr u64 kMergeMid = kMidNT * kMergeIT;
constexpr int kIdxBits = 12;  // log2(kMergeCap)
constexpr int kMidIdxBits = 13;  // log2(kMergeMid)
constexpr int kMaxKeyBits = 64 - 2 * kIdxBits;  // 40: part-rank bits of both sides

// A tile whose sources and keys span at most kDenseCap (source, key) pairs
// ((s1 - s0) << key_bits <= kDenseCap) is merged through a table indexed by
// that pair instead of a sort; this needs key_bits <= kDenseKeyBits.
constexpr u32 kDenseCap = 2048;
constexpr int kDenseKeyBits = 11;  // log2(kDenseCap)

// Arc-pair write pass: 512 threads x 8 records per workgroup, which covers
// kExpandGroup write tiles of kExpandTile records (the LDS staging capacity
// for match descriptors).
constexpr int kExpandNT = 512;
constexpr int kExpandIT = 8;
constexpr u64 kExpandTile = 2048;
constexpr u64 kExpandGroup = kExpandNT * kExpandIT / kExpandTile;

// Write tile t holds records [t kExpandTile, (t + 1) kExpandTile): k0 = the
// match holding its first record, base0 = that match's first record.  The
// emit kernels write the entries of the tiles whose first record falls in a
// match they emit; the matches of tile t are k0(t) .. kend(t) - 1, kend(t)
// following from entry t + 1 (k0(t + 1), plus one unless that match starts
// exactly at the tile boundary; M for the last tile).
struct ExpandTile {
  u64 k0, base0;
};

struct LevelArgs {
  CsrView c1, c2;
  const u32 *sq1, *sq2;  // state id -> q1, q2
  u32 lo, nsrc;          // sources are state ids lo .. lo + nsrc - 1
  u64 *cnt;              // [nsrc] unmerged arcs per source
  u32 *mc;               // [nsrc] matched segment pairs per source
  const u64 *roff;       // [nsrc + 1] exclusive scan of cnt
  const u64 *moff;       // [nsrc + 1] exclusive scan of mc
  u32 *wide, *heavy;     // source lists for wavefront / workgroup joins
  uint4 *wrange;         // [nsrc] segment ranges (b1, e1, b2, e2) of wide[i] at i, of
                         // grp[i] at nsrc - 1 - i (the two lists hold at most nsrc)
  Status *st;
  uint4 *match;          // [M] (M1 arc start, M2 arc start, n1, n2)
  u64 *mrbase;           // [M] first record of each match
  ExpandTile *tiles;     // [ceil(R / kExpandTile)] write-tile entries
  u32 *big;              // [nsrc] sources for the multi-block merge (st->nbig), and
                         // from its end those merged by a workgroup each (st->nmid)
  u32 *pk;               // [nsrc] table entries of a product-merge source, else 0
  uint4 *phdr;           // [2 nsrc] product-merge source header (see ProdHeader)
  u32 prod;              // nonzero: sources may take the product merge
  u64 *tstart, *mend;    // [nsrc] the merge's first / end temp slot per source:
                         // zeroed by the count kernel
  u32 *newc;             // [nsrc] new pairs claimed per source: zeroed by the count
                         // kernel, written by the product merge
  u64 *pflag;            // [nsrc] 1 for a product-merge source, plus 2^32 when it
                         // takes the matrix-core form (summed by the level scan)
  u32 quad;              // nonzero: strided product sources go to the four-source
                         // kernel (dense visited array), the others to glist
  u32 *glist;            // [nsrc] product sources for the one-per-wave kernel (st->ngen)
  u32 *grp;              // [nsrc] sources for the 16-lane joins (st->ngrp)
  HeavyChunk *hchunk;    // [kHeavySplit kHeavyChunks] chunk counts of the heavy joins
  u32 *hdone;            // [kHeavySplit] finished chunks, all 0 between levels
  u32 unred;             // composition without reduction: only strided sources with
                         // the four-source kernel take the product form
};

// Target column marks of a direct product level (MergeArgs::out_src), and
// the source of an entry without a term.
constexpr u32 kDstSlot = 0x80000000u, kDstClaim = 0x40000000u, kDstSlotMask = 0x3fffffffu;
constexpr u32 kHoleSrc = 0xffffffffu;

// Written by the count kernel for a product-merge source u at phdr[2u], [2u+1]:
// (M1 part base, M2 part base, P1 | P2 << 16, matrix-core form), (M1 segment
// range begin, end, M2 segment range begin, end).

// lean: grids for lists expected empty (the previous level had none); the
// list kernels loop over their lists, so a longer list is still counted,
// by fewer workgroups.
void launch_count(const LevelArgs &a, hipStream_t s, bool lean = false);
// The wavefront and workgroup joins' counts alone (after launch_chunk_join).
void launch_count_lists(const LevelArgs &a, hipStream_t s, bool lean = false);
// nwide / nheavy / ngrp: the list lengths the count kernels produced
// (st->nwide, nheavy, ngrp).  thread_joins: the sources in no list too (not
// after launch_chunk_join, which lists all it leaves).
void launch_emit(const LevelArgs &a, u32 nwide, u32 nheavy, u32 ngrp, bool thread_joins,
                 hipStream_t s);
// Writes R records: key = (part1 << b2) | part2 (u32 when key_bits <= 32,
// else u64), weight = p1 * p2.
// tiles: the ceil(R / kExpandTile) write-tile entries written by launch_emit.
void launch_expand(const uint4 *match, const u64 *mrbase, u64 M, u64 R, const CsrView &c1,
                   const CsrView &c2, int b2, bool wide_keys, void *rec_key, float *rec_w,
                   ExpandTile *tiles, u32 *err, hipStream_t s);

// Chunk merge (chunk.hip): a wavefront joins, sorts and sums the records of S
// consecutive sources (at most kChunkS) on the chip, in place of count, scan, match
// emission, write pass and merge tiles.  It takes the sources whose shorter
// symbol list has at most kChunkShort symbols and that join at most kChunkPer
// arc pairs (one record is compared with every other of its source), in
// batches of at most kChunkElems short-list symbols and kChunkRecs records;
// its merged arcs go to `cap` temp slots of its own.  The other sources
// (longer lists, more pairs, no slots left) are listed for the general
// kernels, product merge included, as the count kernel lists them.
constexpr u32 kChunkS = 8;
constexpr u32 kChunkShort = 64;
constexpr u32 kChunkPer = 256;
constexpr u32 kChunkElems = 256;
constexpr u32 kChunkStage = 128;   // longest list staged in LDS,
constexpr u32 kChunkStaged = 512;  // and staged symbols of a batch in all
constexpr u32 kChunkRecs = 256;
constexpr u32 kChunkMinCap = 256, kChunkMaxCap = 512;
constexpr int kChunkKeyBits = 28;  // a source's number above them, and a key of all
                                   // ones marks a merged record
static_assert(kChunkS <= (1u << (31 - kChunkKeyBits)), "no key is all ones");
struct ChunkArgs {
  uint4 *tmp;   // [nblk cap] (., M1 part, M2 part, weight bits) from the join,
                // then (slot or id, a, c, weight bits) after launch_chunk_emit
  uint8_t *src; // [nblk cap] source of each, less the wavefront's first
  u32 *cnt;     // [nblk] merged arcs of each wavefront
  const u64 *off;  // NULL, or (after launch_chunk_pack) wavefront b's first slot
                   // in place of b cap
  u32 *pairs;   // [nsrc] joined pairs of each source merged here, else 0
  u32 S, cap;   // kChunkMinCap .. kChunkMaxCap
  u32 first, nblk;  // wavefronts [first, first + nblk) of the level's ceil(nsrc / S)
};
// Sources per wavefront: fewer on a level that would not fill the chip's
// 8,192 wave slots (a source's steps run one after the other in its wave).
inline u32 chunk_sources(u64 nsrc) {
  u32 s = 1;
  while (s < kChunkS && nsrc > (u64)s * 4096) s <<= 1;
  return s;
}
// Sets tstart / mend (into c.tmp) of the sources it merges, cnt = mc = 0.
void launch_chunk_join(const LevelArgs &a, const ChunkArgs &c, int b2, int key_bits,
                       hipStream_t s);
// Moves the merged arcs of c's wavefronts from their regions to tmp / src
// without the unused slots, wavefront b's to off[b] (exclusive scan of c.cnt),
// and its sources' tstart / mend with them.
void launch_chunk_pack(const LevelArgs &a, const ChunkArgs &c, const u64 *off, uint4 *tmp,
                       uint8_t *src, hipStream_t s);

struct MergeArgs {
  const void *rec_key;
  const float *rec_w;
  u64 R;
  const u64 *roff;
  u32 nsrc, lo;
  const u32 *sq1, *sq2;
  const u32 *pbase1, *pbase2;
  const uint2 *parts1, *parts2;
  int key_bits, b2;
  // visited set: a hash table of pair keys (hkeys, hmask; ids by slot in
  // vis) or, when vn2 != 0, a dense array vis[r1 vn2 + r2] (slot = pair
  // index) holding kUnvisited, kClaimed or the pair's id
  u64 *hkeys;
  u64 hmask;
  u32 *vis;
  u32 vn2;
  u32 *newlist;
  u64 newcap;
  uint4 *temp;     // [R] merged runs: (source, key lo, key hi, weight bits) from the
                   // merge, then (slot, a, c, weight bits) after launch_emit_runs
  u32 *runsrc;     // [R] level-local source of the merged run at each temp slot
                   // (written with the visited-table insert)
  u64 *tstart;     // [nsrc] first temp slot of each source's merged arcs (0 if none)
  u64 *mend;       // [nsrc] one past its last slot (0 if none)
  u64 window;      // W: tile t takes the sources starting in [t W, (t + 1) W)
  uint4 *tiles;    // [ntiles = ceil(R / W) + nmid] scratch: tile descriptors
  u32 *sortlist;   // [ntiles] scratch: tiles left to the sort kernel
  u32 *tile_runs;  // [ntiles] merged runs each tile wrote (zero-filled before the merge)
  u64 ntiles;      // merge tiles: the last nmid hold one source of k_merge_mid each
  u32 nmid;
  Status *st;
  // multi-block path
  u32 *big;        // [nbig] level-local source indices
  // fused expand + merge: the level's matches instead of its records
  const uint4 *match;   // [M] (M1 arc start, M2 arc start, n1, n2)
  const u64 *mrbase;    // [M] first record of each match
  const u64 *moff;      // [nsrc + 1] first match of each source
  const uint2 *arcs1, *arcs2;  // CSR arcs (part rank, weight bits)
  const u32 *wts1, *wts2;      // their weight words alone (Csr::wts)
  // product merge: the sources with pk[u] != 0 own temp slots
  // R + poff[u] .. R + poff[u] + pk[u] - 1 (prodpos slots in all)
  const u32 *pk;
  const uint4 *phdr;
  const u64 *poff;
  u64 prodpos;
  u64 *pcnt;  // [nsrc] joined arc pairs of each product-merge source (written by it)
  u32 *newc;  // [nsrc] new pairs each product-merge source claimed (written by it)
  const u64 *R_dev;  // product merge launched before the host knew R: the level's
                     // record count on the device (the kernel merges only if 0)
  u32 quad;          // the strided product sources are merged four per wave
  const u32 *glist;  // the other product sources (st->ngen of them)
  // direct product level (out_src != NULL; dense visited array only): the
  // product kernel writes source u's merged arcs straight to the result
  // columns at out_base + poff[u] + r instead of to temp, with the target
  // column holding the id when the target had one, else its slot with
  // kDstSlot (and kDstClaim when this entry claimed it); entries past the
  // source's merged count get src = kHoleSrc
  u32 *out_src, *out_dst, *out_il, *out_ol;
  float *out_w;
  u64 out_base;
  const u32 *row1, *seg_sym1, *seg_off1, *row2, *seg_sym2, *seg_off2;
  // composition without reduction, a level of strided product sources
  // (utab != NULL): the four-source kernel resolves only the targets, entry
  // r of source u at utab[poff[u] + r] marked like the target column of a
  // direct level; launch_unreduced_product then writes every joined pair
  u32 *utab;
};

// Small levels in one workgroup (merge.hip, k_small_levels): while a level
// has at most kSmallSources sources and kSmallRecords joined pairs, one
// workgroup joins, sorts and merges its records in LDS, inserts the targets,
// numbers the new pairs in (q1, q2) order and appends the merged arcs, then
// goes on with the next level; it stops at the first level it cannot take
// (too large, or a capacity below), at the depth cap, or when the search
// ends, and publishes the loop state to the host.
constexpr u32 kSmallSources = 512;
constexpr u32 kSmallRecords = 1024;
// Joins it takes: the shorter list at most kSmallShortList symbols, the
// longer at most kSmallLongList, at most kSmallPerSource joined pairs per
// source (longer joins and larger sources are the per-level kernels' work,
// done by many workgroups).
constexpr u32 kSmallShortList = 32, kSmallLongList = 4096, kSmallPerSource = 64;
// Why it stopped: a level too large (sources, joined pairs), a capacity, the
// end of the search, or a source of a shape it does not take (a long list
// or many joined pairs: a property of the inputs' states more than of the
// level).
enum : u32 { kSmallTooLarge = 1, kSmallCapacity = 2, kSmallDone = 3, kSmallShape = 4 };
struct SmallState {
  u64 lo, hi, n_states, arcs, premerge;
  u64 max_frontier, max_level_pre;
  u32 depth, levels, new_levels, reason;
};
struct SmallArgs {
  const u32 *row1, *seg_sym1, *seg_off1, *part_base1;
  const uint2 *arcs1, *parts1;
  const u32 *row2, *seg_sym2, *seg_off2, *part_base2;
  const uint2 *arcs2, *parts2;
  int b2, key_bits;
  MergeArgs va;  // visited set: vis, vn2, hkeys, hmask, st
  u32 *sq1, *sq2;
  u64 state_cap;  // at most this many states after a level (arrays, hash load, caps)
  u64 arc_cap;    // at most this many result arcs after a level
  u32 *out_src, *out_dst, *out_il, *out_ol;
  float *out_w;
  u32 max_levels;
  SmallState init;   // where it starts
  SmallState *out;   // host memory: where it stopped, published with the counters
  Status *host;      // as publication `seq`
  u32 seq;
};
void launch_small_levels(const SmallArgs &a, hipStream_t s);

// Composition without reduction, a level whose sources all took the
// four-source form and whose targets utab holds as ids: source u's joined
// pairs as arcs at out_base + off[u] .. (off: exclusive scan of the joined
// pairs per source) in record order, symbol g and entry (p1, p2) at
// g P1 P2 + p1 P2 + p2, weight the float32 product of the two arc weights.
void launch_unreduced_product(const MergeArgs &a, const u64 *off, hipStream_t s);

// Tile descriptors of the level (a.tiles), then the two tile merges: the
// dense-table kernel (only when a.key_bits <= kDenseKeyBits) and the sort
// kernel, which takes every tile the dense kernel did not merge.
void launch_tile_sources(const MergeArgs &a, hipStream_t s);
void launch_merge_dense(const MergeArgs &a, hipStream_t s);
void launch_merge_sort(const MergeArgs &a, bool wide_keys, hipStream_t s);
// Fused expand + merge of every tile (in place of launch_expand and
// launch_merge_dense; needs key_bits <= kDenseKeyBits, no multi-block
// sources, 32-bit record keys).  narrow: both arc arrays below 2^29 arcs.
void launch_fuse_merge(const MergeArgs &a, bool narrow, hipStream_t s);
// Product merge of the sources with a.pk[u] != 0: their merged arcs, with
// visited-table inserts, at temp[R + poff[u] ...) (or the result, on a
// direct level) and tstart / mend: with a.quad, the strided sources four per
// wave and the listed ones (a.glist) one per wave; else every one of them
// one per wave from the list.  narrow: both arc arrays below 2^29 arcs.
// lean: a grid for a listed-source list expected empty (the previous level
// had none; the waves loop over the list).
void launch_prod_sources(const MergeArgs &a, bool narrow, hipStream_t s, bool lean = false);
// Merge of the a.nmid sources listed from the end of a.big.
void launch_merge_mid(const MergeArgs &a, bool wide_keys, hipStream_t s);
// Multi-block merge of the nbig sources listed in a.big; bigoff has nbig + 1
// entries (exclusive scan of their record counts, total RB).
void launch_big_counts(const u64 *roff, const u32 *big, u32 nbig, u64 *bigcnt, hipStream_t s);
void merge_big(const MergeArgs &a, bool wide_keys, u32 nbig, const u64 *bigoff, u64 RB,
               Arena &T, hipStream_t s);

// vn2 != 0: dense visited array (MergeArgs), hkeys unused.
void launch_insert_start(u64 *hkeys, u64 hmask, u32 *hvals, u32 vn2, u32 s1, u32 s2, u32 *sq1,
                         u32 *sq2, u32 *err, hipStream_t s);
void launch_rehash(const u64 *okeys, const u32 *ovals, u64 ocap, u64 *nkeys, u32 *nvals,
                   u64 nmask, u32 *err, hipStream_t s);
// Dense visited array vis (|Q1| |Q2| entries, already kUnvisited) from the
// state arrays: vis[sq1[i] vn2 + sq2[i]] = i for every state id i < n.
void launch_states_to_dense(const u32 *sq1, const u32 *sq2, u64 n, u32 *vis, u32 vn2,
                            hipStream_t s);
// ids base .. base + nnew - 1 in new-list order (or the order in `order`).
void launch_assign(const u32 *slots, u32 nnew, u32 base, const u64 *hkeys, u32 *hvals, u32 vn2,
                   u32 *sq1, u32 *sq2, hipStream_t s);
// The same for min(*count, cap) new pairs, the count read on the device
// (the host need not know it yet); nothing when count is NULL.
void launch_assign_counted(const u32 *slots, const u32 *count, u32 cap, u32 base,
                           const u64 *hkeys, u32 *hvals, u32 vn2, u32 *sq1, u32 *sq2,
                           hipStream_t s, const u64 *skip_if = nullptr);
void launch_newkeys(const u32 *newlist, u32 nnew, const u64 *hkeys, u32 vn2, int bq2, u64 *keys,
                    u32 *vals, hipStream_t s);
// Result append of the level's merged arcs, so that the output stays grouped
// by source id (aoff: exclusive scan of merged arcs per source): the runs of
// merge tile t go to aoff[first source of t] + r, or, when product-merge
// sources sit between the tile's (mixed), each run to aoff[its source] + its
// number there; those of multi-block source u to aoff[u] + r (bigoff, RB: as
// for merge_big; unused without multi-block sources).  dst ids come from
// hvals.  M: merged arcs of the level (the output arrays' length from osrc).
void launch_compact(const MergeArgs &a, const u64 *aoff, const u64 *bigoff, u32 nbig, u64 RB,
                    bool mixed, u64 M, const u32 *hvals, u32 *osrc, u32 *odst, u32 *oil, u32 *ool,
                    float *ow, hipStream_t s);
// Result append of the product-merge sources (pk[u] != 0): tstart[u] ..
// mend[u] - 1 to aoff[u] ....
void launch_compact_sources(const MergeArgs &a, const u64 *aoff, u64 M, const u32 *hvals,
                            u32 *osrc, u32 *odst, u32 *oil, u32 *ool, float *ow, hipStream_t s);
// Visited-table inserts and labels of the chunk-merged arcs (claims to
// a.newlist; plain: the dense visited array alone is marked, with plain
// stores, and launch_claim_count finds the new pairs: a claim by
// compare-and-swap is performed beyond the L2, 100 ps each against 30 for the
// store, and a level of millions of claims spends most of its time there),
// and their result append (after the level's ids; M: room from osrc on).
// skip_if (may be NULL): nothing is done when that device word is nonzero;
// clear: the append zeroes the level counters of a.st.
void launch_chunk_emit(const MergeArgs &a, const ChunkArgs &c, bool plain, const u64 *skip_if,
                       hipStream_t s);
void launch_chunk_compact(const MergeArgs &a, const ChunkArgs &c, const u64 *aoff, u64 M,
                          const u32 *hvals, u32 *osrc, u32 *odst, u32 *oil, u32 *ool, float *ow,
                          const u64 *skip_if, bool clear, hipStream_t s);
// Visited-table inserts and label lookups for every merged arc of the
// tile-merged sources (merge_big does its own).
void launch_emit_tiles(const MergeArgs &a, hipStream_t s);
// The merge kernels append the slots they claim to a.newlist (a.st->nnew of
// them, in any order); the product merge's kernels only flag them in their
// temp entries, and this adds those to the list.
void launch_newlist_product(const MergeArgs &a, hipStream_t s);
// ids base, base + 1, ... for the *count new pairs of the list in (q1, q2)
// order, nothing when there are more than cap (vn2: as launch_assign).
constexpr u32 kRankMax = 16384;
void launch_rank_assign(const u32 *list, const u32 *count, u32 cap, u32 base, const u64 *hkeys,
                        u32 *hvals, u32 vn2, u32 *sq1, u32 *sq2, hipStream_t s);
// The same for every entry of the dense visited array (n pairs) that the
// level claimed, in two passes: launch_claim_count finds and counts them
// (their number to *nnew when given), launch_claim_assign numbers them;
// launch_claim_ids is both.  temp: claim_temp_bytes(n).  skip_if (may be
// NULL): nothing is done when that device word is nonzero.
size_t claim_temp_bytes(u64 n);
void launch_claim_count(const u32 *vis, u64 n, void *temp, u32 *nnew, const u64 *skip_if,
                        hipStream_t s);
void launch_claim_assign(u32 *vis, u64 n, u32 vn2, u32 base, u32 *sq1, u32 *sq2, void *temp,
                         const u64 *skip_if, hipStream_t s);
void launch_claim_ids(u32 *vis, u64 n, u32 vn2, u32 base, u32 *sq1, u32 *sq2, void *temp,
                      const u64 *skip_if, hipStream_t s);
// Direct product level (see MergeArgs::out_src): ids base + newoff[u] + i for
// the claimed entries of source u in entry order (visited array, state
// arrays and the entries' target column).  The other targets the level
// marked with a slot keep the mark until launch_fix_marked.
void launch_assign_direct(const MergeArgs &a, const u64 *newoff, u32 base, u32 *sq1, u32 *sq2,
                          hipStream_t s);
// The n target entries from a.out_dst + a.out_base: every one still marked
// with a visited-array slot replaced by that slot's id (once every level
// that marked them has assigned its ids; several levels in one pass).
void launch_fix_marked(const MergeArgs &a, u64 n, hipStream_t s);
// Removes the entries without a term (src = kHoleSrc) from the n result rows
// at out_base: source u's merged arcs move from out_base + poff[u] to
// out_base + aoff[u] (aoff: exclusive scan of merged arcs per source), through
// `tmp` (20 n bytes).
void launch_close_holes(const MergeArgs &a, const u64 *aoff, u64 n, void *tmp, hipStream_t s);
// Composition without reduction: every record of the level becomes an arc
// (osrc.. at [0, R)), its target pair claimed in the visited table and each
// new claim appended to a.newlist (a.st->nnew); odst receives table slots
// until launch_fix_dst maps them to ids.
void launch_unreduced(const MergeArgs &a, bool wide_keys, u32 *osrc, u32 *odst, u32 *oil, u32 *ool,
                      float *ow, hipStream_t s);
// dst[k] = hvals[dst[k]] for k < n.
void launch_fix_dst(u32 *dst, u64 n, const u32 *hvals, hipStream_t s);
void launch_finals(const u32 *sq1, const u32 *sq2, u64 n, const uint8_t *f1, const uint8_t *f2,
                   uint8_t *fin, hipStream_t s);
// It also copies *st to `host` (pinned, coherent host memory the device can
// write) and then sets host->seq = seq, so that the host can wait for the
// copy by watching that word (the count scan's last tile does the same
// after the level's first phase, ScanPublish).
// Level total of merged arcs, new pairs (*new_total, when not NULL), the
// product merge's joined pairs (*pair_total: the sum of a.pcnt over the
// level's sources, records included, less st->R) and the dense / sort tile
// statistics of st; after publishing it clears the level counters of *st
// for the next level (what launch_reset_level does).
void launch_merged_total(const u64 *a_total, const u64 *new_total, const u64 *pair_total,
                         const MergeArgs &a, Status *host, u32 seq, hipStream_t s);
void launch_reset_level(Status *st, hipStream_t s);
// The 32-bit words of Status that the level-counter clearing zeroes (bit i:
// word i), for a publication that clears them itself (ScanPublish).
u64 level_clear_mask();

// One-workgroup product level (merge.hip, k_product_level): a level of at
// most kTinySources sources, every one a strided product source (the four-
// source matrix-core form) with the dense visited array, taken whole by one
// workgroup: selection, entry offsets, the product merge, id assignment,
// the level totals and their publication (as `seq`, with the counters
// cleared after), one launch instead of the per-level kernels (the targets
// another source claimed stay marked until launch_fix_marked).
// It changes nothing but the sources' headers when a source is of another
// form: then it publishes the counters with `declined` set (and clears
// nothing) and the level takes the per-level kernels.  The result columns
// must hold out_base + nsrc * 64 rows and the state arrays base + nsrc * 64
// entries; la's pk, phdr, tstart, mend, newc and cnt arrays and poff (also
// ma.poff, written here) nsrc + 1.  ordered: the new pairs' ids in (q1, q2)
// order.
constexpr u32 kTinySources = 64;
void launch_product_level(const LevelArgs &la, const MergeArgs &ma, u64 *poff, u64 *newoff,
                          u32 base, u32 *sq1, u32 *sq2, bool ordered, Status *host, u32 seq,
                          hipStream_t s);

}  // namespace fstc
