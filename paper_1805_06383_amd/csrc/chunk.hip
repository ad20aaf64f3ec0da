// Chunk merge: the records of a run of sources joined, sorted and summed by
// one wavefront.
//
// The paper expands every popped pair, writes its composed arcs, sorts them
// and sums equal keys (section 3.4, Algorithm 2), each step over memory.  A
// sparse source has a few to a few hundred arc pairs, so the steps' launches
// and their dependent loads (two joins, match descriptors, records, merge
// tiles) cost far more than the pairs.  Here a wavefront takes kChunkS
// consecutive sources and keeps everything between the symbol lists and the
// merged arcs in registers and LDS:
//   1. one lane per source reads its two symbol lists' ranges and lists the
//      long joins and the product-merge sources for the general kernels;
//   2. both lists of a batch of sources are staged in LDS by groups of 16
//      lanes (longer ones above kChunkStage symbols stay in memory); the
//      shorter lists' symbols are dealt to the lanes and searched in the
//      longer lists, matches packed in symbol order;
//   3. a lane per match reads its arcs' ranges and writes its arc pairs as
//      records, grouped by source, to LDS;
//   4. a record's key is its source's number and its part ranks, so its place
//      in (source, key) order is the number of smaller keys in the batch: the
//      lanes compare theirs with every key, four to an LDS read that all of
//      them share.  Where keys are equal (most sparse sources have none)
//      the records are put in that order in LDS, and the first of each key
//      sums the run in float64, in record order;
//   5. the merged arcs go, in (source, key) order, to the wavefront's own
//      temp slots, so no counter is shared and nothing is scanned before.
// The visited-set inserts follow in a kernel of their own (k_chunk_emit), at
// full occupancy and once the hash table has room for them.
//
// Bound: the wave's dependent loads (state, row, symbols, segments, arcs: each
// a line of another array) and, at hundreds of records a wavefront, the key
// compares.  A wavefront with its lists in LDS was taken over workgroups of
// 256 threads for 32 sources (barriers over unequal sources: the sparse
// level below 11.2 ms searching in memory, 7.4 ms staged) and over a source's
// records in registers (8.3 ms).  A lane takes a record, not a match: a match
// of 250 arc pairs copied by its lane alone held its wavefront for 100 us
// (1,656 sources of a language model: 127 us, now 54).
// Measured on MI355X: 15.9 M sources with 127 M records in six levels (states
// of degree 20, 5,000 symbols: eight joined pairs a source) 5.3 ms, and the whole composition 19.7 -> 14.9 ms
// against joining, scanning, emitting, expanding and tile-merging them; 29
// levels of 320 to 816,000 sources with two records each 9.5 -> 5.6 ms; a
// lexicon's levels of 5,000 to 44,000 sources 3.35 -> 2.30 ms.
#include "product.hpp"
#include "visited.hpp"

namespace fstc {
namespace {

constexpr u32 NT = kWave;  // a wavefront per workgroup: barriers cost nothing
constexpr u32 kBitWords = kChunkRecs / kWave;
static_assert(kChunkS < (u32)kWave && kWave % kChunkS == 0, "a lane per source");
static_assert(kChunkShort <= kChunkElems && kChunkPer <= kChunkRecs, "a source fits a batch");
static_assert(2 * kChunkElems <= kChunkStaged, "two words a match");
static_assert(kChunkElems <= 65535 && kChunkRecs <= 65535, "16-bit offsets");

struct ChunkLds {
  // per source
  u32 sb[kChunkS], lb[kChunkS], le[kChunkS];  // short list, long list range
  u32 l0[kChunkS + 1];                        // staged symbols of the sources before
  u32 pb1[kChunkS], pb2[kChunkS];             // first parts
  u32 e0[kChunkS + 1];                        // first element (short-list symbol)
  u32 r0[kChunkS], rc[kChunkS];               // first record of the batch; records
  unsigned long long pairs[kChunkS];          // joined pairs
  u32 one[kChunkS];                           // M1's list is the shorter
  u32 shift[kChunkS];                         // records of left sources before
  // per element, staged symbol, match and record
  uint8_t esrc[kChunkElems], hsrc[kChunkElems];
  u32 sht[kChunkElems];                       // short lists; then a match's M2 segment, first arc
  u32 lng[kChunkStaged];                      // long lists; then matches' first records, M2 lengths
  u32 hit[kChunkElems];                       // a match's M1 segment, then its first arc
  __align__(16) u32 key[kChunkRecs];          // source number, part ranks
  float w[kChunkRecs];                        // weights, then the first records' sums
  u64 hb[kBitWords + 1];                      // bit p: record p is the first of its key
  u32 hpre[kBitWords + 1];                    // set bits in the words before
};

// Selects source u (of the lanes with want) for the product merge, as
// k_count_small does: the matrix-core form always, whose products are exact
// where the records here are rounded to float32, and the other one when its
// lists have room for a term or more per entry (A1 A2 / max(n1, n2) pairs
// where the lists agree).  Sources with fewer terms than entries are cheaper
// here, in the same precision; a source of 200 pairs on 25 entries is 6 times as
// dear (a million such sources: 14.9 ms, 2.4 by the product merge), one of 32
// on 4 twice.
__device__ __forceinline__ u32 chunk_product(const LevelArgs &a, bool want, u32 u, u32 q1, u32 q2,
                                             const Ranges &r, bool &mf) {
  u32 pk = want ? select_product(a, u, q1, q2, r, mf) : 0u;
  if (pk && !mf) {
    const u64 a1 = a.c1.seg_off[r.e1] - a.c1.seg_off[r.b1],
              a2 = a.c2.seg_off[r.e2] - a.c2.seg_off[r.b2];
    if (a1 * a2 < (u64)pk * max(r.e1 - r.b1, r.e2 - r.b2)) pk = 0;
  }
  return pk;
}

// Lists source u (of the lanes with pred) in `list`.
__device__ __forceinline__ void list_source(bool pred, u32 u, u32 *list, u32 *counter, uint4 *range,
                                            const uint4 &r) {
  const u64 m = __ballot(pred);
  if (!m) return;
  const u32 leader = (u32)__builtin_ctzll(m);
  u32 at = 0;
  if (lane_id() == leader) at = atomicAdd(counter, (u32)__popcll(m));
  at = __shfl(at, (int)leader, kWave) + count_below(m);
  if (pred) {
    list[at] = u;
    if (range) range[at] = r;
  }
}

// Keys of the n in LDS below `key`, and (le) at most `key`.
__device__ __forceinline__ u32 keys_below(const u32 *keys, u32 n, u32 key, u32 &le) {
  u32 lt = 0, l = 0;
#pragma unroll 4
  for (u32 q = 0; q < n; q += 4) {  // uniform; the keys past n are all ones
    const uint4 k = *reinterpret_cast<const uint4 *>(keys + q);
    lt += k.x < key ? 1u : 0u;
    l += k.x <= key ? 1u : 0u;
    lt += k.y < key ? 1u : 0u;
    l += k.y <= key ? 1u : 0u;
    lt += k.z < key ? 1u : 0u;
    l += k.z <= key ? 1u : 0u;
    lt += k.w < key ? 1u : 0u;
    l += k.w <= key ? 1u : 0u;
  }
  le = l;
  return lt;
}

// Records of the n in LDS before record p, whose key is `key`, in (key,
// record) order.
__device__ __forceinline__ u32 keys_before(const u32 *keys, u32 n, u32 key, u32 p) {
  u32 lt = 0;
#pragma unroll 4
  for (u32 q = 0; q < n; q += 4) {  // uniform
    const uint4 k = *reinterpret_cast<const uint4 *>(keys + q);
    lt += k.x < key || (k.x == key && q < p) ? 1u : 0u;
    lt += k.y < key || (k.y == key && q + 1 < p) ? 1u : 0u;
    lt += k.z < key || (k.z == key && q + 2 < p) ? 1u : 0u;
    lt += k.w < key || (k.w == key && q + 3 < p) ? 1u : 0u;
  }
  return lt;
}

// One batch: sources [i0, i1) of the wavefront, whose En elements begin at
// element eb.  Returns the sources done: [i0, end).  steps: the largest power
// of two that a staged list's length reaches; u, q1, q2, r: lane t's source.
__device__ __forceinline__ u32 chunk_batch(const LevelArgs &a, const ChunkArgs &c, int b2, int kb,
                                           ChunkLds &L, u32 i0, u32 i1, u32 eb, u32 En, u32 steps,
                                           u64 region, u32 &out, u32 u, u32 q1, u32 q2,
                                           const Ranges &r, bool &unfit) {
  const u32 t = lane_id();
  // 2. staging: group g of 16 lanes takes sources i0 + g, i0 + g + 4, ...
  const u32 lbase = L.l0[i0];
#pragma unroll
  for (u32 v = 0; v < kChunkS; v += NT / 16) {
    const u32 i = i0 + v + t / 16, ic = min(i, i1 - 1), l = t % 16;
    const u32 ns = i < i1 ? L.e0[ic + 1] - L.e0[ic] : 0u, so = L.e0[ic] - eb;
    const u32 nl0 = L.l0[ic + 1] - L.l0[ic], lo = L.l0[ic] - lbase;
    const u32 nl = i < i1 && lo + nl0 <= kChunkStaged ? nl0 : 0u;
    const u32 *ss = (L.one[ic] ? a.c1.seg_sym : a.c2.seg_sym) + L.sb[ic];
    const u32 *ls = (L.one[ic] ? a.c2.seg_sym : a.c1.seg_sym) + L.lb[ic];
    // the first 16 and 32 symbols of the lists in flight together
    if (ns) {
      const u32 x = ss[min(l, ns - 1)];
      const u32 y0 = ls[min(l, max(nl, 1u) - 1)], y1 = ls[min(16 + l, max(nl, 1u) - 1)];
      if (l < ns) L.sht[so + l] = x;
      if (l < nl) L.lng[lo + l] = y0;
      if (16 + l < nl) L.lng[lo + 16 + l] = y1;
      for (u32 k = 16 + l; k < ns; k += 16) L.sht[so + k] = ss[k];
      for (u32 k = 32 + l; k < nl; k += 16) L.lng[lo + k] = ls[k];
      for (u32 k = l; k < ns; k += 16) L.esrc[so + k] = (uint8_t)i;
    }
  }
  __syncthreads();
  // search, 64 elements at a time; the matches packed
  u32 H = 0;
  for (u32 e0 = 0; e0 < En; e0 += NT) {
    const u32 e = min(e0 + t, En - 1), i = L.esrc[e];
    const u32 n = L.l0[i + 1] - L.l0[i], o = L.l0[i] - lbase;
    const bool staged = n && o + n <= kChunkStaged;
    const u32 idx = L.sb[i] + (e - (L.e0[i] - eb)), sym = L.sht[e], lb = L.lb[i];
    const bool one = L.one[i];
    u32 pos = 0;  // list symbols below sym
    for (u32 st = steps; st; st >>= 1) {
      const u32 q = pos + st - 1;
      const u32 x = L.lng[staged && q < n ? o + q : 0u];
      pos += staged && q < n && x < sym ? st : 0u;
    }
    bool found = staged && pos < n && L.lng[o + min(pos, n - 1)] == sym;
    if (__ballot(!staged)) {
      const u32 *ls = one ? a.c2.seg_sym : a.c1.seg_sym;
      u32 hi = staged ? 0u : L.le[i] - lb;
      while (__ballot(pos < hi)) {
        const bool live = pos < hi;
        const u32 m = (pos + hi) >> 1;
        const u32 x = ls[live ? lb + m : lb];
        pos = live && x < sym ? m + 1 : pos;
        hi = live && x >= sym ? m : hi;
      }
      if (!staged) found = lb + pos < L.le[i] && ls[min(lb + pos, L.le[i] - 1)] == sym;
    }
    found = found && e0 + t < En;
    const u64 m = __ballot(found);
    if (found) {
      const u32 h = H + count_below(m);
      L.hsrc[h] = (uint8_t)i;
      L.hit[h] = one ? idx : lb + pos;
      L.sht[h] = one ? lb + pos : idx;  // h <= e: the elements up to e are read
    }
    H += (u32)__popcll(m);
    __syncthreads();
  }
  // 3. a lane per match: its segments' arcs; record offsets in match order (a
  //    match's pairs counted up to kChunkPer + 1: its source is left over then)
  if (t >= i0 && t < i1) {
    L.pairs[t] = 0;
    L.rc[t] = 0;
    L.r0[t] = 0;
  }
  __syncthreads();
  // (the staged lists are read no more: their words hold the matches' first
  // records and the lengths of their M2 segments)
  u32 *const first = L.lng, *const len2 = L.lng + kChunkElems;
  u32 R = 0, most = 0;  // most: arc pairs of a match
  for (u32 h0 = 0; h0 < H; h0 += NT) {
    const u32 h = h0 + t;
    const bool v = h < H;
    const u32 s1 = v ? L.hit[h] : 0u, s2 = v ? L.sht[h] : 0u, i = v ? L.hsrc[h] : 0u;
    const u32 a1 = a.c1.seg_off[s1], n1 = a.c1.seg_off[s1 + 1] - a1;
    const u32 a2 = a.c2.seg_off[s2], n2 = a.c2.seg_off[s2 + 1] - a2;
    const u64 nn = v ? (u64)n1 * n2 : 0;
    const u32 n = (u32)min<u64>(nn, (u64)(kChunkPer + 1));
    const u32 inc = wave_inclusive_total(n);
    const u32 ro = R + inc - n;
    R += (u32)__builtin_amdgcn_readlane((int)inc, kWave - 1);
    most = max(most, n);
    if (v) {
      // a source's matches are consecutive: its first one's offset, and its
      // counts added up per source
      if (h == 0 || L.hsrc[h - 1] != i) L.r0[i] = ro;
      atomicAdd(&L.pairs[i], (unsigned long long)nn);
      atomicAdd(&L.rc[i], n);
      L.hit[h] = a1;
      L.sht[h] = a2;
      first[h] = ro;
      len2[h] = n2;
    }
  }
  __syncthreads();
  bool over = false;  // lane t: source t is left over
  if (t >= i0 && t < i1) over = L.rc[t] > kChunkPer;
  u32 end = i1;
  {
    // without the left sources' records; the sources past the records'
    // capacity wait for the next batch
    const bool mine = t >= i0 && t < i1;
    const u32 n = mine && !over ? L.rc[min(t, kChunkS - 1)] : 0u;
    const u32 inc = wave_inclusive_total(n), r0 = inc - n;
    const u64 late = __ballot(mine && inc > kChunkRecs);
    if (late) end = (u32)__builtin_ctzll(late);
    if (mine) {
      L.shift[t] = L.r0[t] - r0;
      L.r0[t] = r0;
      L.rc[t] = over ? 0u : n;
    }
    R = (u32)__builtin_amdgcn_readlane((int)inc, (int)end - 1);
  }
  __syncthreads();
  // records, a lane each: record p is match p's when every match has one arc
  // pair, else of the last match that begins at or before p (a left source's
  // matches begin where the next source's do)
  const bool single = !__ballot(most > 1);
  if (!single) {
    for (u32 h = t; h < H; h += NT) {
      const u32 i = L.hsrc[h];
      first[h] = L.rc[i] ? first[h] - L.shift[i] : L.r0[i];
    }
    __syncthreads();
  }
  for (u32 p = t; p < R; p += NT) {
    u32 h = p, x1 = 0, x2 = 0;
    if (!single) {
      u32 lo = 0, hi = H;  // first[lo] <= p: match 0 begins at record 0
      while (hi - lo > 1) {
        const u32 m = (lo + hi) >> 1;
        if (first[m] <= p) lo = m;
        else hi = m;
      }
      h = lo;
      const u32 k = p - first[h], n2 = len2[h];
      x1 = k / n2;
      x2 = k - x1 * n2;
    }
    const uint2 y1 = a.c1.arcs[L.hit[h] + x1], y2 = a.c2.arcs[L.sht[h] + x2];
    L.key[p] = ((u32)L.hsrc[h] << kb) | (y1.x << b2) | y2.x;
    L.w[p] = __uint_as_float(y1.y) * __uint_as_float(y2.y);
  }
  if (t < 4 && R + t < kChunkRecs) L.key[R + t] = 0xffffffffu;  // above every key
  if (t <= kBitWords) L.hb[t] = 0;
  __syncthreads();
  // 4. places in (source, key) order
  const u32 pmask = (1u << kb) - 1u, p2mask = (1u << b2) - 1u;
  auto put = [&](u32 place, u32 key, float wt) {
    const u32 i = key >> kb, k = key & pmask;
    const u64 o = region + out + place;
    c.tmp[o] = make_uint4(0u, L.pb1[i] + (k >> b2), L.pb2[i] + (k & p2mask), __float_as_uint(wt));
    c.src[o] = (uint8_t)i;
  };
  bool repeats = false, fits = out + R <= c.cap;
  for (u32 p0 = 0; p0 < R; p0 += NT) {
    const u32 p = p0 + t, key = L.key[min(p, R - 1)];
    u32 le;
    const u32 lt = keys_below(L.key, R, key, le);
    const bool eq = __ballot(p < R && le != lt + 1) != 0;
    repeats |= eq;
    // 5. (for nothing when a later record repeats a key: written again below)
    // (+ 0: a sum of one term, as the other merges form it)
    if (!eq && fits && p < R) put(lt, key, L.w[p] + 0.0f);
  }
  u32 M = R;
  auto before = [&](u32 p) {  // merged arcs of the first p records in order
    return !repeats ? p
                    : L.hpre[p / kWave] +
                          (u32)__popcll(L.hb[p / kWave] & ((1ull << (p % kWave)) - 1ull));
  };
  if (repeats) {  // uniform
    // the records in (key, record) order; the first of each key sums the run
    u32 key[kBitWords], place[kBitWords];
    float wt[kBitWords];
#pragma unroll
    for (u32 j = 0; j < kBitWords; ++j) {
      const u32 p = j * NT + t;
      key[j] = 0xffffffffu;
      place[j] = 0;
      wt[j] = 0.0f;
      if (j * NT < R) {
        key[j] = L.key[min(p, R - 1)];
        wt[j] = L.w[min(p, R - 1)];
        place[j] = keys_before(L.key, R, key[j], p);
      }
    }
    __syncthreads();
#pragma unroll
    for (u32 j = 0; j < kBitWords; ++j) {
      if (j * NT + t < R) {
        L.key[place[j]] = key[j];
        L.w[place[j]] = wt[j];
      }
    }
    __syncthreads();
    M = 0;
#pragma unroll
    for (u32 j = 0; j < kBitWords; ++j) {
      const u32 p = j * NT + t;
      key[j] = L.key[min(p, kChunkRecs - 1)];
      const u64 m = __ballot(p < R && (p == 0 || L.key[p - 1] != key[j]));
      place[j] = M + count_below(m);
      if (t == 0) {
        L.hb[j] = m;
        L.hpre[j] = M;
      }
      M += (u32)__popcll(m);
    }
    if (t == 0) L.hpre[kBitWords] = M;
    __syncthreads();
    fits = out + M <= c.cap;
    if (fits) {
#pragma unroll
      for (u32 j = 0; j < kBitWords; ++j) {
        const u32 p = j * NT + t;
        if (!((L.hb[j] >> t) & 1u)) continue;
        double acc = 0.0;
        for (u32 q = p; q < R && L.key[q] == key[j]; ++q) acc += (double)L.w[q];
        put(place[j], key[j], (float)acc);
      }
    }
  }
  // a batch without slots left goes to the general kernels
  const bool mine = t >= i0 && t < end;
  const u64 n = mine ? (u64)L.pairs[min(t, kChunkS - 1)] : 0ull;
  const bool left = mine && (over || (!fits && n != 0));
  if (mine && !left && n) {
    const u32 b = L.r0[t];
    a.tstart[u] = region + out + before(b);
    a.mend[u] = region + out + before(b + L.rc[t]);
    c.pairs[u] = (u32)n;
  }
  unfit |= n > kSmallPerSource;
  if (__ballot(left)) {
    // left over: product-merge sources; short lists with their counts known,
    // for the 16-lane emission; long ones joined again as wide sources
    u32 pk = 0;
    bool mf = false;
    if (left && a.prod && min(r.e1 - r.b1, r.e2 - r.b2) >= kProdMinSymbols) {
      pk = select_product(a, u, q1, q2, r, mf);
      if (pk) {
        a.pk[u] = pk;
        a.pflag[u] = 1ull | ((u64)mf << 32);
        unfit = true;
      }
    }
    // (strided sources go to the four-source kernel when it runs)
    list_source(pk && !(a.quad && (a.phdr[2 * u].w & 4u)), u, a.glist, &a.st->ngen, nullptr,
                make_uint4(0, 0, 0, 0));
    const bool lng = left && !pk && max(r.e1 - r.b1, r.e2 - r.b2) > kGroupLong;
    const bool grp = left && !pk && !lng;
    const uint4 rr = make_uint4(r.b1, r.e1, r.b2, r.e2);
    list_source(lng, u, a.wide, &a.st->nwide, a.wrange, rr);
    const u64 m = __ballot(grp);
    if (m) {
      const u32 leader = (u32)__builtin_ctzll(m);
      u32 at = 0;
      if (t == leader) at = atomicAdd(&a.st->ngrp, (u32)__popcll(m));
      at = __shfl(at, (int)leader, kWave) + count_below(m);
      if (grp) {
        u32 mc = 0;  // its matches
        for (u32 h = 0; h < H; ++h) mc += L.hsrc[h] == t ? 1u : 0u;
        a.grp[at] = u;
        a.wrange[a.nsrc - 1 - at] = rr;
        a.cnt[u] = n;
        a.mc[u] = mc;
        if (n > kMergeSmall) list_large(a, u, n);
        else atomicMax(&a.st->max_small, (u32)n);
      }
    }
    if (t == 0) a.st->general = 1;
  }
  if (fits) out += M;
  __syncthreads();
  return end;
}

__global__ __launch_bounds__(NT) void k_chunk_join(LevelArgs a, ChunkArgs c, int b2, int kb) {
  __shared__ ChunkLds L;
  const u32 t = lane_id();
  const u64 u0 = ((u64)c.first + blockIdx.x) * c.S;
  const u32 ns = (u32)min<u64>(c.S, a.nsrc - u0);
  // 1. classification: lane t < kChunkS holds source u0 + t
  const u32 u = (u32)u0 + t;
  Ranges r{0, 0, 0, 0};
  bool unfit = false;
  u32 E = 0, q1 = 0, q2 = 0;
  bool wide = false, heavy = false, mf = false;
  u32 pk = 0;
  if (t < ns) {
    q1 = a.sq1[a.lo + u];
    q2 = a.sq2[a.lo + u];
    r = Ranges{a.c1.row[q1], a.c1.row[q1 + 1], a.c2.row[q2], a.c2.row[q2 + 1]};
    const u32 pb1 = a.c1.part_base[q1], pb2 = a.c2.part_base[q2];
    const u32 parts = a.c1.part_base[q1 + 1] - pb1 + a.c2.part_base[q2 + 1] - pb2;
    const u32 n1 = r.e1 - r.b1, n2 = r.e2 - r.b2;
    const u32 mn = min(n1, n2), mx = max(n1, n2);
    heavy = mn > kHeavyMin;
    wide = !heavy && mn > kChunkShort;
    // (part counts first, which come with the part bases: most sources have too many)
    pk = chunk_product(a, a.prod && mn >= kProdMinSymbols && mn <= (u32)kWave && parts <= kProdRowSum,
                       u, q1, q2, r, mf);
    if (mn <= kChunkShort && !pk) E = mn;
    unfit = pk || mn > kSmallShortList || mx > kSmallLongList;
    a.tstart[u] = 0;
    a.mend[u] = 0;
    a.newc[u] = 0;
    a.pk[u] = pk;
    a.pflag[u] = pk ? 1ull | ((u64)mf << 32) : 0ull;
    a.cnt[u] = 0;
    a.mc[u] = 0;
    c.pairs[u] = 0;
    const bool one = n1 <= n2;
    L.one[t] = one ? 1u : 0u;
    L.sb[t] = one ? r.b1 : r.b2;
    L.lb[t] = one ? r.b2 : r.b1;
    L.le[t] = one ? r.e2 : r.e1;
    L.pb1[t] = pb1;
    L.pb2[t] = pb2;
  }
  const u32 ln = E ? max(r.e1 - r.b1, r.e2 - r.b2) : 0u, stg = ln <= kChunkStage ? ln : 0u;
  {
    const u32 inc = wave_inclusive_total(E), linc = wave_inclusive_total(stg);
    if (t <= kChunkS) {  // lane kChunkS holds no source: the totals
      L.e0[t] = inc - E;
      L.l0[t] = linc - stg;
    }
  }
  const u32 lens = wave_or(stg);
  const u32 steps = lens ? 1u << (31 - __clz(lens)) : 0u;
  if (__ballot(wide || heavy || pk)) {
    // (strided sources go to the four-source kernel when it runs)
    list_source(pk && !(a.quad && (a.phdr[2 * u].w & 4u)), u, a.glist, &a.st->ngen, nullptr,
                make_uint4(0, 0, 0, 0));
    list_source(heavy, u, a.heavy, &a.st->nheavy, nullptr, make_uint4(0, 0, 0, 0));
    list_source(wide, u, a.wide, &a.st->nwide, a.wrange, make_uint4(r.b1, r.e1, r.b2, r.e2));
    if (t == 0) a.st->general = 1;
  }
  __syncthreads();
  const u64 region = (u64)blockIdx.x * c.cap;
  u32 out = 0;  // merged arcs so far
  u32 i0 = 0;
  while (i0 < ns) {  // uniform
    // the batch: sources [i0, i1) of at most kChunkElems elements
    const u32 eb = L.e0[i0];
    const u32 i = i0 + 1 + t;
    const u32 i1 = i0 + (u32)__popcll(__ballot(i <= ns && L.e0[min(i, kChunkS)] - eb <= kChunkElems));
    // (e0 past the last source is the element total)
    const u32 En = L.e0[i1] - eb;
    i0 = En
            ? chunk_batch(a, c, b2, kb, L, i0, i1, eb, En, steps, region, out, u, q1, q2, r,
                          unfit)
            : i1;
  }
  // (read only on levels about as small as the one-workgroup kernel takes)
  const u32 n = a.nsrc <= 16 * kSmallSources ? (u32)__popcll(__ballot(unfit)) : 0u;
  if (t == 0) {
    c.cnt[blockIdx.x] = out;
    if (n) atomicAdd(&a.st->unfit, n);
  }
}

// First temp slot of wavefront b's merged arcs.
__device__ __forceinline__ u64 region_base(const ChunkArgs &c, u32 b) {
  return c.off ? c.off[b] : (u64)b * c.cap;
}

// Packs the regions (launch_chunk_pack), kPackB of them by a wave at a time:
// their first 64 entries together, then the rest of each.  Bound by the copy,
// 34 B an arc (six runs of up to 15.8 M sparse sources, 1.23 ms each a region at
// a time, a chain of three loads, now 0.97).
constexpr u32 kOutNT = 256, kOutB = 4;
constexpr u32 kPackB = 4;
static_assert(kPackB * kChunkS <= (u32)kWave, "a lane per source");
__global__ __launch_bounds__(kOutNT) void k_chunk_pack(LevelArgs a, ChunkArgs c, const u64 *off,
                                                       uint4 *tmp, uint8_t *src) {
  const u32 lane = lane_id();
  const u32 nw = gridDim.x * (kOutNT / kWave);
  for (u64 b0 = ((u64)blockIdx.x * (kOutNT / kWave) + threadIdx.x / kWave) * kPackB; b0 < c.nblk;
       b0 += (u64)nw * kPackB) {  // wave-uniform
    u32 n[kPackB], most = 0;
    u64 from[kPackB], to[kPackB];
#pragma unroll
    for (u32 j = 0; j < kPackB; ++j) {
      const u32 b = (u32)min<u64>(b0 + j, c.nblk - 1);
      n[j] = b0 + j < c.nblk ? min(c.cnt[b], c.cap) : 0u;  // at most cap by the join
      from[j] = (u64)b * c.cap;
      to[j] = off[b];
      most = max(most, n[j]);
    }
    for (u32 e0 = 0; e0 < most; e0 += kWave) {
      const u32 e = e0 + lane;
      uint4 x[kPackB];
      uint8_t y[kPackB];
#pragma unroll
      for (u32 j = 0; j < kPackB; ++j) {
        x[j] = make_uint4(0, 0, 0, 0);
        y[j] = 0;
        if (e < n[j]) {
          x[j] = c.tmp[from[j] + e];
          y[j] = c.src[from[j] + e];
        }
      }
#pragma unroll
      for (u32 j = 0; j < kPackB; ++j) {
        if (e < n[j]) {
          tmp[to[j] + e] = x[j];
          src[to[j] + e] = y[j];
        }
      }
    }
    // lane j S + i: source i of region j (the sources merged elsewhere have no
    // slots)
    const u32 j = lane / c.S;
    const u64 u = (c.first + b0) * c.S + lane;
    if (j < kPackB && b0 + j < c.nblk && u < a.nsrc && c.pairs[u]) {
      const u64 by = off[b0 + j] - (b0 + j) * c.cap;
      a.tstart[u] += by;
      a.mend[u] += by;
    }
  }
}

// Merged arcs of the chunk merge, a wave per region: part numbers to (r1, a)
// and (r2, c), the target pair inserted in the visited set, claims listed
// (appended when kClaimCap might not hold another round's).  PLAIN (dense
// visited array, launch_chunk_emit): claimed by a plain store instead, and the
// level's new pairs found by a pass over the array.
constexpr u32 kClaimCap = 4096;
static_assert(kOutNT / kWave * kOutB * kChunkMinCap <= kClaimCap &&
                  kOutNT / kWave * 2 * kChunkMaxCap <= kClaimCap,
              "a round's claims fit the list");

// Entries q[j] of this lane where act[j].
template <u32 B, bool PLAIN, class Claims>
__device__ __forceinline__ void emit_entries(const MergeArgs &a, const ChunkArgs &c,
                                             const u64 (&q)[B], const bool (&act)[B], Claims &L) {
  bool is_new[B];
  uint4 x[B];
  uint2 P1[B], P2[B];
  u64 hk[B];
  u32 slot[B], known[B];
#pragma unroll
  for (u32 j = 0; j < B; ++j) x[j] = act[j] ? c.tmp[q[j]] : make_uint4(0, 0, 0, 0);
#pragma unroll
  for (u32 j = 0; j < B; ++j) {
    P1[j] = a.parts1[x[j].y];
    P2[j] = a.parts2[x[j].z];
    hk[j] = ((u64)P1[j].x << 32) | P2[j].x;
  }
  if constexpr (PLAIN) {
    // every lane that finds a pair unvisited stores the same mark
#pragma unroll
    for (u32 j = 0; j < B; ++j) {
      slot[j] = act[j] ? P1[j].x * a.vn2 + P2[j].x : 0u;
      known[j] = act[j] ? __hip_atomic_load(&a.vis[slot[j]], __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_WORKGROUP)
                        : kClaimed;
    }
#pragma unroll
    for (u32 j = 0; j < B; ++j) {
      if (known[j] == kUnvisited)
        __hip_atomic_store(&a.vis[slot[j]], kClaimed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      known[j] = known[j] < kClaimed ? known[j] : kUnvisited;
    }
  } else {
    visit_batch<B>(a, hk, act, slot, is_new, known);
  }
#pragma unroll
  for (u32 j = 0; j < B; ++j) {
    if (act[j])
      c.tmp[q[j]] = make_uint4(known[j] != kUnvisited ? known[j] | kIdFlag : slot[j], P1[j].y,
                               P2[j].y, x[j].w);
    if constexpr (!PLAIN) claims_add(L, is_new[j] ? slot[j] : kNoClaim);
  }
}

// A wave takes B regions at a time, their first 64 entries together, then the
// rest of each: a region of sparse sources holds about 64, one dependent chain
// (parts, visited entry, claim) per lane if taken alone.
template <u32 B, bool PLAIN>
__global__ __launch_bounds__(kOutNT) void k_chunk_emit(MergeArgs a, ChunkArgs c, const u64 *skip_if) {
  __shared__ ClaimLds<PLAIN ? 1u : kClaimCap> L;
  if (skip_if && *skip_if) return;  // uniform
  if (!PLAIN) claims_begin(L);
  constexpr u32 kW = kOutNT / kWave * B;
  const u32 lane = lane_id();
  for (u32 b0 = blockIdx.x * kW; b0 < c.nblk; b0 += gridDim.x * kW) {  // uniform
    if (!PLAIN) {  // room for a round's claims
      __syncthreads();
      const u32 have = L.n;
      __syncthreads();  // every wave has read it before one adds: one decision for all
      if (have + kW * c.cap > kClaimCap) {
        claims_end(a, L);
        __syncthreads();
        claims_begin(L);
      }
    }
    const u32 bw = b0 + threadIdx.x / kWave * B;
    u32 n[B], most = 0;
    u64 q[B];
    bool act[B];
#pragma unroll
    for (u32 j = 0; j < B; ++j) {
      n[j] = bw + j < c.nblk ? min(c.cnt[bw + j], c.cap) : 0u;  // at most cap by the join
      most = max(most, n[j]);
      act[j] = lane < n[j];
      q[j] = (n[j] ? region_base(c, bw + j) : 0ull) + lane;
    }
    if (most == 0) continue;  // wave-uniform
    emit_entries<B, PLAIN>(a, c, q, act, L);
    for (u32 e = kWave; e < most; e += kWave) {
#pragma unroll
      for (u32 j = 0; j < B; ++j) {
        q[j] += kWave;
        act[j] = e + lane < n[j];
      }
      emit_entries<B, PLAIN>(a, c, q, act, L);
    }
  }
  if (!PLAIN) claims_end(a, L);
}

// Result append of the chunk-merged arcs, a wave per region: source u's slots
// [tstart, mend) go to aoff[u] ....
__global__ __launch_bounds__(kOutNT) void k_chunk_compact(MergeArgs a, ChunkArgs c, const u64 *aoff,
                                                          u64 M, const u32 *hvals, u32 *osrc,
                                                          u32 *odst, u32 *oil, u32 *ool, float *ow,
                                                          const u64 *skip_if, u32 clear) {
  if (skip_if && *skip_if) return;
  const u32 lane = lane_id();
  const u32 nw = gridDim.x * (kOutNT / kWave);
  for (u32 b = blockIdx.x * (kOutNT / kWave) + threadIdx.x / kWave; b < c.nblk; b += nw) {
    const u32 n = min(c.cnt[b], c.cap);
    if (n == 0) continue;
    const u64 base = region_base(c, b), u0 = ((u64)c.first + b) * c.S;
    // lane i < S: output position less temp slot (wraps) of source i
    const u64 u = min(u0 + lane % kChunkS, (u64)a.nsrc - 1);
    const u64 to = aoff[u] - a.tstart[u];
    for (u32 e0 = 0; e0 < n; e0 += 2 * kWave) {
      uint4 x[2];
      u32 i[2], d[2];
      u64 k[2];
      bool act[2];
#pragma unroll
      for (u32 j = 0; j < 2; ++j) {
        const u32 e = e0 + j * kWave + lane;
        act[j] = e < n;
        const u64 q = base + min(e, n - 1);
        x[j] = c.tmp[q];
        i[j] = c.src[q];
        k[j] = q;
      }
#pragma unroll
      for (u32 j = 0; j < 2; ++j) {
        k[j] += __shfl(to, (int)(i[j] % kChunkS), kWave);
        if (act[j] && k[j] >= M) {  // impossible: counts agree with aoff
          set_error(&a.st->err, kErrBounds);
          act[j] = false;
        }
        d[j] = act[j] ? target_id(a, x[j].x, hvals) : 0u;
      }
#pragma unroll
      for (u32 j = 0; j < 2; ++j) {
        if (!act[j]) continue;
        osrc[k[j]] = a.lo + (u32)u0 + i[j];
        odst[k[j]] = d[j];
        oil[k[j]] = x[j].y;
        ool[k[j]] = x[j].z;
        ow[k[j]] = __uint_as_float(x[j].w);
      }
    }
  }
  // (no other workgroup of a cleared level reads the counters: skip_if, which
  // they read, is zero and stays so)
  if (clear && blockIdx.x == 0 && threadIdx.x == 0) clear_level(a.st);
}

}  // namespace

void launch_chunk_join(const LevelArgs &a, const ChunkArgs &c, int b2, int key_bits,
                       hipStream_t s) {
  if (key_bits > kChunkKeyBits || !c.S || c.S > kChunkS || !c.nblk ||
      (u64)c.first + c.nblk > ceil_div(a.nsrc, c.S) || c.cap < kChunkMinCap || c.cap > kChunkMaxCap)
    throw Error(FSTC_ERR_INTERNAL, "chunk merge out of its range");
  hipLaunchKernelGGL(k_chunk_join, dim3(c.nblk), dim3(NT), 0, s, a, c, b2, key_bits);
}

void launch_chunk_pack(const LevelArgs &a, const ChunkArgs &c, const u64 *off, uint4 *tmp,
                       uint8_t *src, hipStream_t s) {
  const u64 g = std::min<u64>(ceil_div(c.nblk, kOutNT / kWave * kPackB), 1u << 20);
  hipLaunchKernelGGL(k_chunk_pack, dim3((unsigned)g), dim3(kOutNT), 0, s, a, c, off, tmp, src);
}

void launch_chunk_emit(const MergeArgs &a, const ChunkArgs &c, bool plain, const u64 *skip_if,
                       hipStream_t s) {
  if (!c.nblk) return;
  if (plain && !a.vn2) throw Error(FSTC_ERR_INTERNAL, "plain claims need the dense visited array");
  const u32 B = c.cap <= kChunkMinCap ? kOutB : 2u;
  // a few rounds per workgroup (and append) on large levels
  const u64 rounds = ceil_div(c.nblk, (u64)kOutNT / kWave * B);
  const dim3 g((unsigned)std::max<u64>(1, std::min<u64>(rounds, std::max<u64>((u64)compute_units() * 8,
                                                                            rounds / 4))));
  auto go = [&](auto b, auto pl) {
    hipLaunchKernelGGL((k_chunk_emit<decltype(b)::value, decltype(pl)::value>), g, dim3(kOutNT), 0, s,
                       a, c, skip_if);
  };
  using Four = std::integral_constant<u32, kOutB>;
  using Two = std::integral_constant<u32, 2>;
  if (B == kOutB) plain ? go(Four(), std::true_type()) : go(Four(), std::false_type());
  else plain ? go(Two(), std::true_type()) : go(Two(), std::false_type());
}

void launch_chunk_compact(const MergeArgs &a, const ChunkArgs &c, const u64 *aoff, u64 M,
                          const u32 *hvals, u32 *osrc, u32 *odst, u32 *oil, u32 *ool, float *ow,
                          const u64 *skip_if, bool clear, hipStream_t s) {
  if (!c.nblk) return;
  const u64 g = std::min<u64>(ceil_div(c.nblk, kOutNT / kWave), 1u << 20);
  hipLaunchKernelGGL(k_chunk_compact, dim3((unsigned)g), dim3(kOutNT), 0, s, a, c, aoff, M, hvals,
                     osrc, odst, oil, ool, ow, skip_if, clear ? 1u : 0u);
}

}  // namespace fstc
