// Visited-set inserts and the lists of newly claimed pairs, shared by the
// merge kernels (merge.hip, chunk.hip).  The paper tracks visited pairs in a
// table of |Q1||Q2| entries updated atomically (section 3.4, "Updating
// frontier and visited set").
#pragma once

#include "level.hpp"

namespace fstc {

// Linear-probing insert of B keys at once (lanes with act[i] unset skip
// item i).  Each round issues the probe loads of all pending items before
// testing any, so their latencies overlap.  Slots only ever change from
// kEmptyKey to a key, so a stale read of kEmptyKey is settled by the CAS and
// a plain (workgroup-scope) read is enough.  Bounded by the table size.
template <int B>
__device__ __forceinline__ void hash_insert_batch(u64 *keys, u64 mask, const u64 (&key)[B],
                                                  const bool (&act)[B], u32 (&slot)[B],
                                                  bool (&is_new)[B], u32 *err) {
  u64 h[B];
  bool pend[B];
#pragma unroll
  for (int i = 0; i < B; ++i) {
    pend[i] = act[i];
    is_new[i] = false;
    slot[i] = 0;
    h[i] = mix64(key[i]) & mask;
  }
  for (u64 probe = 0; probe <= mask; ++probe) {
    u64 cur[B];
#pragma unroll
    for (int i = 0; i < B; ++i)
      cur[i] = pend[i] ? __hip_atomic_load(&keys[h[i]], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP)
                       : 0;
    bool any = false;
#pragma unroll
    for (int i = 0; i < B; ++i) {
      if (!pend[i]) continue;
      if (cur[i] == kEmptyKey) {
        cur[i] = atomicCAS((unsigned long long *)&keys[h[i]], (unsigned long long)kEmptyKey,
                           (unsigned long long)key[i]);
        if (cur[i] == kEmptyKey) {
          is_new[i] = true;
          slot[i] = (u32)h[i];
          pend[i] = false;
          continue;
        }
      }
      if (cur[i] == key[i]) {
        slot[i] = (u32)h[i];
        pend[i] = false;
        continue;
      }
      h[i] = (h[i] + 1) & mask;
      any = true;
    }
    if (!any) return;
  }
  set_error(err, kErrHashFull);
}

// Visited-set insert of B target pairs (key = r1 << 32 | r2): the hash
// table, or the dense array when a.vn2 != 0 (slot = r1 vn2 + r2; a claim is
// a CAS from kUnvisited to kClaimed, tried only when a plain read of the
// entry still sees kUnvisited -- entries never return to it).  known[i]:
// the pair's id when an earlier level gave it one and the dense array holds
// it, else kUnvisited.
template <int B>
__device__ __forceinline__ void visit_batch(const MergeArgs &a, const u64 (&key)[B],
                                            const bool (&act)[B], u32 (&slot)[B],
                                            bool (&is_new)[B], u32 (&known)[B]) {
  if (!a.vn2) {
    hash_insert_batch<B>(a.hkeys, a.hmask, key, act, slot, is_new, &a.st->err);
#pragma unroll
    for (int i = 0; i < B; ++i) known[i] = kUnvisited;
    return;
  }
  u32 cur[B];
#pragma unroll
  for (int i = 0; i < B; ++i) {
    slot[i] = act[i] ? (u32)(key[i] >> 32) * a.vn2 + (u32)key[i] : 0u;
    is_new[i] = false;
    cur[i] = act[i] ? __hip_atomic_load(&a.vis[slot[i]], __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_WORKGROUP)
                    : 0u;
  }
#pragma unroll
  for (int i = 0; i < B; ++i) {
    known[i] = cur[i] < kClaimed ? cur[i] : kUnvisited;  // ids are below both markers
    if (act[i] && cur[i] == kUnvisited) is_new[i] = atomicCAS(&a.vis[slot[i]], kUnvisited, kClaimed) == kUnvisited;
  }
}

constexpr u32 kNoClaim = 0xffffffffu;  // slots are below 2^31

// New pairs of a workgroup's merged arcs, collected in LDS and appended to the
// level's new-pair list with one device atomic (same-address atomics
// serialise at about 13 ns each).  The list's order is arbitrary: ids are
// given in list order or by rank (launch_assign, launch_rank_assign).
// Counting and listing the claims in two passes over the merged arcs, with a
// scan between, took 180 us a level of 6M arcs and three launches a level.
template <u32 CAP>
struct ClaimLds {
  u32 slot[CAP];
  u32 n, base;
};

template <u32 CAP>
__device__ __forceinline__ void claims_begin(ClaimLds<CAP> &L) {
  if (threadIdx.x == 0) L.n = 0;
  __syncthreads();
}

// Whole waves; the workgroup adds at most CAP claims in all.
template <u32 CAP>
__device__ __forceinline__ void claims_add(ClaimLds<CAP> &L, u32 claim) {
  const u64 m = __ballot(claim != kNoClaim);
  if (!m) return;
  const u32 leader = (u32)__builtin_ctzll(m);
  u32 at = 0;
  if (lane_id() == leader) at = atomicAdd(&L.n, (u32)__popcll(m));
  at = __shfl(at, (int)leader, kWave) + count_below(m);
  if (claim != kNoClaim && at < CAP) L.slot[at] = claim;
}

template <u32 CAP>
__device__ __forceinline__ void claims_end(const MergeArgs &a, ClaimLds<CAP> &L) {
  __syncthreads();
  const u32 n = L.n;
  if (n == 0) return;  // uniform
  if (threadIdx.x == 0) L.base = atomicAdd(&a.st->nnew, n);
  __syncthreads();
  const u64 base = L.base;
  if (n > CAP || base + n > a.newcap) {  // impossible: the capacities bound both
    if (threadIdx.x == 0) set_error(&a.st->err, kErrNewList);
    return;
  }
  for (u32 i = threadIdx.x; i < n; i += blockDim.x) a.newlist[base + i] = L.slot[i];
}

// Target id of a merged arc's record word x: the id itself when it carries
// kIdFlag (dense visited array only: its slots and ids are below 2^30, while
// hash-table slots use bit 30 themselves), else the id the visited set now
// holds at the slot.
__device__ __forceinline__ u32 target_id(const MergeArgs &a, u32 x, const u32 *hvals) {
  return (a.vn2 && (x & kIdFlag)) ? x & ~kIdFlag : hvals[x & ~kNewFlag];
}

// (level_clear_mask names the same fields, for publications that clear them)
__device__ __forceinline__ void clear_level(Status *st) {
  st->R = st->M = st->merged = st->RB = 0;
  st->nwide = st->nheavy = st->nbig = st->nnew = 0;
  st->max_small = 0;
  st->dense_records = st->dense_runs = st->sort_runs = 0;
  st->nprod = st->nprod_mfma = 0;
  st->prod_records = st->prod_entries = 0;
  st->nsort = 0;
  st->ngen = 0;
  st->ngrp = 0;
  st->unfit = 0;
  st->declined = 0;
  st->general = st->chunk_pairs = 0;
  st->nmid = 0;
}

}  // namespace fstc
