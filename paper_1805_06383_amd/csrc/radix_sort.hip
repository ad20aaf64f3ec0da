// Device-wide stable LSD radix sort of (64-bit key, 32-bit value) pairs.
//
// The paper sorts packed 64-bit keys with a library sort-by-key
// (section 3.4, "Reduction").  Here the sort is written for gfx950: digits of
// at most 8 bits, stable in-tile ranking by wave64 ballots (radix_rank.hpp),
// and only the key bits that can differ (the caller passes the bit range).
//   - Up to kOneTile pairs: one workgroup runs every pass in LDS.
//   - More: one kernel counts every pass's digits, then each pass is one
//     kernel (Merrill & Garland, "Single-pass Parallel Prefix Scan with
//     Decoupled Look-back", 2016, applied per digit; Adinets & Merrill,
//     "Onesweep", 2022): a workgroup takes the next tile from a counter,
//     ranks it, publishes its digit counts, and adds up those of the tiles
//     below until one has published its prefix.
// Bound: at the sizes of one level (10^4 to 10^6 pairs) the launches and the
// gaps between them, not the traffic.  A histogram, a scan and a scatter
// launch per pass took 33 us a pass at 150,000 pairs and 42 us at 372,000.
#include "common.hpp"
#include "radix_rank.hpp"

namespace fstc {
namespace {

constexpr int kNT = 256;
constexpr int kMaxPasses = 8;
constexpr int kOneNT = 1024, kOneIT = 8;
constexpr u64 kOneTile = kOneNT * kOneIT;  // 96 KB of LDS
// Tiles of 2,048 pairs up to this many: more workgroups in flight where a
// level's tiles do not fill the chip, 4,096 above: half the look-back words.
constexpr u64 kFineMax = u64(1) << 20;
constexpr int tile_pairs(bool fine) { return kNT * (fine ? 8 : 16); }
inline u64 tiles_of(u64 n) { return ceil_div(n, tile_pairs(n <= kFineMax)); }

// Control words of one sort, zeroed before it: digit counts of every pass,
// the passes' tile counters, then the tiles' published digit counts (pass
// number and kind of count above the count, so a pass's words never match
// another's).
struct Control {
  u32 hist[kMaxPasses * 256];
  u32 ticket[64];
};
constexpr u32 kAgg = 1, kInc = 2;  // the tile's own counts; with all below it
constexpr u32 kSpins = 1u << 20;   // polls before a tile counts the pairs below itself

struct SortArgs {
  const u64 *ki;
  const u32 *vi;
  u64 *ko;
  u32 *vo;
  u64 n;
  int lo, hi, passes;
  Control *ctl;
  u64 *status;  // [tiles][256]
  u32 nb;
  const u32 *unsorted;  // see SortJob
  u32 epoch;
};
struct SortPair {
  SortArgs j[2];
  u32 split;  // workgroups of the first
  int pass;
};

// Bits of pass p: spread evenly (a digit of b bits takes b ballots per row).
__host__ __device__ inline void pass_bits(const SortArgs &a, int p, int &shift, int &bits) {
  const int w = a.hi - a.lo;
  shift = a.lo + w * p / a.passes;
  bits = a.lo + w * (p + 1) / a.passes - shift;
}

// The job is already in order (see SortJob).
__device__ __forceinline__ bool in_order(const SortArgs &a) {
  return a.unsorted && *a.unsorted != a.epoch;
}

__device__ __forceinline__ const SortArgs &sort_job(const SortPair &p, u32 &blk, u32 &grid) {
  if (blockIdx.x < p.split) {
    blk = blockIdx.x;
    grid = p.split;
    return p.j[0];
  }
  blk = blockIdx.x - p.split;
  grid = gridDim.x - p.split;
  return p.j[1];
}

__global__ __launch_bounds__(kNT) void k_radix_zero(SortPair p) {
  u32 blk, grid;
  const SortArgs &a = sort_job(p, blk, grid);
  if (in_order(a)) return;
  const u64 w = sizeof(Control) / 8, n = w + (u64)a.nb * 256;
  u64 *c = reinterpret_cast<u64 *>(a.ctl);
  for (u64 i = (u64)blk * kNT + threadIdx.x; i < n; i += (u64)grid * kNT) {
    if (i < w) c[i] = 0;
    else a.status[i - w] = 0;
  }
}

// Digit counts of every pass, the keys read once.
__global__ __launch_bounds__(kNT) void k_radix_hist(SortPair p) {
  __shared__ u32 h[kMaxPasses * 256];
  u32 blk, grid;
  const SortArgs &a = sort_job(p, blk, grid);
  if (in_order(a)) return;  // uniform
  for (u32 i = threadIdx.x; i < (u32)a.passes * 256; i += kNT) h[i] = 0;
  __syncthreads();
  constexpr int kB = 8;
  for (u64 b = (u64)blk * (kNT * kB); b < a.n; b += (u64)grid * (kNT * kB)) {
    // every load issued before the first is used (indices clamped)
    u64 k[kB];
#pragma unroll
    for (int j = 0; j < kB; ++j) k[j] = a.ki[min<u64>(b + (u64)j * kNT + threadIdx.x, a.n - 1)];
    for (int q = 0; q < a.passes; ++q) {
      int shift, bits;
      pass_bits(a, q, shift, bits);
      const u32 mask = (1u << bits) - 1u;
#pragma unroll
      for (int j = 0; j < kB; ++j)
        if (b + (u64)j * kNT + threadIdx.x < a.n)
          atomicAdd(&h[q * 256 + ((u32)(k[j] >> shift) & mask)], 1u);
    }
  }
  __syncthreads();
  for (u32 i = threadIdx.x; i < (u32)a.passes * 256; i += kNT)
    if (h[i]) atomicAdd(&a.ctl->hist[i], h[i]);
}

// One pass over one tile of kNT x IT pairs.
template <int IT>
__global__ __launch_bounds__(kNT) void k_radix_pass(SortPair p) {
  constexpr int kTile = kNT * IT;
  constexpr u32 kW = 16;  // published counts read together
  __shared__ u32 s_cnt[(kNT / kWave) * 256];
  __shared__ u32 s_base[256], s_off[256];
  __shared__ u32 s_tmp[kNT / kWave];
  __shared__ u32 s_tile;
  u32 blk, grid;
  const SortArgs &a = sort_job(p, blk, grid);
  if (in_order(a)) {  // uniform
    // its data stays where it is: in the last of an odd number of passes it
    // is copied to the output (the result is then copied back from there)
    if (p.pass == a.passes - 1 && (a.passes & 1)) {
      const u64 base = (u64)blk * kTile;
#pragma unroll
      for (int j = 0; j < IT; ++j) {
        const u64 e = base + (u64)j * kNT + threadIdx.x;
        if (e < a.n) {
          a.ko[e] = a.ki[e];
          a.vo[e] = a.vi[e];
        }
      }
    }
    return;
  }
  // tiles in the order the workgroups start: the tiles below are running
  if (threadIdx.x == 0) s_tile = atomicAdd(&a.ctl->ticket[p.pass], 1u);
  const u32 d = threadIdx.x, lane = lane_id(), w = threadIdx.x / kWave;
  const u32 digits = a.ctl->hist[p.pass * 256 + d];
  u32 total;
  const u32 before = block_exclusive_sum<kNT, u32>(digits, s_tmp, &total);  // barriers
  const u32 tile = s_tile;
  if (tile >= a.nb) return;  // impossible: as many tiles as workgroups
  int shift, bits;
  pass_bits(a, p.pass, shift, bits);
  const u32 mask = (1u << bits) - 1u;
  const u64 t0 = (u64)tile * kTile, base = t0 + (u64)w * (kWave * IT);
  u64 key[IT];
  u32 val[IT], dig[IT], rid[IT];
  u32 valid = 0;
#pragma unroll
  for (int j = 0; j < IT; ++j) {
    const u64 e = base + (u64)j * kWave + lane;
    valid |= (e < a.n ? 1u : 0u) << j;
    key[j] = a.ki[min<u64>(e, a.n - 1)];
    val[j] = a.vi[min<u64>(e, a.n - 1)];
  }
#pragma unroll
  for (int j = 0; j < IT; ++j) dig[j] = (u32)(key[j] >> shift) & mask;
  block_rank_digits<kNT, IT>(dig, valid, bits, rid, s_cnt, s_base, s_tmp);
  const u32 mine = (d < 255 ? s_base[d + 1] : (u32)min<u64>(kTile, a.n - t0)) - s_base[d];
  const u32 tag = (u32)(p.pass + 1) << 2;
  auto publish = [&](u32 kind, u32 v) {
    __hip_atomic_store(&a.status[(u64)tile * 256 + d], (u64)(tag | kind) << 32 | v,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  publish(tile == 0 ? kInc : kAgg, mine);
  u32 below = 0;  // pairs of digit d in the tiles below
  bool failed = false;
  {
    u32 t = tile, polls = 0;  // tiles [t, tile) are added
    bool done = t == 0;
    while (!done && !failed) {
      u64 x[kW];
#pragma unroll
      for (u32 k = 0; k < kW; ++k)
        x[k] = __hip_atomic_load(&a.status[(u64)(t > k ? t - 1 - k : 0u) * 256 + d],
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      bool open = true;
      u32 took = 0;
#pragma unroll
      for (u32 k = 0; k < kW; ++k) {
        const u32 kind = (u32)(x[k] >> 32) ^ tag;
        open = open && !done && k < t && (kind == kAgg || kind == kInc);
        if (open) {
          below += (u32)x[k];
          ++took;
          done = kind == kInc;  // (tile 0 publishes no other)
        }
      }
      t -= took;
      if (!done && took == 0) {
        __builtin_amdgcn_s_sleep(1);
        failed = ++polls > kSpins;
      }
    }
  }
  if (__syncthreads_or(failed ? 1 : 0)) {
    // the pairs below counted again (a workgroup below was held for long)
    s_off[d] = 0;
    __syncthreads();
    for (u64 e = d; e < t0; e += kNT) atomicAdd(&s_off[(u32)(a.ki[e] >> shift) & mask], 1u);
    __syncthreads();
    below = s_off[d];
    __syncthreads();
  }
  if (tile) publish(kInc, below + mine);
  s_off[d] = before + below;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < IT; ++j) {
    if (!((valid >> j) & 1u)) continue;
    const u64 pos = (u64)s_off[dig[j]] + rid[j];
    a.ko[pos] = key[j];
    a.vo[pos] = val[j];
  }
}

// Every pass of a job of at most kOneTile pairs, workgroup i for job i; the
// result replaces the input.
__global__ __launch_bounds__(kOneNT) void k_radix_one(SortPair p) {
  __shared__ u64 s_key[kOneTile];
  __shared__ u32 s_val[kOneTile];
  __shared__ u32 s_cnt[(kOneNT / kWave) * 256];
  __shared__ u32 s_base[256];
  __shared__ u32 s_tmp[kOneNT / kWave];
  const SortArgs &a = p.j[blockIdx.x];
  if (in_order(a)) return;  // uniform
  const u32 lane = lane_id(), w = threadIdx.x / kWave, n = (u32)a.n;
  u64 key[kOneIT];
  u32 val[kOneIT], dig[kOneIT], rid[kOneIT];
  u32 valid = 0;
#pragma unroll
  for (int j = 0; j < kOneIT; ++j) {
    const u32 e = w * (kWave * kOneIT) + j * kWave + lane;
    valid |= (e < n ? 1u : 0u) << j;
    key[j] = a.ki[min(e, n - 1)];
    val[j] = a.vi[min(e, n - 1)];
  }
  for (int q = 0; q < a.passes; ++q) {
    int shift, bits;
    pass_bits(a, q, shift, bits);
    const u32 mask = (1u << bits) - 1u;
#pragma unroll
    for (int j = 0; j < kOneIT; ++j) dig[j] = (u32)(key[j] >> shift) & mask;
    block_rank_digits<kOneNT, kOneIT>(dig, valid, bits, rid, s_cnt, s_base, s_tmp);
#pragma unroll
    for (int j = 0; j < kOneIT; ++j) {
      if (!((valid >> j) & 1u)) continue;
      const u32 pos = s_base[dig[j]] + rid[j];
      s_key[pos] = key[j];
      s_val[pos] = val[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kOneIT; ++j) {
      const u32 e = w * (kWave * kOneIT) + j * kWave + lane;
      key[j] = s_key[min(e, n - 1)];
      val[j] = s_val[min(e, n - 1)];
    }
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < kOneIT; ++j) {
    const u32 e = w * (kWave * kOneIT) + j * kWave + lane;
    if (!((valid >> j) & 1u)) continue;
    a.ko[e] = key[j];
    a.vo[e] = val[j];
  }
}

}  // namespace

size_t radix_temp_bytes(u64 n) { return sizeof(Control) + tiles_of(std::max<u64>(n, 1)) * 256 * 8 + 256; }

void radix_sort_pairs(u64 *keys, u32 *vals, u64 *keys_alt, u32 *vals_alt, u64 n, int lo, int hi,
                      void *temp, hipStream_t s) {
  const SortJob j{keys, keys_alt, vals, vals_alt, n, lo, hi, temp};
  radix_sort_pairs_batch(&j, 1, s);
}

void radix_sort_pairs_batch(const SortJob *jobs, int nj, hipStream_t s) {
  if (nj < 1 || nj > 2) throw Error(FSTC_ERR_INTERNAL, "radix_sort_pairs_batch takes one or two jobs");
  SortPair one{}, many{};
  int n1 = 0, nm = 0, who[2] = {0, 0};
  bool fine = true;
  for (int i = 0; i < nj; ++i) {
    const SortJob &J = jobs[i];
    if (J.n <= 1 || J.hi <= J.lo) continue;
    const u64 nb = tiles_of(J.n);
    // (digit counts and tile offsets are 32-bit)
    if (J.n >= (1ull << 32)) throw Error(FSTC_ERR_CAPACITY, "sort of 2^32 pairs or more");
    SortArgs a{};
    a.ki = J.keys;
    a.vi = J.vals;
    a.n = J.n;
    a.lo = J.lo;
    a.hi = J.hi;
    a.passes = (J.hi - J.lo + 7) / 8;
    a.unsorted = J.unsorted;
    a.epoch = J.epoch;
    if (J.n <= kOneTile) {
      a.ko = J.keys;
      a.vo = J.vals;
      one.j[n1++] = a;
      continue;
    }
    a.ko = J.keys_alt;
    a.vo = J.vals_alt;
    a.ctl = reinterpret_cast<Control *>(((uintptr_t)J.temp + 255) & ~(uintptr_t)255);
    a.status = reinterpret_cast<u64 *>(a.ctl + 1);
    a.nb = (u32)nb;
    fine = fine && J.n <= kFineMax;
    who[nm] = i;
    many.j[nm++] = a;
  }
  if (n1) hipLaunchKernelGGL(k_radix_one, dim3(n1), dim3(kOneNT), 0, s, one);
  if (!nm) return;
  // (both by the larger tiles when one job needs them)
  for (int i = 0; i < nm; ++i) many.j[i].nb = (u32)ceil_div(many.j[i].n, tile_pairs(fine));
  auto grid = [&](auto blocks) {
    many.split = blocks(many.j[0]);
    return dim3(many.split + (nm > 1 ? blocks(many.j[1]) : 0u));
  };
  const dim3 gz = grid([](const SortArgs &a) { return std::min<u32>(a.nb, 256u); });
  hipLaunchKernelGGL(k_radix_zero, gz, dim3(kNT), 0, s, many);
  // (a workgroup adds its counts to the same 256 words per pass as the others)
  hipLaunchKernelGGL(k_radix_hist, gz, dim3(kNT), 0, s, many);
  const int most = std::max(many.j[0].passes, nm > 1 ? many.j[1].passes : 0);
  for (int q = 0; q < most; ++q) {
    SortPair p = many;
    int na = 0;
    for (int i = 0; i < nm; ++i)
      if (q < many.j[i].passes) p.j[na++] = many.j[i];
    p.pass = q;
    p.split = p.j[0].nb;
    const dim3 g(p.split + (na > 1 ? p.j[1].nb : 0u));
    if (fine) hipLaunchKernelGGL(k_radix_pass<8>, g, dim3(kNT), 0, s, p);
    else hipLaunchKernelGGL(k_radix_pass<16>, g, dim3(kNT), 0, s, p);
    for (int i = 0; i < nm; ++i) {
      SortArgs &a = many.j[i];
      if (q >= a.passes) continue;
      u64 *k = const_cast<u64 *>(a.ki);
      u32 *v = const_cast<u32 *>(a.vi);
      a.ki = a.ko;
      a.vi = a.vo;
      a.ko = k;
      a.vo = v;
    }
  }
  for (int i = 0; i < nm; ++i) {
    const SortJob &J = jobs[who[i]];
    if (many.j[i].ki == J.keys) continue;
    FSTC_HIP(hipMemcpyAsync(J.keys, many.j[i].ki, J.n * sizeof(u64), hipMemcpyDeviceToDevice, s));
    FSTC_HIP(hipMemcpyAsync(J.vals, many.j[i].vi, J.n * sizeof(u32), hipMemcpyDeviceToDevice, s));
  }
}

}  // namespace fstc
