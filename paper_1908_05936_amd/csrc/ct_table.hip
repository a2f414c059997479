// ct_table.hip -- gfx950 kernels and the C ABI of the batch hash containers and index pool.
//
// Operation pipelines (every kernel on the caller's stream, in this order):
//   find             : k_find                                  one launch, read-only, lock-free
//   2048 keys or less: k_small                                 the whole insert or erase in one launch
//   speculative      : k_insert_spec or k_erase_spec -> k_spec_clear -> k_spec_build ->
//   insert, erase      k_spec_probe -> k_spec_swap
//   large insert of  : k_part_coarse -> (k_part_fine -> k_part_insert) per group -> k_part_left ->
//   several keys per   k_part_over -> the resolution as above
//   bucket
//   resolve-first    : k_prologue -> k_dedup -> k_insert [-> k_final -> k_fix where FULL can be met]
//   insert
//   insert_alloc     : k_prologue -> k_dedup -> k_insert -> k_final -> k_fix
//   erase            : k_prologue -> k_dedup -> k_erase
//   erase_release    : k_prologue -> k_dedup -> k_erase -> k_final
// Chunks of 2^16 keys or more resolve repeated keys with k_bin_* in the place of k_dedup; grids that do
// not settle their counters themselves are followed by k_apply_count, and large ranked chunks by
// k_tile_count and k_tile_scan.
//
// Index-order semantics, resolve-first.  k_dedup records, per distinct key of the chunk, the lowest
// chunk index holding it (an atomic min in a cache-resident scratch table).  Only that element (the
// "actor") touches the table; later copies are resolved from its outcome, which gives exactly the
// results of a sequential replay.  Distinct actors never race on one key, so a claim CAS can only
// fail because another key took the slot.  When a chunk might reach capacity or empty the pool, or
// when values come from a pool, the new actors are ranked by an exclusive scan in index order and
// k_final hands out capacity and pool entries by rank, so the k-th new key of the chunk is the k-th
// to be stored, as in the sequential replay.
#include <hip/hip_cooperative_groups.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "ct.h"
#include "ct_device.h"
#include "ct_dev_api.h"
#include "ct_probe.h"

using namespace ct;

namespace {

// ---------------------------------------------------------------------------------------------
// value I/O by value kind (0 none, 1 u32, 2 u64); table slots always hold 64-bit values
// ---------------------------------------------------------------------------------------------
template <int VK>
__device__ __forceinline__ uint64_t load_val(const void* vals, int64_t i) {
  if constexpr (VK == 1) return (uint64_t)static_cast<const uint32_t*>(vals)[i];
  else if constexpr (VK == 2) return static_cast<const uint64_t*>(vals)[i];
  else return 0;
}
template <int VK>
__device__ __forceinline__ void store_val(void* out, int64_t i, uint64_t v) {
  if constexpr (VK == 1) static_cast<uint32_t*>(out)[i] = (uint32_t)v;
  else if constexpr (VK == 2) static_cast<uint64_t*>(out)[i] = v;
}
template <int VK>
__device__ __forceinline__ uint64_t sentinel() {
  return VK == 1 ? 0xFFFFFFFFull : ~0ull;
}

// Per lane: lowest chunk index of a key that k_dedup marked as repeated.  The entry is always
// there; the scan is bounded anyway, and a miss makes the element act for itself and raises
// kErrInternal.
__device__ __forceinline__ uint32_t dedup_lookup(const TableView& t, const uint64_t* keys,
                                                 uint64_t key, uint32_t dmask, uint32_t self) {
  const uint64_t mix = dedup_mix(key);
  const uint64_t tag = mix & 0xFFFFFFFF00000000ull;
  uint32_t h = (uint32_t)mix & dmask;
  for (uint32_t step = 0; step <= dmask; ++step) {
    const uint64_t e = t.dd[h];
    if (e == kEmpty) break;
    if ((e & 0xFFFFFFFF00000000ull) == tag && keys[(uint32_t)e] == key) return (uint32_t)e;
    h = (h + 1) & dmask;
  }
  aor32(&t.hdr->err, kErrInternal);
  return self;
}

// ---------------------------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------------------------
// The words that batches count into (spec_count, settle_count).  Every batch relies on them being zero
// when it starts and leaves them so; initialisation, clear, and the first batch after one that
// failed, which may have left its counts, zero them.  One block.
__device__ __forceinline__ void zero_counts(const TableView& t) {
  if (threadIdx.x < kCountStripes) t.stripes[threadIdx.x * kCountStride] = 0;
  if (threadIdx.x == kCountStripes) t.stripes[kSettleWord] = 0;
}

// Empty every slot in [lo, hi) (thread-strided by `step`); `header` also resets the counters.
// Slots are written as 16-byte words, U per thread and round (the stores of a round issue
// back to back; a round that would pass `hi` takes a bounds test per word).
__device__ __forceinline__ void reset_range(const TableView& t, int64_t lo, int64_t hi,
                                            int64_t step, bool header, int zero_err) {
  constexpr int U = 4;
  const uint4 empty = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0u, 0u);
  uint4* slots = reinterpret_cast<uint4*>(t.bk);
  int64_t j = lo * U + threadIdx.x;
  const int64_t span = step * U;
  const int64_t width = blockDim.x;
  for (; j + (U - 1) * width < hi; j += span) {
#pragma unroll
    for (int u = 0; u < U; ++u) slots[j + u * width] = empty;
  }
  for (int u = 0; u < U; ++u)
    if (j + u * width < hi) slots[j + u * width] = empty;
  if (header) zero_counts(t);
  if (header && threadIdx.x == 0) {
    Header* h = t.hdr;
    h->size = 0;
    h->size0 = 0;
    h->spec_val[0] = h->spec_val[1] = 0;
    h->spec_live[0] = h->spec_live[1] = 0;
    h->spec_first[0] = h->spec_first[1] = kNone;
    if (zero_err) {
      h->err = 0;
      h->inject = 0;
    }
    // an empty table starts a fresh history: its next insert and erase chunks speculate
    h->fbd[0] = h->fbd[1] = 0;
    if (t.fb) {
      __hip_atomic_store(t.fb, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      __hip_atomic_store(t.fb + 1, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    h->fast = 0;
    h->spec = 0;
    h->ndup = 0;
    h->nnew = 0;
    h->dump_count = 0;
    h->live_count = 0;
    h->violations = 0;
    h->dagg = 0;
    h->dskew = 0;
    h->dskew_age = 0;
  }
}

__global__ __launch_bounds__(kBlock) void k_table_reset(TableView t, int zero_header) {
  reset_range(t, (int64_t)blockIdx.x * blockDim.x, (int64_t)t.nb * kSlots,
              (int64_t)gridDim.x * blockDim.x, blockIdx.x == 0, zero_header);
}

__global__ __launch_bounds__(64) void k_zero_counts(TableView t) { zero_counts(t); }

// Per chunk: clear the dedup scratch, snapshot the counters, decide whether the chunk can reach
// capacity (or empty the pool).
// Units [lo, hi) of a chunk's scratch clear: the first dslots/2 units are 16-byte dedup-entry
// pairs, the rest 16-byte groups of repeated-key marks.  `header`: snapshot the counters and
// decide whether the chunk can reach capacity (or empty the pool).
__device__ __forceinline__ int64_t prologue_units(uint32_t dslots, int64_t q) {
  return (int64_t)dslots / 2 + (q + 15) / 16;
}

// Per-chunk counters: snapshot size (and pool top), reset the chunk's lists, decide whether the
// chunk can reach capacity (or empty the pool), and record how repeated keys are resolved.
__device__ __forceinline__ void chunk_header(const TableView& t, PoolHeader* pool, int64_t q,
                                             uint32_t dmode) {
  Header* h = t.hdr;
  h->size0 = h->size;
  h->spec_first[0] = h->spec_first[1] = kNone;
  h->ndup = 0;
  h->nnew = 0;
  bool fast = h->size + (uint64_t)q <= t.cap;
  if (pool) {
    pool->top0 = pool->top;
    fast = fast && pool->top >= q;
  }
  h->fast = fast ? 1u : 0u;
  h->spec = 0u;
  h->dmode = dmode;
  h->dovf = 0;
  // binned chunks of a table whose keys recently overflowed the bins fold each tile's repeated
  // keys before scattering; every 16th such chunk tries without, and ends the hint if it fits
  uint32_t agg = 0;
  if (dmode && h->dskew) agg = (++h->dskew_age & 15u) != 0u ? 1u : 0u;
  h->dagg = agg;
}

__device__ __forceinline__ void prologue_range(const TableView& t, PoolHeader* pool,
                                               uint32_t dslots, int64_t q, int64_t lo, int64_t hi,
                                               int64_t step, bool header) {
  const uint4 empty = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
  const int64_t nd = (int64_t)dslots / 2;
  for (int64_t j = lo + threadIdx.x; j < hi; j += step) {
    if (j < nd) reinterpret_cast<uint4*>(t.dd)[j] = empty;
    else reinterpret_cast<uint4*>(t.dmark)[j - nd] = make_uint4(0, 0, 0, 0);
  }
  if (header && threadIdx.x == 0) chunk_header(t, pool, q, 0u);
}

// A chunk with a pool, or a small one that may meet FULL: its insert or erase kernel adds to the tile
// sums.
__device__ __forceinline__ void zero_tile_sums(const TableView& t, int64_t q) {
  for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < (q + kTile - 1) / kTile;
       j += (int64_t)gridDim.x * kBlock)
    t.tsum[j] = 0;
}

__global__ __launch_bounds__(kBlock) void k_prologue(TableView t, PoolHeader* pool,
                                                     uint32_t dslots, int64_t q, int ranked) {
  if (ranked) zero_tile_sums(t, q);
  prologue_range(t, pool, dslots, q, (int64_t)blockIdx.x * blockDim.x, prologue_units(dslots, q),
                 (int64_t)gridDim.x * blockDim.x, blockIdx.x == 0);
}

// Lowest index per distinct key of the chunk.  The block takes 256 consecutive elements at a time
// and first resolves them among themselves in LDS: every element of a key repeated inside the
// window is marked, and only the window's lowest copy of each key (its representative) goes on
// to the chunk-wide table dd.  There the first representative to arrive claims an empty entry
// with one CAS; a later one marks itself and the holder, and lowers the entry's index with an
// atomic min when its own index is lower (the index only decreases, so a representative above
// the index it reads cannot lower it).  Every element of a key that occurs more than once ends
// up marked, unique keys stay unmarked, and the entry ends at the key's lowest index.  All
// indices held by one entry belong to one key, so the fingerprint plus one look at that
// element's key identifies the entry exactly.  A key repeated many times therefore costs one
// global operation per window, not per copy.  Needs blockDim.x == kBlock.  Bound by latency at the
// sizes that come here: keys and skip bytes are asked for before the LDS table is cleared, and the
// entries of dd before the window is resolved (2^15 keys 9.8 us without that, 8.4 with).
// `skip` (nullable): elements with a nonzero byte there take no part (a masked insert).
__device__ __forceinline__ void dedup_range(const TableView& t, const uint64_t* __restrict__ keys,
                                            const uint8_t* __restrict__ skip, uint32_t dmask,
                                            int64_t lo, int64_t hi, int64_t step) {
  constexpr uint32_t kW = 2 * kBlock;  // LDS slots of a window's table
  __shared__ unsigned long long wk[kW];
  __shared__ uint32_t wmin[kW], wcnt[kW];
  for (int64_t b0 = lo; b0 < hi; b0 += step) {  // uniform trip count: barriers below
    const int64_t i = b0 + threadIdx.x;
    const uint64_t key = keys[min(i, hi - 1)];
    const uint8_t out = skip ? skip[min(i, hi - 1)] : 0;
    for (uint32_t j = threadIdx.x; j < kW; j += kBlock) {
      wk[j] = kEmpty;
      wmin[j] = kNone;
      wcnt[j] = 0;
    }
    __syncthreads();
    const bool valid = i < hi && !out;
    const bool normal = valid && key < kTomb;
    if (valid && !normal) amin32(&t.hdr->spec_first[key - kTomb], (uint32_t)i);
    const uint64_t mix = dedup_mix(key);
    uint32_t s = (uint32_t)(mix >> 32) & (kW - 1);
    uint32_t h = (uint32_t)mix & dmask;
    uint64_t e = normal ? t.dd[h] : 0;
    if (normal) {
      for (;;) {  // at most kBlock keys in kW slots: a free or matching slot exists
        const unsigned long long old = atomicCAS(&wk[s], (unsigned long long)kEmpty,
                                                 (unsigned long long)key);
        if (old == kEmpty || old == key) break;
        s = (s + 1) & (kW - 1);
      }
      atomicMin(&wmin[s], (uint32_t)i);
      atomicAdd(&wcnt[s], 1u);
    }
    __syncthreads();
    if (normal) {
      if (wcnt[s] > 1) t.dmark[i] = 1;
      if (wmin[s] == (uint32_t)i) {  // the window's representative of this key
        const uint64_t tag = mix & 0xFFFFFFFF00000000ull;
        const uint64_t mine = tag | (uint64_t)i;
        for (uint32_t probe = 0; probe <= dmask; ++probe) {
          if (e == kEmpty) {
            uint64_t expected = kEmpty;
            if (cas64(&t.dd[h], expected, mine)) break;
            e = expected;
          }
          if ((e & 0xFFFFFFFF00000000ull) == tag && keys[(uint32_t)e] == key) {
            const uint32_t held = (uint32_t)e;
            uint32_t prev = held;
            if ((uint32_t)i < held) prev = (uint32_t)amin64(&t.dd[h], mine);
            t.dmark[i] = 1;
            if (!t.dmark[prev]) t.dmark[prev] = 1;
            break;
          }
          h = (h + 1) & dmask;
          e = t.dd[h];
        }
      }
    }
    __syncthreads();  // the window's LDS table is reused by the next window
  }
}

__global__ __launch_bounds__(kBlock) void k_dedup(TableView t, const uint64_t* __restrict__ keys,
                                                  const uint8_t* __restrict__ skip, int64_t q,
                                                  uint32_t dmask) {
  dedup_range(t, keys, skip, dmask, (int64_t)blockIdx.x * kBlock, q, (int64_t)gridDim.x * kBlock);
}

// ---------------------------------------------------------------------------------------------
// Binned dedup: what dedup_range finds, as each repeated element's first occurrence in dfirst (kNone
// for an element that is not repeated), without a device-scope atomic per element.  Keys move into 64 coarse bins and then into P fine bins by the high bits
// of dedup_mix, so all copies of a key share a fine bin; each fine bin (about 1024 elements)
// finds its repeated keys in an LDS hash table.  The only global atomics reserve room in a bin,
// one per block and non-empty bin.  A bin that would overflow its capacity sets dovf; the chunk
// then clears dd and runs dedup_range instead, so results never depend on the key distribution.
// ---------------------------------------------------------------------------------------------
// Exclusive block-wide scan of one value per thread (kBlock threads); returns the prefix and
// writes the block total to *total.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* total) {
  __shared__ uint32_t wsum[kBlock / 64];
  const int lane = wave_lane();
  uint32_t x = v;
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  if (lane == 63) wsum[threadIdx.x >> 6] = x;
  __syncthreads();
  uint32_t before = 0, all = 0;
  for (int w = 0; w < kBlock / 64; ++w) {
    if (w < (int)(threadIdx.x >> 6)) before += wsum[w];
    all += wsum[w];
  }
  *total = all;
  __syncthreads();
  return before + x - v;
}

// The chunk's overflow flag and one fill count, read once for the whole block.  Other blocks of
// the same launch may raise the flag while this block starts, so a per-wave read could let some
// waves of a block leave and others stay; the staying waves would then meet the block's barriers
// and scans without the leavers' contributions (the scan words those waves never wrote hold stale
// LDS contents).  One reader and a barrier make the decision uniform across the block.
__device__ __forceinline__ bool block_overflowed(const TableView& t, const uint32_t* count,
                                                 uint32_t* fill) {
  __shared__ uint32_t flag_and_fill[2];
  if (threadIdx.x == 0) {
    const uint32_t o = t.hdr->dovf;
    const uint32_t f = *count;
    flag_and_fill[0] = o;
    flag_and_fill[1] = f;
  }
  __syncthreads();
  *fill = flag_and_fill[1];
  return flag_and_fill[0] != 0;
}

__device__ __forceinline__ uint32_t fine_bin(const TableView& t, uint64_t mix) {
  return (uint32_t)(mix >> (64 - t.lp));
}

// Units [lo, hi) of a binned chunk's prologue: the marks (16 per unit), then the bin counts
// (4 per unit); `header` also takes the chunk's counter snapshot.
__device__ __forceinline__ int64_t bin_prologue_units(const TableView& t, int64_t q) {
  return (q + 15) / 16 + ((int64_t)kCoarseCtrWords + ((int64_t)1 << t.lp)) / 4;
}

// The kernels of the path that resolves repeated keys first leave at once when the chunk went the
// speculative way (decided on the device, k_spec_decide); `decided`: the flag is this chunk's.
__global__ __launch_bounds__(kBlock) void k_bin_prologue(TableView t, PoolHeader* pool, int64_t q,
                                                         int ranked, int decided) {
  if (decided && t.hdr->spec) return;
  if (ranked) zero_tile_sums(t, q);
  const int64_t nm = (q + 15) / 16;
  const int64_t hi = bin_prologue_units(t, q);
  const uint4 zero = make_uint4(0, 0, 0, 0);
  for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < hi; j += (int64_t)gridDim.x * kBlock) {
    if (j < nm) reinterpret_cast<uint4*>(t.dmark)[j] = zero;
    else reinterpret_cast<uint4*>(t.bcur)[j - nm] = zero;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) chunk_header(t, pool, q, 1u);
}

// Both scatters: the block's elements, ranked within their bin (code = rank << 8 | bin, or ~0 for
// none), are staged in LDS in bin order and each bin's run is written by consecutive threads, so
// the stores of a wave go to consecutive positions of one bin.  cnt[b] holds the block's count
// for bin b; this reserves the runs (bin b's fill count at bcur[cur0 + b * cur_stride]), flags an
// overflow of `cap`, and writes bin b of the block to out[(gbin0 + b * gstride) * cap + position].
struct BinStage {
  uint64_t k[kBinTile];
  uint32_t i[kBinTile];
  uint8_t b[kBinTile];
  uint32_t cnt[kMaxFinePerCoarse];
  uint32_t base[kMaxFinePerCoarse];
  uint32_t loc[kMaxFinePerCoarse];
};

template <int PER>
__device__ __forceinline__ void bin_write(const TableView& t, BinStage& S, uint32_t nbins,
                                          const uint64_t (&k)[PER], const uint32_t (&ix)[PER],
                                          const uint32_t (&code)[PER], uint32_t cur0,
                                          uint32_t cur_stride, uint32_t gbin0, uint32_t gstride,
                                          uint32_t cap, uint64_t* __restrict__ outk,
                                          uint32_t* __restrict__ outi) {
  const uint32_t c = threadIdx.x < nbins ? S.cnt[threadIdx.x] : 0u;
  uint32_t total;
  const uint32_t pre = block_exclusive_scan(c, &total);
  if (threadIdx.x < nbins) {
    uint32_t o = 0;
    if (c) {
      o = aadd32(&t.bcur[cur0 + threadIdx.x * cur_stride], c);
      if (o + c > cap) t.hdr->dovf = 1u;
    }
    S.base[threadIdx.x] = o;
    S.loc[threadIdx.x] = pre;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    if (code[e] == ~0u) continue;
    const uint32_t b = code[e] & 0xFFu;
    const uint32_t p = S.loc[b] + (code[e] >> 8);
    S.k[p] = k[e];
    S.i[p] = ix[e];
    S.b[p] = (uint8_t)b;
  }
  __syncthreads();
  // a block stages at most kBinTile elements; the bound also keeps p from wrapping
  const uint32_t staged = min(total, (uint32_t)kBinTile);
  for (uint32_t p = threadIdx.x; p < staged; p += kBlock) {
    const uint32_t b = S.b[p];
    const uint32_t pos = S.base[b] + (p - S.loc[b]);
    if (pos < cap) {
      const int64_t at = (int64_t)(gbin0 + b * gstride) * cap + pos;
      outk[at] = S.k[p];
      outi[at] = S.i[p];
    }
  }
}

// Coarse scatter: block b takes elements [b * kBinTile, (b + 1) * kBinTile) into segment
// b mod kBinSub of the 64 coarse bins.  The out-of-band keys take their lowest index directly, as
// in dedup_range.
// When the chunk folds (dagg: its table's recent chunks overflowed the bins, i.e. skewed keys),
// the tile first finds its own repeated keys in an LDS table.  Only each key's first copy in the
// tile goes to the bins; when the tile holds other copies it is marked with dfirst = itself (the
// fine bins replace that if an earlier tile holds the key), and every other copy is marked with
// dfirst = kIndirect | that first copy.  A key repeated thousands of times then reaches its fine
// bin once per tile instead of once per copy.  A copy that finds no slot within kFoldProbe probes
// simply goes to the bins unfolded: the fine bins resolve whatever reaches them exactly.
constexpr int kFoldProbe = 32;

__global__ __launch_bounds__(kBlock) void k_bin_scatter1(TableView t, const uint64_t* __restrict__ keys,
                                                         int64_t q) {
  if (t.hdr->spec) return;
  constexpr int kPer = kBinTile / kBlock;
  constexpr uint32_t kFolded = ~0u - 1u;  // hs entry of a copy that stays out of the bins
  __shared__ BinStage S;
  const int64_t t0 = (int64_t)blockIdx.x * kBinTile;
  uint64_t k[kPer];
  uint32_t ix[kPer], code[kPer], hs[kPer], first[kPer];
  // all loads first, from clamped (in-bounds) positions: a load under a branch would make the
  // compiler wait for it before the next one is issued.  The chunk's mode comes with them.
#pragma unroll
  for (int e = 0; e < kPer; ++e) k[e] = keys[min(t0 + e * kBlock + (int64_t)threadIdx.x, q - 1)];
  const uint32_t agg = t.hdr->dagg;
  if (threadIdx.x < kBinCoarse) S.cnt[threadIdx.x] = 0;
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    hs[e] = ~0u;
    first[e] = kNone;  // not repeated, as far as the tile knows
  }
  if (agg) {
    // H[s] (in S.i): tile position of a copy of slot s's key, the lowest once all have arrived;
    // D[s] (in S.b): the key occurs more than once in the tile.  S.k holds the tile's keys by
    // position.  All three are free until the bins are written.
    uint32_t* H = S.i;
    uint8_t* D = S.b;
    for (uint32_t j = threadIdx.x; j < (uint32_t)kBinTile; j += kBlock) {
      H[j] = ~0u;
      D[j] = 0;
    }
#pragma unroll
    for (int e = 0; e < kPer; ++e) S.k[e * kBlock + threadIdx.x] = k[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      const uint32_t local = e * kBlock + threadIdx.x;
      if (t0 + local < q && k[e] < kTomb) {
        uint32_t s = (uint32_t)dedup_mix(k[e]) & (kBinTile - 1u);
        for (int probe = 0; probe < kFoldProbe; ++probe) {
          const uint32_t prev = atomicCAS(&H[s], ~0u, local);
          if (prev == ~0u) {
            hs[e] = s;
            break;
          }
          if (S.k[prev] == k[e]) {
            atomicMin(&H[s], local);
            D[s] = 1;
            hs[e] = s;
            break;
          }
          s = (s + 1u) & (kBinTile - 1u);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      if (hs[e] == ~0u || !D[hs[e]]) continue;
      const uint32_t local = e * kBlock + threadIdx.x;
      const uint32_t i = (uint32_t)(t0 + local);
      const uint32_t rep = H[hs[e]];
      if (rep == local) {
        first[e] = i;
      } else {
        first[e] = kIndirect | (uint32_t)(t0 + rep);
        hs[e] = kFolded;
      }
    }
  }
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int64_t i = t0 + e * kBlock + threadIdx.x;
    if (i < q) t.dfirst[i] = first[e];
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int64_t i = t0 + e * kBlock + threadIdx.x;
    code[e] = ~0u;
    ix[e] = (uint32_t)i;
    if (i < q) {
      if (k[e] >= kTomb) {
        amin32(&t.hdr->spec_first[k[e] - kTomb], (uint32_t)i);
      } else if (hs[e] != kFolded) {
        const uint32_t b = (uint32_t)(dedup_mix(k[e]) >> (64 - t.lp1));
        code[e] = (atomicAdd(&S.cnt[b], 1u) << 8) | b;
      }
    }
  }
  __syncthreads();
  const uint32_t seg = blockIdx.x % kBinSub;
  bin_write<kPer>(t, S, kBinCoarse, k, ix, code, seg * kCtrStride, kBinSub * kCtrStride, seg,
                  kBinSub, t.c1, t.r1k, t.r1i);
}

// Fine scatter: the blocks of segment g of coarse bin c = g / kBinSub take its tiles in turn
// (tile r, r + blocks_per_seg, ...) and move each into the 2^(lp - lp1) fine bins of c, the same
// way.
__global__ __launch_bounds__(kBlock) void k_bin_scatter2(TableView t, int blocks_per_seg) {
  if (t.hdr->spec) return;
  constexpr int kPer = kBinTile / kBlock;
  __shared__ BinStage S;
  const int g = (int)blockIdx.x / blocks_per_seg;
  const int c = g / kBinSub;
  uint32_t fill;
  if (block_overflowed(t, &t.bcur[g * kCtrStride], &fill)) return;
  const uint32_t n1 = min(fill, t.c1);
  const int lp2 = t.lp - t.lp1;
  const uint32_t p2 = 1u << lp2;
  const int64_t src = (int64_t)g * t.c1;
  for (uint32_t j0 = (uint32_t)((int)blockIdx.x % blocks_per_seg) * kBinTile; j0 < n1;
       j0 += (uint32_t)blocks_per_seg * kBinTile) {
    uint64_t k[kPer];
    uint32_t ix[kPer], code[kPer];
#pragma unroll
    for (int e = 0; e < kPer; ++e) {   // loads first, clamped (n1 > j0 >= 0)
      const uint32_t j = min(j0 + e * kBlock + threadIdx.x, n1 - 1u);
      k[e] = t.r1k[src + j];
      ix[e] = t.r1i[src + j];
    }
    // (the previous tile's writes read S.k, S.i, S.b, S.base and S.loc only: cnt is free)
    for (uint32_t j = threadIdx.x; j < p2; j += kBlock) S.cnt[j] = 0;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      const uint32_t j = j0 + e * kBlock + threadIdx.x;
      code[e] = ~0u;
      if (j < n1) {
        const uint32_t f2 = fine_bin(t, dedup_mix(k[e])) & (p2 - 1u);
        code[e] = (atomicAdd(&S.cnt[f2], 1u) << 8) | f2;
      }
    }
    __syncthreads();
    bin_write<kPer>(t, S, p2, k, ix, code, kCoarseCtrWords + ((uint32_t)c << lp2), 1u,
                    (uint32_t)c << lp2, 1u, t.c2, t.r2k, t.r2i);
  }
}

// One fine bin per block: insert its keys into an LDS table (CAS on the key word, atomic min on
// the index, a flag when a key arrives again), then mark every element of a repeated key and
// give it the key's lowest index.  A bin holds up to c2 entries but the table has kBinLds slots:
// it needs fewer distinct keys than slots, which the bins of folded (skewed) chunks meet by far.
// A bin with more distinct keys (no probe finds a free or matching slot) flags an overflow, and
// the chunk takes the exact fallback.  Bound by its scattered stores, one per repeated element: with
// a mark beside each first occurrence, 4 M repeated keys into a set took 380 us, now 337.
__global__ __launch_bounds__(kBlock) void k_bin_dedup(TableView t) {
  if (t.hdr->spec) return;
  __shared__ unsigned long long hk[kBinLds];
  __shared__ uint32_t hm[kBinLds];
  __shared__ uint8_t hx[kBinLds];
  const uint32_t f = blockIdx.x;
  uint32_t fill;
  if (block_overflowed(t, &t.bcur[kCoarseCtrWords + f], &fill)) return;
  const uint32_t n = min(fill, t.c2);
  if (n == 0) return;
  const uint64_t* rk = t.r2k + (int64_t)f * t.c2;
  const uint32_t* ri = t.r2i + (int64_t)f * t.c2;
  // a bin holds at most c2 <= kPer * kBlock elements: each thread keeps its own in registers.
  // The loads are issued first, from clamped positions, and overlap the table's initialisation.
  // The first kPer0 rows cover any bin of uniform keys (1.75 x the mean); the rest are loaded
  // only when the fill reaches them (a uniform test).
  constexpr int kPer = (kBinFineCap + kBlock - 1) / kBlock;
  constexpr int kPer0 = 7;
  uint64_t kk[kPer];
  uint32_t slot[kPer], idx[kPer];
#pragma unroll
  for (int e = 0; e < kPer0; ++e) {
    const uint32_t j = min(threadIdx.x + e * kBlock, n - 1u);
    kk[e] = rk[j];
    idx[e] = ri[j];
  }
#pragma unroll
  for (int e = kPer0; e < kPer; ++e) {
    kk[e] = kEmpty;
    idx[e] = 0;
  }
  if (n > (uint32_t)(kPer0 * kBlock)) {
#pragma unroll
    for (int e = kPer0; e < kPer; ++e) {
      const uint32_t j = min(threadIdx.x + e * kBlock, n - 1u);
      kk[e] = rk[j];
      idx[e] = ri[j];
    }
  }
  for (uint32_t j = threadIdx.x; j < (uint32_t)kBinLds; j += kBlock) {
    hk[j] = kEmpty;
    hm[j] = kNone;
    hx[j] = 0;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const uint32_t j = threadIdx.x + e * kBlock;
    slot[e] = kNone;
    if (j < n) {
      const uint64_t key = kk[e];
      uint32_t s = (uint32_t)dedup_mix(key) & (kBinLds - 1);
      for (int probe = 0; probe < kBinLds; ++probe) {
        const unsigned long long old = atomicCAS(&hk[s], (unsigned long long)kEmpty,
                                                 (unsigned long long)key);
        if (old == kEmpty || old == key) {
          if (old == key) hx[s] = 1;
          atomicMin(&hm[s], idx[e]);
          slot[e] = s;
          break;
        }
        s = (s + 1) & (kBinLds - 1);
      }
      if (slot[e] == kNone) t.hdr->dovf = 1u;  // every slot holds another key
    }
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    if (slot[e] != kNone && hx[slot[e]]) t.dfirst[idx[e]] = hm[slot[e]];
  }
}

// Overflow path: clear dd (it aliases the coarse bins) and switch the chunk to dedup_range.
__global__ __launch_bounds__(kBlock) void k_bin_fallback_clear(TableView t, uint32_t dslots) {
  if (t.hdr->spec) return;
  if (!t.hdr->dovf) {
    // the bins held: a chunk scattered without folding ends the skew hint
    if (blockIdx.x == 0 && threadIdx.x == 0 && !t.hdr->dagg) t.hdr->dskew = 0;
    return;
  }
  const uint4 empty = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
  for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < (int64_t)dslots / 2;
       j += (int64_t)gridDim.x * kBlock)
    reinterpret_cast<uint4*>(t.dd)[j] = empty;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    t.hdr->dmode = 0;
    t.hdr->dskew = 1;   // later chunks of this table fold each tile's repeats first
    t.hdr->dskew_age = 0;
  }
}

__global__ __launch_bounds__(kBlock) void k_bin_fallback_dedup(TableView t,
                                                               const uint64_t* __restrict__ keys,
                                                               int64_t q, uint32_t dmask) {
  if (!t.hdr->dovf || t.hdr->spec) return;
  dedup_range(t, keys, nullptr, dmask, (int64_t)blockIdx.x * kBlock, q, (int64_t)gridDim.x * kBlock);
}

// What is known of element i's repetition, loaded by the caller together with its key (one memory
// round trip instead of two): in a binned chunk (dmode) dfirst[i], kNone for an element that is not
// repeated; else dmark[i].
__device__ __forceinline__ uint32_t load_mark(const TableView& t, int64_t i, bool binned) {
  return binned ? t.dfirst[i] : t.dmark[i];
}

// Whether a mark says that the element is repeated (in a binned chunk also a mark that is its first
// copy's alone).
__device__ __forceinline__ bool repeated(uint32_t mark, bool binned) {
  return binned ? mark != kNone : mark != 0;
}

// Index-order role of this lane's element: its own index when it is the first copy of its key in
// the chunk, else the index of that first copy.
__device__ __forceinline__ uint32_t first_copy(const TableView& t, const uint64_t* keys,
                                               uint64_t key, int64_t i, uint32_t dmask,
                                               uint32_t mark, bool binned) {
  if (key >= kTomb) return t.hdr->spec_first[key - kTomb];
  if (!repeated(mark, binned)) return (uint32_t)i;
  if (!binned) return dedup_lookup(t, keys, key, dmask, (uint32_t)i);
  return (mark & kIndirect) ? t.dfirst[mark & ~kIndirect] : mark;
}

// Insert actors, one element per lane.  fast: claim directly with one CAS per new key (all CASes of
// the wave in flight together).  Otherwise (or with a pool) flag new keys for the ranked
// completion.  Elements [lo, hi) of a chunk, 64 per wave, the block's waves striding by `step`.
// `skip` (nullable): elements with a nonzero byte there take no part and keep their outputs.
// Returns this thread's count of stored keys.
template <int VK, bool ALLOC, bool AHEAD>
__device__ __forceinline__ int64_t insert_range(const TableView& t, WaveLds* w,
                                                const uint64_t* __restrict__ keys,
                                                const uint8_t* __restrict__ skip,
                                                const void* __restrict__ vals, uint32_t dmask,
                                                uint8_t* __restrict__ status,
                                                int32_t* __restrict__ vout, int64_t lo, int64_t hi,
                                                int64_t step) {
  const bool fast = t.hdr->fast != 0;
  const uint32_t inject = __builtin_amdgcn_readfirstlane(t.hdr->inject);
  const bool flags = ALLOC || !fast;
  const bool binned = t.hdr->dmode != 0;
  int64_t ins = 0;
  for (int64_t w0 = lo + (int64_t)(threadIdx.x & ~63u); w0 < hi; w0 += step) {
    const int64_t i = w0 + wave_lane();
    const bool valid = i < hi;
    const uint64_t key = keys[min(i, hi - 1)];
    // the value is loaded with the key (coalesced) so that its latency hides behind the probe
    const uint64_t val = (!ALLOC && valid) ? load_val<VK>(vals, i) : 0;
    const uint32_t mark = load_mark(t, min(i, hi - 1), binned);
    const uint32_t out = skip ? skip[min(i, hi - 1)] : 0;
    asm volatile("" ::"v"(mark), "v"(out));  // keep the loads here, issued with the key's
    const bool active = valid && !out;
    const uint32_t first = active ? first_copy(t, keys, key, i, dmask, mark, binned) : 0u;
    const bool actor = active && first == (uint32_t)i;
    const bool dup = active && !actor;
    // what k_fix reads: the mark says that the key is repeated, dup[i] names its first copy.  A later
    // copy whose first copy can neither meet FULL nor draw a value has its outcome here.
    if (flags && active && (repeated(mark, binned) || dup)) {
      t.dup[i] = first;
      t.dmark[i] = 1;  // (so far only known in dfirst, or a later copy of an out-of-band key)
    }

    uint8_t st = dup && !flags ? kPresent : kNoStatus;
    uint8_t newf = 0;
    uint64_t ref = 0;
    if (actor && key >= kTomb) {  // out-of-band key: this lane alone
      const int s = (int)(key - kTomb);
      if (t.hdr->spec_live[s]) {
        st = kPresent;
        if (ALLOC && vout) vout[i] = (int32_t)(uint32_t)t.hdr->spec_val[s];
      } else if (!fast) {
        newf = 1;
      } else if (ALLOC) {
        t.hdr->spec_live[s] = 1;
        ref = kSpecRef + (uint64_t)s;
        newf = 1;
      } else {
        t.hdr->spec_live[s] = 1;
        t.hdr->spec_val[s] = val;
        st = kInserted;
        ++ins;
      }
    }
    const bool look = actor && key < kTomb;
    const Place p = place_keys<true, ALLOC, AHEAD>(t, w, look, key, fast, inject);
    if (look) {
      if (p.found) {
        st = kPresent;
        if (ALLOC && vout) vout[i] = (int32_t)(uint32_t)p.val;
      } else if (!fast) {
        newf = 1;
      } else if (p.pos == kNoPos) {
        st = kFull;  // no free slot anywhere: cannot happen while size + chunk <= capacity
        aor32(&t.hdr->err, kErrFull);
      } else if (ALLOC) {
        ref = p.pos;
        newf = 1;
      } else {
        if (VK) t.bk[p.pos >> 3].s[p.pos & 7].val = val;
        st = kInserted;
        ++ins;
      }
    }
    if (valid) {
      if (flags) t.flag[i] = newf;
      if (ALLOC && newf) t.ref[i] = ref;
      if (status && st != kNoStatus) status[i] = st;
    }
  }
  return ins;
}

// The host's view of how an insert chunk of q keys went: q and the keys it stored, one 64-bit
// store to host-mapped memory (read without synchronising; a stale or torn read only changes
// which path the next chunk takes, never a result).
// Word 0 reports insert chunks (keys stored), word 1 erase chunks (keys removed).
__device__ __forceinline__ void chunk_feedback(const TableView& t, int word, int64_t q,
                                               int64_t changed) {
  if (q <= 0) return;
  const uint64_t w = ((uint64_t)q << 32) | (uint64_t)(uint32_t)(changed < 0 ? 0 : changed);
  t.hdr->fbd[word] = w;
  if (t.fb) __hip_atomic_store(t.fb + word, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The last block of a small grid settles the live count: every block adds (change << 20 | 1) to one
// word of the table, and the one that completes the grid's number has the total in its answer and
// puts the word back to zero.  Saves the launch of k_apply_count (4 us of the host, which bounds
// batches of this size: 96 requests through the server, a third of them updates, went from 2.45 to
// 2.2 ms with this, the counts and the outcomes below taken into the insert and erase kernels).
// One same-address atomic takes 12.6 ns, so grids of more than kSettleBlocks leave partials instead.
__device__ __forceinline__ void settle_count(const TableView& t, int64_t tot, int64_t q, int word) {
  const uint64_t old = __hip_atomic_fetch_add(&t.stripes[kSettleWord], ((uint64_t)tot << 20) | 1u,
                                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if ((old & 0xFFFFFu) + 1u != gridDim.x) return;
  Header* h = t.hdr;
  const int64_t sum = (int64_t)(old >> 20) + tot;
  t.stripes[kSettleWord] = 0;
  h->size = word ? h->size - (uint64_t)sum : h->size + (uint64_t)sum;
  // (an insert chunk that may meet capacity stores more keys in its ranked pass: no report)
  if (word || h->fast) chunk_feedback(t, word, q, sum);
}

// The rank flags per tile, by the kernel that wrote them: each pass of the block covers 256
// consecutive elements, all in one tile, and each thread re-reads the flag it wrote itself; the
// tile sums were zeroed by the chunk's prologue.
__device__ __forceinline__ void count_flags(const TableView& t, int64_t q) {
  for (int64_t b0 = (int64_t)blockIdx.x * kBlock; b0 < q; b0 += (int64_t)gridDim.x * kBlock) {
    __syncthreads();  // block_sum's partials are reused
    const int64_t i = b0 + threadIdx.x;
    const int64_t c = block_sum((int64_t)(i < q ? t.flag[i] : 0));
    if (threadIdx.x == 0 && c) aadd32(&t.tsum[b0 / kTile], (uint32_t)c);
  }
}

// Held to 5 waves per SIMD (96 VGPRs, no spills), as are the speculative kernels below; the compiler
// takes 98 to 109 VGPRs, 4 waves.  Of the large-table churn (2^24 keys erased and inserted again,
// load 0.8) one round took 2.75 ms at 5 waves, 2.83 at 4, 2.78 at 6 and 2.98 at 7, which spill; with
// eight keys per 8-lane group and claims retried one key at a time it took 2.89 ms.
template <int VK, bool ALLOC, bool AHEAD>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(AHEAD ? 1 : 5))) void k_insert(TableView t, const uint64_t* __restrict__ keys,
                                                   const void* __restrict__ vals, int64_t q,
                                                   uint32_t dmask, uint8_t* __restrict__ status,
                                                   int32_t* __restrict__ vout,
                                                   const uint8_t* __restrict__ skip, int settle) {
  if (t.hdr->spec) return;
  const int64_t ins = insert_range<VK, ALLOC, AHEAD>(t, wave_lds<kBlock>(), keys, skip, vals, dmask, status, vout,
                                              (int64_t)blockIdx.x * kBlock, q,
                                              (int64_t)gridDim.x * kBlock);
  if (!ALLOC) {
    const int64_t tot = block_sum(ins);
    if (threadIdx.x == 0) {
      if (settle) settle_count(t, tot, q, 0);
      else t.bcnt[blockIdx.x] = tot;  // summed by k_apply_count
    }
  }
  if (ALLOC || (settle && !t.hdr->fast)) count_flags(t, q);
}

// Host-side resizing (a table's capacity is fixed when it is created, Section 4; it grows by a
// copy into a larger table): every live pair of src is inserted into dst.  A wave takes 64 slots of
// src (8 buckets).  The keys of src are distinct and the host has checked that dst has room for
// all of them, so a new key claims a slot directly; a key dst already holds stays unchanged.
// Counts per block, summed by k_apply_count.
__global__ __launch_bounds__(kBlock) void k_rehash(TableView src, TableView dst) {
  const int64_t nslots = (int64_t)src.nb * kSlots;
  const uint32_t inject = __builtin_amdgcn_readfirstlane(dst.hdr->inject);
  int64_t ins = 0;
  for (int64_t w0 = (int64_t)blockIdx.x * kBlock + (threadIdx.x & ~63u); w0 < nslots;
       w0 += (int64_t)gridDim.x * kBlock) {
    const int64_t j = w0 + wave_lane();
    Slot sl;
    sl.key = kEmpty;
    sl.val = 0;
    if (j < nslots) sl = src.bk[j >> 3].s[j & 7];
    const bool live = sl.key < kTomb;
    const Place p = place_keys<true, false, false>(dst, wave_lds<kBlock>(), live, sl.key, true, inject);
    if (live && !p.found) {
      if (p.pos != kNoPos) {
        dst.bk[p.pos >> 3].s[p.pos & 7].val = sl.val;
        ++ins;
      } else {
        aor32(&dst.hdr->err, kErrFull);  // not reached while dst has the room the host checked
      }
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {  // the out-of-band keys
    for (int s = 0; s < 2; ++s) {
      if (src.hdr->spec_live[s] && !dst.hdr->spec_live[s]) {
        dst.hdr->spec_live[s] = 1;
        dst.hdr->spec_val[s] = src.hdr->spec_val[s];
        ++ins;
      }
    }
  }
  const int64_t tot = block_sum(ins);
  if (threadIdx.x == 0) dst.bcnt[blockIdx.x] = tot;
}

// Erase actors, one element per lane.  RELEASE: the removed value is kept for the ordered push.
template <bool RELEASE, bool AHEAD>
__device__ __forceinline__ int64_t erase_range(const TableView& t, WaveLds* w,
                                               const uint64_t* __restrict__ keys, uint32_t dmask,
                                               uint8_t* __restrict__ erased, int64_t lo, int64_t hi,
                                               int64_t step) {
  const bool binned = t.hdr->dmode != 0;
  int64_t del = 0;
  for (int64_t w0 = lo + (int64_t)(threadIdx.x & ~63u); w0 < hi; w0 += step) {
    const int64_t i = w0 + wave_lane();
    const bool valid = i < hi;
    const uint64_t key = keys[min(i, hi - 1)];
    const uint32_t mark = load_mark(t, min(i, hi - 1), binned);
    asm volatile("" ::"v"(mark));  // keep the load here, issued with the key's
    const bool actor = valid && first_copy(t, keys, key, i, dmask, mark, binned) == (uint32_t)i;
    uint8_t hit = 0;
    uint64_t val = 0;
    if (actor && key >= kTomb) {
      const int s = (int)(key - kTomb);
      if (t.hdr->spec_live[s]) {
        t.hdr->spec_live[s] = 0;
        val = t.hdr->spec_val[s];
        hit = 1;
      }
    }
    const Place p = place_keys<false, RELEASE, AHEAD>(t, w, actor && key < kTomb, key, false, 0);
    if (p.found) {
      // kEmpty only where the bucket already holds one: no probe sequence runs through it
      t.bk[p.pos >> 3].s[p.pos & 7].key = p.had_empty ? kEmpty : kTomb;
      val = p.val;
      hit = 1;
    }
    if (valid) {
      if (erased) erased[i] = hit;
      if (RELEASE) {
        t.flag[i] = hit;
        t.ref[i] = val;
      }
      del += hit;
    }
  }
  return del;
}

template <bool RELEASE, bool AHEAD>
__global__ __launch_bounds__(kBlock) void k_erase(TableView t, const uint64_t* __restrict__ keys,
                                                  int64_t q, uint32_t dmask,
                                                  uint8_t* __restrict__ erased, int settle) {
  const int64_t del = erase_range<RELEASE, AHEAD>(t, wave_lds<kBlock>(), keys, dmask, erased, (int64_t)blockIdx.x * kBlock, q,
                                           (int64_t)gridDim.x * kBlock);
  if (RELEASE) {  // the removals are the rank flags: their total settles the live count
    count_flags(t, q);
    return;
  }
  const int64_t tot = block_sum(del);
  if (threadIdx.x == 0) {
    if (settle) settle_count(t, tot, q, 1);
    else t.bcnt[blockIdx.x] = -tot;
  }
}

// Add the per-block partials of the preceding insert/erase kernel to the live count.
// Returns the change (valid on thread 0).
__device__ __forceinline__ int64_t apply_count_block(const TableView& t, int nparts) {
  int64_t v = 0;
  for (int j = threadIdx.x; j < nparts; j += blockDim.x) v += t.bcnt[j];
  v = (int64_t)wave_sum((uint64_t)v);
  __shared__ int64_t part[16];
  if (wave_lane() == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  int64_t s = 0;
  if (threadIdx.x == 0) {
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += part[w];
    if (s) t.hdr->size = (uint64_t)((int64_t)t.hdr->size + s);
  }
  __syncthreads();
  return s;
}

// fb_q > 0: the partials are the count changes of an insert (fb_word 0) or erase (fb_word 1)
// chunk of fb_q keys: report how many keys the chunk stored or removed.
__global__ __launch_bounds__(1024) void k_apply_count(TableView t, int nblocks, int64_t fb_q,
                                                      int fb_word, int decided) {
  if (decided && t.hdr->spec) return;
  const int64_t s = apply_count_block(t, nblocks);
  // (an insert chunk that may meet capacity stores more keys in its ranked pass: no report)
  if (threadIdx.x == 0 && fb_q && (fb_word || t.hdr->fast))
    chunk_feedback(t, fb_word, fb_q, fb_word ? -s : s);
}

// ---------------------------------------------------------------------------------------------
// Speculative insert: repeated keys resolved after the table update instead of before it.
//
// When the host can prove that a chunk cannot reach capacity, no element can meet FULL and the
// index order matters only among copies of one key.  Every element then probes and claims for
// itself.  Claims only turn free slots into keys during the kernel, and every copy of a key takes
// the first free slot of the same probe sequence, so a key is stored at most once: a copy either
// claims the slot, sees the key in a bucket, or loses its CAS to the key (the rescan after a lost
// CAS looks for the key as well as for free slots).  The claimer is whichever copy got there
// first, not necessarily the lowest index, and a copy that sees the key cannot tell whether it
// was there before the chunk.  Such elements are "listed" (flag 2; claimers have flag 1): they
// report PRESENT.  After the kernel, a key needs a fix only when it has a claimer and a listed
// copy of lower index; that copy becomes the inserter (its value goes into the slot, the statuses
// swap).  A listed key without a claimer was present before the chunk, so PRESENT was right.
//
// The resolution pairs claimers with listed copies through the dd table, in the direction that
// puts fewer keys into it: with few listed elements (a batch of mostly new keys), the listed keys
// enter dd with their lowest index and the claimers look themselves up; with mostly listed
// elements (keys that are mostly present already), the claimers enter dd and each listed copy
// lowers the index beside its claimer's entry, which the claimer checks afterwards.  The
// out-of-band keys are always listed and resolved by one thread.  With distinct keys absent from
// the table nothing is listed, and the resolution kernels return at once.
// ---------------------------------------------------------------------------------------------
enum : uint8_t { kFlagNone = 0, kFlagClaimed = 1, kFlagListed = 2, kFlagLeft = 3, kFlagSure = 4 };

// A speculative chunk's counts: every block adds (elements stored or removed << 32 | listed) to one
// of kCountStripes words on separate 128-byte lines of the table, which are zero between batches.
// (Per-block partials summed by one block took 10.8 us per 2^23-key chunk, and zeroing the words
// first another launch.)
__device__ __forceinline__ void spec_count(const TableView& t, int64_t block, int64_t tot) {
  if (tot) aadd64(&t.stripes[(block % kCountStripes) * kCountStride], (uint64_t)tot);
}

// Their sum; the first wave of a block calls it.
__device__ __forceinline__ uint64_t spec_total(const TableView& t) {
  const int lane = wave_lane();
  return wave_sum(lane < kCountStripes ? t.stripes[lane * kCountStride] : 0ull);
}

__device__ __forceinline__ void spec_zero(const TableView& t) {
  if (threadIdx.x < kCountStripes) t.stripes[threadIdx.x * kCountStride] = 0;
}

// Elements [lo, hi) of a chunk, 64 per wave.  Returns this thread's (stored, listed) counts.
template <int VK, bool AHEAD>
__device__ __forceinline__ uint2 insert_spec_range(const TableView& t, WaveLds* w,
                                                   const uint64_t* __restrict__ keys,
                                                   const void* __restrict__ vals,
                                                   uint8_t* __restrict__ status, int64_t lo,
                                                   int64_t hi, int64_t step) {
  const uint32_t inject = __builtin_amdgcn_readfirstlane(t.hdr->inject);
  uint32_t ins = 0, listed = 0;
  for (int64_t w0 = lo + (int64_t)(threadIdx.x & ~63u); w0 < hi; w0 += step) {
    const int64_t i = w0 + wave_lane();
    const bool valid = i < hi;
    const uint64_t key = keys[min(i, hi - 1)];
    const uint64_t val = valid ? load_val<VK>(vals, i) : 0;
    bool amb = valid && key >= kTomb;  // out-of-band keys: resolved after the kernel
    uint8_t st = kPresent;
    uint8_t claimed = 0;
    const bool look = valid && key < kTomb;
    const Place p = place_keys<true, false, AHEAD>(t, w, look, key, true, inject);
    if (look) {
      if (p.found) {
        amb = true;
      } else if (p.pos == kNoPos) {
        st = kFull;  // no free slot anywhere: cannot happen while size + chunk <= capacity
        aor32(&t.hdr->err, kErrFull);
      } else {
        if (VK) t.bk[p.pos >> 3].s[p.pos & 7].val = val;
        st = kInserted;
        claimed = 1;
        ++ins;
      }
    }
    if (valid) {
      t.flag[i] = claimed ? kFlagClaimed : (amb ? kFlagListed : kFlagNone);
      if (status) status[i] = st;
      listed += amb ? 1u : 0u;
    }
  }
  return make_uint2(ins, listed);
}

template <int VK, bool AHEAD>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(AHEAD ? 1 : 5))) void k_insert_spec(TableView t, const uint64_t* __restrict__ keys,
                                                        const void* __restrict__ vals, int64_t q,
                                                        uint8_t* __restrict__ status, int decided) {
  if (decided && !t.hdr->spec) return;
  const uint2 c = insert_spec_range<VK, AHEAD>(t, wave_lds<kBlock>(), keys, vals, status, (int64_t)blockIdx.x * kBlock, q,
                                        (int64_t)gridDim.x * kBlock);
  const int64_t tot = block_sum(((int64_t)c.x << 32) + (int64_t)c.y);
  if (threadIdx.x == 0) spec_count(t, blockIdx.x, tot);
}

// Speculative erase: every element probes; a found key is removed with one CAS (key -> kEmpty
// where its bucket holds an empty slot, else kTomb), so of several copies exactly one removes it
// (flag 1, reports 1).  A copy that loses that CAS or finds no key is listed (flag 2, reports 0):
// afterwards the lowest listed copy takes the removal over from a higher remover.  A copy cannot
// miss a key that is still there: an erase writes kEmpty only into buckets that already hold one,
// so no probe sequence is cut short.  Out-of-band keys are always listed.
template <bool AHEAD>
__device__ __forceinline__ uint2 erase_spec_range(const TableView& t, WaveLds* w,
                                                  const uint64_t* __restrict__ keys,
                                                  uint8_t* __restrict__ erased, int64_t lo,
                                                  int64_t hi, int64_t step) {
  uint32_t del = 0, listed = 0;
  for (int64_t w0 = lo + (int64_t)(threadIdx.x & ~63u); w0 < hi; w0 += step) {
    const int64_t i = w0 + wave_lane();
    const bool valid = i < hi;
    const uint64_t key = keys[min(i, hi - 1)];
    const Place p = place_keys<false, false, AHEAD>(t, w, valid && key < kTomb, key, false, 0);
    uint8_t hit = 0;
    if (p.found) {
      uint64_t expected = key;
      hit = cas64(&t.bk[p.pos >> 3].s[p.pos & 7].key, expected, p.had_empty ? kEmpty : kTomb) ? 1 : 0;
    }
    if (valid) {
      t.flag[i] = hit ? kFlagClaimed : kFlagListed;
      if (erased) erased[i] = hit;
      del += hit;
      listed += hit ^ 1u;
    }
  }
  return make_uint2(del, listed);
}

template <bool AHEAD>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(AHEAD ? 1 : 5))) void k_erase_spec(TableView t, const uint64_t* __restrict__ keys,
                                                       int64_t q, uint8_t* __restrict__ erased) {
  const uint2 c = erase_spec_range<AHEAD>(t, wave_lds<kBlock>(), keys, erased, (int64_t)blockIdx.x * kBlock, q,
                                   (int64_t)gridDim.x * kBlock);
  const int64_t tot = block_sum(((int64_t)c.x << 32) + (int64_t)c.y);
  if (threadIdx.x == 0) spec_count(t, blockIdx.x, tot);
}

// Whether the table's last insert (word 0) or erase (word 1) chunk changed at least half its keys.
__device__ __forceinline__ bool mostly_changed(const Header* h, int word) {
  const uint64_t f = h->fbd[word];
  const uint64_t fq = f >> 32, changed = f & 0xFFFFFFFFull;
  return fq == 0 || 2 * changed >= fq;
}

// The host could not prove that a large insert chunk stays below capacity: decide from the live
// count itself, and (unless `always`) from how the last chunk went.  One thread.
__global__ void k_spec_decide(TableView t, int64_t q, int always) {
  const Header* h = t.hdr;
  const bool spec = h->size + (uint64_t)q <= t.cap && (always || mostly_changed(h, 0));
  if (threadIdx.x == 0) {
    t.hdr->spec = spec ? 1u : 0u;
    t.hdr->fast = spec ? 1u : 0u;  // (the ranked completion leaves at once)
    t.hdr->ndup = 0;
  }
}

// Resolution direction and dd entries for `nd` listed elements of a q-element chunk.
struct SpecPlan {
  bool by_claimers;  // claimers enter dd (mostly listed elements)
  uint32_t slots;    // dd entries in use: a power of two >= 2 x the keys entering dd
};

__device__ __forceinline__ SpecPlan spec_plan(uint32_t nd, int64_t q) {
  SpecPlan p;
  p.by_claimers = 2 * (int64_t)nd > q;
  const uint32_t enter = p.by_claimers ? (uint32_t)(q - nd) : nd;
  uint32_t s = 2;
  while (s < 2 * enter) s <<= 1;
  p.slots = s;
  return p;
}

// In the claimer direction, the lowest listed index per claimer entry sits behind the entries.
__device__ __forceinline__ uint32_t* spec_low(const TableView& t, const SpecPlan& p) {
  return reinterpret_cast<uint32_t*>(t.dd + p.slots);
}

// The counters after a speculative insert or erase of q elements whose counts are `tot`: live count,
// feedback words, and what the resolution reads.  One thread.  An insert ran because its chunk
// cannot reach capacity; a live count that says otherwise is a library bug.
__device__ __forceinline__ void spec_settle(const TableView& t, int64_t q, bool erase, uint64_t tot) {
  Header* h = t.hdr;
  const uint64_t changed = tot >> 32;
  if (!erase && h->size + (uint64_t)q > t.cap) h->err |= kErrInternal;
  h->size = erase ? h->size - changed : h->size + changed;
  chunk_feedback(t, erase, q, (int64_t)changed);
  h->spec_first[0] = h->spec_first[1] = kNone;
  h->ndup = (uint32_t)tot;
}

// Clears the dd entries (and, in the claimer direction, the lowest-index words) the resolution of
// `nd` listed elements uses; nothing when no element is listed.
// (The resolution stages take their block b of nb as arguments, so that the grouped plan can run
// them per step; the single-table kernels pass blockIdx.x and gridDim.x.)
__device__ __forceinline__ void spec_clear_range(const TableView& t, int64_t q, uint32_t nd, int64_t b,
                                                 int64_t nb) {
  if (nd == 0) return;
  const SpecPlan p = spec_plan(nd, q);
  const int64_t units = p.slots / 2;
  const uint4 ones = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
  for (int64_t j = b * kBlock + threadIdx.x; j < units; j += nb * kBlock) {
    reinterpret_cast<uint4*>(t.dd)[j] = ones;
    if (p.by_claimers && j < units / 2) reinterpret_cast<uint4*>(spec_low(t, p))[j] = ones;
  }
  if (p.by_claimers && units == 1 && b == 0 && threadIdx.x == 0) {
    spec_low(t, p)[0] = kNone;
    spec_low(t, p)[1] = kNone;
  }
}

// Every block sums the counts for itself; the first also settles the counters.
__global__ __launch_bounds__(kBlock) void k_spec_clear(TableView t, int64_t q, int erase, int decided) {
  if (decided && !t.hdr->spec) return;
  __shared__ uint64_t tot;
  if (threadIdx.x < 64) {
    const uint64_t v = spec_total(t);
    if (threadIdx.x == 0) {
      tot = v;
      if (blockIdx.x == 0) spec_settle(t, q, erase != 0, v);
    }
  }
  __syncthreads();
  spec_clear_range(t, q, (uint32_t)tot, blockIdx.x, gridDim.x);
}

// dd slot of `key` among entries (tag | chunk index); kNone when absent.
__device__ __forceinline__ uint32_t dd_find(const TableView& t, const uint64_t* keys, uint64_t key,
                                           uint32_t dmask, uint32_t* idx) {
  const uint64_t mix = dedup_mix(key);
  const uint64_t tag = mix & 0xFFFFFFFF00000000ull;
  uint32_t h = (uint32_t)mix & dmask;
  for (uint32_t probe = 0; probe <= dmask; ++probe) {
    const uint64_t e = t.dd[h];
    if (e == kEmpty) return kNone;
    if ((e & 0xFFFFFFFF00000000ull) == tag && keys[(uint32_t)e] == key) {
      *idx = (uint32_t)e;
      return h;
    }
    h = (h + 1) & dmask;
  }
  return kNone;
}

// Build: the keys that enter dd.  Listed direction: windows of 1024 elements first resolve their
// listed keys in LDS, so a key listed many times costs one CAS or atomic min per window (skipped
// when the held index is already lower).  Claimer direction: every claimer's key is distinct, so
// each takes an empty entry with one CAS.  Out-of-band listed copies take an atomic min on their
// header word in both directions.  Windows that list nothing, most of those of a batch of mostly
// new keys, cost their flags alone.
__device__ __forceinline__ void spec_build_range(const TableView& t, const uint64_t* __restrict__ keys,
                                                 int64_t q, int64_t blk, int64_t nblk) {
  const uint32_t nd = t.hdr->ndup;  // written by spec_settle
  if (nd == 0) return;
  const SpecPlan p = spec_plan(nd, q);
  const uint32_t dmask = p.slots - 1;
  constexpr int kPer = 4;
  constexpr uint32_t kW = 2 * kPer * kBlock;
  __shared__ unsigned long long wk[kW];
  __shared__ uint32_t wmin[kW];
  for (int64_t b0 = blk * kBlock * kPer; b0 < q; b0 += nblk * kBlock * kPer) {
    uint8_t f[kPer];
    uint64_t key[kPer];
    bool any = false;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int64_t i = b0 + k * kBlock + threadIdx.x;
      f[k] = i < q ? t.flag[i] : kFlagNone;
      any |= f[k] == kFlagListed;
    }
    if (!p.by_claimers && !__syncthreads_or(any)) continue;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int64_t i = b0 + k * kBlock + threadIdx.x;
      key[k] = f[k] == kFlagListed || (p.by_claimers && f[k] == kFlagClaimed) ? keys[i] : 0;
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int64_t i = b0 + k * kBlock + threadIdx.x;
      if (f[k] == kFlagListed && key[k] >= kTomb) amin32(&t.hdr->spec_first[key[k] - kTomb], (uint32_t)i);
      if (p.by_claimers && f[k] == kFlagClaimed) {
        const uint64_t mix = dedup_mix(key[k]);
        uint32_t h = (uint32_t)mix & dmask;
        for (uint32_t probe = 0; probe <= dmask; ++probe) {
          uint64_t expected = kEmpty;
          if (cas64(&t.dd[h], expected, (mix & 0xFFFFFFFF00000000ull) | (uint64_t)i)) break;
          h = (h + 1) & dmask;
        }
      }
    }
    // listed direction (uniform per block: p depends only on nd and q)
    if (p.by_claimers) continue;
    for (uint32_t j = threadIdx.x; j < kW; j += kBlock) {
      wk[j] = kEmpty;
      wmin[j] = kNone;
    }
    __syncthreads();
    uint32_t s[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int64_t i = b0 + k * kBlock + threadIdx.x;
      s[k] = kNone;
      if (f[k] != kFlagListed || key[k] >= kTomb) continue;
      uint32_t at = (uint32_t)(dedup_mix(key[k]) >> 32) & (kW - 1);
      for (;;) {  // at most kW / 2 keys in kW slots: a free or matching slot exists
        const unsigned long long old = atomicCAS(&wk[at], (unsigned long long)kEmpty,
                                                 (unsigned long long)key[k]);
        if (old == kEmpty || old == key[k]) break;
        at = (at + 1) & (kW - 1);
      }
      atomicMin(&wmin[at], (uint32_t)i);
      s[k] = at;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int64_t i = b0 + k * kBlock + threadIdx.x;
      if (s[k] == kNone || wmin[s[k]] != (uint32_t)i) continue;
      const uint64_t mix = dedup_mix(key[k]);
      const uint64_t tag = mix & 0xFFFFFFFF00000000ull;
      const uint64_t mine = tag | (uint64_t)i;
      uint32_t h = (uint32_t)mix & dmask;
      for (uint32_t probe = 0; probe <= dmask; ++probe) {
        uint64_t e = t.dd[h];
        if (e == kEmpty) {
          uint64_t expected = kEmpty;
          if (cas64(&t.dd[h], expected, mine)) break;
          e = expected;
        }
        if ((e & 0xFFFFFFFF00000000ull) == tag && keys[(uint32_t)e] == key[k]) {
          if ((uint32_t)i < (uint32_t)e) amin64(&t.dd[h], mine);
          break;
        }
        h = (h + 1) & dmask;
      }
    }
    __syncthreads();  // the window's LDS table is reused by the next window
  }
}

__global__ __launch_bounds__(kBlock) void k_spec_build(TableView t, const uint64_t* __restrict__ keys,
                                                       int64_t q) {
  spec_build_range(t, keys, q, blockIdx.x, gridDim.x);
}

// Slot of a key that is known to be stored (one lane alone, eight key loads per bucket).
__device__ __forceinline__ uint64_t lane_slot_of(const TableView& t, uint64_t key) {
  const Seq q = probe_seq(t, key);
  uint64_t b = q.home;
  for (uint64_t step = 0; step < t.nb; ++step) {
    for (int c = 0; c < kSlots; ++c)
      if (t.bk[b].s[c].key == key) return b * kSlots + (uint64_t)c;
    b = next_bucket(t, b, q.step);
  }
  return kNoPos;
}

// Claimer c hands the insert of its key to listed copy m < c: m's value into the slot, statuses
// swapped.
// An erase only moves the outcome: m reports the removal, c reports none (both statuses are the
// insert's INSERTED / PRESENT values, 1 / 0).
template <int VK, bool ERASE>
__device__ __forceinline__ void hand_over(const TableView& t, const void* __restrict__ vals,
                                          uint8_t* __restrict__ status, uint64_t key, uint32_t c,
                                          uint32_t m) {
  if (ERASE) {
    if (status) {
      status[m] = 1;
      status[c] = 0;
    }
    return;
  }
  const uint64_t pos = lane_slot_of(t, key);
  if (pos == kNoPos) {
    aor32(&t.hdr->err, kErrInternal);
    return;
  }
  if (VK) t.bk[pos >> 3].s[pos & 7].val = load_val<VK>(vals, m);
  if (status) {
    status[m] = kInserted;
    status[c] = kPresent;
  }
}

// Probe: listed direction: every claimer looks its key up and hands over to a lower listed copy.
// Claimer direction: every listed copy of a claimed key lowers the index word beside the entry
// (windows of 256 elements combine copies of one entry in LDS first; skipped when the word is
// already lower).
template <int VK, bool ERASE>
__device__ __forceinline__ void spec_probe_range(const TableView& t, const uint64_t* __restrict__ keys,
                                                 const void* __restrict__ vals, int64_t q,
                                                 uint8_t* __restrict__ status, int64_t blk,
                                                 int64_t nblk) {
  const uint32_t nd = t.hdr->ndup;  // written by spec_settle
  if (nd == 0) return;
  const SpecPlan p = spec_plan(nd, q);
  const uint32_t dmask = p.slots - 1;
  uint32_t* low = spec_low(t, p);
  constexpr uint32_t kW = 2 * kBlock;
  __shared__ uint32_t wh[kW], wmin[kW];
  if (!p.by_claimers) {  // four look-ups per thread in flight: flag, key and entry depend on each other
    constexpr int kPer = 4;
    for (int64_t b0 = blk * kBlock * kPer; b0 < q; b0 += nblk * kBlock * kPer) {
      uint8_t f[kPer];
      uint64_t key[kPer], e[kPer];
      uint32_t h[kPer];
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        const int64_t i = b0 + k * kBlock + threadIdx.x;
        f[k] = i < q ? t.flag[i] : kFlagNone;
      }
#pragma unroll
      for (int k = 0; k < kPer; ++k)
        key[k] = f[k] == kFlagClaimed ? keys[b0 + k * kBlock + threadIdx.x] : 0;
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        h[k] = (uint32_t)dedup_mix(key[k]) & dmask;
        e[k] = f[k] == kFlagClaimed ? t.dd[h[k]] : kEmpty;
      }
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        const uint64_t i = (uint64_t)(b0 + k * kBlock + threadIdx.x);
        const uint64_t tag = dedup_mix(key[k]) & 0xFFFFFFFF00000000ull;
        for (uint32_t probe = 0; probe <= dmask && e[k] != kEmpty; ++probe) {
          if ((e[k] & 0xFFFFFFFF00000000ull) == tag && keys[(uint32_t)e[k]] == key[k]) {
            if ((uint32_t)e[k] < (uint32_t)i)
              hand_over<VK, ERASE>(t, vals, status, key[k], (uint32_t)i, (uint32_t)e[k]);
            break;
          }
          h[k] = (h[k] + 1) & dmask;
          e[k] = t.dd[h[k]];
        }
      }
    }
    return;
  }
  for (int64_t b0 = blk * kBlock; b0 < q; b0 += nblk * kBlock) {
    const int64_t i = b0 + threadIdx.x;
    const uint8_t f = i < q ? t.flag[i] : kFlagNone;
    for (uint32_t j = threadIdx.x; j < kW; j += kBlock) {
      wh[j] = kNone;
      wmin[j] = kNone;
    }
    __syncthreads();
    uint32_t h = kNone, s = 0;
    if (f == kFlagListed) {
      const uint64_t key = keys[i];
      uint32_t c = 0;
      if (key < kTomb) {
        h = dd_find(t, keys, key, dmask, &c);
        if (h != kNone && (uint32_t)i > c) h = kNone;  // the claimer is lower: nothing to do
      }
    }
    if (h != kNone) {
      s = (h * 2654435761u) & (kW - 1);
      for (;;) {  // at most kBlock entries in kW slots
        const uint32_t old = atomicCAS(&wh[s], kNone, h);
        if (old == kNone || old == h) break;
        s = (s + 1) & (kW - 1);
      }
      atomicMin(&wmin[s], (uint32_t)i);
    }
    __syncthreads();
    if (h != kNone && wmin[s] == (uint32_t)i && (uint32_t)i < low[h]) amin32(&low[h], (uint32_t)i);
    __syncthreads();
  }
}

template <int VK, bool ERASE>
__global__ __launch_bounds__(kBlock) void k_spec_probe(TableView t, const uint64_t* __restrict__ keys,
                                                       const void* __restrict__ vals, int64_t q,
                                                       uint8_t* __restrict__ status) {
  spec_probe_range<VK, ERASE>(t, keys, vals, q, status, blockIdx.x, gridDim.x);
}

// Swap (claimer direction): a claimer whose entry holds a lower listed index hands over.  Thread
// 0 of the first block settles each out-of-band key on its lowest copy (an insert stores it when
// it was absent, an erase removes it when it was there).
template <int VK, bool ERASE>
__device__ __forceinline__ void spec_swap_range(const TableView& t, const uint64_t* __restrict__ keys,
                                                const void* __restrict__ vals, int64_t q,
                                                uint8_t* __restrict__ status, int64_t blk,
                                                int64_t nblk) {
  const uint32_t nd = t.hdr->ndup;  // written by spec_settle
  if (nd == 0) return;
  if (blk == 0 && threadIdx.x == 0) {
    Header* h = t.hdr;
    for (int s = 0; s < 2; ++s) {
      const uint32_t m = h->spec_first[s];
      if (m == kNone) continue;
      if (ERASE) {  // the lowest copy removes the key when it was there
        if (!h->spec_live[s]) continue;
        h->spec_live[s] = 0;
        h->size -= 1;
        if (status) status[m] = 1;
      } else {      // the lowest copy stores the key when it was absent
        if (h->spec_live[s]) continue;
        h->spec_live[s] = 1;
        h->spec_val[s] = load_val<VK>(vals, m);
        h->size += 1;
        if (status) status[m] = kInserted;
      }
    }
  }
  const SpecPlan p = spec_plan(nd, q);
  if (!p.by_claimers) return;
  const uint32_t dmask = p.slots - 1;
  const uint32_t* low = spec_low(t, p);
  for (int64_t c = blk * kBlock + threadIdx.x; c < q; c += nblk * kBlock) {
    if (t.flag[c] != kFlagClaimed) continue;
    const uint64_t key = keys[c];
    uint32_t self = 0;
    const uint32_t h = dd_find(t, keys, key, dmask, &self);
    if (h == kNone) {
      aor32(&t.hdr->err, kErrInternal);
      continue;
    }
    const uint32_t m = low[h];
    if (m < (uint32_t)c) hand_over<VK, ERASE>(t, vals, status, key, (uint32_t)c, m);
  }
}

template <int VK, bool ERASE>
__global__ __launch_bounds__(kBlock) void k_spec_swap(TableView t, const uint64_t* __restrict__ keys,
                                                      const void* __restrict__ vals, int64_t q,
                                                      uint8_t* __restrict__ status) {
  if (blockIdx.x == 0) spec_zero(t);  // for the next batch
  spec_swap_range<VK, ERASE>(t, keys, vals, q, status, blockIdx.x, gridDim.x);
}

// ---------------------------------------------------------------------------------------------
// Partitioned insert: a speculative insert of a large batch with several keys per bucket.
//
// What bounds the plain one is the claim: a gather, a 64-bit compare-and-swap at the memory side and a
// store into a random line, 18 G/s on this chip at most.  When the batch holds several keys per
// bucket, it is cheaper to bring the keys to the buckets: they move, by the high bits of their home
// bucket, into coarse and then fine bins of kPartBuckets buckets each; a workgroup loads a fine
// bin's buckets into LDS, claims slots there with LDS compare-and-swaps, and writes the buckets back.
// Every access to memory is a stream.  2^26 keys with 64-bit values filling a table to load 0.8
// (clearing it and looking 2^22 keys up included): 4.33 ms plain, 2.98 partitioned.
//
// An element whose home bucket holds its key is present; one whose home bucket shows an empty slot is
// absent from the table and claims there.  Copies of a key meet in one fine bin: while a bucket is
// in LDS, the value word of a slot claimed from the batch holds the lowest batch index that
// asked for its key, and that element stores the key and its value.  (Leaving copies to the
// speculative insert's resolution: 2^24 keys of 2^21 distinct took 2.7 ms, 1.1 plain.)
// Every other element is left over and placed by the ordinary probe afterwards: those whose home bucket
// is full (one in fourteen at load 0.8) through a list per coarse bin, which takes the place of the
// bin's own elements, and the rare rest (home bucket full but for tombstones; no room in a bin,
// which takes keys repeated very often) by a mark in their flags.  Only copies of those can be left
// unresolved; they end listed, and the speculative insert's resolution pairs them with the claimers.
// The buckets of a fine bin belong to one workgroup while the bins are inserted, and nothing else
// runs on the table.
// Copies of a key may meet in different kernels, each of which sees the claims of those before it.
// Within one, free slots of a bucket only become keys, and all copies ask for them in the same
// order, so a copy finds the key, loses its claim to it, or finds the bucket full like every later
// copy.
// ---------------------------------------------------------------------------------------------
constexpr int kPartBits = 8;
constexpr int kPartBuckets = 1 << kPartBits;   // buckets of a fine bin: 34 KB of LDS
constexpr int kPartStride = 2 * kSlots + 1;    // u64 words of a bucket in LDS (odd: lanes spread)
constexpr int kPartThreads = 512;
constexpr int kPartPer = 5;                    // elements of a fine bin a thread, at most
constexpr int kPartLeft = 512;                 // left-over positions gathered in LDS per fine bin
constexpr int kPartWindow = 8 * kBlock;        // flags that a block looks over at a time
constexpr int kPartXcds = 8;                   // blocks go to the chip's L2 domains in turn
constexpr int kPartCtr = kBinSub * kCtrStride; // counter words of a coarse bin (one line a segment)

struct PartView {
  uint64_t *r1k, *r2k;   // keys, values and batch indices of the coarse and the fine bins
  void *r1v, *r2v;
  uint32_t *r1i, *r2i;
  uint32_t *cur1, *cur2; // fill counts: coarse segments kCtrStride words apart, fine bins
  uint32_t *nleft;       // left-over elements of each coarse bin, kCtrStride words apart
  uint32_t *nover;       // 1: some element is marked kFlagLeft, or listed
  uint8_t* flag;         // by batch index: kFlagLeft for elements that found no room in a bin;
                         // kFlagSure for claimers while no copy of any key may be listed
  uint32_t c1, c2;       // capacities of a coarse segment and of a fine bin
  int lp2;               // log2 of the fine bins of a coarse bin
};

__device__ __forceinline__ uint32_t home32(const TableView& t, uint64_t key) {
  return (uint32_t)scale32(fmix64(key), t.nb);
}

template <int VK>
struct PartStage {
  uint64_t k[kBinTile];
  typename std::conditional<VK == 1, uint32_t, uint64_t>::type v[VK ? kBinTile : 1];
  uint32_t i[kBinTile];
  uint8_t b[kBinTile];
  uint32_t cnt[256], base[256], loc[256];
};

// The block's staged elements (code = rank << 8 | bin, ~0 for none) go to the bins in runs of
// consecutive positions, as bin_write does; an element past a bin's capacity is left over.
template <int VK, int PER>
__device__ __forceinline__ void part_write(const PartView& P, PartStage<VK>& S, uint32_t nbins,
                                           const uint64_t (&k)[PER], const uint64_t (&v)[PER],
                                           const uint32_t (&ix)[PER], const uint32_t (&code)[PER],
                                           uint32_t* cur, uint32_t cur_stride, int64_t bin0,
                                           uint32_t bin_stride, uint32_t cap, uint64_t* outk,
                                           void* outv, uint32_t* outi) {
  const uint32_t c = threadIdx.x < nbins ? S.cnt[threadIdx.x] : 0u;
  uint32_t total;
  const uint32_t pre = block_exclusive_scan(c, &total);
  if (threadIdx.x < nbins) {
    S.base[threadIdx.x] = c ? aadd32(&cur[threadIdx.x * cur_stride], c) : 0u;
    S.loc[threadIdx.x] = pre;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    if (code[e] == ~0u) continue;
    const uint32_t b = code[e] & 0xFFu;
    const uint32_t p = S.loc[b] + (code[e] >> 8);
    S.k[p] = k[e];
    if (VK) S.v[p] = (decltype(S.v[0] + 0))v[e];
    S.i[p] = ix[e];
    S.b[p] = (uint8_t)b;
  }
  __syncthreads();
  const uint32_t staged = min(total, (uint32_t)kBinTile);
  for (uint32_t p = threadIdx.x; p < staged; p += kBlock) {
    const uint32_t b = S.b[p];
    const uint32_t pos = S.base[b] + (p - S.loc[b]);
    if (pos < cap) {
      const int64_t at = (bin0 + (int64_t)b * bin_stride) * cap + pos;
      outk[at] = S.k[p];
      if (VK) store_val<VK>(outv, at, S.v[p]);
      outi[at] = S.i[p];
    } else {
      P.flag[S.i[p]] = kFlagLeft;
      *P.nover = 1;
    }
  }
}

// Coarse scatter, one tile of kBinTile elements per block into segment block mod kBinSub.  Statuses and
// flags start as those of a claimer; the kernels that follow write the exceptions.  Bound by
// memory: 38 bytes a key with 64-bit values, 2^26 keys in 0.65 ms, 3.9 TB/s.
template <int VK>
__global__ __launch_bounds__(kBlock) void k_part_coarse(TableView t, PartView P,
                                                        const uint64_t* __restrict__ keys,
                                                        const void* __restrict__ vals, int64_t n,
                                                        int ncoarse, uint8_t* __restrict__ status) {
  constexpr int kPer = kBinTile / kBlock;
  __shared__ PartStage<VK> S;
  const int64_t t0 = (int64_t)blockIdx.x * kBinTile;
  uint64_t k[kPer], v[kPer];
  uint32_t ix[kPer], code[kPer];
#pragma unroll
  for (int e = 0; e < kPer; ++e) {   // loads first, clamped
    const int64_t i = min(t0 + e * kBlock + (int64_t)threadIdx.x, n - 1);
    k[e] = keys[i];
    v[e] = load_val<VK>(vals, i);
  }
  S.cnt[threadIdx.x] = 0;
  __syncthreads();
  int64_t special = 0;
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int64_t i = t0 + e * kBlock + threadIdx.x;
    code[e] = ~0u;
    ix[e] = (uint32_t)i;
    if (i >= n) continue;
    const bool normal = k[e] < kTomb;
    P.flag[i] = normal ? kFlagSure : kFlagListed;
    if (status) status[i] = normal ? kInserted : kPresent;
    if (normal) {
      const uint32_t b = home32(t, k[e]) >> (kPartBits + P.lp2);
      code[e] = (atomicAdd(&S.cnt[b], 1u) << 8) | b;
    } else {
      ++special;
    }
  }
  const int64_t listed = block_sum(special);  // (a barrier between the counts and their use)
  if (threadIdx.x == 0) spec_count(t, blockIdx.x, listed);
  __syncthreads();
  const uint32_t seg = blockIdx.x % kBinSub;
  part_write<VK, kPer>(P, S, (uint32_t)ncoarse, k, v, ix, code, P.cur1 + seg * kCtrStride, kPartCtr, seg,
                       kBinSub, P.c1, P.r1k, P.r1v, P.r1i);
}

// Fine scatter of the coarse bins from `coarse0` on: the blocks of a segment take its tiles in turn.
// The fine bins of these coarse bins start at r2's beginning.  A tile leaves about eight elements
// to each fine bin, half a line; blocks of one coarse bin share an L2 (blockIdx modulo kPartXcds),
// where those halves meet before they go to memory: 2^26 keys took 1.08 ms with the segments'
// blocks on all of them and take 0.67, 4.0 TB/s.
template <int VK>
__global__ __launch_bounds__(kBlock) void k_part_fine(TableView t, PartView P, int coarse0,
                                                      int ncoarse, int blocks_per_seg) {
  constexpr int kPer = kBinTile / kBlock;
  __shared__ PartStage<VK> S;
  const int r = (int)blockIdx.x / kPartXcds, per = kBinSub * blocks_per_seg;
  const int c = coarse0 + r / per * kPartXcds + (int)blockIdx.x % kPartXcds;
  if (c >= ncoarse) return;
  const int64_t seg = (int64_t)c * kBinSub + r % per / blocks_per_seg;
  const uint32_t n1 = min(P.cur1[seg * kCtrStride], P.c1);
  const int64_t src = seg * P.c1;
  const uint32_t nf = 1u << P.lp2;
  for (uint32_t j0 = (uint32_t)(r % blocks_per_seg) * kBinTile; j0 < n1;
       j0 += (uint32_t)blocks_per_seg * kBinTile) {
    uint64_t k[kPer], v[kPer];
    uint32_t ix[kPer], code[kPer];
#pragma unroll
    for (int e = 0; e < kPer; ++e) {   // loads first, clamped (n1 > j0 >= 0)
      const uint32_t j = min(j0 + e * kBlock + threadIdx.x, n1 - 1u);
      k[e] = P.r1k[src + j];
      v[e] = load_val<VK>(P.r1v, src + j);
      ix[e] = P.r1i[src + j];
    }
    S.cnt[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      code[e] = ~0u;
      if (j0 + e * kBlock + threadIdx.x < n1) {
        const uint32_t b = (home32(t, k[e]) >> kPartBits) & (nf - 1u);
        code[e] = (atomicAdd(&S.cnt[b], 1u) << 8) | b;
      }
    }
    __syncthreads();
    part_write<VK, kPer>(P, S, nf, k, v, ix, code, P.cur2 + ((uint32_t)c << P.lp2), 1u,
                         (int64_t)(c - coarse0) << P.lp2, 1u, P.c2, P.r2k, P.r2v, P.r2i);
    __syncthreads();  // the stage is refilled by the next tile
  }
}

// One fine bin per block: its buckets in LDS, claims there, buckets back.  Bound by memory: 20
// bytes a key and the buckets both ways, 2^26 keys into 2^26/0.8 slots in 0.89 ms, 4.5 TB/s.
// Reading the elements ahead of the buckets' barrier gained nothing: four blocks a CU cover it.
template <int VK>
__global__ __launch_bounds__(kPartThreads) void k_part_insert(TableView t, PartView P, int coarse0,
                                                              uint8_t* __restrict__ status) {
  __shared__ uint64_t L[kPartBuckets * kPartStride];
  __shared__ uint32_t left[kPartLeft], nleft, lbase;
  const int64_t fl = ((int64_t)(blockIdx.x / (kPartXcds << P.lp2) * kPartXcds + blockIdx.x % kPartXcds) << P.lp2) +
                     (blockIdx.x / kPartXcds & ((1u << P.lp2) - 1u));  // fine bin within the group
  const int64_t f = ((int64_t)coarse0 << P.lp2) + fl;
  const int64_t b0 = f << kPartBits;
  if (b0 >= (int64_t)t.nb) return;
  const uint32_t n = min(P.cur2[f], P.c2);
  if (n == 0) return;
  const int64_t src = fl * P.c2;
  const int nslots = (int)min((int64_t)kPartBuckets, (int64_t)t.nb - b0) * kSlots;
  Slot* slots = t.bk[b0].s;  // the bin's buckets are contiguous
  for (int j = threadIdx.x; j < nslots; j += kPartThreads) {
    const Slot sl = slots[j];
    uint64_t* w = &L[(j >> 3) * kPartStride + 2 * (j & 7)];
    const bool taken = sl.key < kTomb;
    w[0] = sl.key;
    w[1] = taken ? sl.val : ~0ull;
    const uint64_t mask = __ballot(taken) >> (threadIdx.x & 56u);  // the bucket's slots taken before
    if ((j & 7) == 0) L[(j >> 3) * kPartStride + 2 * kSlots] = mask & 0xFFu;
  }
  if (threadIdx.x == 0) nleft = 0;
  __syncthreads();
  const uint32_t inject = __builtin_amdgcn_readfirstlane(t.hdr->inject);
  uint32_t claimed = 0;
  uint64_t val[kPartPer];
  uint32_t idx[kPartPer], slot[kPartPer];  // slot: LDS word of the value; 0: none
#pragma unroll
  for (int e = 0; e < kPartPer; ++e) {
    slot[e] = 0;
    const uint32_t j = threadIdx.x + e * kPartThreads;
    if (j >= n) continue;
    const uint64_t key = P.r2k[src + j];
    val[e] = load_val<VK>(P.r2v, src + j);
    idx[e] = P.r2i[src + j];
    const uint32_t at = (home32(t, key) & (kPartBuckets - 1u)) * kPartStride;
    unsigned long long* w = reinterpret_cast<unsigned long long*>(&L[at]);
    uint32_t m = 0, em = 0, tb = 0;
#pragma unroll
    for (int c = 0; c < kSlots; ++c) {
      const uint64_t x = w[2 * c];
      m |= x == key ? 1u << c : 0u;
      em |= x == kEmpty ? 1u << c : 0u;
      tb |= x == kTomb ? 1u << c : 0u;
    }
    uint32_t c = m ? (uint32_t)__builtin_ctz(m) : 0u;
    bool met = m != 0, over = !met && !em, full = over && !tb;
    bool won = false;
    const uint32_t rot = (uint32_t)(key >> 61);
    uint32_t lose = injected_loss(key, inject, rot), late = 0;  // test hook, as in place_keys
    uint32_t fs = em | tb << 8;
    while (!met && !over && !won) {  // absent: every pass takes a slot or learns that it is gone
      const uint32_t fr = fs >> 8 ? fs >> 8 : fs;
      c = ((uint32_t)__builtin_ctz((fr * 0x101u) >> rot) + rot) & 7u;
      const unsigned long long want = (fs >> 8 != 0) != (c == lose) ? kTomb : kEmpty;
      const unsigned long long got = atomicCAS(&w[2 * c], want, (unsigned long long)key);
      won = got == want;
      met = got == key;
      if (c == lose) {
        late = fs & kFreeSlot << c;
        lose = kSlots;
      }
      fs &= ~(kFreeSlot << c);
      if (!fs) {
        fs = late;
        late = 0;
      }
      over = full = !met && !won && !fs;
    }
    claimed += won;
    if (over) {
      const uint32_t p = full ? atomicAdd(&nleft, 1u) : ~0u;
      if (p < (uint32_t)kPartLeft) {
        left[p] = j;
      } else {
        P.flag[idx[e]] = kFlagLeft;
        *P.nover = 1;
      }
    } else if (w[2 * kSlots] >> c & 1u) {  // there before the batch
      P.flag[idx[e]] = kFlagNone;
      if (status) status[idx[e]] = kPresent;
    } else {
      slot[e] = at + 2 * c + 1;
      atomicMin(&w[2 * c + 1], (unsigned long long)idx[e]);
    }
  }
  __syncthreads();
  const uint32_t c = (uint32_t)(f >> P.lp2);
  const uint32_t nl = min(nleft, (uint32_t)kPartLeft);
  if (threadIdx.x == 0 && nl) lbase = aadd32(&P.nleft[c * kCtrStride], nl);
#pragma unroll
  for (int e = 0; e < kPartPer; ++e) {
    if (slot[e] && L[slot[e]] != idx[e]) {  // a lower copy stores the key
      slot[e] = 0;
      P.flag[idx[e]] = kFlagNone;
      if (status) status[idx[e]] = kPresent;
    }
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kPartPer; ++e)
    if (slot[e]) L[slot[e]] = VK ? val[e] : 0;
  __syncthreads();
  for (int j = threadIdx.x; j < nslots; j += kPartThreads) {
    const uint64_t* w = &L[(j >> 3) * kPartStride + 2 * (j & 7)];
    Slot sl;
    sl.key = w[0];
    sl.val = sl.key < kTomb ? w[1] : 0;
    slots[j] = sl;
  }
  const int64_t tot = block_sum<kPartThreads>((int64_t)claimed);
  if (threadIdx.x == 0) spec_count(t, blockIdx.x, tot << 32);
  const int64_t dst = (int64_t)c * kBinSub * P.c1 + lbase;  // the coarse bin has been taken apart
  for (uint32_t j = threadIdx.x; j < nl; j += kPartThreads) {
    P.r1k[dst + j] = P.r2k[src + left[j]];
    if (VK) store_val<VK>(P.r1v, dst + j, load_val<VK>(P.r2v, src + left[j]));
    P.r1i[dst + j] = P.r2i[src + left[j]];
  }
}

// One left-over element per lane, by the ordinary probe.  Returns (stored, listed).
template <int VK>
__device__ __forceinline__ uint2 part_place(const TableView& t, const PartView& P, bool mine, uint64_t key,
                                            uint64_t val, int64_t i, uint32_t inject, bool home_full,
                                            uint8_t* __restrict__ status) {
  const Place p = place_keys<true, false, false>(t, wave_lds<kBlock>(), mine, key, true, inject,
                                                 home_full);
  if (!mine) return make_uint2(0, 0);
  uint8_t f = kFlagClaimed;
  if (p.found) {
    f = kFlagListed;
    if (status) status[i] = kPresent;
  } else if (p.pos == kNoPos) {
    f = kFlagNone;  // no free slot anywhere: cannot happen below capacity
    if (status) status[i] = kFull;
    aor32(&t.hdr->err, kErrFull);
  } else if (VK) {
    t.bk[p.pos >> 3].s[p.pos & 7].val = val;
  }
  if (!home_full || f != kFlagClaimed) P.flag[i] = f;  // (else it is kFlagSure)
  return make_uint2(f == kFlagClaimed, f == kFlagListed);
}

// The left-over lists of the coarse bins, `blocks` blocks each: keys whose home bucket is full.
// Random claims again, 4.6 million of 2^26 keys in 0.36 ms; with their indices alone in the lists,
// keys and values gathered from the batch and the home bucket probed again, 0.78.
template <int VK>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(5))) void k_part_left(TableView t, PartView P, int blocks,
                                                                         uint8_t* __restrict__ status) {
  const uint32_t c = blockIdx.x / (uint32_t)blocks;
  const uint32_t m = P.nleft[c * kCtrStride];
  const int64_t src = (int64_t)c * kBinSub * P.c1;
  const uint32_t inject = __builtin_amdgcn_readfirstlane(t.hdr->inject);
  uint32_t claimed = 0, listed = 0;
  for (uint32_t j0 = blockIdx.x % (uint32_t)blocks * kBlock + (threadIdx.x & ~63u); j0 < m;
       j0 += (uint32_t)blocks * kBlock) {
    const uint32_t j = min(j0 + (uint32_t)wave_lane(), m - 1u);
    const uint2 n = part_place<VK>(t, P, j0 + wave_lane() < m, P.r1k[src + j], load_val<VK>(P.r1v, src + j),
                                   P.r1i[src + j], inject, true, status);
    claimed += n.x;
    listed += n.y;
  }
  if (listed) *P.nover = 1;
  const int64_t tot = block_sum(((int64_t)claimed << 32) + (int64_t)listed);
  if (threadIdx.x == 0) spec_count(t, blockIdx.x, tot);
}

// The elements marked kFlagLeft: a block gathers those of a window of flags.  Copies of a key may be
// listed from here on, so every claimer's flag becomes kFlagClaimed.
template <int VK>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(5))) void k_part_over(TableView t, PartView P,
                                                                         const uint64_t* __restrict__ keys,
                                                                         const void* __restrict__ vals, int64_t n,
                                                                         uint8_t* __restrict__ status) {
  if (*P.nover == 0) return;
  __shared__ uint16_t list[kPartWindow];
  __shared__ uint32_t m;
  const uint32_t inject = __builtin_amdgcn_readfirstlane(t.hdr->inject);
  uint32_t claimed = 0, listed = 0;
  for (int64_t w0 = (int64_t)blockIdx.x * kPartWindow; w0 < n; w0 += (int64_t)gridDim.x * kPartWindow) {
    if (threadIdx.x == 0) m = 0;
    __syncthreads();
    const int64_t i0 = w0 + 8 * (int)threadIdx.x;
    // (the flags are laid out to a multiple of 8)
    const uint64_t f = i0 < n ? *reinterpret_cast<const uint64_t*>(P.flag + i0) : 0;
    uint64_t is = f & (f >> 1) & 0x0101010101010101ull;  // kFlagLeft alone has both bits
    if (n - i0 < 8 && i0 < n) is &= (1ull << (8 * (int)(n - i0))) - 1;
    const uint64_t sure = f & 0x0404040404040404ull;
    if (sure) *reinterpret_cast<uint64_t*>(P.flag + i0) = (f ^ sure) | sure >> 2;
    uint32_t at = is ? atomicAdd(&m, (uint32_t)__popcll(is)) : 0u;
    for (; is; is &= is - 1) list[at++] = (uint16_t)(8 * threadIdx.x + (__builtin_ctzll(is) >> 3));
    __syncthreads();
    const uint32_t mm = m;
    for (uint32_t j0 = threadIdx.x & ~63u; j0 < mm; j0 += kBlock) {
      const uint32_t j = j0 + wave_lane();
      const int64_t i = w0 + list[min(j, mm - 1u)];
      const uint2 c = part_place<VK>(t, P, j < mm, keys[i], load_val<VK>(vals, i), i, inject, false, status);
      claimed += c.x;
      listed += c.y;
    }
    __syncthreads();  // the list is refilled
  }
  const int64_t tot = block_sum(((int64_t)claimed << 32) + (int64_t)listed);
  if (threadIdx.x == 0) spec_count(t, blockIdx.x, tot);
}

// Flagged count per tile of kTile elements, for grids that do not settle (a launch costs these less than
// counting in the insert kernel: 4 M repeated keys into a set, 380 us against 386).
__global__ __launch_bounds__(kBlock) void k_tile_count(TableView t, int64_t q) {
  if (t.hdr->fast) return;
  __shared__ uint32_t part[kBlock / 64];
  const int64_t t0 = (int64_t)blockIdx.x * kTile;
  uint64_t c = 0;
  for (int j = threadIdx.x; j < kTile; j += kBlock) {
    const int64_t i = t0 + j;
    if (i < q) c += t.flag[i];
  }
  c = wave_sum(c);
  if (wave_lane() == 0) part[threadIdx.x >> 6] = (uint32_t)c;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t s = 0;
    for (int w = 0; w < kBlock / 64; ++w) s += part[w];
    t.tsum[blockIdx.x] = s;
  }
}

// One block of NT threads: exclusive scan of the tile counts, then the counter updates the ranks
// imply.  mode 0: insert near capacity; 1: insert with pool values; 2: erase releasing to the pool.
// A chunk's totals once its nnew new actors are ranked: the live count, the pool top and the
// error bits (mode 0 insert near capacity, 1 insert with pool values, 2 erase releasing to the
// pool).  One thread.
__device__ __forceinline__ void rank_totals(const TableView& t, PoolHeader* pool, uint64_t nnew,
                                            int mode) {
  Header* h = t.hdr;
  h->nnew = (uint32_t)nnew;
  const uint64_t room = t.cap - h->size0;
  if (mode == 0) {
    const uint64_t ins = nnew < room ? nnew : room;
    h->size = h->size0 + ins;
    if (nnew > room) h->err |= kErrFull;
  } else if (mode == 1) {
    const uint64_t avail = (uint64_t)pool->top0;
    const uint64_t lim = room < avail ? room : avail;
    const uint64_t ins = nnew < lim ? nnew : lim;
    h->size = h->size0 + ins;
    pool->top = pool->top0 - (int64_t)ins;
    if (nnew > lim) {
      if (room <= avail) h->err |= kErrFull;
      else h->err |= kErrPool;
    }
  } else {
    h->size = h->size0 - nnew;  // every flagged element removed its key
    const uint64_t room_p = (uint64_t)(pool->cap - pool->top0);
    const uint64_t pushed = nnew < room_p ? nnew : room_p;
    pool->top = pool->top0 + (int64_t)pushed;
    if (nnew > room_p) pool->err |= kErrPool;
  }
}

template <int NT>
__device__ __forceinline__ void scan_tiles_block(const TableView& t, PoolHeader* pool, int ntiles,
                                                 int mode) {
  __shared__ uint32_t carry;
  __shared__ uint32_t ws[NT / 64];
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int base = 0; base < ntiles; base += NT) {
    const int j = base + (int)threadIdx.x;
    const uint32_t v = j < ntiles ? t.tsum[j] : 0u;
    const int lane = wave_lane();
    uint32_t x = v;
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t y = __shfl_up(x, off, 64);
      if (lane >= off) x += y;
    }
    if (lane == 63) ws[threadIdx.x >> 6] = x;
    __syncthreads();
    uint32_t before = 0, all = 0;
    for (int w = 0; w < NT / 64; ++w) {
      if (w < (int)(threadIdx.x >> 6)) before += ws[w];
      all += ws[w];
    }
    if (j < ntiles) t.tsum[j] = carry + before + x - v;
    __syncthreads();
    if (threadIdx.x == 0) carry += all;
    __syncthreads();
  }
  if (threadIdx.x == 0) rank_totals(t, pool, carry, mode);
  __syncthreads();
}

__global__ __launch_bounds__(1024) void k_tile_scan(TableView t, PoolHeader* pool, int ntiles,
                                                    int mode) {
  if (mode == 0 && t.hdr->fast) return;
  scan_tiles_block<1024>(t, pool, ntiles, mode);
}

// Ranked completion of flagged elements, one tile per block.
// MODE 0: insert near capacity (rank < room -> claim, else FULL)
// MODE 1: insert with pool values (rank < min(room, pool) -> value = pool element top0-1-rank)
// MODE 2: erase releasing to the pool (pool element top0+rank = value)
// (the batch moves only the back of the pool: head is fixed while it runs)
template <int VK, int MODE>
__device__ __forceinline__ void final_tile(const TableView& t, WaveLds* w, PoolHeader* pool,
                                           int32_t* __restrict__ pstack,
                                           const uint64_t* __restrict__ keys,
                                           const void* __restrict__ vals, int64_t q,
                                           uint8_t* __restrict__ status,
                                           int32_t* __restrict__ vout, int64_t tile,
                                           int inline_tiles) {
  const bool fast = t.hdr->fast != 0;
  if (MODE == 0 && fast) return;
  __shared__ uint16_t list[kTile];
  const int64_t t0 = tile * kTile;
  uint32_t f[kTile / kBlock];
  uint32_t cnt = 0;
#pragma unroll
  for (int k = 0; k < kTile / kBlock; ++k) {
    const int64_t i = t0 + (int64_t)threadIdx.x * (kTile / kBlock) + k;
    f[k] = i < q ? t.flag[i] : 0u;
    cnt += f[k];
  }
  uint32_t total;
  uint32_t o = block_exclusive_scan(cnt, &total);
#pragma unroll
  for (int k = 0; k < kTile / kBlock; ++k)
    if (f[k]) list[o++] = (uint16_t)(threadIdx.x * (kTile / kBlock) + k);
  __syncthreads();
  // inline_tiles == 0: the tile sums hold the rank scan's exclusive prefixes.  inline_tiles = n > 0
  // (small chunks, no scan launched): they hold the n tiles' counts; each block adds those before
  // its tile, and the block of tile 0 also settles the chunk's totals as the scan would.
  uint64_t rbase;
  if (inline_tiles > 0) {
    __shared__ uint64_t rb_shared;
    uint64_t before = 0, all = 0;
    for (int j = threadIdx.x; j < inline_tiles; j += kBlock) {
      const uint64_t c = t.tsum[j];
      all += c;
      if (j < tile) before += c;
    }
    before = (uint64_t)block_sum((int64_t)before);
    __syncthreads();  // block_sum's partials are reused
    all = (uint64_t)block_sum((int64_t)all);
    if (threadIdx.x == 0) {
      rb_shared = before;
      if (tile == 0) rank_totals(t, pool, all, MODE);
    }
    __syncthreads();
    rbase = rb_shared;
  } else {
    rbase = t.tsum[tile];
  }
  const Header* h = t.hdr;
  const uint64_t room = t.cap - h->size0;
  // One lane per element throughout.  Where nothing is left to claim (a release, or new keys that
  // hold their slot already), the elements only move values: eight lanes per element took 20.5 us
  // for the 26,214 releases of a voxel frame, now 5.4.  New keys that still need a slot are placed
  // 64 at a time: 4 M repeated keys into a set took 127 us here with eight lanes per key, now 80.
  const bool moves = MODE == 2 || (MODE == 1 && fast);
  int64_t top0 = 0, head = 0, pcap = 0;
  if (MODE != 0) {
    top0 = pool->top0;
    head = pool->head;
    pcap = pool->cap;
  }
  const uint64_t lim = MODE == 1 && (uint64_t)top0 < room ? (uint64_t)top0 : room;
  for (uint32_t j0 = threadIdx.x & ~63u; j0 < total; j0 += kBlock) {
    const uint32_t j = j0 + (uint32_t)wave_lane();
    const bool mine = j < total;
    const int64_t i = t0 + (mine ? list[j] : list[0]);
    const uint64_t rank = rbase + j;
    if constexpr (MODE == 2) {
      const int64_t pos = top0 + (int64_t)rank;
      if (mine && pos < pcap) pstack[ring_pos(head, pcap, pos)] = (int32_t)(uint32_t)t.ref[i];
    } else {
      const bool stored = mine && rank < lim;
      uint64_t v = 0;
      if (stored) {
        if constexpr (MODE == 1) v = (uint64_t)(uint32_t)pstack[ring_pos(head, pcap, top0 - 1 - (int64_t)rank)];
        else v = load_val<VK>(vals, i);
      }
      uint64_t pos = kNoPos;
      if (moves) {
        if (stored) pos = t.ref[i];
      } else {
        const uint64_t key = keys[i];
        const Place p = place_keys<true, false, false>(t, w, stored && key < kTomb, key, true, 0);
        pos = p.pos;
        if (stored && key >= kTomb) {
          pos = kSpecRef + (key - kTomb);
          t.hdr->spec_live[key - kTomb] = 1;
        }
      }
      if (stored && pos != kNoPos) {
        if (pos >= kSpecRef) t.hdr->spec_val[pos - kSpecRef] = v;
        else if (VK || MODE == 1) t.bk[pos >> 3].s[pos & 7].val = v;
      }
      if (mine) {
        if (status) status[i] = pos == kNoPos ? kFull : kInserted;
        if (MODE == 1 && vout) vout[i] = pos == kNoPos ? -1 : (int32_t)(uint32_t)v;
      }
    }
  }
  __syncthreads();  // the tile list is reused by the caller's next tile
}

template <int VK, int MODE>
__global__ __launch_bounds__(kBlock) void k_final(TableView t, PoolHeader* pool,
                                                  int32_t* __restrict__ pstack,
                                                  const uint64_t* __restrict__ keys,
                                                  const void* __restrict__ vals, int64_t q,
                                                  uint8_t* __restrict__ status,
                                                  int32_t* __restrict__ vout, int inline_tiles) {
  final_tile<VK, MODE>(t, MODE == 2 ? nullptr : wave_lds<kBlock>(), pool, pstack, keys, vals, q, status, vout, blockIdx.x, inline_tiles);
}

// Later copies of a key take the outcome of its first occurrence: PRESENT (or its value), unless
// the first occurrence met FULL, which a later copy meets again.  Reads the marks of all q
// elements, four per thread (they are cleared in units of 16): a list of the later copies would
// cost the insert kernel one atomic on one address per wave, 12.6 ns each (a pool-valued insert of
// 2^19 samples, each block met four times, took 131 us with such a list and takes 19 without; this
// kernel went from 9 to 11).
// A thread's four look-ups of a first copy are in flight together, and while the chunk cannot meet
// FULL nothing reads the first copy's status.
__device__ __forceinline__ void fix_range(const TableView& t, int64_t q, uint8_t* __restrict__ status,
                                          int32_t* __restrict__ vout, int64_t lo, int64_t step) {
  const int64_t units = (q + 3) / 4;
  const bool fast = t.hdr->fast != 0;
  for (int64_t j = lo + threadIdx.x; j < units; j += step) {
    const uint32_t m = reinterpret_cast<const uint32_t*>(t.dmark)[j];
    if (!m) continue;
    const uint4 d = reinterpret_cast<const uint4*>(t.dup)[j];
    const uint32_t i = (uint32_t)(4 * j);
    uint32_t f[4] = {d.x, d.y, d.z, d.w};
    int32_t v[4] = {};
    uint8_t st[4] = {};
#pragma unroll
    for (int k = 0; k < 4; ++k)  // the first copy, or this element where there is no other
      if (!((m >> (8 * k)) & 0xFFu) || (int64_t)i + k >= q) f[k] = i;
    if (vout)
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = vout[f[k]];
    if (status && !fast)
#pragma unroll
      for (int k = 0; k < 4; ++k) st[k] = status[f[k]];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (!((m >> (8 * k)) & 0xFFu) || (int64_t)i + k >= q || f[k] == i + k) continue;
      if (vout) vout[i + k] = v[k];
      if (status) status[i + k] = st[k] == kFull ? kFull : kPresent;
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_fix(TableView t, int64_t q, uint8_t* __restrict__ status,
                                                int32_t* __restrict__ vout, int alloc) {
  if (t.hdr->spec) return;
  if (!alloc && t.hdr->fast) return;  // the insert kernel knew their outcome
  fix_range(t, q, status, vout, (int64_t)blockIdx.x * kBlock, (int64_t)gridDim.x * kBlock);
}

// ---------------------------------------------------------------------------------------------
// Small batches: the whole operation in one launch of one workgroup.
//
// What bounds a batch of some hundred keys is launches, not work: the pipelines above take 5 to 8
// of them, 3 to 4 us each.  Here one workgroup finds the repeated keys in LDS, places the first
// copies, ranks the new ones in index order where capacity or a pool asks for it, gives the later
// copies their outcome, and settles the counters.  kSmallPer elements per thread, element
// e * blockDim + tid, so index order is (e, wave, lane).
// ---------------------------------------------------------------------------------------------
enum SmallOp : int { sInsert, sAlloc, sErase, sRelease };
constexpr int kSmallPer = 2;
constexpr int kSmallMax = 1024 * kSmallPer;

// hslots: a power of two >= 2 n (repeated-key table, load at most one half).
// The loops over a thread's elements stay rolled, with the elements' state in LDS, and both placing
// passes share one copy of place_keys: such a launch runs its code once, so instruction fetch is
// part of its time.  500 keys erased, inserted and partly looked up: 62 us as 15 launches, 28 as 3,
// of which the inserts' kernel is 16.7 us and the erases' 9 (22 and 9.6 without reading ahead).
template <int VK, int OP>
__global__ __launch_bounds__(1024) void k_small(TableView t, PoolHeader* pool,
                                                int32_t* __restrict__ pstack,
                                                const uint64_t* __restrict__ keys,
                                                const uint8_t* __restrict__ skip,
                                                const void* __restrict__ vals, int32_t n,
                                                uint32_t hslots, uint8_t* __restrict__ status,
                                                int32_t* __restrict__ vout) {
  constexpr bool kIns = OP == sInsert || OP == sAlloc;
  constexpr bool kPool = OP == sAlloc || OP == sRelease;
  __shared__ uint64_t lk[kSmallMax];       // by index: key
  __shared__ uint64_t rf[kSmallMax];       //   slot of a new key, value released, value allocated
  __shared__ uint32_t H[2 * kSmallMax];    // repeated-key table: lowest index of the slot's key
  __shared__ uint16_t fst[kSmallMax];      //   H slot of the key, then index of its first copy
  __shared__ uint16_t rk[kSmallMax];       //   rank among the flagged
  __shared__ uint8_t ost[kSmallMax];       //   outcome
  __shared__ uint8_t flg[kSmallMax];       //   takes part in the ranking
  __shared__ uint32_t sfirst[2], flagged[kSmallPer][16], changed_sum;
  constexpr uint16_t kSkipped = 0xFFFF;
  WaveLds* w = wave_lds<1024>();
  Header* hdr = t.hdr;
  const int bd = (int)blockDim.x, tid = (int)threadIdx.x, wave = tid >> 6;
  const uint64_t size0 = hdr->size;
  const uint64_t room = t.cap - size0;
  const uint32_t inject = kIns ? __builtin_amdgcn_readfirstlane(hdr->inject) : 0u;
  int64_t top0 = 0, head = 0, pcap = 0;
  if (kPool) {
    top0 = pool->top;
    head = pool->head;
    pcap = pool->cap;
  }
  // no element can meet FULL: a new key claims its slot at once
  const bool fast = size0 + (uint64_t)n <= t.cap && (OP != sAlloc || top0 >= n);
  const uint64_t lim = OP == sAlloc && (uint64_t)top0 < room ? (uint64_t)top0 : room;

  for (uint32_t j = tid; j < hslots; j += bd) H[j] = kNone;
  if (tid < 2) sfirst[tid] = kNone;
  if (tid == 2) changed_sum = 0;
#pragma unroll 1
  for (int i = tid; i < n; i += bd) lk[i] = keys[i];
  __syncthreads();
#pragma unroll 1
  for (int i = tid; i < n; i += bd) {
    const uint64_t key = lk[i];
    uint32_t s = 0;
    if (skip && skip[i]) {
      s = kSkipped;
    } else if (key >= kTomb) {
      atomicMin(&sfirst[key - kTomb], (uint32_t)i);
    } else {
      s = (uint32_t)dedup_mix(key) & (hslots - 1);
      for (;;) {  // at most n keys in 2 n slots: a free or matching slot exists
        const uint32_t prev = atomicCAS(&H[s], kNone, (uint32_t)i);
        if (prev == kNone) break;
        if (lk[prev] == key) {
          atomicMin(&H[s], (uint32_t)i);
          break;
        }
        s = (s + 1) & (hslots - 1);
      }
    }
    fst[i] = (uint16_t)s;
  }
  __syncthreads();

  uint32_t changed = 0, nnew = 0;
  const bool ranked = kPool || !fast;
  // pass 0: probe the first copies (and claim, while FULL is out of the question); pass 1, for
  // inserts that may meet FULL: the first `lim` new keys in index order claim
  const int passes = kIns && !fast ? 2 : 1;
#pragma unroll 1
  for (int pass = 0; pass < passes; ++pass) {
#pragma unroll 1
    for (int e = 0; e * bd < n; ++e) {
      const int i = e * bd + tid;
      const uint64_t key = i < n ? lk[i] : 0;
      const bool special = key >= kTomb;
      bool mine = false;
      if (i < n) {
        if (pass == 0) {
          const uint32_t s = fst[i];
          const uint32_t first = s == kSkipped ? (uint32_t)kSkipped
                                 : special ? sfirst[key - kTomb] : H[s];
          fst[i] = (uint16_t)first;
          mine = first == (uint32_t)i;
        } else {
          mine = flg[i] && rk[i] < lim;
        }
      }
      const Place p = place_keys<kIns, kPool, true>(t, w, mine && !special, key, kIns && (fast || pass),
                                                    inject);
      bool found = p.found;
      uint64_t val = p.val, pos = p.pos;
      if (mine && special) {
        found = pass == 0 && hdr->spec_live[key - kTomb] != 0;
        val = hdr->spec_val[key - kTomb];
        pos = kSpecRef + (key - kTomb);
      }
      bool flag = false;
      uint8_t st = kIns ? (uint8_t)kPresent : (uint8_t)0;
      if (mine) {
        if constexpr (kIns) {
          if (!found && !fast && pass == 0) {
            flag = true;      // FULL unless pass 1 stores it
            st = kFull;
            val = ~0ull;
          } else if (!found && pos == kNoPos) {
            st = kFull;       // no free slot anywhere: cannot happen below capacity
            aor32(&hdr->err, kErrFull);
          } else if (!found) {
            st = kInserted;
            flag = true;
            ++changed;
            val = pos;
            if (OP == sInsert) {
              const uint64_t v = load_val<VK>(vals, i);
              if (special) {
                hdr->spec_live[key - kTomb] = 1;
                hdr->spec_val[key - kTomb] = v;
              } else if (VK) {
                t.bk[pos >> 3].s[pos & 7].val = v;
              }
            }
          }
        } else if (found) {
          if (special) hdr->spec_live[key - kTomb] = 0;
          // kEmpty only where the bucket already holds one: no probe sequence runs through it
          else t.bk[pos >> 3].s[pos & 7].key = p.had_empty ? kEmpty : kTomb;
          st = 1;
          flag = true;
          ++changed;
        }
        rf[i] = val;
        ost[i] = st;
      }
      if (pass == 0 && ranked) {
        if (i < n) flg[i] = flag;
        const uint64_t m = __ballot(flag);
        if (wave_lane() == 0) flagged[e][wave] = (uint32_t)__builtin_popcountll(m);
        if (flag) rk[i] = (uint16_t)__builtin_popcountll(m & ((1ull << wave_lane()) - 1ull));
      }
    }
    if (pass == 0 && ranked) {  // ranks in index order: (element, wave, lane)
      __syncthreads();
#pragma unroll 1
      for (int e = 0; e * bd < n; ++e) {
        const int i = e * bd + tid;
        for (int v = 0; v < (bd >> 6); ++v) {
          if (v == wave && i < n && flg[i]) rk[i] = (uint16_t)(rk[i] + nnew);
          nnew += flagged[e][v];
        }
      }
    }
  }
  if (kPool) {  // (each thread's own elements: no barrier needed)
#pragma unroll 1
    for (int i = tid; i < n; i += bd) {
      if (!flg[i]) continue;
      const int64_t r = rk[i];
      if (OP == sRelease) {
        const int64_t at = top0 + r;
        if (at < pcap) pstack[ring_pos(head, pcap, at)] = (int32_t)(uint32_t)rf[i];
      } else if (ost[i] == kInserted) {
        const uint32_t v = (uint32_t)pstack[ring_pos(head, pcap, top0 - 1 - r)];
        const uint64_t pos = rf[i];
        if (pos >= kSpecRef) {
          hdr->spec_live[pos - kSpecRef] = 1;
          hdr->spec_val[pos - kSpecRef] = v;
        } else {
          t.bk[pos >> 3].s[pos & 7].val = v;
        }
        rf[i] = v;
      }
    }
  }
  const uint64_t sum = wave_sum(changed);
  if (wave_lane() == 0 && sum) atomicAdd(&changed_sum, (uint32_t)sum);
  __syncthreads();
#pragma unroll 1
  for (int i = tid; i < n; i += bd) {  // later copies take the outcome of the first
    const uint32_t f = fst[i];
    if (f == kSkipped) continue;
    uint8_t st = ost[f];
    if (f != (uint32_t)i) st = kIns ? (st == kFull ? kFull : kPresent) : 0;
    if (status) status[i] = st;
    if (OP == sAlloc && vout) vout[i] = (int32_t)(uint32_t)rf[f];
  }
  if (tid == 0) {
    hdr->size0 = size0;
    if (kPool) pool->top0 = top0;
    if (OP == sAlloc) rank_totals(t, pool, nnew, 1);
    else if (OP == sRelease) rank_totals(t, pool, nnew, 2);
    else if (kIns && !fast) rank_totals(t, nullptr, nnew, 0);
    else hdr->size = kIns ? size0 + changed_sum : size0 - changed_sum;
    if (OP == sErase) chunk_feedback(t, 1, n, changed_sum);
    if (OP == sInsert && fast) chunk_feedback(t, 0, n, changed_sum);
  }
}

// find / contains: a wave takes 64 consecutive keys, one per lane (coalesced loads and stores), and
// probes them in rounds until every lane has its answer.
template <int VK>
__device__ __forceinline__ void find_range(const TableView& t, WaveLds* w,
                                           const uint64_t* __restrict__ keys, void* __restrict__ out,
                                           uint8_t* __restrict__ found_out, int64_t lo, int64_t hi,
                                           int64_t step) {
  for (int64_t w0 = lo + (int64_t)(threadIdx.x & ~63u); w0 < hi; w0 += step) {
    const int64_t i = w0 + wave_lane();
    const bool valid = i < hi;
    const uint64_t key = keys[min(i, hi - 1)];
    bool look = valid && key < kTomb;
    bool hit = false;
    uint64_t v = 0;
    if (valid && !look) {
      hit = t.hdr->spec_live[key - kTomb] != 0;
      v = t.hdr->spec_val[key - kTomb];
    }
    const Seq q = probe_seq(t, key);
    uint32_t b = (uint32_t)q.home;
    uint32_t left = (uint32_t)t.nb;
    for (uint64_t mask = __ballot(look); mask; mask = __ballot(look)) {
      uint64_t val = 0;
      const ProbeRound<false, VK != 0, false> round(t, w, mask, look, key, b, 0);
      const uint32_t x = round.answer(0, &val);
      if (look) {
        if (x & kBitsMatch) {
          hit = true;
          v = val;
        }
        look = x == 0 && --left != 0;
        b = next_bucket32(t, b, (uint32_t)q.step);
      }
    }
    if (valid) {
      if (out) store_val<VK>(out, i, hit ? v : sentinel<VK>());
      if (found_out) found_out[i] = hit ? 1 : 0;
    }
  }
}

// Held to 7 waves per SIMD (72 VGPRs, no spills): 2^27 Zipf lookups in the 2^26-key table took
// 2.27 ms at 7 waves, 2.37 at 6, 2.60 at 5 (the compiler's choice) and 2.66 at 8, which spills;
// probing eight keys per 8-lane group with a ballot per key and no packing took 3.51 ms.  Uniform
// lookups (2^26 keys): 2.04 ms at 6 and 7, 2.33 ms before; 2^24 in a 2^20-key table 0.31, 0.40 before.
template <int VK>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(7))) void k_find(TableView t, const uint64_t* __restrict__ keys,
                                                 int64_t n, void* __restrict__ out,
                                                 uint8_t* __restrict__ found_out) {
  find_range<VK>(t, wave_lds<kBlock>(), keys, out, found_out, (int64_t)blockIdx.x * kBlock, n,
                 (int64_t)gridDim.x * kBlock);
}

// Range selection (Section 3.6: a range of the container becomes a vector through a copy_if),
// and the dump, which selects every live pair.  Appending through one shared counter serialises
// (every append is an atomic on the same address), so block b owns a contiguous slot range:
// k_sel_count writes its count to bcnt[b], k_sel_scan turns the counts into offsets (and the
// total, out-of-band keys included, into dump_count), and k_sel_write reads the range again and
// writes each accepted pair at its block's offset plus its rank in the block.  The out-of-band
// keys go last.  Predicates see the key only.
struct AllKeys {
  __device__ bool operator()(uint64_t) const { return true; }
};
struct KeyRange {
  uint64_t lo, hi;  // lo <= key < hi, unsigned
  __device__ bool operator()(uint64_t key) const { return key >= lo && key < hi; }
};
struct VoxelBox {
  int32_t lo[3], hi[3];  // packed block coordinates in [lo, hi], bounds included
  __device__ bool operator()(uint64_t key) const {
    if (key >> 63) return false;  // packs no block
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const uint32_t f = (uint32_t)(key >> (21 * d)) & 0x1FFFFFu;
      const int32_t c = (int32_t)(f << 11) >> 11;  // sign-extend the 21-bit field
      if (c < lo[d] || c > hi[d]) return false;
    }
    return true;
  }
};

constexpr int kSelPer = 8;                       // slots per thread and round
constexpr int64_t kSelRound = (int64_t)kBlock * kSelPer;

template <class Pred>
__device__ __forceinline__ uint32_t sel_round(const TableView& t, const Pred& pred, int64_t r0,
                                              int64_t hi, Slot (&sl)[kSelPer]) {
  uint32_t take = 0;
#pragma unroll
  for (int e = 0; e < kSelPer; ++e) {   // loads first (clamped), then the tests
    const int64_t j = min(r0 + e * kBlock + (int64_t)threadIdx.x, hi - 1);
    sl[e] = t.bk[j >> 3].s[j & 7];
  }
#pragma unroll
  for (int e = 0; e < kSelPer; ++e) {
    const int64_t j = r0 + e * kBlock + (int64_t)threadIdx.x;
    if (j < hi && sl[e].key != kEmpty && sl[e].key != kTomb && pred(sl[e].key)) take |= 1u << e;
  }
  return take;
}

template <class Pred>
__global__ __launch_bounds__(kBlock) void k_sel_count(TableView t, Pred pred, int64_t per) {
  const int64_t nslots = (int64_t)t.nb * kSlots;
  const int64_t lo = (int64_t)blockIdx.x * per;
  const int64_t hi = min(lo + per, nslots);
  int64_t c = 0;
  Slot sl[kSelPer];
  for (int64_t r0 = lo; r0 < hi; r0 += kSelRound) c += __builtin_popcount(sel_round(t, pred, r0, hi, sl));
  const int64_t tot = block_sum(c);
  if (threadIdx.x == 0) t.bcnt[blockIdx.x] = tot;
}

template <class Pred>
__global__ __launch_bounds__(1024) void k_sel_scan(TableView t, Pred pred, int nblocks) {
  __shared__ int64_t wsum[16];
  const int per = (nblocks + 1023) / 1024;
  const int b0 = (int)threadIdx.x * per;
  int64_t loc = 0;
  for (int j = 0; j < per; ++j)
    if (b0 + j < nblocks) loc += t.bcnt[b0 + j];
  const int lane = wave_lane();
  int64_t x = loc;
  for (int off = 1; off < 64; off <<= 1) {
    const int64_t y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  if (lane == 63) wsum[threadIdx.x >> 6] = x;
  __syncthreads();
  int64_t before = 0, total = 0;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
    if (w < (int)(threadIdx.x >> 6)) before += wsum[w];
    total += wsum[w];
  }
  int64_t run = before + x - loc;
  for (int j = 0; j < per; ++j) {
    if (b0 + j >= nblocks) break;
    const int64_t c = t.bcnt[b0 + j];
    t.bcnt[b0 + j] = run;
    run += c;
  }
  if (threadIdx.x == 0) {
    for (int sp = 0; sp < 2; ++sp)
      if (t.hdr->spec_live[sp] && pred(kTomb + (uint64_t)sp)) ++total;
    t.hdr->dump_count = (uint64_t)total;
  }
}

template <class Pred>
__global__ __launch_bounds__(kBlock) void k_sel_write(TableView t, Pred pred, int64_t per,
                                                      uint64_t* __restrict__ kout,
                                                      uint64_t* __restrict__ vout, int64_t cap) {
  const int64_t nslots = (int64_t)t.nb * kSlots;
  const int64_t lo = (int64_t)blockIdx.x * per;
  const int64_t hi = min(lo + per, nslots);
  int64_t off = t.bcnt[blockIdx.x];
  Slot sl[kSelPer];
  for (int64_t r0 = lo; r0 < hi; r0 += kSelRound) {
    const uint32_t take = sel_round(t, pred, r0, hi, sl);
    uint32_t total;
    uint32_t p = block_exclusive_scan((uint32_t)__builtin_popcount(take), &total);
#pragma unroll
    for (int e = 0; e < kSelPer; ++e) {
      if (!((take >> e) & 1u)) continue;
      const int64_t at = off + p++;
      if (at < cap) {
        kout[at] = sl[e].key;
        if (vout) vout[at] = sl[e].val;
      }
    }
    off += total;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {  // the out-of-band keys, after every bucket's
    int64_t at = (int64_t)t.hdr->dump_count;
    for (int sp = 0; sp < 2; ++sp)
      if (t.hdr->spec_live[sp] && pred(kTomb + (uint64_t)sp)) --at;
    for (int sp = 0; sp < 2; ++sp) {
      if (!t.hdr->spec_live[sp] || !pred(kTomb + (uint64_t)sp)) continue;
      if (at < cap) {
        kout[at] = kTomb + (uint64_t)sp;
        if (vout) vout[at] = t.hdr->spec_val[sp];
      }
      ++at;
    }
  }
}

// Set-up and fold of a striped launch of the reference kernels below: zero the stripes and decide
// whether the launch can meet the capacity (the live count plus `maxins` inserts), then add the
// stripes to the live count.  The decision is one word that every wave of the launch reads.
__global__ __launch_bounds__(64) void k_dev_prep(TableView t, uint64_t maxins) {
  t.bcnt[threadIdx.x * kStripeStride] = 0;
  if (threadIdx.x == 0) {
    const uint64_t n = t.hdr->size;
    t.bcnt[kStripeFlag] = (n <= t.cap && maxins <= t.cap - n) ? 1 : 0;
  }
}

__global__ __launch_bounds__(64) void k_dev_fold(TableView t) {
  if (!t.bcnt[kStripeFlag]) return;
  const uint64_t s = wave_sum((uint64_t)t.bcnt[threadIdx.x * kStripeStride]);
  if (threadIdx.x == 0) t.hdr->size += s;
}

// One element of the reference kernels below: operation `op` on keys[i] through the device
// functions, its status (and found value) written at i.
__device__ __forceinline__ void dev_apply_one(const DevView& v, int32_t op, int64_t i, uint64_t key,
                                              const void* __restrict__ vals, int32_t vk,
                                              void* __restrict__ vout, uint8_t* __restrict__ status) {
  if (op == CT_OP_INSERT) {
    const uint64_t val = vk == 2 ? static_cast<const uint64_t*>(vals)[i]
                         : vk == 1 ? (uint64_t)static_cast<const uint32_t*>(vals)[i] : 0ull;
    const uint8_t st = dev_insert(v, key, val);
    if (status) status[i] = st;
  } else if (op == CT_OP_ERASE) {
    const bool hit = dev_erase(v, key);
    if (status) status[i] = hit ? 1 : 0;
  } else {
    uint64_t val = 0;
    const bool hit = dev_find(v, key, &val);
    if (status) status[i] = hit ? 1 : 0;
    if (vout) {
      if (vk == 2) static_cast<uint64_t*>(vout)[i] = hit ? val : ~0ull;
      else if (vk == 1) static_cast<uint32_t*>(vout)[i] = hit ? (uint32_t)val : ~0u;
    }
  }
}

// Per-thread operations through the device-side API (ct_dev_api.h): element i is handled by one
// thread, all concurrently and in no particular order.  The reference user kernel, and what the
// tests drive the device API with.
__global__ __launch_bounds__(kBlock) void k_dev_apply(DevView v, int32_t op, const uint64_t* __restrict__ keys,
                                                      const void* __restrict__ vals, int32_t vk,
                                                      int64_t n, void* __restrict__ vout,
                                                      uint8_t* __restrict__ status) {
  if (v.striped) v.striped = (int32_t)v.t.bcnt[kStripeFlag];
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    dev_apply_one(v, op, i, keys[i], vals, vk, vout, status);
}

// The mixed-mode reference kernel: element i does operation ops[i], every element concurrently.
// A workgroup takes a window of kSortWin elements and sorts their indices by operation into LDS
// queues, then runs each queue on consecutive threads, so most waves call one device function
// with all 64 lanes and their probes go as a team.  An unknown code leaves the table alone and
// reports kNoStatus; non-find elements get the absent sentinel as their value.
constexpr int kSortWin = 4 * kBlock;

__global__ __launch_bounds__(kBlock) void k_dev_apply_sorted(DevView v, const uint8_t* __restrict__ ops,
                                                             const uint64_t* __restrict__ keys,
                                                             const void* __restrict__ vals, int32_t vk,
                                                             int64_t n, void* __restrict__ vout,
                                                             uint8_t* __restrict__ status) {
  constexpr int32_t kKind[3] = {CT_OP_FIND, CT_OP_INSERT, CT_OP_ERASE};
  __shared__ uint16_t q[3][kSortWin];
  __shared__ uint32_t qn[3];
  if (v.striped) v.striped = (int32_t)v.t.bcnt[kStripeFlag];
  const uint64_t below = (1ull << wave_lane()) - 1ull;
  const int64_t nwin = (n + kSortWin - 1) / kSortWin;
  for (int64_t w = blockIdx.x; w < nwin; w += gridDim.x) {  // the same trips for the whole block
    if (threadIdx.x < 3) qn[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortWin / kBlock; ++r) {
      const int slot = r * kBlock + (int)threadIdx.x;
      const int64_t i = w * kSortWin + slot;
      int kind = -1;
      if (i < n) {
        const int32_t op = ops[i];
        kind = op == CT_OP_FIND ? 0 : op == CT_OP_INSERT ? 1 : op == CT_OP_ERASE ? 2 : -1;
        if (vout && op != CT_OP_FIND) {
          if (vk == 2) static_cast<uint64_t*>(vout)[i] = ~0ull;
          else if (vk == 1) static_cast<uint32_t*>(vout)[i] = ~0u;
        }
        if (kind < 0 && status) status[i] = kNoStatus;
      }
      // one LDS add per wave and kind; order inside the wave by rank among the kind's lanes
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const uint64_t m = __ballot(kind == k);
        if (!m) continue;
        uint32_t base = 0;
        if (wave_lane() == __builtin_ctzll(m)) base = atomicAdd(&qn[k], (uint32_t)__builtin_popcountll(m));
        base = __shfl(base, __builtin_ctzll(m), 64);
        if (kind == k) q[k][base + (uint32_t)__builtin_popcountll(m & below)] = (uint16_t)slot;
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const uint32_t cnt = qn[k];
      for (uint32_t j = threadIdx.x; j < cnt; j += kBlock) {
        const int64_t e = w * kSortWin + q[k][j];
        dev_apply_one(v, kKind[k], e, keys[e], vals, vk, vout, status);
      }
    }
    __syncthreads();  // the queues are read before the next window refills them
  }
}

// The neighbour update of a block map (the allocation step of the reconstruction workload behind
// Section 4.1's voxel-block example): every block of `blocks` makes sure that its 6 face
// neighbours (ndirs 6) or all 26 neighbours (ndirs 26) are in the table, each new one with the
// index of a block that asked for it as its value, or (ALLOC) with pop_back() of the index pool,
// as a reconstruction allocates voxel blocks.  Coordinates wrap in their 21-bit fields.
template <bool ALLOC>
__global__ __launch_bounds__(kBlock) void k_voxel_neighbours(DevView v, DevPool pool,
                                                             const uint64_t* __restrict__ blocks,
                                                             int64_t n, int32_t ndirs) {
  if (v.striped) v.striped = (int32_t)v.t.bcnt[kStripeFlag];
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const uint64_t b = blocks[i];
    const int32_t x = sfield21(b), y = sfield21(b >> 21), z = sfield21(b >> 42);
    for (int d = 0; d < 27; ++d) {
      const int dx = d % 3 - 1, dy = (d / 3) % 3 - 1, dz = d / 9 - 1;
      const int nz = (dx != 0) + (dy != 0) + (dz != 0);
      if (nz == 0 || (ndirs == 6 && nz != 1)) continue;
      const uint64_t k = ((uint64_t)(uint32_t)(x + dx) & 0x1FFFFFull) |
                         (((uint64_t)(uint32_t)(y + dy) & 0x1FFFFFull) << 21) |
                         (((uint64_t)(uint32_t)(z + dz) & 0x1FFFFFull) << 42);
      if (dev_contains(v, k)) continue;
      if constexpr (ALLOC) {
        int32_t got;
        dev_insert_alloc(v, pool, k, &got);
      } else {
        dev_insert(v, k, (uint64_t)(uint32_t)i);
      }
    }
  }
}

// The two-container step of the reconstruction example of Section 4.1: every thread asks the
// block map whether its key is there (contains, read-only on `map`) and, if so, inserts the key
// into the update set `set` (an unordered_set, many threads may insert the same key).  status[i]:
// kNoStatus when the map lacks the key, else the set insert's PRESENT / INSERTED / FULL.
__global__ __launch_bounds__(kBlock) void k_dev_update_set(DevView map, DevView set,
                                                           const uint64_t* __restrict__ keys,
                                                           int64_t n, uint8_t* __restrict__ status) {
  if (set.striped) set.striped = (int32_t)set.t.bcnt[kStripeFlag];
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const uint64_t key = keys[i];
    uint8_t st = kNoStatus;
    if (dev_contains(map, key)) st = dev_insert(set, key, 0);
    if (status) status[i] = st;
  }
}

// Per-thread push_back / pop_back through the device-side API: element i by one thread, all
// concurrently.
__global__ __launch_bounds__(kBlock) void k_dev_pool_apply(DevPool p, int32_t op,
                                                           const int32_t* __restrict__ in, int64_t n,
                                                           int32_t* __restrict__ out,
                                                           uint8_t* __restrict__ status) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    bool ok;
    if (op == CT_DEV_PUSH_BACK) {
      ok = dev_push_back(p, in[i]);
    } else {
      int32_t v = -1;
      ok = dev_pop_back(p, &v);
      if (out) out[i] = ok ? v : -1;
    }
    if (status) status[i] = ok ? 1 : 2;
  }
}

__global__ void k_check_begin(TableView t) {
  Header* h = t.hdr;
  h->live_count = 0;
  h->violations = 0;
  h->dup_count = 0;
  h->pool_bad = 0;
  h->pool_count = 0;
  h->pool_h1 = 0;
  h->pool_h2 = 0;
}

// Two independent 64-bit fingerprints of a pool index.  Sums of them over a multiset (wrapping)
// are equal for equal multisets; a multiset that differs from {0 .. P-1} (an index missing,
// repeated, or replaced) changes both sums except with probability about 2^-64 each.
__device__ __forceinline__ uint64_t check_h1(uint64_t v) { return fmix64(v + 0x9E3779B97F4A7C15ull); }
__device__ __forceinline__ uint64_t check_h2(uint64_t v) {
  return fmix64(v * 0xD1B54A32D192ED03ull + 0x632BE59BD9B4E019ull);
}

struct CheckSums {
  uint64_t live = 0, unreach = 0, dup = 0, pbad = 0, h1 = 0, h2 = 0;
  int64_t pcnt = 0;
};

__device__ __forceinline__ void check_pool_value(CheckSums& c, uint64_t v, int64_t pool_cap) {
  if (v >= (uint64_t)pool_cap) {
    ++c.pbad;
  } else {
    ++c.pcnt;
    c.h1 += check_h1(v);
    c.h2 += check_h2(v);
  }
}

__device__ __forceinline__ void check_flush(const TableView& t, CheckSums c) {
  c.live = wave_sum(c.live);
  c.unreach = wave_sum(c.unreach);
  c.dup = wave_sum(c.dup);
  c.pbad = wave_sum(c.pbad);
  c.h1 = wave_sum(c.h1);
  c.h2 = wave_sum(c.h2);
  c.pcnt = (int64_t)wave_sum((uint64_t)c.pcnt);
  if (wave_lane() == 0) {
    Header* h = t.hdr;
    if (c.live) aadd64(&h->live_count, c.live);
    if (c.unreach) aadd64(&h->violations, c.unreach);
    if (c.dup) aadd64(&h->dup_count, c.dup);
    if (c.pbad) aadd64(&h->pool_bad, c.pbad);
    if (c.pcnt) aadd64(reinterpret_cast<uint64_t*>(&h->pool_count), (uint64_t)c.pcnt);
    if (c.h1) aadd64(&h->pool_h1, c.h1);
    if (c.h2) aadd64(&h->pool_h2, c.h2);
  }
}

// Every live key must be reachable (no bucket between its home and its own bucket holds a kEmpty
// slot, so a lookup finds it) and stored once: a second copy of a key lies on the same probe
// path, so the walk of the later copy passes the earlier one (or an earlier slot of its own
// bucket).  With pool_cap > 0 the live values are pool indices and enter the fingerprint sums.
__global__ __launch_bounds__(kBlock) void k_check(TableView t, int64_t pool_cap) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nt = (int64_t)gridDim.x * blockDim.x;
  const int64_t nslots = (int64_t)t.nb * kSlots;
  CheckSums c;
  for (int64_t j = tid; j < nslots; j += nt) {
    const Slot sl = t.bk[j >> 3].s[j & 7];
    if (sl.key == kEmpty || sl.key == kTomb) continue;
    ++c.live;
    const uint64_t at = (uint64_t)(j >> 3);
    const int own = (int)(j & 7);
    const Seq q = probe_seq(t, sl.key);
    uint64_t b = q.home;
    bool unreachable = false, dup = false;
    for (uint64_t step = 0;; ++step) {
      if (step >= t.nb) { unreachable = true; break; }
      const bool last = b == at;
      bool has_empty = false;
      for (int s = 0; s < kSlots; ++s) {
        const uint64_t k2 = t.bk[b].s[s].key;
        has_empty |= k2 == kEmpty;
        dup |= k2 == sl.key && (!last || s < own);
      }
      if (last) break;
      if (has_empty) { unreachable = true; break; }
      b = next_bucket(t, b, q.step);
    }
    c.unreach += unreachable;
    c.dup += dup;
    if (pool_cap > 0) check_pool_value(c, sl.val, pool_cap);
  }
  if (pool_cap > 0 && tid == 0) {
    for (int s = 0; s < 2; ++s)
      if (t.hdr->spec_live[s]) check_pool_value(c, t.hdr->spec_val[s], pool_cap);
  }
  check_flush(t, c);
}

// The pool's entries enter the fingerprint sums, and every index 0 .. cap-1 leaves them once: the
// sums and the count end at zero exactly when the pool and the table's live values together hold
// each index once.
__global__ __launch_bounds__(kBlock) void k_check_pool(TableView t, const PoolHeader* ph,
                                                       const int32_t* __restrict__ stack) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nt = (int64_t)gridDim.x * blockDim.x;
  const int64_t top = ph->top, head = ph->head, cap = ph->cap;
  CheckSums c;
  for (int64_t j = tid; j < cap; j += nt) {
    if (j < top) {
      const int32_t v = stack[ring_pos(head, cap, j)];
      check_pool_value(c, v < 0 ? ~0ull : (uint64_t)v, cap);
    }
    --c.pcnt;
    c.h1 -= check_h1((uint64_t)j);
    c.h2 -= check_h2((uint64_t)j);
  }
  check_flush(t, c);
}

// ---------------------------------------------------------------------------------------------
// table health and purge.  An erase leaves a tombstone where its bucket holds no empty slot, and
// inserts turn tombstones back into keys; nothing turns a tombstone back into an empty slot, so
// under long churn the buckets without an empty slot grow in number, and lookups of absent keys
// walk past more of them.  The purge reopens every bucket that no live key's probe path passes:
// its tombstones become empty slots.  A bucket that some live key passes (one before that key's
// own bucket on its path) keeps its tombstones, so every live key stays reachable.
// ---------------------------------------------------------------------------------------------
// Buckets without an empty slot, and tombstones; 8 lanes per bucket.
__global__ __launch_bounds__(kBlock) void k_health(TableView t) {
  const int sub = threadIdx.x & 7;
  const int64_t ngroups = (int64_t)gridDim.x * (kBlock / 8);
  uint64_t closed = 0, tombs = 0;
  const int64_t nbk = (int64_t)t.nb;
  const int64_t span = ((nbk + ngroups - 1) / ngroups) * ngroups;   // equal trips: ballots below
  for (int64_t b = (int64_t)blockIdx.x * (kBlock / 8) + (threadIdx.x >> 3); b < span; b += ngroups) {
    const uint64_t key = b < nbk ? t.bk[b].s[sub].key : 0;
    const uint32_t e = group_bits(__ballot(b < nbk && key == kEmpty));
    if (b < nbk && sub == 0 && !e) ++closed;
    if (b < nbk && key == kTomb) ++tombs;
  }
  closed = wave_sum(closed);
  tombs = wave_sum(tombs);
  if (wave_lane() == 0) {
    if (closed) aadd64(&t.hdr->closed_count, closed);
    if (tombs) aadd64(&t.hdr->tomb_count, tombs);
  }
}

__global__ void k_health_begin(TableView t) {
  t.hdr->closed_count = 0;
  t.hdr->tomb_count = 0;
}

__global__ __launch_bounds__(kBlock) void k_purge_clear(uint32_t* __restrict__ bits, int64_t words) {
  for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < words;
       j += (int64_t)gridDim.x * kBlock)
    bits[j] = 0;
}

// Bit (b - w0) for every bucket b in [w0, w1) that a live key's probe path passes before the
// key's own bucket.
__global__ __launch_bounds__(kBlock) void k_purge_mark(TableView t, uint32_t* __restrict__ bits,
                                                       int64_t w0, int64_t w1) {
  const int64_t nslots = (int64_t)t.nb * kSlots;
  for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < nslots;
       j += (int64_t)gridDim.x * kBlock) {
    const uint64_t key = t.bk[j >> 3].s[j & 7].key;
    if (key == kEmpty || key == kTomb) continue;
    const uint64_t at = (uint64_t)(j >> 3);
    const Seq q = probe_seq(t, key);
    uint64_t b = q.home;
    for (uint64_t step = 0; b != at && step < t.nb; ++step) {
      if ((int64_t)b >= w0 && (int64_t)b < w1) {
        const uint64_t r = b - (uint64_t)w0;
        atomicOr(&bits[r >> 5], 1u << (r & 31));
      }
      b = next_bucket(t, b, q.step);
    }
  }
}

// Every bucket of [w0, w1) that no live key passes: its tombstones become empty slots.
__global__ __launch_bounds__(kBlock) void k_purge_reopen(TableView t, const uint32_t* __restrict__ bits,
                                                         int64_t w0, int64_t w1) {
  const int64_t nslots = (w1 - w0) * kSlots;
  for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < nslots;
       j += (int64_t)gridDim.x * kBlock) {
    const uint64_t r = (uint64_t)(j >> 3);
    if ((bits[r >> 5] >> (r & 31)) & 1u) continue;
    uint64_t* k = &t.bk[(uint64_t)w0 + r].s[j & 7].key;
    if (*k == kTomb) *k = kEmpty;
  }
}

// ---------------------------------------------------------------------------------------------
// pool kernels
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_pool_init(PoolHeader* ph, int32_t* stack, int64_t cap) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nt = (int64_t)gridDim.x * blockDim.x;
  for (int64_t j = tid; j < cap; j += nt) stack[j] = (int32_t)(cap - 1 - j);
  if (tid == 0) {
    ph->top = cap;
    ph->top0 = cap;
    ph->cap = cap;
    ph->err = 0;
    ph->head = 0;
    ph->head0 = 0;
  }
}

__global__ void k_pool_snapshot(PoolHeader* ph) {
  ph->top0 = ph->top;
  ph->head0 = ph->head;
}

__global__ __launch_bounds__(kBlock) void k_pool_pop(PoolHeader* ph, const int32_t* __restrict__ stack,
                                                     int64_t n, int32_t* __restrict__ out,
                                                     uint8_t* __restrict__ status) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nt = (int64_t)gridDim.x * blockDim.x;
  const int64_t top0 = ph->top0, head0 = ph->head0, cap = ph->cap;
  for (int64_t i = tid; i < n; i += nt) {
    const bool ok = i < top0;
    if (out) out[i] = ok ? stack[ring_pos(head0, cap, top0 - 1 - i)] : -1;
    if (status) status[i] = ok ? 1 : 2;
  }
  if (tid == 0) {
    ph->top = n < top0 ? top0 - n : 0;
    if (n > top0) ph->err |= kErrPool;
  }
}

__global__ __launch_bounds__(kBlock) void k_pool_push(PoolHeader* ph, int32_t* __restrict__ stack,
                                                      const int32_t* __restrict__ in, int64_t n,
                                                      uint8_t* __restrict__ status) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nt = (int64_t)gridDim.x * blockDim.x;
  const int64_t top0 = ph->top0, head0 = ph->head0, cap = ph->cap;
  for (int64_t i = tid; i < n; i += nt) {
    const bool ok = top0 + i < cap;
    if (ok) stack[ring_pos(head0, cap, top0 + i)] = in[i];
    if (status) status[i] = ok ? 1 : 2;
  }
  if (tid == 0) {
    ph->top = (top0 + n < cap) ? top0 + n : cap;
    if (top0 + n > cap) ph->err |= kErrPool;
  }
}

__global__ __launch_bounds__(kBlock) void k_pool_copy(const PoolHeader* ph, const int32_t* __restrict__ stack,
                                                      int32_t* __restrict__ out, int64_t cap) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nt = (int64_t)gridDim.x * blockDim.x;
  const int64_t m = ph->top < cap ? ph->top : cap;
  for (int64_t j = tid; j < m; j += nt) out[j] = stack[ring_pos(ph->head, ph->cap, j)];
}

// Deque front operations (Section 4.3).  pop_front: element i of the batch removes pool element i
// (front first), -1 once the pool is empty.  push_front: element i goes just in front of the
// previous one, so the last value pushed ends up first.
__global__ __launch_bounds__(kBlock) void k_pool_pop_front(PoolHeader* ph, const int32_t* __restrict__ stack,
                                                           int64_t n, int32_t* __restrict__ out,
                                                           uint8_t* __restrict__ status) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nt = (int64_t)gridDim.x * blockDim.x;
  const int64_t top0 = ph->top0, head0 = ph->head0, cap = ph->cap;
  for (int64_t i = tid; i < n; i += nt) {
    const bool ok = i < top0;
    if (out) out[i] = ok ? stack[ring_pos(head0, cap, i)] : -1;
    if (status) status[i] = ok ? 1 : 2;
  }
  if (tid == 0) {
    const int64_t m = n < top0 ? n : top0;
    ph->head = m ? ring_pos(head0, cap, m) : head0;
    ph->top = top0 - m;
    if (n > top0) ph->err |= kErrPool;
  }
}

__global__ __launch_bounds__(kBlock) void k_pool_push_front(PoolHeader* ph, int32_t* __restrict__ stack,
                                                            const int32_t* __restrict__ in, int64_t n,
                                                            uint8_t* __restrict__ status) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nt = (int64_t)gridDim.x * blockDim.x;
  const int64_t top0 = ph->top0, head0 = ph->head0, cap = ph->cap;
  for (int64_t i = tid; i < n; i += nt) {
    const bool ok = top0 + i < cap;
    if (ok) stack[ring_pos(head0, cap, -1 - i)] = in[i];
    if (status) status[i] = ok ? 1 : 2;
  }
  if (tid == 0) {
    const int64_t room = cap - top0;
    const int64_t m = n < room ? n : room;
    ph->head = m ? ring_pos(head0, cap, -m) : head0;
    ph->top = top0 + m;
    if (n > room) ph->err |= kErrPool;
  }
}

// ---------------------------------------------------------------------------------------------
// grouped execution of a plan: one launch per pipeline stage covers the same stage of many
// tables.  A plan is cut into levels holding at most one chunk-step per table (the k-th step of
// every table); within a level the steps touch disjoint tables, scratch and arrays, so a stage's
// blocks of all steps can run in one grid.  Block b of a stage launch finds its step from the
// launch's entry list (first block of each step, ascending) and then runs exactly the range code
// of the single-table kernel with the step's own block index and block count.
// ---------------------------------------------------------------------------------------------
// Plan operation kinds (the CT_OP_* values).
enum : int32_t { kOpClear = 0, kOpInsert = 1, kOpFind = 2, kOpErase = 3 };

// Stages of the grouped pipeline, in launch order within a level.
enum GStage : int32_t {
  gReset, gPro, gDedup, gFind, gInsert, gErase, gApply,
  gSClear, gSBuild, gSProbe, gSSwap,  // resolution of speculative steps
  gCount, gScan, gFinal, gFix, gStages,
  gCopy = 100  // copy stage of merged operations (before the first and after the last level)
};

struct GStep {
  TableView v;
  const uint64_t* keys;
  const void* vals;
  void* vout;
  uint8_t* flags;
  int64_t q;      // elements of this step (at most the table's chunk for insert and erase)
  uint32_t db;    // dedup slots of the step's chunk
  int32_t vk;     // value kind of the table
  int32_t type;   // plan operation
  int32_t gb;     // blocks of the step's insert / erase / find stage
  int32_t ntiles; // rank-scan tiles
  int32_t spath;  // insert or erase: 0 resolve repeated keys first; 1 speculate when the table's
                  // last chunk of the kind changed at least half its keys; 2 speculate always
                  // (an insert only when it cannot reach capacity)
};

struct GEntry {
  int32_t first;  // first block of the step in this launch
  int32_t step;   // index into the step array
};

struct GLoc {
  int32_t step, lb, nblk;
};

// Step of block b of a launch of nb blocks: the last entry whose first block is <= b.  Uniform per
// block.
__device__ __forceinline__ GLoc g_locate_at(const GEntry* __restrict__ e, int32_t n, int32_t b,
                                            int32_t nb) {
  int32_t lo = 0, hi = n - 1;
  while (lo < hi) {
    const int32_t mid = (lo + hi + 1) >> 1;
    if (e[mid].first <= b) lo = mid;
    else hi = mid - 1;
  }
  const int32_t end = lo + 1 < n ? e[lo + 1].first : nb;
  return GLoc{e[lo].step, b - e[lo].first, end - e[lo].first};
}

__device__ __forceinline__ GLoc g_locate(const GEntry* __restrict__ e, int32_t n) {
  return g_locate_at(e, n, (int32_t)blockIdx.x, (int32_t)gridDim.x);
}

// A pointer read from memory may point anywhere for all the compiler knows, and an access through
// it goes by the unit that also serves LDS, whose answers the probe rounds wait for.  These point
// to global memory, and are read as what they are.
template <typename T>
__device__ __forceinline__ T* in_global(T* const& field) {
  typedef __attribute__((address_space(1))) T* Global;
  return (T*)*static_cast<Global const*>(static_cast<const void*>(&field));
}

// The step of block L.
__device__ __forceinline__ GStep g_step(const GStep* __restrict__ st, const GLoc& L) {
  const GStep& m = st[L.step];
  GStep g = m;
  g.v.bk = in_global(m.v.bk);
  g.v.hdr = in_global(m.v.hdr);
  g.v.dd = in_global(m.v.dd);
  g.v.dmark = in_global(m.v.dmark);
  g.v.dup = in_global(m.v.dup);
  g.v.flag = in_global(m.v.flag);
  g.v.ref = in_global(m.v.ref);
  g.v.tsum = in_global(m.v.tsum);
  g.v.bcnt = in_global(m.v.bcnt);
  g.v.stripes = in_global(m.v.stripes);
  g.v.dfirst = in_global(m.v.dfirst);
  g.v.fb = in_global(m.v.fb);
  g.keys = in_global(m.keys);
  g.vals = in_global(m.vals);
  g.vout = in_global(m.vout);
  g.flags = in_global(m.flags);
  return g;
}

__device__ __forceinline__ void g_reset_body(const GStep* __restrict__ st, const GLoc L) {
  const TableView t = g_step(st, L).v;
  reset_range(t, (int64_t)L.lb * kBlock, (int64_t)t.nb * kSlots, (int64_t)L.nblk * kBlock,
              L.lb == 0, 0);
}

// Whether an insert or erase step speculates, decided on the device from the table's state when
// the step starts, so that a plan replayed later decides afresh.  Every block of the prologue
// stage computes it from words that no block of the stage writes, so all agree.
__device__ __forceinline__ bool g_speculates(const GStep& g) {
  if (g.spath == 0 || g.q <= 0 || (g.type != kOpInsert && g.type != kOpErase)) return false;
  const Header* h = g.v.hdr;
  const bool ins = g.type == kOpInsert;
  if (ins && h->size + (uint64_t)g.q > g.v.cap) return false;   // FULL must be ranked
  return g.spath == 2 || mostly_changed(h, ins ? 0 : 1);
}

// Prologue: a speculative step needs only its header words (the dd entries are cleared after the
// claims, and only when something is listed).  Its count words are zero already: g_apply_body zeroes
// what it has summed, as k_spec_swap does for single-table batches.  Otherwise the dedup scratch is
// cleared and the header decides as for a single-table chunk.
__device__ __forceinline__ void g_prologue_body(const GStep* __restrict__ st, const GLoc L) {
  const GStep g = g_step(st, L);
  const TableView t = g.v;
  if (g_speculates(g)) {
    if (L.lb == 0 && threadIdx.x == 0) {
      t.hdr->ndup = 0;
      t.hdr->fast = 1u;
      t.hdr->spec = 1u;
    }
    return;
  }
  prologue_range(t, nullptr, g.db, g.q, (int64_t)L.lb * kBlock, prologue_units(g.db, g.q),
                 (int64_t)L.nblk * kBlock, L.lb == 0);
}

__device__ __forceinline__ void g_dedup_body(const GStep* __restrict__ st, const GLoc L) {
  const GStep g = g_step(st, L);
  const TableView t = g.v;
  if (t.hdr->spec) return;
  dedup_range(t, g.keys, nullptr, g.db - 1, (int64_t)L.lb * kBlock, g.q, (int64_t)L.nblk * kBlock);
}

// The grouped find / insert / erase stages run with BS threads per block (the plan's block size):
// the range code strides by the step's blocks times BS.
template <int BS>
__device__ __forceinline__ void g_insert_body(const GStep* __restrict__ st, const GLoc L) {
  const GStep g = g_step(st, L);
  const TableView t = g.v;
  const int64_t lo = (int64_t)L.lb * BS, step = (int64_t)L.nblk * BS;
  WaveLds* w = wave_lds<BS>();
  if (t.hdr->spec) {
    uint2 c;
    if (g.vk == 1) c = insert_spec_range<1, false>(t, w, g.keys, g.vals, g.flags, lo, g.q, step);
    else if (g.vk == 2) c = insert_spec_range<2, false>(t, w, g.keys, g.vals, g.flags, lo, g.q, step);
    else c = insert_spec_range<0, false>(t, w, g.keys, nullptr, g.flags, lo, g.q, step);
    const int64_t tot = block_sum<BS>(((int64_t)c.x << 32) + (int64_t)c.y);
    if (threadIdx.x == 0) spec_count(t, L.lb, tot);
    return;
  }
  int64_t ins;
  if (g.vk == 1)
    ins = insert_range<1, false, false>(t, w, g.keys, nullptr, g.vals, g.db - 1, g.flags, nullptr, lo, g.q, step);
  else if (g.vk == 2)
    ins = insert_range<2, false, false>(t, w, g.keys, nullptr, g.vals, g.db - 1, g.flags, nullptr, lo, g.q, step);
  else
    ins = insert_range<0, false, false>(t, w, g.keys, nullptr, nullptr, g.db - 1, g.flags, nullptr, lo, g.q, step);
  const int64_t tot = block_sum<BS>(ins);
  if (threadIdx.x == 0) t.bcnt[L.lb] = tot;
}

template <int BS>
__device__ __forceinline__ void g_erase_body(const GStep* __restrict__ st, const GLoc L) {
  const GStep g = g_step(st, L);
  const TableView t = g.v;
  if (t.hdr->spec) {
    const uint2 c = erase_spec_range<false>(t, wave_lds<BS>(), g.keys, g.flags, (int64_t)L.lb * BS, g.q,
                                     (int64_t)L.nblk * BS);
    const int64_t tot = block_sum<BS>(((int64_t)c.x << 32) + (int64_t)c.y);
    if (threadIdx.x == 0) spec_count(t, L.lb, tot);
    return;
  }
  const int64_t del = erase_range<false, false>(t, wave_lds<BS>(), g.keys, g.db - 1, g.flags, (int64_t)L.lb * BS,
                                         g.q, (int64_t)L.nblk * BS);
  const int64_t tot = block_sum<BS>(del);
  if (threadIdx.x == 0) t.bcnt[L.lb] = -tot;
}

template <int BS>
__device__ __forceinline__ void g_find_body(const GStep* __restrict__ st, const GLoc L) {
  const GStep g = g_step(st, L);
  const TableView t = g.v;
  const int64_t lo = (int64_t)L.lb * BS, step = (int64_t)L.nblk * BS;
  WaveLds* w = wave_lds<BS>();
  if (g.vk == 1) find_range<1>(t, w, g.keys, g.vout, g.flags, lo, g.q, step);
  else if (g.vk == 2) find_range<2>(t, w, g.keys, g.vout, g.flags, lo, g.q, step);
  else find_range<0>(t, w, g.keys, nullptr, g.flags, lo, g.q, step);
}

// The count change into the live count and the feedback words; for a speculative step also the
// listed total, which the resolution stages read.
__device__ __forceinline__ void g_apply_body(const GStep* __restrict__ st, const GLoc L) {
  const GStep g = g_step(st, L);
  const TableView t = g.v;
  const bool erase = g.type == kOpErase;
  if (t.hdr->spec) {
    if (threadIdx.x < 64) {
      const uint64_t tot = spec_total(t);
      if (threadIdx.x == 0) spec_settle(t, g.q, erase, tot);
      spec_zero(t);
    }
    return;
  }
  const int64_t change = apply_count_block(t, g.gb);
  if (threadIdx.x == 0) chunk_feedback(t, erase ? 1 : 0, g.q, erase ? -change : change);
}

// Resolution of a speculative step (the single-table kernels' range code, per step).
__device__ __forceinline__ void g_sclear_body(const GStep* __restrict__ st, const GLoc L) {
  const GStep g = g_step(st, L);
  if (!g.v.hdr->spec) return;
  spec_clear_range(g.v, g.q, g.v.hdr->ndup, L.lb, L.nblk);
}

__device__ __forceinline__ void g_sbuild_body(const GStep* __restrict__ st, const GLoc L) {
  const GStep g = g_step(st, L);
  if (!g.v.hdr->spec) return;
  spec_build_range(g.v, g.keys, g.q, L.lb, L.nblk);
}

template <bool SWAP>
__device__ __forceinline__ void g_sfix_body(const GStep* __restrict__ st, const GLoc L) {
  const GStep g = g_step(st, L);
  const TableView t = g.v;
  if (!t.hdr->spec) return;
  if (g.type == kOpErase) {
    if (SWAP) spec_swap_range<0, true>(t, g.keys, nullptr, g.q, g.flags, L.lb, L.nblk);
    else spec_probe_range<0, true>(t, g.keys, nullptr, g.q, g.flags, L.lb, L.nblk);
  } else if (g.vk == 1) {
    if (SWAP) spec_swap_range<1, false>(t, g.keys, g.vals, g.q, g.flags, L.lb, L.nblk);
    else spec_probe_range<1, false>(t, g.keys, g.vals, g.q, g.flags, L.lb, L.nblk);
  } else if (g.vk == 2) {
    if (SWAP) spec_swap_range<2, false>(t, g.keys, g.vals, g.q, g.flags, L.lb, L.nblk);
    else spec_probe_range<2, false>(t, g.keys, g.vals, g.q, g.flags, L.lb, L.nblk);
  } else {
    if (SWAP) spec_swap_range<0, false>(t, g.keys, nullptr, g.q, g.flags, L.lb, L.nblk);
    else spec_probe_range<0, false>(t, g.keys, nullptr, g.q, g.flags, L.lb, L.nblk);
  }
}

__device__ __forceinline__ void g_tile_count_body(const GStep* __restrict__ st, const GLoc L) {
  const GStep g = g_step(st, L);
  const TableView t = g.v;
  if (t.hdr->fast) return;
  __shared__ uint32_t part[kBlock / 64];
  const int64_t t0 = (int64_t)L.lb * kTile;
  uint64_t c = 0;
  for (int j = threadIdx.x; j < kTile; j += kBlock) {
    const int64_t i = t0 + j;
    if (i < g.q) c += t.flag[i];
  }
  c = wave_sum(c);
  if (wave_lane() == 0) part[threadIdx.x >> 6] = (uint32_t)c;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t sum = 0;
    for (int w = 0; w < kBlock / 64; ++w) sum += part[w];
    t.tsum[L.lb] = sum;
  }
}

template <int NT>
__device__ __forceinline__ void g_tile_scan_body(const GStep* __restrict__ st, const GLoc L) {
  const TableView t = g_step(st, L).v;
  if (t.hdr->fast) return;
  scan_tiles_block<NT>(t, nullptr, st[L.step].ntiles, 0);
}

__device__ __forceinline__ void g_final_body(const GStep* __restrict__ st, const GLoc L) {
  const GStep g = g_step(st, L);
  const TableView t = g.v;
  if (t.hdr->fast) return;   // nothing to rank: leave before any of the tile code
  if (g.vk == 1)
    final_tile<1, 0>(t, wave_lds<kBlock>(), nullptr, nullptr, g.keys, g.vals, g.q, g.flags, nullptr, L.lb, 0);
  else if (g.vk == 2)
    final_tile<2, 0>(t, wave_lds<kBlock>(), nullptr, nullptr, g.keys, g.vals, g.q, g.flags, nullptr, L.lb, 0);
  else
    final_tile<0, 0>(t, wave_lds<kBlock>(), nullptr, nullptr, g.keys, nullptr, g.q, g.flags, nullptr, L.lb, 0);
}

// A byte range moved by the grouped plan's copy stages (operations merged into one step).
struct GCopy {
  const void* src;
  void* dst;
  int64_t bytes;
};

// Segment of this block's entry, copied by the entry's blocks: single bytes up to the destination's
// first 16-byte boundary and past its last one, 16-byte stores between, four loads per thread in
// flight.  Operations of odd sizes leave sources and destinations (of one-byte flags above all) at
// any alignment to each other, and a load may have any.  70 million operations' arrays of 256 tables
// (0.9 GB in 5000 segments) take 0.38 ms, 0.55 with one unit of the widest common alignment at a time.
typedef uint32_t Unaligned16 __attribute__((ext_vector_type(4), aligned(1)));

__device__ __forceinline__ void g_copy_body(const GCopy* __restrict__ segs, const GLoc L) {
  const GCopy& g = segs[L.step];
  const uint8_t* s = static_cast<const uint8_t*>(in_global(g.src));
  uint8_t* d = static_cast<uint8_t*>(in_global(g.dst));
  const int64_t bytes = g.bytes;
  const int64_t first = (int64_t)L.lb * kBlock + threadIdx.x;
  const int64_t stride = (int64_t)L.nblk * kBlock;
  const int64_t head = min((int64_t)(-reinterpret_cast<uintptr_t>(d) & 15u), bytes);
  const int64_t units = (bytes - head) / 16, tail = head + units * 16;
  if (first < head) d[first] = s[first];
  if (tail + first < bytes) d[tail + first] = s[tail + first];
  s += head;
  uint4* d16 = reinterpret_cast<uint4*>(d + head);
  for (int64_t i = first; i < units; i += 4 * stride) {
    Unaligned16 x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      x[k] = *reinterpret_cast<const Unaligned16*>(s + 16 * min(i + k * stride, units - 1));
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (i + k * stride < units) d16[i + k * stride] = make_uint4(x[k].x, x[k].y, x[k].z, x[k].w);
  }
}

__device__ __forceinline__ void g_fix_body(const GStep* __restrict__ st, const GLoc L) {
  const GStep g = g_step(st, L);
  const TableView t = g.v;
  if (t.hdr->spec || t.hdr->fast) return;   // the outcomes are known already
  fix_range(t, g.q, g.flags, nullptr, (int64_t)L.lb * kBlock, (int64_t)L.nblk * kBlock);
}

// One launch per stage: block b of the launch runs the stage's body for its own step.
__global__ __launch_bounds__(kBlock) void k_g_reset(const GStep* __restrict__ st,
                                                    const GEntry* __restrict__ e, int32_t n) {
  g_reset_body(st, g_locate(e, n));
}
__global__ __launch_bounds__(kBlock) void k_g_prologue(const GStep* __restrict__ st,
                                                       const GEntry* __restrict__ e, int32_t n) {
  g_prologue_body(st, g_locate(e, n));
}
__global__ __launch_bounds__(kBlock) void k_g_dedup(const GStep* __restrict__ st,
                                                    const GEntry* __restrict__ e, int32_t n) {
  g_dedup_body(st, g_locate(e, n));
}
// (5 waves per SIMD as in k_insert: the large multi-table schedule 5.85 ms without, 5.80 with)
template <int BS>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(5))) void k_g_insert(const GStep* __restrict__ st,
                                                 const GEntry* __restrict__ e, int32_t n) {
  g_insert_body<BS>(st, g_locate(e, n));
}
template <int BS>
__global__ __launch_bounds__(BS) void k_g_erase(const GStep* __restrict__ st,
                                                const GEntry* __restrict__ e, int32_t n) {
  g_erase_body<BS>(st, g_locate(e, n));
}
template <int BS>
__global__ __launch_bounds__(BS) void k_g_find(const GStep* __restrict__ st,
                                               const GEntry* __restrict__ e, int32_t n) {
  g_find_body<BS>(st, g_locate(e, n));
}
__global__ __launch_bounds__(1024) void k_g_apply(const GStep* __restrict__ st,
                                                  const GEntry* __restrict__ e, int32_t n) {
  g_apply_body(st, g_locate(e, n));
}
__global__ __launch_bounds__(kBlock) void k_g_tile_count(const GStep* __restrict__ st,
                                                         const GEntry* __restrict__ e, int32_t n) {
  g_tile_count_body(st, g_locate(e, n));
}
__global__ __launch_bounds__(1024) void k_g_tile_scan(const GStep* __restrict__ st,
                                                      const GEntry* __restrict__ e, int32_t n) {
  g_tile_scan_body<1024>(st, g_locate(e, n));
}
__global__ __launch_bounds__(kBlock) void k_g_final(const GStep* __restrict__ st,
                                                    const GEntry* __restrict__ e, int32_t n) {
  g_final_body(st, g_locate(e, n));
}
__global__ __launch_bounds__(kBlock) void k_g_copy(const GCopy* __restrict__ segs,
                                                   const GEntry* __restrict__ e, int32_t n) {
  g_copy_body(segs, g_locate(e, n));
}
__global__ __launch_bounds__(kBlock) void k_g_fix(const GStep* __restrict__ st,
                                                  const GEntry* __restrict__ e, int32_t n) {
  g_fix_body(st, g_locate(e, n));
}
__global__ __launch_bounds__(kBlock) void k_g_sclear(const GStep* __restrict__ st,
                                                     const GEntry* __restrict__ e, int32_t n) {
  g_sclear_body(st, g_locate(e, n));
}
__global__ __launch_bounds__(kBlock) void k_g_sbuild(const GStep* __restrict__ st,
                                                     const GEntry* __restrict__ e, int32_t n) {
  g_sbuild_body(st, g_locate(e, n));
}
template <bool SWAP>
__global__ __launch_bounds__(kBlock) void k_g_sfix(const GStep* __restrict__ st,
                                                   const GEntry* __restrict__ e, int32_t n) {
  g_sfix_body<SWAP>(st, g_locate(e, n));
}

// The whole grouped schedule in one cooperative launch.  Every workgroup of the grid is resident
// at once (the runtime refuses a cooperative launch that cannot be), so a grid-wide barrier
// between stages cannot wait for a workgroup that never runs.  Stage by stage, the grid's blocks
// take the stage's blocks in turn (block b runs b, b + grid, ...) with the same bodies as the
// per-stage launches, 256 threads each, then meet at the barrier, whose device-scope fences make
// the stage's stores visible to every XCD before the next stage reads them.  No workgroup waits
// for another in any other way, and every workgroup reaches every barrier.
struct GLaunchDev {
  int32_t stage, n, blocks, pad;
  int64_t entry_off;
};

__global__ __launch_bounds__(kBlock) void k_g_persistent(const GLaunchDev* __restrict__ ls,
                                                         int32_t nl, const GStep* __restrict__ st,
                                                         const GEntry* __restrict__ en,
                                                         const GCopy* __restrict__ cp) {
  cooperative_groups::grid_group grid = cooperative_groups::this_grid();
  for (int32_t l = 0; l < nl; ++l) {
    const GLaunchDev L = ls[l];
    const GEntry* e = en + L.entry_off;
    for (int32_t b = (int32_t)blockIdx.x; b < L.blocks; b += (int32_t)gridDim.x) {
      const GLoc g = g_locate_at(e, L.n, b, L.blocks);
      switch (L.stage) {
        case gReset: g_reset_body(st, g); break;
        case gPro: g_prologue_body(st, g); break;
        case gDedup: g_dedup_body(st, g); break;
        case gFind: g_find_body<kBlock>(st, g); break;
        case gInsert: g_insert_body<kBlock>(st, g); break;
        case gErase: g_erase_body<kBlock>(st, g); break;
        case gApply: g_apply_body(st, g); break;
        case gCount: g_tile_count_body(st, g); break;
        case gScan: g_tile_scan_body<kBlock>(st, g); break;
        case gFinal: g_final_body(st, g); break;
        case gFix: g_fix_body(st, g); break;
        case gSClear: g_sclear_body(st, g); break;
        case gSBuild: g_sbuild_body(st, g); break;
        case gSProbe: g_sfix_body<false>(st, g); break;
        case gSSwap: g_sfix_body<true>(st, g); break;
        case gCopy: g_copy_body(cp, g); break;
        default: break;
      }
      __syncthreads();  // the next block's body reuses this workgroup's LDS
    }
    grid.sync();
  }
}

}  // namespace

// =============================================================================================
// host side
// =============================================================================================
// Per-table kernel timing: while enabled, each kernel launched for the table is bracketed by two
// HIP events recorded on the caller's stream; read-out waits for them and sums per kernel kind.
struct Profiler {
  bool on = false;
  std::vector<hipEvent_t> events;  // pairs (start, end)
  std::vector<int> kinds;          // kind of each recorded pair
  size_t used = 0;
  double total_ms[CT_KERNEL_KINDS] = {};
  int64_t launches[CT_KERNEL_KINDS] = {};
};

struct ct_table {
  Profiler prof;
  ct_table_desc desc;
  uint8_t* base;
  int64_t bytes;
  TableView v;
  int64_t chunk;      // Q: elements per chunk (power of two)
  bool chunk_chosen;  // the caller chose it: batches are cut into such chunks, workspace or not
  uint64_t size_ub;   // upper bound of the live count known to the host
  int64_t dd_bytes;   // bytes of the dedup scratch region at v.dd (the purge's bitmap)
  int32_t insert_path = CT_INSERT_AUTO;  // how insert chunks resolve repeated keys
  uint64_t* fb_host = nullptr;           // host side of v.fb (pinned, mapped), or null
  bool counts_stale = false;             // a batch failed: its counts may still be in v.stripes
};

struct ct_pool {
  uint8_t* base;
  int64_t cap;
  PoolHeader* hdr;
  int32_t* stack;
};

namespace {

constexpr int64_t kAlign = 256;

int64_t align_up(int64_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

bool is_prime(int64_t x) {
  if (x < 2) return false;
  if (x % 2 == 0) return x == 2;
  for (int64_t d = 3; d * d <= x; d += 2)
    if (x % d == 0) return false;
  return true;
}

// Smallest prime >= x (x >= 1); a prime bucket count lets every probe step visit all buckets.
int64_t next_prime(int64_t x) {
  if (x <= 2) return 2;
  while (!is_prime(x)) ++x;
  return x;
}

int64_t pow2ceil(int64_t x) {
  int64_t p = 1;
  while (p < x) p <<= 1;
  return p;
}

struct Layout {
  int64_t nb, chunk, dslots, ntiles;
  int64_t off_bk, off_dd, off_dmark, off_dup, off_flag, off_ref, off_tsum, off_bcnt, off_stripes, total;
  // binned dedup (chunk >= kBinMinChunk; otherwise bins == false and the offsets are unused)
  bool bins;
  int64_t nfine, c1, c2;
  int lp, lp1;
  int64_t off_r1k, off_r1i, off_r2k, off_r2i, off_bcur, off_dfirst;
};

static_assert(kBinFineCap % kBlock == 0, "fine-bin entries are held kBlock per register row");

bool layout_scratch(Layout* L, int64_t q, int64_t off);

bool make_layout(const ct_table_desc* d, Layout* L) {
  if (!d || d->capacity < 0) return false;
  if (d->val_kind < 0 || d->val_kind > 2 || d->hash_kind < 0 || d->hash_kind > 1) return false;
  int64_t nb = d->bucket_count;
  if (nb == 0) nb = next_prime(std::max<int64_t>(1, (d->capacity + kSlots - 1) / kSlots));
  if (nb < 1) nb = 1;
  if (nb >= ((int64_t)1 << 31)) return false;  // 32-bit bucket arithmetic in the probes
  if (nb * kSlots < d->capacity) return false;
  int64_t q = d->chunk;
  if (q == 0) {
    // one chunk per ~capacity/8 keys: long kernels amortise launch and drain, and the scratch
    // (about 78 bytes per chunk element at these sizes) stays below two thirds of the buckets'
    // 16 bytes per slot
    int64_t f = 1024;
    while (f * 2 <= d->capacity / 8 && f < ((int64_t)1 << 23)) f *= 2;
    q = f;
  }
  if (q < 1024 || q > ((int64_t)1 << 24) || (q & (q - 1))) return false;
  L->nb = nb;
  int64_t off = align_up((int64_t)sizeof(Header));
  L->off_bk = off;
  off = align_up(off + nb * (int64_t)sizeof(Bucket));
  if (!layout_scratch(L, q, off)) return false;
  L->off_stripes = L->total;  // the table's own, whatever scratch a batch runs on
  L->total = align_up(L->total + kStripeRegion);
  return true;
}

// The per-chunk scratch of chunks of q elements (a power of two in [1024, 2^24]), from offset `off`.
bool layout_scratch(Layout* L, int64_t q, int64_t off) {
  L->chunk = q;
  L->dslots = 2 * q;
  L->ntiles = (q + kTile - 1) / kTile;
  L->bins = q >= kBinMinChunk;
  if (L->bins) {
    L->nfine = q / kBinFine;
    L->lp = 0;
    while (((int64_t)1 << L->lp) < L->nfine) ++L->lp;
    L->lp1 = 0;
    while ((1 << L->lp1) < kBinCoarse) ++L->lp1;
    const int64_t nseg = (int64_t)kBinCoarse * kBinSub;
    L->c1 = 2 * (q / nseg) + 256;
    L->c2 = kBinFineCap;
    if (L->nfine / kBinCoarse > kMaxFinePerCoarse) return false;
    if (nseg * L->c1 < L->dslots) return false;  // dd (8 bytes per slot) must fit in r1k
    L->off_r1k = off;
    L->off_dd = off;
    off = align_up(off + nseg * L->c1 * 8);
    L->off_r1i = off;
    off = align_up(off + nseg * L->c1 * 4);
    L->off_r2k = off;
    off = align_up(off + L->nfine * L->c2 * 8);
    L->off_r2i = off;
    off = align_up(off + L->nfine * L->c2 * 4);
    L->off_bcur = off;
    off = align_up(off + (kCoarseCtrWords + L->nfine) * 4);
    L->off_dfirst = off;
    off = align_up(off + q * 4);
  } else {
    L->off_dd = off;
    off = align_up(off + L->dslots * 8);
  }
  L->off_dmark = off;
  off = align_up(off + q);
  L->off_dup = off;
  off = align_up(off + q * 4);
  L->off_flag = off;
  off = align_up(off + q);
  L->off_ref = off;
  off = align_up(off + q * 8);
  L->off_tsum = off;
  off = align_up(off + L->ntiles * 4);
  L->off_bcnt = off;
  off = align_up(off + kMaxGroupBlocks * 8);
  L->total = off;
  return true;
}

// Point the view's scratch at the arrays that L lays out from `base`.
void scratch_view(TableView* v, uint8_t* base, const Layout& L) {
  v->dd = reinterpret_cast<uint64_t*>(base + L.off_dd);
  v->dmark = base + L.off_dmark;
  v->dup = reinterpret_cast<uint32_t*>(base + L.off_dup);
  v->flag = base + L.off_flag;
  v->ref = reinterpret_cast<uint64_t*>(base + L.off_ref);
  v->tsum = reinterpret_cast<uint32_t*>(base + L.off_tsum);
  v->bcnt = reinterpret_cast<int64_t*>(base + L.off_bcnt);
  v->r1k = L.bins ? reinterpret_cast<uint64_t*>(base + L.off_r1k) : nullptr;
  v->r1i = L.bins ? reinterpret_cast<uint32_t*>(base + L.off_r1i) : nullptr;
  v->r2k = L.bins ? reinterpret_cast<uint64_t*>(base + L.off_r2k) : nullptr;
  v->r2i = L.bins ? reinterpret_cast<uint32_t*>(base + L.off_r2i) : nullptr;
  v->bcur = L.bins ? reinterpret_cast<uint32_t*>(base + L.off_bcur) : nullptr;
  v->dfirst = L.bins ? reinterpret_cast<uint32_t*>(base + L.off_dfirst) : nullptr;
  v->c1 = L.bins ? (uint32_t)L.c1 : 0u;
  v->c2 = L.bins ? (uint32_t)L.c2 : 0u;
  v->lp = L.bins ? L.lp : 0;
  v->lp1 = L.bins ? L.lp1 : 0;
}

inline hipStream_t S(void* s) { return reinterpret_cast<hipStream_t>(s); }

// Sum the recorded pairs into the per-kind totals (waits for the last recorded event).
ct_status prof_drain(Profiler& P) {
  ct_status r = CT_OK;
  for (size_t j = 0; j < P.kinds.size(); ++j) {
    float ms = 0.f;
    if (hipEventSynchronize(P.events[2 * j + 1]) != hipSuccess ||
        hipEventElapsedTime(&ms, P.events[2 * j], P.events[2 * j + 1]) != hipSuccess) {
      r = CT_E_HIP;
      continue;
    }
    P.total_ms[P.kinds[j]] += ms;
    P.launches[P.kinds[j]] += 1;
  }
  P.kinds.clear();
  P.used = 0;
  return r;
}

// Launch `f` (a kernel launch on stream s) for table t, timed when profiling is on.
template <typename F>
void launch(ct_table* t, int kind, hipStream_t s, F&& f) {
  hipEvent_t end = nullptr;
  if (t && t->prof.on) {
    Profiler& P = t->prof;
    if (P.used + 2 > P.events.size()) prof_drain(P);
    if (hipEventRecord(P.events[P.used], s) == hipSuccess) {  // else this launch goes untimed
      end = P.events[P.used + 1];
      P.kinds.push_back(kind);
      P.used += 2;
    }
  }
  f();
  if (end && hipEventRecord(end, s) != hipSuccess) {  // drop the half-recorded pair
    t->prof.kinds.pop_back();
    t->prof.used -= 2;
  }
}

int64_t bin_prologue_units_host(const TableView& v, int64_t q) {
  return (q + 15) / 16 + ((int64_t)kCoarseCtrWords + ((int64_t)1 << v.lp)) / 4;
}

// Blocks of `bs` threads for n groups of eight keys (at most kMaxGroupBlocks: the count
// partials of one launch).
int group_blocks(int64_t n, int bs = kBlock) {
  const int64_t b = (n + (bs / 8) - 1) / (bs / 8);
  return (int)std::max<int64_t>(1, std::min<int64_t>(b, kMaxGroupBlocks));
}

// Chunks of at most this many rank tiles skip the one-block rank scan: each ranked-completion
// block sums the tile counts before its own tile (at most four loads a thread), and the first settles the
// chunk's totals.  Blocks allocated for n new keys and released again (two ranked batches), with
// the scan and without: 270,000 keys (264 tiles) 105.5 and 101.7 us, 2^19 136.3 and 132.5, 700,000
// 160.3 and 156.3, 2^20 (1024 tiles) 209.3 and 206.5; a set filled beyond its capacity by 2^20 keys
// 111.9 and 109.1.  From there to 2048 tiles the gain ends: 217.1 and 214.8 us at 1,100,000 keys
// allocated, 160.2 and 162.2 at 2^21 keys into the set, where every block sums eight counts a thread.
constexpr int kInlineRankTiles = 1024;

int flat_blocks(int64_t n) {
  const int64_t b = (n + kBlock - 1) / kBlock;
  return (int)std::max<int64_t>(1, std::min<int64_t>(b, 8192));
}

ct_status launched() { return hipGetLastError() == hipSuccess ? CT_OK : CT_E_HIP; }

// The same after launches that count into the table's words.
ct_status counted(ct_table* t) {
  const ct_status r = launched();
  if (r != CT_OK) t->counts_stale = true;
  return r;
}

// Before launches that count: zero what a failed batch may have left.  (While `s` is captured nothing
// runs, so the mark stays.)
void fresh_counts(ct_table* t, hipStream_t s) {
  if (!t->counts_stale) return;
  hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
  t->counts_stale = hipStreamIsCapturing(s, &c) != hipSuccess || c != hipStreamCaptureStatusNone;
  k_zero_counts<<<1, 64, 0, s>>>(t->v);
}

// dedup entries for a chunk of q elements: a power of two >= 2q (load at most one half)
uint32_t dedup_slots_for(int64_t q) { return (uint32_t)std::max<int64_t>(2, pow2ceil(2 * q)); }

template <typename T>
ct_status read_back(const T* dev, T* host, hipStream_t s) {
  if (hipMemcpyAsync(host, dev, sizeof(T), hipMemcpyDeviceToHost, s) != hipSuccess) return CT_E_HIP;
  return hipStreamSynchronize(s) == hipSuccess ? CT_OK : CT_E_HIP;
}

// ---------------------------------------------------------------------------------------------
// insert / erase drivers
// ---------------------------------------------------------------------------------------------
// The scratch a batch runs on: the table's own with its chunk, or a caller's workspace with larger
// chunks.
struct BatchScratch {
  TableView v;
  int64_t chunk;
  bool spec;  // it holds what speculative chunks need, and no more
};

// Chunk of a batch of n keys given a workspace: the whole batch up to 2^21 keys (165 MB), when that
// is more than the table's own chunk and the caller left the chunk to the library; else 0.  A
// default table cuts a batch that fills it into eight or more chunks of 6 to 12 launches each,
// which is what small and middle tables spend their time on: 4 M repeated keys into a set of 10^6
// took 1.59 ms in chunks of 2^17 and take 0.42 in chunks of 2^21; building, reading and erasing a
// map of 2^16 keys (four chunks) 143 us, now 78.  At 2^21 keys a chunk's kernels run several times longer than their
// launches take; the own chunks of the largest tables (2^23) stay.
constexpr int64_t kWorkspaceChunk = (int64_t)1 << 21;

int64_t workspace_chunk(const ct_table* t, int64_t n) {
  if (t->chunk_chosen || n <= t->chunk) return 0;
  const int64_t q = pow2ceil(std::min<int64_t>(n, kWorkspaceChunk));
  return q > t->chunk ? q : 0;
}

// Resolve the repeated keys of one chunk: binned for large chunks, dd otherwise.  ranked: the kernel
// that follows adds to the tile sums.
void dedup_chunk(ct_table* t, const TableView& v, PoolHeader* pool, const uint64_t* kc, int64_t q,
                 hipStream_t s, int ranked, int decided = 0) {
  const uint32_t db = dedup_slots_for(q);
  if (v.r1k && q >= kBinMinChunk) {
    // blocks per coarse segment: enough for its expected fill (about c1 / 2) in one tile each
    const int blocks_per_seg = (int)std::max<int64_t>(1, (v.c1 / 2 + kBinTile - 1) / kBinTile);
    const int nfine = 1 << v.lp;
    launch(t, CT_KERNEL_PROLOGUE, s, [&] { k_bin_prologue<<<flat_blocks(bin_prologue_units_host(v, q)), kBlock, 0, s>>>(v, pool, q, ranked, decided); });
    launch(t, CT_KERNEL_DEDUP, s, [&] { k_bin_scatter1<<<(int)((q + kBinTile - 1) / kBinTile), kBlock, 0, s>>>(v, kc, q); });
    launch(t, CT_KERNEL_DEDUP, s, [&] { k_bin_scatter2<<<kBinCoarse * kBinSub * blocks_per_seg, kBlock, 0, s>>>(v, blocks_per_seg); });
    launch(t, CT_KERNEL_DEDUP, s, [&] { k_bin_dedup<<<nfine, kBlock, 0, s>>>(v); });
    launch(t, CT_KERNEL_DEDUP, s, [&] { k_bin_fallback_clear<<<flat_blocks(db / 2), kBlock, 0, s>>>(v, db); });
    launch(t, CT_KERNEL_DEDUP, s, [&] { k_bin_fallback_dedup<<<flat_blocks(q), kBlock, 0, s>>>(v, kc, q, db - 1); });
  } else {
    launch(t, CT_KERNEL_PROLOGUE, s, [&] { k_prologue<<<flat_blocks(db / 2), kBlock, 0, s>>>(v, pool, db, q, ranked); });
    launch(t, CT_KERNEL_DEDUP, s, [&] { k_dedup<<<flat_blocks(q), kBlock, 0, s>>>(v, kc, nullptr, q, db - 1); });
  }
}

// Whether a chunk that cannot reach capacity is inserted speculatively.  AUTO follows the
// table's last insert chunk (reported through the mapped feedback word, possibly stale): keys
// mostly new -> speculative; mostly present or repeated -> repeated keys resolved first, where
// only one copy of each key probes the table.
bool use_speculation(const ct_table* t, int word) {
  if (t->insert_path == CT_INSERT_RESOLVE_FIRST) return false;
  if (t->insert_path == CT_INSERT_SPECULATIVE || !t->fb_host) return true;
  const uint64_t f = __atomic_load_n(t->fb_host + word, __ATOMIC_RELAXED);
  const uint64_t fq = f >> 32, changed = f & 0xFFFFFFFFull;
  return fq == 0 || 2 * changed >= fq;
}

// The scratch of speculative chunks of q elements: the resolution's entries and the flags.
int64_t spec_bytes(int64_t q) { return align_up(12 * q) + align_up(q); }

// Whether a whole batch can and should run speculatively: it cannot reach capacity (an erase never
// does), and the table's last chunk changed most of its keys.
bool spec_wanted(const ct_table* t, bool erase, int64_t n) {
  return (erase || t->size_ub + (uint64_t)n <= (uint64_t)t->desc.capacity) &&
         use_speculation(t, erase ? 1 : 0);
}

// Chunk of a speculative batch given a workspace.  13 bytes a key instead of 79 make chunks of 2^23
// keys affordable (109 MB): 6,000,000 keys into an empty map took 500 us in chunks of 2^21, 475 in
// one; 2^22 keys erased and inserted again in a table of 2^24 800, now 779.
constexpr int64_t kSpecChunk = (int64_t)1 << 23;

int64_t spec_chunk(const ct_table* t, int64_t n) {
  if (t->chunk_chosen || n <= t->chunk) return 0;
  const int64_t q = pow2ceil(std::min<int64_t>(n, kSpecChunk));
  return q > t->chunk ? q : 0;
}

enum BatchKind : int { bInsert, bErase, bPool };  // bPool: insert_alloc and erase_release

// What a batch of n keys can use.
int64_t batch_bytes(const ct_table* t, BatchKind kind, int64_t n) {
  if (kind != bPool && spec_wanted(t, kind == bErase, n)) {
    const int64_t q = spec_chunk(t, n);
    return q ? spec_bytes(q) : 0;
  }
  Layout L;
  const int64_t q = workspace_chunk(t, n);
  return q && layout_scratch(&L, q, 0) ? L.total : 0;
}

// The table's own scratch, or `ws` when it holds what the batch can use now (batch_bytes).
BatchScratch batch_scratch(const ct_table* t, BatchKind kind, int64_t n, void* ws, int64_t ws_bytes) {
  BatchScratch b = {t->v, t->chunk, false};
  if (!ws) return b;
  uint8_t* base = static_cast<uint8_t*>(ws);
  Layout L;
  if (kind != bPool && spec_wanted(t, kind == bErase, n)) {
    const int64_t q = spec_chunk(t, n);
    if (q && ws_bytes >= spec_bytes(q)) {
      b.v.dd = reinterpret_cast<uint64_t*>(base);
      b.v.flag = base + align_up(12 * q);
      b.chunk = q;
      b.spec = true;
    }
  } else if (const int64_t q = workspace_chunk(t, n);
             q && layout_scratch(&L, q, 0) && ws_bytes >= L.total) {
    scratch_view(&b.v, base, L);
    b.chunk = q;
  }
  return b;
}

// A chunk of at least this many keys that the host cannot prove to stay below capacity enqueues both
// paths and k_spec_decide picks one on the device: a program that enqueues rounds of erases and
// inserts ahead of the device never gives the host a bound it can use.  The path not taken costs its
// launches (about 30 us); the speculative path saves 230 us per 2^23 keys that are mostly new.
// Batches of 2^21 keys would gain no more than those launches.
constexpr int64_t kDeviceDecides = (int64_t)1 << 22;

// Inserts and erases of at most this many keys read ahead on their probe paths (ProbeRound): their
// waves do not fill the chip, so a lane waits for one bucket after another while the memory has
// room.  60,000 keys erased and inserted again at load 0.8 took 86 us without and 79 with; at 2^18
// keys (a voxel frame) the extra lines cost as much as they save (61 us without, 66 with).  Finds
// walk shorter paths and gained nothing.
constexpr int64_t kAheadMax = 65536;

void find_kernel(int vk, hipStream_t s, const TableView& v, const uint64_t* keys, int64_t n, void* out,
                 uint8_t* found) {
  const int gb = group_blocks((n + kSlots - 1) / kSlots);
  if (vk == CT_VAL_U32) k_find<1><<<gb, kBlock, 0, s>>>(v, keys, n, out, found);
  else if (vk == CT_VAL_U64) k_find<2><<<gb, kBlock, 0, s>>>(v, keys, n, out, found);
  else k_find<0><<<gb, kBlock, 0, s>>>(v, keys, n, nullptr, found);
}

// Batches (and last chunks) of at most this many keys run as one workgroup's launch: 2048 keys erased,
// inserted and partly looked up took 66 us as separate launches and take 50; the limit is what one
// workgroup holds at two keys per thread.  The price is in tables filled to their last slots, where
// absent keys walk hundreds of buckets or all of them and one compute unit walks them alone: 2000
// absent keys erased from a full default table of 2^16 took 0.56 ms as separate launches and take
// 0.75, and 7.6 and 16.5 ms where no bucket at all is open; up to load 0.95 none was slower.
constexpr int64_t kSmallBatch = kSmallMax;

template <int VK, int OP>
ct_status small_batch(ct_table* t, const TableView& v, ct_pool* p, const uint64_t* keys,
                      const uint8_t* skip, const void* vals, int64_t n, uint8_t* status,
                      int32_t* vout, hipStream_t s) {
  const int threads = (int)std::min<int64_t>(1024, std::max<int64_t>(64, pow2ceil(n)));
  launch(t, OP == sInsert || OP == sAlloc ? CT_KERNEL_INSERT : CT_KERNEL_ERASE, s, [&] {
    k_small<VK, OP><<<1, threads, 0, s>>>(v, p ? p->hdr : nullptr, p ? p->stack : nullptr, keys, skip,
                                          vals, (int32_t)n, dedup_slots_for(n), status, vout);
  });
  return launched();
}

// The resolution kernels of a speculative chunk (after its insert or erase kernel).
// The resolution kernels stride over their elements with at most kSpecGrid blocks: they read one
// header word and leave when nothing is listed, and a small grid keeps that cheap.
constexpr int kSpecGrid = 1024;

template <int VK, bool ERASE>
void spec_resolve(ct_table* t, const TableView& v, const uint64_t* kc, const void* vc, int64_t q,
                  uint8_t* sc, uint32_t db, hipStream_t s, int decided = 0) {
  const int g = std::min(flat_blocks(q), kSpecGrid);
  launch(t, CT_KERNEL_APPLY, s, [&] { k_spec_clear<<<std::min(flat_blocks(db / 2), kSpecGrid), kBlock, 0, s>>>(v, q, ERASE ? 1 : 0, decided); });
  launch(t, CT_KERNEL_DEDUP, s, [&] { k_spec_build<<<g, kBlock, 0, s>>>(v, kc, q); });
  launch(t, CT_KERNEL_FIX, s, [&] { k_spec_probe<VK, ERASE><<<g, kBlock, 0, s>>>(v, kc, vc, q, sc); });
  launch(t, CT_KERNEL_FIX, s, [&] { k_spec_swap<VK, ERASE><<<g, kBlock, 0, s>>>(v, kc, vc, q, sc); });
}

// The workspace of a partitioned insert.
struct PartLayout {
  int64_t ncoarse, nfine, group;   // group: coarse bins whose fine bins r2 holds at a time
  int64_t c1, c2, blocks_per_seg;
  int lp2;
  int64_t off_r1k, off_r1v, off_r1i, off_r2k, off_r2v, off_r2i, off_flag, off_ctr, ctr_words;
  int64_t total;
};

// Which batches take the partitioned path: speculative ones (they cannot reach capacity, and the
// table's last chunk stored most of its keys) of at least three keys per bucket and 2^23 keys.
// Measured with 64-bit values into an empty table, plain against partitioned: at three keys per
// bucket 2^22 keys 235 us against 244, 2^24 keys 1070 against 797; at two, 2^24 keys 1035 against
// 949, which its workspace of 30 bytes a key outweighs; at one, 1052 against 1432 (each bucket
// goes both ways whole).  Smaller batches end up in the caches, where random claims are cheap.  Tables
// beyond 2^24 buckets would need a third level of bins.  Generic keys only: the spatial hash fills
// its bins unevenly.
constexpr int64_t kPartMinKeys = (int64_t)1 << 23;
constexpr int64_t kPartMinRatio = 3;
// The fine bins are filled and inserted in this many groups, which share their memory: one group
// would save 1 % of the time for another 10 bytes of workspace a key, four cost 2 %.
constexpr int kPartGroups = 2;

bool part_layout(const ct_table* t, int64_t n, PartLayout* L) {
  const int64_t nb = (int64_t)t->v.nb;
  if (t->chunk_chosen || t->v.hash != CT_HASH_MIX64 || n < kPartMinKeys || n < kPartMinRatio * nb ||
      n > ((int64_t)1 << 30))
    return false;
  const int vb = t->desc.val_kind == CT_VAL_U64 ? 8 : t->desc.val_kind == CT_VAL_U32 ? 4 : 0;
  L->nfine = (nb + kPartBuckets - 1) / kPartBuckets;
  int bits = 0;
  while (((int64_t)1 << bits) < L->nfine) ++bits;
  L->lp2 = std::min(8, bits / 2);
  L->ncoarse = (L->nfine + ((int64_t)1 << L->lp2) - 1) >> L->lp2;
  if (L->ncoarse > 256) return false;
  // capacities: the mean of uniform hashes and eight standard deviations
  auto cap_for = [](double mean) { return (int64_t)(mean + 8.0 * std::sqrt(mean)) + 64; };
  const double per_bucket = (double)n / (double)nb;
  L->c1 = cap_for(per_bucket * kPartBuckets * (double)((int64_t)1 << L->lp2) / kBinSub * 1.02);
  L->c2 = std::min<int64_t>(cap_for(per_bucket * kPartBuckets), kPartPer * kPartThreads);
  L->group = (L->ncoarse + kPartGroups * kPartXcds - 1) / (kPartGroups * kPartXcds) * kPartXcds;
  L->blocks_per_seg = std::max<int64_t>(1, (L->c1 + kBinTile - 1) / kBinTile);
  const int64_t n1 = L->ncoarse * kBinSub * L->c1, n2 = (L->group << L->lp2) * L->c2;
  int64_t off = 0;
  auto take = [&](int64_t bytes) {
    const int64_t o = off;
    off = align_up(off + bytes);
    return o;
  };
  L->off_r1k = take(n1 * 8);
  L->off_r1v = take(n1 * vb);
  L->off_r1i = take(n1 * 4);
  // the resolution's entries take r1's place: at most pow2ceil(n) of them, 12 bytes each
  off = std::max(off, align_up(12 * pow2ceil(n)));
  L->off_r2k = take(n2 * 8);
  L->off_r2v = take(n2 * vb);
  L->off_r2i = take(n2 * 4);
  L->off_flag = take(n);
  L->ctr_words = L->ncoarse * (kPartCtr + kCtrStride) + kCtrStride + (L->ncoarse << L->lp2);
  L->off_ctr = take(L->ctr_words * 4);
  L->total = off;
  return true;
}

bool part_wanted(const ct_table* t, int64_t n, PartLayout* L) {
  return t->size_ub + (uint64_t)n <= (uint64_t)t->desc.capacity && use_speculation(t, 0) &&
         part_layout(t, n, L);
}

template <int VK>
ct_status part_insert(ct_table* t, const PartLayout& L, uint8_t* ws, const uint64_t* keys,
                      const void* vals, int64_t n, uint8_t* status, hipStream_t s) {
  PartView P;
  P.r1k = reinterpret_cast<uint64_t*>(ws + L.off_r1k);
  P.r1v = ws + L.off_r1v;
  P.r1i = reinterpret_cast<uint32_t*>(ws + L.off_r1i);
  P.r2k = reinterpret_cast<uint64_t*>(ws + L.off_r2k);
  P.r2v = ws + L.off_r2v;
  P.r2i = reinterpret_cast<uint32_t*>(ws + L.off_r2i);
  P.flag = ws + L.off_flag;
  P.cur1 = reinterpret_cast<uint32_t*>(ws + L.off_ctr);
  P.nleft = P.cur1 + L.ncoarse * kPartCtr;
  P.nover = P.nleft + L.ncoarse * kCtrStride;
  P.cur2 = P.nover + kCtrStride;
  P.c1 = (uint32_t)L.c1;
  P.c2 = (uint32_t)L.c2;
  P.lp2 = L.lp2;
  TableView v = t->v;  // the resolution reads the flags and its entries from the workspace
  v.flag = P.flag;
  v.dd = P.r1k;
  t->size_ub = std::min<uint64_t>(t->size_ub + (uint64_t)n, (uint64_t)t->desc.capacity);
  fresh_counts(t, s);
  launch(t, CT_KERNEL_PROLOGUE, s, [&] { k_purge_clear<<<flat_blocks(L.ctr_words), kBlock, 0, s>>>(P.cur1, L.ctr_words); });
  launch(t, CT_KERNEL_INSERT, s, [&] { k_part_coarse<VK><<<(int)((n + kBinTile - 1) / kBinTile), kBlock, 0, s>>>(v, P, keys, vals, n, (int)L.ncoarse, status); });
  for (int64_t c0 = 0; c0 < L.ncoarse; c0 += L.group) {
    const int64_t nc = (std::min(L.group, L.ncoarse - c0) + kPartXcds - 1) / kPartXcds * kPartXcds;
    launch(t, CT_KERNEL_INSERT, s, [&] { k_part_fine<VK><<<(int)(nc * kBinSub * L.blocks_per_seg), kBlock, 0, s>>>(v, P, (int)c0, (int)L.ncoarse, (int)L.blocks_per_seg); });
    launch(t, CT_KERNEL_INSERT, s, [&] { k_part_insert<VK><<<(int)(nc << L.lp2), kPartThreads, 0, s>>>(v, P, (int)c0, status); });
  }
  const int lb = (int)std::max<int64_t>(1, 2048 / L.ncoarse);
  launch(t, CT_KERNEL_INSERT, s, [&] { k_part_left<VK><<<(int)L.ncoarse * lb, kBlock, 0, s>>>(v, P, lb, status); });
  launch(t, CT_KERNEL_INSERT, s, [&] { k_part_over<VK><<<(int)std::min<int64_t>((n + kPartWindow - 1) / kPartWindow, kSpecGrid), kBlock, 0, s>>>(v, P, keys, vals, n, status); });
  spec_resolve<VK, false>(t, v, keys, vals, n, status, dedup_slots_for(std::min<int64_t>(n, (int64_t)1 << 26)), s);
  return counted(t);
}

// Insert of n keys in the chunks and with the scratch of B.
template <int VK>
ct_status insert_chunks(ct_table* t, const BatchScratch& B, const uint64_t* keys,
                        const void* vals, int64_t n, uint8_t* status, hipStream_t s) {
  const TableView& v = B.v;
  fresh_counts(t, s);
  const int vb = VK == 1 ? 4 : 8;
  for (int64_t c0 = 0; c0 < n; c0 += B.chunk) {
    const int64_t q = std::min<int64_t>(B.chunk, n - c0);
    const uint32_t db = dedup_slots_for(q);
    const uint64_t* kc = keys + c0;
    const void* vc = VK ? static_cast<const void*>(static_cast<const uint8_t*>(vals) + c0 * vb) : nullptr;
    uint8_t* sc = status ? status + c0 : nullptr;
    const int gb = group_blocks((q + kSlots - 1) / kSlots);
    const int ntiles = (int)((q + kTile - 1) / kTile);
    // the host bound proves that no element can meet FULL: the rank pass is not needed
    const bool surely_fast = t->size_ub + (uint64_t)q <= (uint64_t)t->desc.capacity;
    t->size_ub = std::min<uint64_t>(t->size_ub + (uint64_t)q, (uint64_t)t->desc.capacity);
    if (q <= kSmallBatch) {
      ct_status r = small_batch<VK, sInsert>(t, v, nullptr, kc, nullptr, vc, q, sc, nullptr, s);
      if (r != CT_OK) return r;
      continue;
    }
    if (surely_fast && (B.spec || use_speculation(t, 0))) {
      // speculative: insert first, then resolve the copies of keys listed as ambiguous
      launch(t, CT_KERNEL_INSERT, s, [&] { (q <= kAheadMax ? k_insert_spec<VK, true> : k_insert_spec<VK, false>)<<<gb, kBlock, 0, s>>>(v, kc, vc, q, sc, 0); });
      spec_resolve<VK, false>(t, v, kc, vc, q, sc, db, s);
      ct_status r = counted(t);
      if (r != CT_OK) return r;
      continue;
    }
    const int settle = gb <= kSettleBlocks;
    const int decided = !surely_fast && t->insert_path != CT_INSERT_RESOLVE_FIRST &&
                        v.r1k && q >= kDeviceDecides;
    if (decided) {  // the speculative kernels first; whichever path is not taken leaves at once
      const int always = t->insert_path == CT_INSERT_SPECULATIVE;
      launch(t, CT_KERNEL_PROLOGUE, s, [&] { k_spec_decide<<<1, 1, 0, s>>>(v, q, always); });
      launch(t, CT_KERNEL_INSERT, s, [&] { k_insert_spec<VK, false><<<gb, kBlock, 0, s>>>(v, kc, vc, q, sc, 1); });
      spec_resolve<VK, false>(t, v, kc, vc, q, sc, db, s, 1);
    }
    dedup_chunk(t, v, nullptr, kc, q, s, settle && !surely_fast, decided);
    launch(t, CT_KERNEL_INSERT, s, [&] { (q <= kAheadMax ? k_insert<VK, false, true> : k_insert<VK, false, false>)<<<gb, kBlock, 0, s>>>(v, kc, vc, q, db - 1, sc, nullptr, nullptr, settle); });
    if (!settle) launch(t, CT_KERNEL_APPLY, s, [&] { k_apply_count<<<1, 1024, 0, s>>>(v, gb, q, 0, decided); });
    if (!surely_fast) {
      if (!settle) launch(t, CT_KERNEL_RANK, s, [&] { k_tile_count<<<ntiles, kBlock, 0, s>>>(v, q); });
      const int inl = ntiles <= kInlineRankTiles ? ntiles : 0;
      if (!inl) launch(t, CT_KERNEL_RANK, s, [&] { k_tile_scan<<<1, 1024, 0, s>>>(v, nullptr, ntiles, 0); });
      launch(t, CT_KERNEL_FINAL, s, [&] { k_final<VK, 0><<<ntiles, kBlock, 0, s>>>(v, nullptr, nullptr, kc, vc, q, sc, nullptr, inl); });
    }
    if (sc && !surely_fast) launch(t, CT_KERNEL_FIX, s, [&] { k_fix<<<flat_blocks((q + 3) / 4), kBlock, 0, s>>>(v, q, sc, nullptr, 0); });
    ct_status r = counted(t);
    if (r != CT_OK) return r;
  }
  return CT_OK;
}

ct_status insert_any(ct_table* t, const BatchScratch& B, const uint64_t* keys, const void* vals,
                     int64_t n, uint8_t* status, hipStream_t s) {
  const int vk = t->desc.val_kind;
  if (vk == CT_VAL_U32) return insert_chunks<1>(t, B, keys, vals, n, status, s);
  if (vk == CT_VAL_U64) return insert_chunks<2>(t, B, keys, vals, n, status, s);
  return insert_chunks<0>(t, B, keys, nullptr, n, status, s);
}

template <bool RELEASE>
ct_status erase_chunks(ct_table* t, const BatchScratch& B, ct_pool* p, const uint64_t* keys,
                       int64_t n, uint8_t* erased, hipStream_t s) {
  const TableView& v = B.v;
  fresh_counts(t, s);
  for (int64_t c0 = 0; c0 < n; c0 += B.chunk) {
    const int64_t q = std::min<int64_t>(B.chunk, n - c0);
    const uint32_t db = dedup_slots_for(q);
    const uint64_t* kc = keys + c0;
    uint8_t* ec = erased ? erased + c0 : nullptr;
    const int gb = group_blocks((q + kSlots - 1) / kSlots);
    const int ntiles = (int)((q + kTile - 1) / kTile);
    if (q <= kSmallBatch) {
      ct_status r = small_batch<1, RELEASE ? sRelease : sErase>(t, v, p, kc, nullptr, nullptr, q, ec,
                                                                nullptr, s);
      if (r != CT_OK) return r;
      continue;
    }
    if (!RELEASE && (B.spec || use_speculation(t, 1))) {
      // speculative: remove first, then move each removal to the lowest copy of its key
      launch(t, CT_KERNEL_ERASE, s, [&] { (q <= kAheadMax ? k_erase_spec<true> : k_erase_spec<false>)<<<gb, kBlock, 0, s>>>(v, kc, q, ec); });
      spec_resolve<0, true>(t, v, kc, nullptr, q, ec, db, s);
      ct_status r = counted(t);
      if (r != CT_OK) return r;
      continue;
    }
    const int settle = gb <= kSettleBlocks;
    dedup_chunk(t, v, RELEASE ? p->hdr : nullptr, kc, q, s, RELEASE);
    launch(t, CT_KERNEL_ERASE, s, [&] { (q <= kAheadMax ? k_erase<RELEASE, true> : k_erase<RELEASE, false>)<<<gb, kBlock, 0, s>>>(v, kc, q, db - 1, ec, settle); });
    if (!RELEASE) {
      if (!settle) launch(t, CT_KERNEL_APPLY, s, [&] { k_apply_count<<<1, 1024, 0, s>>>(v, gb, q, 1, 0); });
    } else {
      const int inl = ntiles <= kInlineRankTiles ? ntiles : 0;
      if (!inl) launch(t, CT_KERNEL_RANK, s, [&] { k_tile_scan<<<1, 1024, 0, s>>>(v, p->hdr, ntiles, 2); });
      launch(t, CT_KERNEL_FINAL, s, [&] { k_final<0, 2><<<ntiles, kBlock, 0, s>>>(v, p->hdr, p->stack, kc, nullptr, q, nullptr, nullptr, inl); });
    }
    ct_status r = counted(t);
    if (r != CT_OK) return r;
  }
  return CT_OK;
}

ct_status check_batch(const ct_table* t, const void* keys, int64_t n, const void* ws = nullptr,
                      int64_t ws_bytes = 0) {
  if (!t || n < 0 || ws_bytes < 0) return CT_E_INVALID;
  if (n > 0 && !keys) return CT_E_INVALID;
  if (reinterpret_cast<uintptr_t>(ws) % kAlign) return CT_E_INVALID;
  return CT_OK;
}

}  // namespace

namespace {
template <class Pred>
ct_status select_into(ct_table* t, const Pred& pred, uint64_t* keys_out, uint64_t* vals_out,
                      int64_t cap, int64_t* h_count, void* stream) {
  if (!t || !h_count || cap < 0 || (cap > 0 && !keys_out)) return CT_E_INVALID;
  if (t->desc.val_kind == CT_VAL_NONE) vals_out = nullptr;
  hipStream_t s = S(stream);
  const int64_t nslots = (int64_t)t->v.nb * kSlots;
  const int64_t rounds = (nslots + kSelRound - 1) / kSelRound;
  const int64_t g0 = std::max<int64_t>(1, std::min<int64_t>(rounds, kMaxGroupBlocks));
  const int64_t per = ((rounds + g0 - 1) / g0) * kSelRound;   // whole rounds per block
  const int grid = (int)((nslots + per - 1) / per);
  k_sel_count<Pred><<<grid, kBlock, 0, s>>>(t->v, pred, per);
  k_sel_scan<Pred><<<1, 1024, 0, s>>>(t->v, pred, grid);
  k_sel_write<Pred><<<grid, kBlock, 0, s>>>(t->v, pred, per, keys_out, vals_out, cap);
  if (launched() != CT_OK) return CT_E_HIP;
  uint64_t c = 0;
  ct_status r = read_back(&t->v.hdr->dump_count, &c, s);
  if (r != CT_OK) return r;
  *h_count = (int64_t)c;
  return CT_OK;
}
}  // namespace

extern "C" {

const char* ct_status_str(ct_status s) {
  switch (s) {
    case CT_OK: return "ok";
    case CT_E_INVALID: return "invalid argument";
    case CT_E_FULL: return "capacity exhausted";
    case CT_E_EMPTY: return "pool empty";
    case CT_E_NOMEM: return "host allocation failed";
    case CT_E_HIP: return "HIP runtime error";
  }
  return "unknown status";
}

ct_status ct_table_bytes(const ct_table_desc* d, int64_t* bytes) {
  Layout L;
  if (!bytes || !make_layout(d, &L)) return CT_E_INVALID;
  *bytes = L.total;
  return CT_OK;
}

ct_status ct_table_init(void* d_buf, int64_t bytes, const ct_table_desc* d, void* stream,
                        ct_table** out) {
  Layout L;
  if (!out || !d_buf || !make_layout(d, &L) || bytes < L.total) return CT_E_INVALID;
  if (reinterpret_cast<uintptr_t>(d_buf) % kAlign) return CT_E_INVALID;
  ct_table* t = new (std::nothrow) ct_table;
  if (!t) return CT_E_NOMEM;
  uint8_t* base = static_cast<uint8_t*>(d_buf);
  t->desc = *d;
  t->desc.bucket_count = L.nb;
  t->desc.chunk = L.chunk;
  t->base = base;
  t->bytes = bytes;
  t->chunk = L.chunk;
  t->chunk_chosen = d->chunk != 0;
  t->size_ub = 0;
  t->dd_bytes = L.bins ? (int64_t)kBinCoarse * kBinSub * L.c1 * 8 : L.dslots * 8;
  TableView& v = t->v;
  v.hdr = reinterpret_cast<Header*>(base);
  v.bk = reinterpret_cast<Bucket*>(base + L.off_bk);
  v.nb = (uint64_t)L.nb;
  v.cap = (uint64_t)d->capacity;
  scratch_view(&v, base, L);
  v.stripes = reinterpret_cast<uint64_t*>(base + L.off_stripes);
  v.hash = d->hash_kind;
  v.nb_pow2 = (L.nb & (L.nb - 1)) == 0;
  v.step_mode = v.nb_pow2 ? 1 : (is_prime(L.nb) ? 2 : 0);
  // the insert-path feedback word; without it every provable chunk is speculative
  v.fb = nullptr;
  void* fbh = nullptr;
  if (hipHostMalloc(&fbh, 64, hipHostMallocMapped) == hipSuccess) {
    void* fbd = nullptr;
    if (hipHostGetDevicePointer(&fbd, fbh, 0) == hipSuccess) {
      t->fb_host = static_cast<uint64_t*>(fbh);
      *t->fb_host = 0;
      v.fb = static_cast<uint64_t*>(fbd);
    } else {
      (void)hipHostFree(fbh);
    }
  }
  (void)hipGetLastError();  // a failed pinned allocation only disables the feedback
  k_table_reset<<<flat_blocks(L.nb * kSlots), kBlock, 0, S(stream)>>>(v, 1);
  if (launched() != CT_OK) {
    if (t->fb_host) (void)hipHostFree(t->fb_host);
    delete t;
    return CT_E_HIP;
  }
  *out = t;
  return CT_OK;
}

ct_status ct_table_destroy(ct_table* t) {
  if (!t) return CT_E_INVALID;
  for (hipEvent_t e : t->prof.events) (void)hipEventDestroy(e);
  if (t->fb_host) (void)hipHostFree(t->fb_host);
  delete t;
  return CT_OK;
}

ct_status ct_table_set_profiling(ct_table* t, int enable) {
  if (!t) return CT_E_INVALID;
  Profiler& P = t->prof;
  if (enable && !P.on) {
    if (P.events.empty()) {
      P.events.resize(8192);
      for (hipEvent_t& e : P.events)
        if (hipEventCreate(&e) != hipSuccess) return CT_E_HIP;
    }
    P.on = true;
  } else if (!enable && P.on) {
    P.on = false;
    return prof_drain(P);
  }
  return CT_OK;
}

ct_status ct_table_profile(ct_table* t, int32_t kind, double* total_ms, int64_t* launches) {
  if (!t || kind < 0 || kind >= CT_KERNEL_KINDS) return CT_E_INVALID;
  ct_status r = prof_drain(t->prof);
  if (total_ms) *total_ms = t->prof.total_ms[kind];
  if (launches) *launches = t->prof.launches[kind];
  return r;
}

ct_status ct_table_profile_reset(ct_table* t) {
  if (!t) return CT_E_INVALID;
  ct_status r = prof_drain(t->prof);
  for (int k = 0; k < CT_KERNEL_KINDS; ++k) {
    t->prof.total_ms[k] = 0.0;
    t->prof.launches[k] = 0;
  }
  return r;
}

ct_status ct_table_info(const ct_table* t, int64_t* bucket_count, int64_t* chunk) {
  if (!t) return CT_E_INVALID;
  if (bucket_count) *bucket_count = (int64_t)t->v.nb;
  if (chunk) *chunk = t->chunk;
  return CT_OK;
}

ct_status ct_table_value_bytes(const ct_table* t, int32_t* bytes) {
  if (!t || !bytes) return CT_E_INVALID;
  *bytes = t->desc.val_kind == CT_VAL_U64 ? 8 : t->desc.val_kind == CT_VAL_U32 ? 4 : 0;
  return CT_OK;
}

ct_status ct_insert_batch_ws(ct_table* t, const uint64_t* keys, const void* vals, int64_t n,
                             uint8_t* status, void* ws, int64_t ws_bytes, void* stream) {
  ct_status r = check_batch(t, keys, n, ws, ws_bytes);
  if (r != CT_OK) return r;
  if (n == 0) return CT_OK;
  const int vk = t->desc.val_kind;
  if (vk != CT_VAL_NONE && !vals) return CT_E_INVALID;
  PartLayout P;
  if (ws && part_wanted(t, n, &P)) {
    uint8_t* w = static_cast<uint8_t*>(ws);
    if (ws_bytes < P.total)
      return insert_any(t, BatchScratch{t->v, t->chunk, false}, keys, vals, n, status, S(stream));
    if (vk == CT_VAL_U32) return part_insert<1>(t, P, w, keys, vals, n, status, S(stream));
    if (vk == CT_VAL_U64) return part_insert<2>(t, P, w, keys, vals, n, status, S(stream));
    return part_insert<0>(t, P, w, keys, nullptr, n, status, S(stream));
  }
  return insert_any(t, batch_scratch(t, bInsert, n, ws, ws_bytes), keys, vals, n, status, S(stream));
}

ct_status ct_insert_batch(ct_table* t, const uint64_t* keys, const void* vals, int64_t n,
                          uint8_t* status, void* stream) {
  return ct_insert_batch_ws(t, keys, vals, n, status, nullptr, 0, stream);
}

ct_status ct_workspace_bytes(const ct_table* t, int32_t op, int32_t pool, int64_t n, int64_t* bytes) {
  if (!t || n < 0 || !bytes || (op != CT_OP_INSERT && op != CT_OP_ERASE)) return CT_E_INVALID;
  PartLayout P;
  *bytes = op == CT_OP_INSERT && !pool && part_wanted(t, n, &P)
               ? P.total
               : batch_bytes(t, pool ? bPool : op == CT_OP_ERASE ? bErase : bInsert, n);
  return CT_OK;
}

ct_status ct_find_batch(ct_table* t, const uint64_t* keys, int64_t n, void* vals_out,
                        uint8_t* found, void* stream) {
  ct_status r = check_batch(t, keys, n);
  if (r != CT_OK) return r;
  const int vk = t->desc.val_kind;
  if (vk == CT_VAL_NONE && vals_out) return CT_E_INVALID;
  if (n == 0) return CT_OK;
  launch(t, CT_KERNEL_FIND, S(stream), [&] { find_kernel(vk, S(stream), t->v, keys, n, vals_out, found); });
  return launched();
}

ct_status ct_erase_batch_ws(ct_table* t, const uint64_t* keys, int64_t n, uint8_t* erased, void* ws,
                            int64_t ws_bytes, void* stream) {
  ct_status r = check_batch(t, keys, n, ws, ws_bytes);
  if (r != CT_OK) return r;
  if (n == 0) return CT_OK;
  return erase_chunks<false>(t, batch_scratch(t, bErase, n, ws, ws_bytes), nullptr, keys, n, erased,
                             S(stream));
}

ct_status ct_erase_batch(ct_table* t, const uint64_t* keys, int64_t n, uint8_t* erased,
                         void* stream) {
  return ct_erase_batch_ws(t, keys, n, erased, nullptr, 0, stream);
}

ct_status ct_size(ct_table* t, int64_t* h_size, void* stream) {
  if (!t || !h_size) return CT_E_INVALID;
  uint64_t v = 0;
  ct_status r = read_back(&t->v.hdr->size, &v, S(stream));
  if (r != CT_OK) return r;
  *h_size = (int64_t)v;
  t->size_ub = v;
  return CT_OK;
}

ct_status ct_clear(ct_table* t, void* stream) {
  if (!t) return CT_E_INVALID;
  launch(t, CT_KERNEL_CLEAR, S(stream), [&] { k_table_reset<<<flat_blocks((int64_t)t->v.nb * kSlots), kBlock, 0, S(stream)>>>(t->v, 0); });
  t->size_ub = 0;
  return launched();
}

ct_status ct_table_device_view(ct_table* t, int32_t mode, void* out, int64_t bytes) {
  if (!t || !out || bytes < (int64_t)sizeof(DevView) || mode < kDevRead || mode > kDevMixed)
    return CT_E_INVALID;
  DevView v{};
  v.t = t->v;
  v.mode = mode;
  std::memcpy(out, &v, sizeof(v));
  // device inserts grow the table behind the host's back
  if (mode == kDevInsert || mode == kDevMixed) t->size_ub = (uint64_t)t->desc.capacity;
  return CT_OK;
}

ct_status ct_dev_apply(ct_table* t, int32_t op, const uint64_t* keys, const void* vals, int64_t n,
                       void* vals_out, uint8_t* status, void* stream) {
  if (!t || n < 0 || (n > 0 && !keys)) return CT_E_INVALID;
  if (op != CT_OP_INSERT && op != CT_OP_FIND && op != CT_OP_ERASE) return CT_E_INVALID;
  const int32_t vk = t->desc.val_kind;
  if (op == CT_OP_INSERT && vk != CT_VAL_NONE && n > 0 && !vals) return CT_E_INVALID;
  if (n == 0) return CT_OK;
  DevView v{};
  v.t = t->v;
  v.mode = op == CT_OP_INSERT ? kDevInsert : op == CT_OP_ERASE ? kDevErase : kDevRead;
  if (op == CT_OP_INSERT)
    t->size_ub = std::min<uint64_t>(t->size_ub + (uint64_t)n, (uint64_t)t->desc.capacity);
  v.striped = op != CT_OP_FIND;
  if (v.striped) k_dev_prep<<<1, kStripes, 0, S(stream)>>>(t->v, op == CT_OP_INSERT ? (uint64_t)n : 0);
  k_dev_apply<<<flat_blocks(n), kBlock, 0, S(stream)>>>(v, op, keys, vals, vk, n, vals_out, status);
  if (v.striped) k_dev_fold<<<1, kStripes, 0, S(stream)>>>(t->v);
  return launched();
}

ct_status ct_dev_apply_mixed(ct_table* t, const uint8_t* ops, const uint64_t* keys, const void* vals,
                             int64_t n, void* vals_out, uint8_t* status, void* stream) {
  if (!t || n < 0 || (n > 0 && (!keys || !ops))) return CT_E_INVALID;
  const int32_t vk = t->desc.val_kind;
  if (vk != CT_VAL_NONE && n > 0 && !vals) return CT_E_INVALID;
  if (n == 0) return CT_OK;
  DevView v{};
  v.t = t->v;
  v.mode = kDevMixed;
  t->size_ub = std::min<uint64_t>(t->size_ub + (uint64_t)n, (uint64_t)t->desc.capacity);
  v.striped = 1;
  k_dev_prep<<<1, kStripes, 0, S(stream)>>>(t->v, (uint64_t)n);
  const int sorted_blocks = (int)std::max<int64_t>(1, std::min<int64_t>((n + kSortWin - 1) / kSortWin, 8192));
  k_dev_apply_sorted<<<sorted_blocks, kBlock, 0, S(stream)>>>(v, ops, keys, vals, vk, n, vals_out,
                                                               status);
  k_dev_fold<<<1, kStripes, 0, S(stream)>>>(t->v);
  return launched();
}

ct_status ct_voxel_insert_neighbours(ct_table* t, const uint64_t* blocks, int64_t n, int32_t ndirs,
                                     void* stream) {
  if (!t || n < 0 || (n > 0 && !blocks) || (ndirs != 6 && ndirs != 26)) return CT_E_INVALID;
  if (t->desc.val_kind == CT_VAL_NONE) return CT_E_INVALID;
  if (n == 0) return CT_OK;
  DevView v{};
  v.t = t->v;
  v.mode = kDevInsert;
  t->size_ub = std::min<uint64_t>(t->size_ub + (uint64_t)n * (uint64_t)ndirs,
                                  (uint64_t)t->desc.capacity);
  v.striped = 1;
  k_dev_prep<<<1, kStripes, 0, S(stream)>>>(t->v, (uint64_t)n * (uint64_t)ndirs);
  k_voxel_neighbours<false><<<flat_blocks(n), kBlock, 0, S(stream)>>>(v, DevPool{}, blocks, n, ndirs);
  k_dev_fold<<<1, kStripes, 0, S(stream)>>>(t->v);
  return launched();
}

ct_status ct_voxel_insert_neighbours_alloc(ct_table* t, ct_pool* p, const uint64_t* blocks,
                                           int64_t n, int32_t ndirs, void* stream) {
  if (!t || !p || n < 0 || (n > 0 && !blocks) || (ndirs != 6 && ndirs != 26)) return CT_E_INVALID;
  if (t->desc.val_kind == CT_VAL_NONE) return CT_E_INVALID;
  if (n == 0) return CT_OK;
  DevView v{};
  v.t = t->v;
  v.mode = kDevInsert;
  t->size_ub = std::min<uint64_t>(t->size_ub + (uint64_t)n * (uint64_t)ndirs,
                                  (uint64_t)t->desc.capacity);
  v.striped = 1;
  k_dev_prep<<<1, kStripes, 0, S(stream)>>>(t->v, (uint64_t)n * (uint64_t)ndirs);
  k_voxel_neighbours<true><<<flat_blocks(n), kBlock, 0, S(stream)>>>(v, DevPool{p->hdr, p->stack},
                                                                     blocks, n, ndirs);
  k_dev_fold<<<1, kStripes, 0, S(stream)>>>(t->v);
  return launched();
}

ct_status ct_dev_update_set(ct_table* map, ct_table* set, const uint64_t* keys, int64_t n,
                            uint8_t* status, void* stream) {
  if (!map || !set || map == set || n < 0 || (n > 0 && !keys)) return CT_E_INVALID;
  if (n == 0) return CT_OK;
  hipStream_t s = S(stream);
  DevView mv{};
  mv.t = map->v;
  mv.mode = kDevRead;
  DevView sv{};
  sv.t = set->v;
  sv.mode = kDevInsert;
  sv.striped = 1;
  set->size_ub = std::min<uint64_t>(set->size_ub + (uint64_t)n, (uint64_t)set->desc.capacity);
  k_dev_prep<<<1, kStripes, 0, s>>>(set->v, (uint64_t)n);
  k_dev_update_set<<<flat_blocks(n), kBlock, 0, s>>>(mv, sv, keys, n, status);
  k_dev_fold<<<1, kStripes, 0, s>>>(set->v);
  return launched();
}

ct_status ct_pool_device_view(ct_pool* p, void* out, int64_t bytes) {
  if (!p || !out || bytes < (int64_t)sizeof(DevPool)) return CT_E_INVALID;
  const DevPool d{p->hdr, p->stack};
  std::memcpy(out, &d, sizeof(d));
  return CT_OK;
}

ct_status ct_dev_pool_apply(ct_pool* p, int32_t op, const int32_t* in, int64_t n, int32_t* out,
                            uint8_t* status, void* stream) {
  if (!p || n < 0 || (op != CT_DEV_PUSH_BACK && op != CT_DEV_POP_BACK)) return CT_E_INVALID;
  if (op == CT_DEV_PUSH_BACK && n > 0 && !in) return CT_E_INVALID;
  if (n == 0) return CT_OK;
  k_dev_pool_apply<<<flat_blocks(n), kBlock, 0, S(stream)>>>(DevPool{p->hdr, p->stack}, op, in, n,
                                                             out, status);
  return launched();
}

ct_status ct_table_rehash(ct_table* src, ct_table* dst, void* stream) {
  if (!src || !dst || src == dst || src->desc.val_kind != dst->desc.val_kind) return CT_E_INVALID;
  int64_t ns = 0, nd = 0;
  ct_status r = ct_size(src, &ns, stream);
  if (r == CT_OK) r = ct_size(dst, &nd, stream);
  if (r != CT_OK) return r;
  if (nd + ns > dst->desc.capacity) return CT_E_FULL;
  if (ns == 0) return CT_OK;
  const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(((int64_t)src->v.nb + kBlock / 8 - 1) / (kBlock / 8), kMaxGroupBlocks));
  hipStream_t s = S(stream);
  launch(dst, CT_KERNEL_INSERT, s, [&] { k_rehash<<<grid, kBlock, 0, s>>>(src->v, dst->v); });
  launch(dst, CT_KERNEL_APPLY, s, [&] { k_apply_count<<<1, 1024, 0, s>>>(dst->v, grid, 0, 0, 0); });
  dst->size_ub = (uint64_t)(nd + ns);
  return launched();
}

ct_status ct_dump(ct_table* t, uint64_t* keys_out, uint64_t* vals_out, int64_t cap,
                  int64_t* h_count, void* stream) {
  return select_into(t, AllKeys{}, keys_out, vals_out, cap, h_count, stream);
}

ct_status ct_select_key_range(ct_table* t, uint64_t lo, uint64_t hi, uint64_t* keys_out,
                              uint64_t* vals_out, int64_t cap, int64_t* h_count, void* stream) {
  return select_into(t, KeyRange{lo, hi}, keys_out, vals_out, cap, h_count, stream);
}

ct_status ct_select_voxel_box(ct_table* t, const int32_t* h_lo3, const int32_t* h_hi3,
                              uint64_t* keys_out, uint64_t* vals_out, int64_t cap, int64_t* h_count,
                              void* stream) {
  if (!h_lo3 || !h_hi3) return CT_E_INVALID;
  VoxelBox box;
  for (int d = 0; d < 3; ++d) {
    box.lo[d] = h_lo3[d];
    box.hi[d] = h_hi3[d];
  }
  return select_into(t, box, keys_out, vals_out, cap, h_count, stream);
}

ct_status ct_check_invariants_detail(ct_table* t, const ct_pool* p, int64_t* h_violations,
                                     uint32_t* h_what, void* stream) {
  if (!t || !h_violations) return CT_E_INVALID;
  if (p && t->desc.val_kind != CT_VAL_U32) return CT_E_INVALID;
  hipStream_t s = S(stream);
  const int64_t pool_cap = p ? std::max<int64_t>(p->cap, 1) : 0;
  k_check_begin<<<1, 1, 0, s>>>(t->v);
  k_check<<<flat_blocks((int64_t)t->v.nb * kSlots), kBlock, 0, s>>>(t->v, pool_cap);
  if (p) k_check_pool<<<flat_blocks(p->cap), kBlock, 0, s>>>(t->v, p->hdr, p->stack);
  if (launched() != CT_OK) return CT_E_HIP;
  Header h;
  if (hipMemcpyAsync(&h, t->v.hdr, sizeof(Header), hipMemcpyDeviceToHost, s) != hipSuccess)
    return CT_E_HIP;
  if (hipStreamSynchronize(s) != hipSuccess) return CT_E_HIP;
  const uint64_t specs = (uint64_t)(h.spec_live[0] != 0) + (uint64_t)(h.spec_live[1] != 0);
  int64_t bad = 0;
  uint32_t what = 0;
  if (h.live_count + specs != h.size || h.size > t->v.cap) {
    ++bad;
    what |= CT_CHECK_SIZE;
  }
  if (h.dup_count) {
    bad += (int64_t)h.dup_count;
    what |= CT_CHECK_DUPLICATE;
  }
  if (h.violations) {
    bad += (int64_t)h.violations;
    what |= CT_CHECK_REACH;
  }
  if (p && (h.pool_bad || h.pool_count != 0 || h.pool_h1 != 0 || h.pool_h2 != 0)) {
    bad += h.pool_bad ? (int64_t)h.pool_bad : 1;
    what |= CT_CHECK_POOL;
  }
  *h_violations = bad;
  if (h_what) *h_what = what;
  return CT_OK;
}

ct_status ct_check_invariants(ct_table* t, const ct_pool* p, int64_t* h_violations, void* stream) {
  return ct_check_invariants_detail(t, p, h_violations, nullptr, stream);
}

ct_status ct_table_health(ct_table* t, int64_t* h_closed, int64_t* h_tombstones, void* stream) {
  if (!t || (!h_closed && !h_tombstones)) return CT_E_INVALID;
  hipStream_t s = S(stream);
  k_health_begin<<<1, 1, 0, s>>>(t->v);
  k_health<<<group_blocks((int64_t)t->v.nb), kBlock, 0, s>>>(t->v);
  if (launched() != CT_OK) return CT_E_HIP;
  Header h;
  if (hipMemcpyAsync(&h, t->v.hdr, sizeof(Header), hipMemcpyDeviceToHost, s) != hipSuccess)
    return CT_E_HIP;
  if (hipStreamSynchronize(s) != hipSuccess) return CT_E_HIP;
  if (h_closed) *h_closed = (int64_t)h.closed_count;
  if (h_tombstones) *h_tombstones = (int64_t)h.tomb_count;
  return CT_OK;
}

ct_status ct_table_purge(ct_table* t, void* stream) {
  if (!t) return CT_E_INVALID;
  hipStream_t s = S(stream);
  uint32_t* bits = reinterpret_cast<uint32_t*>(t->v.dd);
  const int64_t window = t->dd_bytes / 4 * 32;   // buckets per pass: one bit each
  const int64_t nb = (int64_t)t->v.nb;
  for (int64_t w0 = 0; w0 < nb; w0 += window) {
    const int64_t w1 = std::min(nb, w0 + window);
    const int64_t words = (w1 - w0 + 31) / 32;
    k_purge_clear<<<flat_blocks(words), kBlock, 0, s>>>(bits, words);
    k_purge_mark<<<flat_blocks(nb * kSlots), kBlock, 0, s>>>(t->v, bits, w0, w1);
    k_purge_reopen<<<flat_blocks((w1 - w0) * kSlots), kBlock, 0, s>>>(t->v, bits, w0, w1);
    if (launched() != CT_OK) return CT_E_HIP;
  }
  return CT_OK;
}

ct_status ct_get_error(ct_table* t, uint32_t* h_err, void* stream) {
  if (!t || !h_err) return CT_E_INVALID;
  uint32_t e = 0;
  ct_status r = read_back(&t->v.hdr->err, &e, S(stream));
  if (r != CT_OK) return r;
  *h_err = e;
  const uint32_t zero = 0;
  if (hipMemcpyAsync(&t->v.hdr->err, &zero, sizeof(zero), hipMemcpyHostToDevice, S(stream)) != hipSuccess)
    return CT_E_HIP;
  return hipStreamSynchronize(S(stream)) == hipSuccess ? CT_OK : CT_E_HIP;
}

__global__ void k_set_inject(TableView t, uint32_t every) { t.hdr->inject = every; }

ct_status ct_table_debug_inject_claim_losses(ct_table* t, uint32_t every, void* stream) {
  if (!t) return CT_E_INVALID;
  k_set_inject<<<1, 1, 0, S(stream)>>>(t->v, every);
  return launched();
}

ct_status ct_table_dedup_skewed(ct_table* t, int32_t* h_skewed, void* stream) {
  if (!t || !h_skewed) return CT_E_INVALID;
  uint32_t v = 0;
  ct_status r = read_back(&t->v.hdr->dskew, &v, S(stream));
  if (r != CT_OK) return r;
  *h_skewed = v ? 1 : 0;
  return CT_OK;
}

ct_status ct_table_set_insert_path(ct_table* t, int32_t path) {
  if (!t || path < CT_INSERT_AUTO || path > CT_INSERT_SPECULATIVE) return CT_E_INVALID;
  t->insert_path = path;
  return CT_OK;
}

// --- pools -------------------------------------------------------------------------------------
ct_status ct_pool_bytes(int64_t capacity, int64_t* bytes) {
  if (!bytes || capacity < 0 || capacity > 0x7FFFFFFFll) return CT_E_INVALID;
  *bytes = align_up((int64_t)sizeof(PoolHeader)) + align_up(capacity * 4);
  return CT_OK;
}

ct_status ct_pool_init(void* d_buf, int64_t bytes, int64_t capacity, void* stream, ct_pool** out) {
  int64_t need = 0;
  if (!out || !d_buf || ct_pool_bytes(capacity, &need) != CT_OK || bytes < need) return CT_E_INVALID;
  if (reinterpret_cast<uintptr_t>(d_buf) % kAlign) return CT_E_INVALID;
  ct_pool* p = new (std::nothrow) ct_pool;
  if (!p) return CT_E_NOMEM;
  p->base = static_cast<uint8_t*>(d_buf);
  p->cap = capacity;
  p->hdr = reinterpret_cast<PoolHeader*>(p->base);
  p->stack = reinterpret_cast<int32_t*>(p->base + align_up((int64_t)sizeof(PoolHeader)));
  k_pool_init<<<flat_blocks(capacity), kBlock, 0, S(stream)>>>(p->hdr, p->stack, capacity);
  if (launched() != CT_OK) {
    delete p;
    return CT_E_HIP;
  }
  *out = p;
  return CT_OK;
}

ct_status ct_pool_destroy(ct_pool* p) {
  if (!p) return CT_E_INVALID;
  delete p;
  return CT_OK;
}

ct_status ct_pool_pop_batch(ct_pool* p, int64_t n, int32_t* out, uint8_t* status, void* stream) {
  if (!p || n < 0) return CT_E_INVALID;
  if (n == 0) return CT_OK;
  k_pool_snapshot<<<1, 1, 0, S(stream)>>>(p->hdr);
  k_pool_pop<<<flat_blocks(n), kBlock, 0, S(stream)>>>(p->hdr, p->stack, n, out, status);
  return launched();
}

ct_status ct_pool_pop_front_batch(ct_pool* p, int64_t n, int32_t* out, uint8_t* status,
                                  void* stream) {
  if (!p || n < 0) return CT_E_INVALID;
  if (n == 0) return CT_OK;
  k_pool_snapshot<<<1, 1, 0, S(stream)>>>(p->hdr);
  k_pool_pop_front<<<flat_blocks(n), kBlock, 0, S(stream)>>>(p->hdr, p->stack, n, out, status);
  return launched();
}

ct_status ct_pool_push_front_batch(ct_pool* p, const int32_t* in, int64_t n, uint8_t* status,
                                   void* stream) {
  if (!p || n < 0 || (n > 0 && !in)) return CT_E_INVALID;
  if (n == 0) return CT_OK;
  k_pool_snapshot<<<1, 1, 0, S(stream)>>>(p->hdr);
  k_pool_push_front<<<flat_blocks(n), kBlock, 0, S(stream)>>>(p->hdr, p->stack, in, n, status);
  return launched();
}

ct_status ct_pool_push_batch(ct_pool* p, const int32_t* in, int64_t n, uint8_t* status,
                             void* stream) {
  if (!p || n < 0 || (n > 0 && !in)) return CT_E_INVALID;
  if (n == 0) return CT_OK;
  k_pool_snapshot<<<1, 1, 0, S(stream)>>>(p->hdr);
  k_pool_push<<<flat_blocks(n), kBlock, 0, S(stream)>>>(p->hdr, p->stack, in, n, status);
  return launched();
}

ct_status ct_pool_size(ct_pool* p, int64_t* h_size, void* stream) {
  if (!p || !h_size) return CT_E_INVALID;
  return read_back(&p->hdr->top, h_size, S(stream));
}

ct_status ct_pool_dump(ct_pool* p, int32_t* out, int64_t cap, int64_t* h_count, void* stream) {
  if (!p || !h_count || cap < 0 || (cap > 0 && !out)) return CT_E_INVALID;
  if (cap > 0) k_pool_copy<<<flat_blocks(cap), kBlock, 0, S(stream)>>>(p->hdr, p->stack, out, cap);
  if (launched() != CT_OK) return CT_E_HIP;
  return read_back(&p->hdr->top, h_count, S(stream));
}

ct_status ct_pool_get_error(ct_pool* p, uint32_t* h_err, void* stream) {
  if (!p || !h_err) return CT_E_INVALID;
  uint32_t e = 0;
  ct_status r = read_back(&p->hdr->err, &e, S(stream));
  if (r != CT_OK) return r;
  *h_err = e;
  const uint32_t zero = 0;
  if (hipMemcpyAsync(&p->hdr->err, &zero, sizeof(zero), hipMemcpyHostToDevice, S(stream)) != hipSuccess)
    return CT_E_HIP;
  return hipStreamSynchronize(S(stream)) == hipSuccess ? CT_OK : CT_E_HIP;
}

}  // extern "C"

namespace {

// Pool-valued insert of n keys; with `skip`, only the elements whose byte there is zero take part,
// in index order among themselves (masked batches are sparse: their repeated keys are resolved
// through dd, whatever the chunk size).
ct_status insert_alloc_chunks(ct_table* t, const BatchScratch& B, ct_pool* p, const uint64_t* keys,
                              const uint8_t* skip, int64_t n, int32_t* vals_out, uint8_t* status,
                              hipStream_t s) {
  const TableView& v = B.v;
  ct_status r = CT_OK;
  for (int64_t c0 = 0; c0 < n; c0 += B.chunk) {
    const int64_t q = std::min<int64_t>(B.chunk, n - c0);
    const uint32_t db = dedup_slots_for(q);
    const uint64_t* kc = keys + c0;
    const uint8_t* mc = skip ? skip + c0 : nullptr;
    uint8_t* sc = status ? status + c0 : nullptr;
    int32_t* vc = vals_out ? vals_out + c0 : nullptr;
    if (q <= kSmallBatch) {
      r = small_batch<1, sAlloc>(t, v, p, kc, mc, nullptr, q, sc, vc, s);
      if (r != CT_OK) return r;
      t->size_ub = std::min<uint64_t>(t->size_ub + (uint64_t)q, (uint64_t)t->desc.capacity);
      continue;
    }
    t->size_ub = std::min<uint64_t>(t->size_ub + (uint64_t)q, (uint64_t)t->desc.capacity);
    const int gb = group_blocks((q + kSlots - 1) / kSlots);
    const int ntiles = (int)((q + kTile - 1) / kTile);
    if (mc) {
      launch(t, CT_KERNEL_PROLOGUE, s, [&] { k_prologue<<<flat_blocks(db / 2), kBlock, 0, s>>>(v, p->hdr, db, q, 1); });
      launch(t, CT_KERNEL_DEDUP, s, [&] { k_dedup<<<flat_blocks(q), kBlock, 0, s>>>(v, kc, mc, q, db - 1); });
    } else {
      dedup_chunk(t, v, p->hdr, kc, q, s, 1);
    }
    launch(t, CT_KERNEL_INSERT, s, [&] { (q <= kAheadMax ? k_insert<1, true, true> : k_insert<1, true, false>)<<<gb, kBlock, 0, s>>>(v, kc, nullptr, q, db - 1, sc, vc, mc, 0); });
    const int inl = ntiles <= kInlineRankTiles ? ntiles : 0;
    if (!inl) launch(t, CT_KERNEL_RANK, s, [&] { k_tile_scan<<<1, 1024, 0, s>>>(v, p->hdr, ntiles, 1); });
    launch(t, CT_KERNEL_FINAL, s, [&] { k_final<1, 1><<<ntiles, kBlock, 0, s>>>(v, p->hdr, p->stack, kc, nullptr, q, sc, vc, inl); });
    if (sc || vc) launch(t, CT_KERNEL_FIX, s, [&] { k_fix<<<flat_blocks((q + 3) / 4), kBlock, 0, s>>>(v, q, sc, vc, 1); });
    r = launched();
    if (r != CT_OK) return r;
  }
  return CT_OK;
}

}  // namespace

extern "C" {

ct_status ct_insert_alloc_batch_ws(ct_table* t, ct_pool* p, const uint64_t* keys,
                                   const uint8_t* skip, int64_t n, int32_t* vals_out,
                                   uint8_t* status, void* ws, int64_t ws_bytes, void* stream) {
  ct_status r = check_batch(t, keys, n, ws, ws_bytes);
  if (r != CT_OK || !p) return CT_E_INVALID;
  if (t->desc.val_kind != CT_VAL_U32) return CT_E_INVALID;
  if (n == 0) return CT_OK;
  return insert_alloc_chunks(t, batch_scratch(t, bPool, n, ws, ws_bytes), p, keys, skip, n, vals_out,
                             status, S(stream));
}

ct_status ct_insert_alloc_batch(ct_table* t, ct_pool* p, const uint64_t* keys, int64_t n,
                                int32_t* vals_out, uint8_t* status, void* stream) {
  return ct_insert_alloc_batch_ws(t, p, keys, nullptr, n, vals_out, status, nullptr, 0, stream);
}

ct_status ct_insert_alloc_batch_masked(ct_table* t, ct_pool* p, const uint64_t* keys,
                                       const uint8_t* skip, int64_t n, int32_t* vals_out,
                                       uint8_t* status, void* stream) {
  if (n > 0 && !skip) return CT_E_INVALID;
  return ct_insert_alloc_batch_ws(t, p, keys, skip, n, vals_out, status, nullptr, 0, stream);
}

ct_status ct_erase_release_batch_ws(ct_table* t, ct_pool* p, const uint64_t* keys, int64_t n,
                                    uint8_t* erased, void* ws, int64_t ws_bytes, void* stream) {
  ct_status r = check_batch(t, keys, n, ws, ws_bytes);
  if (r != CT_OK || !p) return CT_E_INVALID;
  if (t->desc.val_kind != CT_VAL_U32) return CT_E_INVALID;
  if (n == 0) return CT_OK;
  return erase_chunks<true>(t, batch_scratch(t, bPool, n, ws, ws_bytes), p, keys, n, erased, S(stream));
}

ct_status ct_erase_release_batch(ct_table* t, ct_pool* p, const uint64_t* keys, int64_t n,
                                 uint8_t* erased, void* stream) {
  return ct_erase_release_batch_ws(t, p, keys, n, erased, nullptr, 0, stream);
}

}  // extern "C"

// --- multi-table plans ----------------------------------------------------------------------
// A plan replays a schedule of single-table operations.  Tables are spread over `lanes` side
// streams forked from the caller's stream (a table's operations stay on one stream, so their
// order holds) and joined back at the end; each operation runs the same kernel pipeline as the
// single-table call.  The whole fork/join sequence captures into one HIP graph.
namespace {
struct PlanOp {
  ct_table* t;
  int32_t type;
  const uint64_t* keys;
  const void* vals;
  void* vout;
  uint8_t* flags;
  int64_t n;
};
}  // namespace

namespace ct_group {
// One kernel launch of a grouped plan: `n` entries from `entry_off` of the entry array.
struct Launch {
  int32_t stage, n, blocks;
  int64_t entry_off;
};
}  // namespace ct_group

struct ct_plan {
  std::vector<PlanOp> ops;
  std::vector<ct_table*> tables;  // distinct tables in first-use order
  std::vector<hipStream_t> side;
  std::vector<hipEvent_t> ev;     // fork event + one join event per side stream
  // grouped form (ct_plan_group): valid while the plan still has `grouped_ops` operations
  std::vector<ct_group::Launch> glaunch;
  const void* gsteps = nullptr;    // device: GStep[]
  const void* gentries = nullptr;  // device: GEntry[]
  const void* gcopies = nullptr;   // device: GCopy[] of the merged operations' copy stages
  size_t grouped_ops = (size_t)-1;
  int gblock = kBlock;             // threads per block of its find / insert / erase stages
  const void* glaunch_dev = nullptr;  // device: GLaunchDev[] for the single-launch form
  int32_t gwidest = 1;             // most blocks of any one stage launch
};

namespace {

ct_status plan_streams(ct_plan* p, int32_t lanes) {
  while ((int32_t)p->side.size() < lanes) {
    hipStream_t s;
    if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) return CT_E_HIP;
    p->side.push_back(s);
  }
  while (p->ev.size() < p->side.size() + 1) {
    hipEvent_t e;
    if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) return CT_E_HIP;
    p->ev.push_back(e);
  }
  return CT_OK;
}

ct_status run_op(const PlanOp& o, hipStream_t s) {
  ct_table* t = o.t;
  const int vk = t->desc.val_kind;
  switch (o.type) {
    case kOpClear:
      launch(t, CT_KERNEL_CLEAR, s, [&] { k_table_reset<<<flat_blocks((int64_t)t->v.nb * kSlots), kBlock, 0, s>>>(t->v, 0); });
      return launched();
    case kOpInsert:
      return insert_any(t, BatchScratch{t->v, t->chunk, false}, o.keys, o.vals, o.n, o.flags, s);
    case kOpErase:
      return erase_chunks<false>(t, BatchScratch{t->v, t->chunk, false}, nullptr, o.keys, o.n, o.flags, s);
    default: {
      launch(t, CT_KERNEL_FIND, s, [&] { find_kernel(vk, s, t->v, o.keys, o.n, o.vout, o.flags); });
      return launched();
    }
  }
}

// Copy-stage blocks for a segment: enough 256-thread blocks for 16-byte units, at most 2048.
int copy_blocks(int64_t bytes) {
  const int64_t b = (bytes / 16 + kBlock - 1) / kBlock;
  return (int)std::max<int64_t>(1, std::min<int64_t>(b, 2048));
}

bool inserts_or_erases(const GStep& g) { return g.type == kOpInsert || g.type == kOpErase; }

// Blocks of a grouped stage whose blocks stride over n units of work and usually find little
// or nothing to do (the resolution of a speculative step, the repeated-key outcomes, the
// prologue's scratch clear): 8 units per thread, at most 1024 blocks per step.
int spec_blocks(int64_t n) {
  const int64_t b = (n + 8 * kBlock - 1) / (8 * kBlock);
  return (int)std::max<int64_t>(1, std::min<int64_t>(b, 1024));
}

// Units of a chunk's scratch clear (as prologue_units on the device).
int64_t prologue_units_host(uint32_t dslots, int64_t q) { return (int64_t)dslots / 2 + (q + 15) / 16; }

// Blocks of step `g` in stage `stage` (0: the step has no such stage); the same grids as the
// single-table pipeline.
int stage_blocks(int stage, const GStep& g) {
  switch (stage) {
    case gReset: return g.type == kOpClear ? flat_blocks((int64_t)g.v.nb * kSlots) : 0;
    case gPro: return inserts_or_erases(g) ? spec_blocks(prologue_units_host(g.db, g.q)) : 0;
    case gDedup: return inserts_or_erases(g) ? flat_blocks(g.q) : 0;
    case gFind: return g.type == kOpFind ? g.gb : 0;
    case gInsert: return g.type == kOpInsert ? g.gb : 0;
    case gErase: return g.type == kOpErase ? g.gb : 0;
    case gApply: return inserts_or_erases(g) ? 1 : 0;
    // resolution of a speculative step: a few elements per thread when something is listed; the
    // blocks leave at once otherwise
    case gSClear: return inserts_or_erases(g) && g.spath ? spec_blocks((int64_t)g.db / 2) : 0;
    case gSBuild:
    case gSProbe:
    case gSSwap: return inserts_or_erases(g) && g.spath ? spec_blocks(g.q) : 0;
    case gCount: return g.type == kOpInsert ? g.ntiles : 0;
    case gScan: return g.type == kOpInsert ? 1 : 0;
    case gFinal: return g.type == kOpInsert ? g.ntiles : 0;
    case gFix: return g.type == kOpInsert && g.flags ? spec_blocks(g.q) : 0;
  }
  return 0;
}

// The grouped form of a plan, built on the host.  `base` is the device buffer the form will live
// in (null while only sizing it): steps, entries, copy segments, then the merge area.
struct GroupForm {
  std::vector<GStep> steps;
  std::vector<GEntry> entries;
  std::vector<GCopy> copies;
  std::vector<ct_group::Launch> launches;
  int64_t merge_bytes = 0;
  int64_t steps_off = 0, entries_off = 0, copies_off = 0, launches_off = 0, merge_off = 0,
          total = 0;
};

// Cut the plan into chunk-steps, assign each the per-table ordinal as its level, and lay out one
// launch per (level, stage) that has steps.  With CT_GROUP_MERGE_RUNS, a run of consecutive
// operations of one kind on one table becomes one operation over a contiguous copy of its arrays
// in the merge area (a batch equals its parts applied in order), gathered before the first level
// and scattered back after the last.  Host only.
// Threads per block of the grouped find / insert / erase stages encoded in `options`.
int group_block_size(int32_t options) {
  const int code = (options >> CT_GROUP_BLOCK_SHIFT) & 0xF;
  return code ? (1 << code) : kBlock;
}

bool group_options_valid(int32_t options) {
  if (options & ~(CT_GROUP_MERGE_RUNS | (0xF << CT_GROUP_BLOCK_SHIFT))) return false;
  const int code = (options >> CT_GROUP_BLOCK_SHIFT) & 0xF;
  return code == 0 || (code >= 7 && code <= 10);   // 128 .. 1024 threads
}

ct_status group_build(const ct_plan* p, int32_t options, uint8_t* base, GroupForm& F) {
  const bool merge = (options & CT_GROUP_MERGE_RUNS) != 0;
  const int bs = group_block_size(options);
  struct Eff {  // an operation of one table as it will be cut into steps
    PlanOp op;
    size_t first, count;  // its run of plan operations
  };
  std::vector<std::vector<Eff>> per(p->tables.size());
  for (size_t k = 0; k < p->ops.size(); ++k) {
    const PlanOp& o = p->ops[k];
    const size_t ti = (size_t)(std::find(p->tables.begin(), p->tables.end(), o.t) - p->tables.begin());
    std::vector<Eff>& v = per[ti];
    if (merge && o.type != kOpClear && !v.empty() && v.back().op.type == o.type) {
      v.back().count += 1;
      v.back().op.n += o.n;
    } else {
      v.push_back(Eff{o, k, 1});
    }
  }
  // merge area: contiguous arrays for every run of two or more operations
  std::vector<GCopy> copy_out;
  int64_t moff = 0;
  auto take = [&](int64_t bytes) {
    const int64_t o = moff;
    moff += align_up(bytes);
    return o;
  };
  struct Fix {  // device addresses of a merged run's arrays, as offsets into the merge area
    int64_t keys = -1, vals = -1, flags = -1, vout = -1;
  };
  std::vector<std::vector<Fix>> fixes(per.size());
  for (size_t ti = 0; ti < per.size(); ++ti) {
    fixes[ti].resize(per[ti].size());
    for (size_t r = 0; r < per[ti].size(); ++r) {
      const Eff& e = per[ti][r];
      if (e.count < 2) continue;
      const ct_table* t = e.op.t;
      const int vk = t->desc.val_kind;
      const int64_t vb = vk == CT_VAL_U32 ? 4 : 8;
      bool want_flags = false, want_vout = false;
      for (size_t k = e.first, c = 0; c < e.count; ++k) {
        const PlanOp& o = p->ops[k];
        if (o.t != t) continue;
        want_flags = want_flags || o.flags;
        want_vout = want_vout || o.vout;
        ++c;
      }
      Fix& f = fixes[ti][r];
      f.keys = take(e.op.n * 8);
      if (e.op.type == kOpInsert && vk != CT_VAL_NONE) f.vals = take(e.op.n * vb);
      if (want_flags) f.flags = take(e.op.n);
      if (e.op.type == kOpFind && vk != CT_VAL_NONE && want_vout) f.vout = take(e.op.n * vb);
    }
  }
  F.merge_bytes = moff;
  // device layout: steps | entries | copies | merge area (filled in below once counts are known)
  // while only sizing, a placeholder base keeps every merged array non-null, so the steps and
  // their stages (a fix stage needs a status array) are the same as when building
  uint8_t* const b0 = base ? base : reinterpret_cast<uint8_t*>((uintptr_t)kAlign);
  auto dev = [&](int64_t merge_off) -> uint8_t* { return b0 + F.merge_off + merge_off; };

  std::vector<int32_t> level;
  std::vector<GCopy> copy_in;
  // first pass only counts steps and copies so the layout offsets are known; the second fills
  for (int pass = 0; pass < 2; ++pass) {
    F.steps.clear();
    level.clear();
    copy_in.clear();
    copy_out.clear();
    for (size_t ti = 0; ti < per.size(); ++ti) {
      int32_t lev = 0;
      for (size_t r = 0; r < per[ti].size(); ++r) {
        const Eff& e = per[ti][r];
        PlanOp o = e.op;
        ct_table* t = o.t;
        const int vk = t->desc.val_kind;
        const int64_t vb = vk == CT_VAL_U32 ? 4 : 8;
        if (e.count >= 2) {
          const Fix& f = fixes[ti][r];
          uint8_t* mk = dev(f.keys);
          uint8_t* mv = f.vals >= 0 ? dev(f.vals) : nullptr;
          uint8_t* mf = f.flags >= 0 ? dev(f.flags) : nullptr;
          uint8_t* mo = f.vout >= 0 ? dev(f.vout) : nullptr;
          int64_t pos = 0;
          for (size_t k = e.first, c = 0; c < e.count; ++k) {
            const PlanOp& part = p->ops[k];
            if (part.t != t) continue;
            ++c;
            copy_in.push_back(GCopy{part.keys, mk + pos * 8, part.n * 8});
            if (mv) copy_in.push_back(GCopy{part.vals, mv + pos * vb, part.n * vb});
            if (mf && part.flags) copy_out.push_back(GCopy{mf + pos, part.flags, part.n});
            if (mo && part.vout) copy_out.push_back(GCopy{mo + pos * vb, part.vout, part.n * vb});
            pos += part.n;
          }
          o.keys = reinterpret_cast<const uint64_t*>(mk);
          o.vals = mv;
          o.flags = mf;
          o.vout = mo;
        }
        const bool ie = o.type == kOpInsert || o.type == kOpErase;
        const int64_t span = ie ? t->chunk : std::max<int64_t>(o.n, 1);
        for (int64_t c0 = 0; c0 < std::max<int64_t>(o.n, 1); c0 += span) {
          const int64_t q = o.type == kOpClear ? 0 : std::min<int64_t>(span, o.n - c0);
          GStep g{};
          g.v = t->v;
          g.type = o.type;
          g.vk = vk;
          g.q = q;
          g.keys = o.keys ? o.keys + c0 : nullptr;
          g.vals = (o.type == kOpInsert && vk != CT_VAL_NONE)
                       ? static_cast<const uint8_t*>(o.vals) + c0 * vb : nullptr;
          g.vout = (o.type == kOpFind && o.vout) ? static_cast<uint8_t*>(o.vout) + c0 * vb : nullptr;
          g.flags = o.flags ? o.flags + c0 : nullptr;
          g.db = ie ? dedup_slots_for(q) : 0u;
          g.spath = !ie || t->insert_path == CT_INSERT_RESOLVE_FIRST ? 0
                    : t->insert_path == CT_INSERT_SPECULATIVE ? 2 : 1;
          g.gb = group_blocks((q + kSlots - 1) / kSlots, bs);
          g.ntiles = (int32_t)((q + kTile - 1) / kTile);
          F.steps.push_back(g);
          level.push_back(lev++);
        }
      }
    }
    F.copies = copy_in;
    F.copies.insert(F.copies.end(), copy_out.begin(), copy_out.end());
    F.steps_off = 0;
    F.entries_off = align_up((int64_t)(F.steps.size() * sizeof(GStep)));
    // entries: one per (level, stage, step) plus one per copy segment (bounded by a count pass)
    int64_t nent = (int64_t)F.copies.size();
    for (const GStep& g : F.steps)
      for (int stage = 0; stage < gStages; ++stage) nent += stage_blocks(stage, g) ? 1 : 0;
    F.copies_off = F.entries_off + align_up(nent * (int64_t)sizeof(GEntry));
    // launch list for the single-launch form: at most a copy launch on each side of the levels
    int32_t nlev_max = 0;
    for (int32_t l : level) nlev_max = std::max(nlev_max, l + 1);
    const int64_t max_launches = 2 + (int64_t)nlev_max * gStages;
    F.launches_off = F.copies_off + align_up((int64_t)(F.copies.size() * sizeof(GCopy)));
    F.merge_off = F.launches_off + align_up(max_launches * (int64_t)sizeof(GLaunchDev));
    F.total = std::max<int64_t>(kAlign, F.merge_off + F.merge_bytes);
  }
  // Keys per thread of the find / insert / erase stages, per level: a level with much work runs
  // its steps with fewer, longer-running blocks (each block pays its step lookup and partial count
  // once), as long as the level still offers about 2^20 threads; at most 16 keys per thread.
  {
    int32_t nl = 0;
    for (int32_t l : level) nl = std::max(nl, l + 1);
    std::vector<int64_t> keys_at(nl, 0);
    auto probes = [](const GStep& g) {
      return g.type == kOpInsert || g.type == kOpErase || g.type == kOpFind;
    };
    for (size_t i = 0; i < F.steps.size(); ++i)
      if (probes(F.steps[i])) keys_at[level[i]] += F.steps[i].q;
    for (size_t i = 0; i < F.steps.size(); ++i) {
      GStep& g = F.steps[i];
      if (!probes(g)) continue;
      int64_t per = 1;
      while (per < 16 && keys_at[level[i]] >= (per * 2) << 20) per *= 2;
      g.gb = group_blocks((g.q + kSlots * per - 1) / (kSlots * per), bs);
    }
  }
  // launches: copy in, the levels, copy out
  F.entries.clear();
  F.launches.clear();
  auto copy_launch = [&](size_t from, size_t to) {
    if (from == to) return CT_OK;
    int64_t blocks = 0;
    const int64_t off = (int64_t)F.entries.size();
    for (size_t i = from; i < to; ++i) {
      F.entries.push_back(GEntry{(int32_t)blocks, (int32_t)i});
      blocks += copy_blocks(F.copies[i].bytes);
      if (blocks > (int64_t)INT32_MAX / 2) return CT_E_INVALID;
    }
    F.launches.push_back(ct_group::Launch{gCopy, (int32_t)(to - from), (int32_t)blocks, off});
    return CT_OK;
  };
  if (copy_launch(0, copy_in.size()) != CT_OK) return CT_E_INVALID;
  int32_t nlev = 0;
  for (int32_t l : level) nlev = std::max(nlev, l + 1);
  std::vector<std::vector<int32_t>> by_level(nlev);
  for (size_t i = 0; i < F.steps.size(); ++i) by_level[level[i]].push_back((int32_t)i);
  for (int32_t l = 0; l < nlev; ++l) {
    for (int stage = 0; stage < gStages; ++stage) {
      int64_t blocks = 0;
      const int64_t off = (int64_t)F.entries.size();
      for (int32_t i : by_level[l]) {
        const int b = stage_blocks(stage, F.steps[i]);
        if (!b) continue;
        F.entries.push_back(GEntry{(int32_t)blocks, i});
        blocks += b;
        if (blocks > (int64_t)INT32_MAX / 2) return CT_E_INVALID;
      }
      const int64_t n = (int64_t)F.entries.size() - off;
      if (n) F.launches.push_back(ct_group::Launch{stage, (int32_t)n, (int32_t)blocks, off});
    }
  }
  if (copy_launch(copy_in.size(), F.copies.size()) != CT_OK) return CT_E_INVALID;
  return CT_OK;
}

// One launch of a grouped find / insert / erase stage with BS threads per block.
template <int BS>
void probe_stage(int32_t stage, hipStream_t s, const ct_group::Launch& L, const GStep* st,
                 const GEntry* e) {
  if (stage == gFind) k_g_find<BS><<<L.blocks, BS, 0, s>>>(st, e, L.n);
  else if (stage == gInsert) k_g_insert<BS><<<L.blocks, BS, 0, s>>>(st, e, L.n);
  else k_g_erase<BS><<<L.blocks, BS, 0, s>>>(st, e, L.n);
}

}  // namespace

extern "C" {

ct_status ct_plan_group_bytes(ct_plan* p, int32_t options, int64_t* bytes) {
  if (!p || !bytes || !group_options_valid(options)) return CT_E_INVALID;
  GroupForm F;
  ct_status r = group_build(p, options, nullptr, F);
  if (r != CT_OK) return r;
  *bytes = F.total;
  return CT_OK;
}

ct_status ct_plan_group(ct_plan* p, int32_t options, void* d_buf, int64_t bytes) {
  if (!p || !d_buf || reinterpret_cast<uintptr_t>(d_buf) % kAlign) return CT_E_INVALID;
  if (!group_options_valid(options)) return CT_E_INVALID;
  uint8_t* base = static_cast<uint8_t*>(d_buf);
  GroupForm F;
  ct_status r = group_build(p, options, base, F);
  if (r != CT_OK) return r;
  if (bytes < F.total) return CT_E_INVALID;
  if (!F.steps.empty() && hipMemcpy(base + F.steps_off, F.steps.data(), F.steps.size() * sizeof(GStep),
                                    hipMemcpyHostToDevice) != hipSuccess)
    return CT_E_HIP;
  if (!F.entries.empty() && hipMemcpy(base + F.entries_off, F.entries.data(),
                                      F.entries.size() * sizeof(GEntry), hipMemcpyHostToDevice) != hipSuccess)
    return CT_E_HIP;
  if (!F.copies.empty() && hipMemcpy(base + F.copies_off, F.copies.data(),
                                     F.copies.size() * sizeof(GCopy), hipMemcpyHostToDevice) != hipSuccess)
    return CT_E_HIP;
  std::vector<GLaunchDev> ld;
  int32_t widest = 1;
  for (const ct_group::Launch& L : F.launches) {
    ld.push_back(GLaunchDev{L.stage, L.n, L.blocks, 0, L.entry_off});
    widest = std::max(widest, L.blocks);
  }
  if (!ld.empty() && hipMemcpy(base + F.launches_off, ld.data(), ld.size() * sizeof(GLaunchDev),
                               hipMemcpyHostToDevice) != hipSuccess)
    return CT_E_HIP;
  p->glaunch_dev = base + F.launches_off;
  p->gwidest = widest;
  p->glaunch = std::move(F.launches);
  p->gsteps = base + F.steps_off;
  p->gentries = base + F.entries_off;
  p->gcopies = base + F.copies_off;
  p->grouped_ops = p->ops.size();
  p->gblock = group_block_size(options);
  return CT_OK;
}

ct_status ct_plan_launch_grouped(ct_plan* p, void* stream) {
  if (!p || p->grouped_ops != p->ops.size()) return CT_E_INVALID;
  hipStream_t s = S(stream);
  const GStep* st = static_cast<const GStep*>(p->gsteps);
  const GEntry* en = static_cast<const GEntry*>(p->gentries);
  for (ct_table* t : p->tables) fresh_counts(t, s);
  for (const ct_group::Launch& L : p->glaunch) {
    const GEntry* e = en + L.entry_off;
    switch (L.stage) {
      case gReset: k_g_reset<<<L.blocks, kBlock, 0, s>>>(st, e, L.n); break;
      case gPro: k_g_prologue<<<L.blocks, kBlock, 0, s>>>(st, e, L.n); break;
      case gDedup: k_g_dedup<<<L.blocks, kBlock, 0, s>>>(st, e, L.n); break;
      case gFind:
      case gInsert:
      case gErase:
        if (p->gblock == 128) probe_stage<128>(L.stage, s, L, st, e);
        else if (p->gblock == 512) probe_stage<512>(L.stage, s, L, st, e);
        else if (p->gblock == 1024) probe_stage<1024>(L.stage, s, L, st, e);
        else probe_stage<kBlock>(L.stage, s, L, st, e);
        break;
      case gApply: k_g_apply<<<L.blocks, 1024, 0, s>>>(st, e, L.n); break;
      case gCount: k_g_tile_count<<<L.blocks, kBlock, 0, s>>>(st, e, L.n); break;
      case gScan: k_g_tile_scan<<<L.blocks, 1024, 0, s>>>(st, e, L.n); break;
      case gFinal: k_g_final<<<L.blocks, kBlock, 0, s>>>(st, e, L.n); break;
      case gFix: k_g_fix<<<L.blocks, kBlock, 0, s>>>(st, e, L.n); break;
      case gSClear: k_g_sclear<<<L.blocks, kBlock, 0, s>>>(st, e, L.n); break;
      case gSBuild: k_g_sbuild<<<L.blocks, kBlock, 0, s>>>(st, e, L.n); break;
      case gSProbe: k_g_sfix<false><<<L.blocks, kBlock, 0, s>>>(st, e, L.n); break;
      case gSSwap: k_g_sfix<true><<<L.blocks, kBlock, 0, s>>>(st, e, L.n); break;
      case gCopy:
        k_g_copy<<<L.blocks, kBlock, 0, s>>>(static_cast<const GCopy*>(p->gcopies), e, L.n);
        break;
      default: return CT_E_INVALID;
    }
    if (launched() != CT_OK) {
      for (ct_table* t : p->tables) t->counts_stale = true;
      return CT_E_HIP;
    }
  }
  return CT_OK;
}

ct_status ct_plan_launch_single(ct_plan* p, int32_t max_blocks, void* stream) {
  if (!p || p->grouped_ops != p->ops.size() || p->gblock != kBlock || max_blocks < 0)
    return CT_E_INVALID;
  if (p->glaunch.empty()) return CT_OK;
  int dev = 0, coop = 0, ncu = 0, per_cu = 0;
  hipStream_t s = S(stream);
  if (s) {
    if (hipStreamGetDevice(s, &dev) != hipSuccess) return CT_E_HIP;
  } else if (hipGetDevice(&dev) != hipSuccess) {
    return CT_E_HIP;
  }
  if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess ||
      hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_g_persistent, kBlock, 0) != hipSuccess)
    return CT_E_HIP;
  if (!coop || per_cu < 1 || ncu < 1) return CT_E_HIP;
  // every workgroup must be resident at once: at most what the device holds, and no more than
  // the widest stage can use
  int64_t grid = std::min<int64_t>((int64_t)per_cu * ncu, p->gwidest);
  if (max_blocks > 0) grid = std::min<int64_t>(grid, max_blocks);
  grid = std::max<int64_t>(grid, 1);
  const GLaunchDev* ls = static_cast<const GLaunchDev*>(p->glaunch_dev);
  int32_t nl = (int32_t)p->glaunch.size();
  const GStep* st = static_cast<const GStep*>(p->gsteps);
  const GEntry* en = static_cast<const GEntry*>(p->gentries);
  const GCopy* cp = static_cast<const GCopy*>(p->gcopies);
  for (ct_table* t : p->tables) fresh_counts(t, s);
  void* args[] = {&ls, &nl, &st, &en, &cp};
  if (hipLaunchCooperativeKernel(reinterpret_cast<const void*>(k_g_persistent), dim3((unsigned)grid),
                                 dim3(kBlock), args, 0, s) != hipSuccess) {
    (void)hipGetLastError();  // a refused launch must not fail the caller's next call
    return CT_E_HIP;
  }
  return CT_OK;
}

ct_status ct_plan_group_info(ct_plan* p, int64_t* nlaunches, int64_t* nsteps) {
  if (!p || p->grouped_ops != p->ops.size()) return CT_E_INVALID;
  if (nlaunches) *nlaunches = (int64_t)p->glaunch.size();
  if (nsteps) {
    int64_t m = 0;
    for (const ct_group::Launch& L : p->glaunch)
      if (L.stage == gReset || L.stage == gPro || L.stage == gFind) m += L.n;
    *nsteps = m;
  }
  return CT_OK;
}

ct_status ct_plan_create(ct_plan** out) {
  if (!out) return CT_E_INVALID;
  ct_plan* p = new (std::nothrow) ct_plan;
  if (!p) return CT_E_NOMEM;
  *out = p;
  return CT_OK;
}

ct_status ct_plan_destroy(ct_plan* p) {
  if (!p) return CT_E_INVALID;
  for (hipStream_t s : p->side) (void)hipStreamDestroy(s);
  for (hipEvent_t e : p->ev) (void)hipEventDestroy(e);
  delete p;
  return CT_OK;
}

ct_status ct_plan_add(ct_plan* p, ct_table* t, int32_t op, const uint64_t* keys, const void* vals,
                      void* vals_out, uint8_t* flags_out, int64_t n) {
  if (!p || !t || n < 0) return CT_E_INVALID;
  if (op < kOpClear || op > kOpErase) return CT_E_INVALID;
  const int vk = t->desc.val_kind;
  if (op != kOpClear && n > 0 && !keys) return CT_E_INVALID;
  if (op == kOpInsert && vk != CT_VAL_NONE && n > 0 && !vals) return CT_E_INVALID;
  if (op == kOpFind && vk == CT_VAL_NONE && vals_out) return CT_E_INVALID;
  if (op != kOpClear && n == 0) return CT_OK;
  p->ops.push_back(PlanOp{t, op, keys, vals, vals_out, flags_out, op == kOpClear ? 0 : n});
  if (std::find(p->tables.begin(), p->tables.end(), t) == p->tables.end()) p->tables.push_back(t);
  // the plan may run any number of times later: the host no longer bounds this table's size
  t->size_ub = (uint64_t)t->desc.capacity;
  return CT_OK;
}

ct_status ct_plan_info(ct_plan* p, int64_t* nops, int64_t* ntables) {
  if (!p) return CT_E_INVALID;
  if (nops) *nops = (int64_t)p->ops.size();
  if (ntables) *ntables = (int64_t)p->tables.size();
  return CT_OK;
}

ct_status ct_plan_launch(ct_plan* p, int32_t lanes, void* stream) {
  if (!p || lanes < 1 || lanes > 8) return CT_E_INVALID;
  ct_status r = plan_streams(p, lanes);
  if (r != CT_OK) return r;
  hipStream_t s = S(stream);
  if (hipEventRecord(p->ev[0], s) != hipSuccess) return CT_E_HIP;
  for (int32_t i = 0; i < lanes; ++i)
    if (hipStreamWaitEvent(p->side[i], p->ev[0], 0) != hipSuccess) return CT_E_HIP;
  for (const PlanOp& o : p->ops) {
    const size_t ti = (size_t)(std::find(p->tables.begin(), p->tables.end(), o.t) - p->tables.begin());
    r = run_op(o, p->side[ti % (size_t)lanes]);
    if (r != CT_OK) return r;
  }
  for (int32_t i = 0; i < lanes; ++i) {
    if (hipEventRecord(p->ev[1 + i], p->side[i]) != hipSuccess) return CT_E_HIP;
    if (hipStreamWaitEvent(s, p->ev[1 + i], 0) != hipSuccess) return CT_E_HIP;
  }
  return CT_OK;
}

ct_status ct_plan_capture(ct_plan* p, int32_t lanes, void* stream, void** graph_exec) {
  if (!p || !graph_exec || !stream || lanes < 1 || lanes > 8) return CT_E_INVALID;
  ct_status r = plan_streams(p, lanes);
  if (r != CT_OK) return r;
  hipStream_t s = S(stream);
  if (hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal) != hipSuccess) return CT_E_HIP;
  r = ct_plan_launch(p, lanes, stream);
  hipGraph_t g = nullptr;
  const hipError_t e = hipStreamEndCapture(s, &g);
  if (r != CT_OK || e != hipSuccess) {
    if (g) (void)hipGraphDestroy(g);
    return r != CT_OK ? r : CT_E_HIP;
  }
  hipGraphExec_t x = nullptr;
  const hipError_t ie = hipGraphInstantiate(&x, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (ie != hipSuccess) return CT_E_HIP;
  *graph_exec = x;
  return CT_OK;
}

ct_status ct_plan_capture_grouped(ct_plan* p, void* stream, void** graph_exec) {
  if (!p || !graph_exec || !stream || p->grouped_ops != p->ops.size()) return CT_E_INVALID;
  hipStream_t s = S(stream);
  if (hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal) != hipSuccess) return CT_E_HIP;
  ct_status r = ct_plan_launch_grouped(p, stream);
  hipGraph_t g = nullptr;
  const hipError_t e = hipStreamEndCapture(s, &g);
  if (r != CT_OK || e != hipSuccess) {
    if (g) (void)hipGraphDestroy(g);
    return r != CT_OK ? r : CT_E_HIP;
  }
  hipGraphExec_t x = nullptr;
  const hipError_t ie = hipGraphInstantiate(&x, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (ie != hipSuccess) return CT_E_HIP;
  *graph_exec = x;
  return CT_OK;
}

ct_status ct_graph_launch(void* graph_exec, void* stream) {
  if (!graph_exec) return CT_E_INVALID;
  return hipGraphLaunch(static_cast<hipGraphExec_t>(graph_exec), S(stream)) == hipSuccess ? CT_OK : CT_E_HIP;
}

ct_status ct_graph_destroy(void* graph_exec) {
  if (!graph_exec) return CT_E_INVALID;
  return hipGraphExecDestroy(static_cast<hipGraphExec_t>(graph_exec)) == hipSuccess ? CT_OK : CT_E_HIP;
}

}  // extern "C"

// ---------------------------------------------------------------------------------------------
// Allocation-free insert: the per-chunk scratch lives in a static device array, not in the
// table's buffer.  One array per GPU (each device holds its own copy), shared by every call on
// that GPU: calls that overlap on one GPU race on it.  Every kernel that needs part of it cleared
// clears it itself at the start of each chunk (the prologue kernels), so a call never depends on
// what the previous call left there.
// ---------------------------------------------------------------------------------------------
namespace {

constexpr int64_t kStaticChunk = 1 << 15;  // elements per chunk: below the binned-dedup size

struct StaticScratch {
  int64_t dd, dmark, dup, flag, ref, tsum, bcnt, total;
};

constexpr StaticScratch static_scratch_layout() {
  StaticScratch L{};
  int64_t off = 0;
  L.dd = off;
  off += 2 * kStaticChunk * 8;
  L.dmark = off;
  off += kStaticChunk;
  L.dup = off;
  off += kStaticChunk * 4;
  L.flag = off;
  off += kStaticChunk;
  L.ref = off;
  off += kStaticChunk * 8;
  L.tsum = off;
  off += 256;  // kStaticChunk / kTile tile sums, 4 bytes each
  L.bcnt = off;
  off += (int64_t)kMaxGroupBlocks * 8;
  L.total = off;
  return L;
}

constexpr StaticScratch kStaticLayout = static_scratch_layout();
static_assert(kStaticChunk / kTile * 4 <= 256, "tile sums fit their region");
static_assert(kStaticLayout.dd % 256 == 0 && kStaticLayout.dmark % 256 == 0 &&
                  kStaticLayout.dup % 256 == 0 && kStaticLayout.flag % 256 == 0 &&
                  kStaticLayout.ref % 256 == 0 && kStaticLayout.tsum % 256 == 0 &&
                  kStaticLayout.bcnt % 256 == 0,
              "every region starts on a 256-byte boundary");

}  // namespace

static __device__ __align__(256) uint8_t scratch[kStaticLayout.total];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
uint8_t* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the device that runs `s`, looked up once per device with that
// device current.  The array's name is a host-side stand-in and never reaches a kernel.
ct_status scratch_for_stream(hipStream_t s, uint8_t** out) {
  int dev = -1;
  if (s) {
    if (hipStreamGetDevice(s, &dev) != hipSuccess) return CT_E_HIP;
  } else if (hipGetDevice(&dev) != hipSuccess) {
    return CT_E_HIP;
  }
  if (dev < 0 || dev >= kMaxDevices) return CT_E_INVALID;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    int prev = -1;
    if (hipGetDevice(&prev) != hipSuccess) return CT_E_HIP;
    if (prev != dev && hipSetDevice(dev) != hipSuccess) return CT_E_HIP;
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (prev != dev) (void)hipSetDevice(prev);
    if (e != hipSuccess || !p) return CT_E_HIP;
    g_scratch_ptr[dev] = static_cast<uint8_t*>(p);
  }
  *out = g_scratch_ptr[dev];
  return CT_OK;
}

}  // namespace

extern "C" {

ct_status ct_insert_batch_noalloc(ct_table* t, const uint64_t* keys, const void* vals, int64_t n,
                                  uint8_t* status, void* stream) {
  ct_status r = check_batch(t, keys, n);
  if (r != CT_OK) return r;
  const int vk = t->desc.val_kind;
  if (vk != CT_VAL_NONE && !vals) return CT_E_INVALID;
  if (n == 0) return CT_OK;
  hipStream_t s = S(stream);
  uint8_t* base = nullptr;
  r = scratch_for_stream(s, &base);
  if (r != CT_OK) return r;
  TableView w = t->v;  // the table's slots and header, the static array's scratch
  w.dd = reinterpret_cast<uint64_t*>(base + kStaticLayout.dd);
  w.dmark = base + kStaticLayout.dmark;
  w.dup = reinterpret_cast<uint32_t*>(base + kStaticLayout.dup);
  w.flag = base + kStaticLayout.flag;
  w.ref = reinterpret_cast<uint64_t*>(base + kStaticLayout.ref);
  w.tsum = reinterpret_cast<uint32_t*>(base + kStaticLayout.tsum);
  w.bcnt = reinterpret_cast<int64_t*>(base + kStaticLayout.bcnt);
  w.r1k = nullptr;  // chunks below the binned size resolve repeats through dd
  w.r1i = nullptr;
  w.r2k = nullptr;
  w.r2i = nullptr;
  w.bcur = nullptr;
  w.dfirst = nullptr;
  const int64_t chunk = std::min<int64_t>(t->chunk, kStaticChunk);
  return insert_any(t, BatchScratch{w, chunk, false}, keys, vals, n, status, s);
}

}  // extern "C"
