// ct_probe.h -- the wave-cooperative probe round of the batch kernels (gfx950, wave64).
//
// Every lane owns one key and the bucket it reads next.  A round reads the bucket of every lane
// that is still looking, eight lanes to a bucket (lane v & 7 reads slot v & 7: one 16-byte load per
// lane, one 128-byte line per group), and hands each owner the comparisons of its eight slots.
//
// What bounds it.  At the large table (1.34 GB, load 0.8) a lookup reads 1.3 lines at random; the
// chip serves about 38 G such lines/s from HBM, so a lookup may cost a SIMD only some 60 cycles
// per key before instructions, not memory, set the pace.  Hence:
//   * owners hand (key, bucket offset) to the reading group through two 8-byte LDS words instead
//     of four cross-lane moves per key;
//   * after the first round the lanes still looking (about a third, then a tenth) are packed, so a
//     round issues ceil(lanes / 8) loads and compares instead of eight;
//   * the comparisons of a round are collected as bits per lane and turned into bits per owner by
//     three lane exchanges (an 8 x 8 bit transpose), not by a ballot and shifts per key.
#pragma once

#include "ct_device.h"

namespace ct {

struct WaveLds {
  uint64_t off[64];  // byte offset of the bucket and key of the lanes that look
  uint64_t key[64];
  uint64_t val[64];  // value beside the matching key, per item
};

typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));

constexpr uint32_t kBitsMatch = 0xFFu;      // bits of an answer: slots holding the key
constexpr int kEmptyShift = 8;              //   slots holding kEmpty
constexpr int kTombShift = kEmptyShift + 8; //   slots holding kTomb (FREE rounds only)

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}

// Every byte of x is a row of an 8 x 8 bit matrix over the 8 lanes of a group: bit j of lane s
// becomes bit s of lane j.  Each step swaps the off-diagonal blocks of one size with the lane
// 1, 2 or 4 away.
__device__ __forceinline__ uint32_t transpose8(uint32_t x, int sub) {
  auto step = [&](uint32_t other, uint32_t low, int k) {
    const bool hi = (sub & k) != 0;
    const uint32_t keep = hi ? ~low : low;
    const uint32_t moved = __builtin_amdgcn_alignbit(other, other, hi ? (uint32_t)k : 32u - (uint32_t)k);
    return (x & keep) | (moved & ~keep);
  };
  x = step(dpp<0xB1>(x), 0x55555555u, 1);               // quad_perm [1,0,3,2]
  x = step(dpp<0x4E>(x), 0x33333333u, 2);               // quad_perm [2,3,0,1]
  x = step(dpp<0x1B>(dpp<0x141>(x)), 0x0F0F0F0Fu, 4);   // row_half_mirror, then quad_perm [3,2,1,0]
  return x;
}

// NJ bucket reads of this lane's group: items j * 8 + g for j < NJ (CLAMP: of n; past the last, it is
// read again).
template <bool FREE, bool VAL, int NJ, bool CLAMP>
__device__ __forceinline__ uint32_t probe_lines(const Bucket* bk, WaveLds* w, uint32_t n, uint32_t g,
                                                int sub) {
  u64x2 sl[NJ];  // .y is loaded only with VAL
  const char* base = reinterpret_cast<const char*>(bk) + sub * (int)sizeof(Slot);
  uint32_t r[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    r[j] = CLAMP ? min((uint32_t)j * 8u + g, n - 1u) : (uint32_t)j * 8u + g;
    if (VAL) sl[j] = *reinterpret_cast<const u64x2*>(base + w->off[r[j]]);
    else sl[j].x = *reinterpret_cast<const uint64_t*>(base + w->off[r[j]]);
  }
  // the keys are read back here rather than held across the loads: sixteen registers fewer
  asm volatile("" ::: "memory");
  uint32_t x = 0;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const bool hit = sl[j].x == w->key[r[j]];
    if (VAL) {
      if (hit) w->val[j * 8 + g] = sl[j].y;
    }
    x |= hit ? 1u << j : 0u;
    x |= sl[j].x == kEmpty ? 1u << (kEmptyShift + j) : 0u;
    if (FREE) x |= sl[j].x == kTomb ? 1u << (kTombShift + j) : 0u;
  }
  return x;
}

// Bucket after b on a key's probe path.  Both terms are below 2^31.
__device__ __forceinline__ uint32_t next_bucket32(const TableView& t, uint32_t b, uint32_t step) {
  const uint32_t nb = (uint32_t)t.nb;
  const uint32_t nx = b + step;
  return nx >= nb ? nx - nb : nx;
}

// One round of the lanes with `look` set.  Called by all 64 lanes of the wave together; `mask` is the
// ballot of `look`, not zero.  Each looking lane gets the answers of `steps` buckets of its path, from
// `b` on; answer(s) are the slot bits (kBitsMatch, kEmptyShift, kTombShift) of the s-th.
//
// AHEAD (batches too small to fill the chip, which wait for memory one bucket after another): when
// half the lanes or fewer look, the round's 64 bucket reads go to the next 2, 4 or 8 buckets of
// each.  Otherwise a lane reads one bucket and the looking lanes are packed, so that no line is
// read in vain.
template <bool FREE, bool VAL, bool AHEAD>
struct ProbeRound {
  WaveLds* w;
  uint32_t x, rank, shift;  // packed answers, this lane's rank, log2 of steps
  bool packed;

  __device__ __forceinline__ ProbeRound(const TableView& t, WaveLds* lds, uint64_t mask, bool look,
                                        uint64_t key, uint32_t b, uint32_t step)
      : w(lds), shift(0) {
    const int lane = wave_lane();
    const int sub = lane & 7;
    const uint32_t g = (uint32_t)lane >> 3;
    const uint32_t n = (uint32_t)__builtin_popcountll(mask);
    // more than half the lanes look: item = lane, in an order that leaves each answer on its owner
    // after the transpose
    packed = n <= 32;
    rank = packed ? __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                              __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0))
                  : (uint32_t)sub * 8u + g;
    if (AHEAD) shift = n > 32 ? 0u : n > 16 ? 1u : n > 8 ? 2u : 3u;
    __builtin_amdgcn_wave_barrier();  // the items of the round before have been read
    if (look || !packed) {
      uint32_t nx = b;
      for (uint32_t s = 0; s < (1u << shift); ++s) {
        const uint32_t at = (rank << shift) + s;
        w->off[at] = (uint64_t)nx * sizeof(Bucket);
        w->key[at] = key;
        if (AHEAD) nx = next_bucket32(t, nx, step);
      }
    }
    __builtin_amdgcn_wave_barrier();
    const uint32_t items = packed ? n << shift : 64u;
    if (AHEAD) x = items > 32 ? probe_lines<FREE, VAL, 8, true>(t.bk, w, items, g, sub)
                                         : probe_lines<FREE, VAL, 4, true>(t.bk, w, items, g, sub);
    else if (n > 32) x = probe_lines<FREE, VAL, 8, false>(t.bk, w, n, g, sub);
    else if (n > 16) x = probe_lines<FREE, VAL, 4, true>(t.bk, w, n, g, sub);
    else if (n > 8) x = probe_lines<FREE, VAL, 2, true>(t.bk, w, n, g, sub);
    else x = probe_lines<FREE, VAL, 1, true>(t.bk, w, n, g, sub);
    __builtin_amdgcn_wave_barrier();
    x = transpose8(x, sub);  // lane (g, s) now answers item s * 8 + g
  }

  __device__ __forceinline__ uint32_t steps() const { return 1u << shift; }

  // All 64 lanes call it together.
  __device__ __forceinline__ uint32_t answer(uint32_t s, uint64_t* val) const {
    const uint32_t at = (rank << shift) + s;
    if (VAL) *val = w->val[at & 63u];
    if (!packed) return x;
    return (uint32_t)__shfl((int)x, (int)(((at & 7u) << 3) | ((at >> 3) & 7u)), 64);
  }
};

// The WaveLds of this thread's wave in a block of BS threads (one array per kernel).
template <int BS>
__device__ __forceinline__ WaveLds* wave_lds() {
  __shared__ WaveLds w[BS / 64];
  return &w[threadIdx.x >> 6];
}

// Where a wave's keys are, or where they go.  Every lane with `look` set walks its key's probe path
// to the key, or to the first bucket that holds an empty slot; with CLAIM an absent key then takes
// the first free slot on the path (one CAS per lane, all lanes of the wave at once).
//
// Inside a bucket the order of the free slots is fixed per key: tombstones first (an empty slot
// keeps the bucket open for lookups), and from a slot that depends on the key, so that keys of one
// bucket that claim at the same time mostly ask for different slots.  With the lowest slot first,
// 2^14 keys filling 2^14 buckets lost every third claim and retried one key at a time.
//
// A claim that loses to another key goes on to the next slot that the probe saw free in that bucket,
// without reading it again, and past the last of them to the next bucket.  Slots only change from
// free to a key while a kernel inserts, and all copies of a key ask for free slots in the same
// order: a slot that one copy found taken before its claim is a slot that a copy with an older
// view asks for and loses.  So a copy either claims, sees the key, or loses its CAS to the key, and
// a key is stored once.  Every bucket is asked at most once per slot, so each lane ends.
// (Probing the bucket again after each lost claim: 2^16 keys into an empty map of 2^17 took 23 us.)
//
// The test hook (`inject`, 0 = off) makes keys chosen by their hash lose their claim of one slot per
// bucket, the first in their order (their compare-and-swap expects the other kind of free slot there),
// and ask for it again once the bucket's other free slots are gone.  Key and slot alone decide, not
// what a copy saw, so all copies still ask in the same order.  The slot, or kSlots for none:
__device__ __forceinline__ uint32_t injected_loss(uint64_t key, uint32_t inject, uint32_t first) {
  return inject && (uint32_t)(dedup_mix(key) >> 32) % inject == 0 ? first : (uint32_t)kSlots;
}

constexpr uint32_t kFreeSlot = 0x101u;  // slot 0 of a bucket's free slots: bits 0-7 empty, 8-15 tombstones

struct Place {
  bool found;      // the key is there (with CLAIM: or another copy of it got the slot)
  bool had_empty;  // its bucket holds an empty slot
  uint64_t pos;    // slot of the key or of the claim; kNoPos: none (!found)
  uint64_t val;    // value beside the key found (VAL)
};

template <bool CLAIM, bool VAL, bool AHEAD>
__device__ __forceinline__ Place place_keys(const TableView& t, WaveLds* w, bool look, uint64_t key,
                                            bool claim, uint32_t inject, bool home_full = false) {
  Place r = {false, false, kNoPos, 0};
  const Seq q = probe_seq(t, key);
  const uint32_t step = (uint32_t)q.step;
  uint32_t b = (uint32_t)q.home, left = (uint32_t)t.nb;
  uint32_t fb = kNone, fleft = 0;           // first bucket with a free slot on the path
  uint32_t fs = 0;                          // its free slots: bits 0-7 empty, 8-15 tombstones
  if (home_full) {  // known: begin at the second bucket of the path
    b = next_bucket32(t, b, step);
    look = look && --left != 0;
  }
  for (uint64_t mask = __ballot(look); mask; mask = __ballot(look)) {
    const ProbeRound<CLAIM, VAL, AHEAD> round(t, w, mask, look, key, b, step);
    bool claiming = false;
    bool here = look;       // still on the buckets of this round
    const uint32_t steps = AHEAD ? round.steps() : 1u;
    for (uint32_t s = 0; s < steps; ++s) {
      uint64_t val = 0;
      const uint32_t x = round.answer(s, &val);
      if (!here) continue;
      if (x & kBitsMatch) {
        r.found = true;
        r.had_empty = ((x >> kEmptyShift) & 0xFFu) != 0;
        r.pos = (uint64_t)b * kSlots + (uint64_t)__builtin_ctz(x & kBitsMatch);
        if (VAL) r.val = val;
        look = here = false;
        continue;
      }
      const uint32_t e = (x >> kEmptyShift) & 0xFFu;
      if constexpr (CLAIM) {
        const uint32_t fr = (x >> kEmptyShift) & 0xFFFFu;
        if (fb == kNone && fr) {
          fb = b;
          fleft = left;
          fs = fr;
        }
      }
      if (!e && --left != 0) {
        b = next_bucket32(t, b, step);
        continue;
      }
      look = here = false;
      claiming = CLAIM && claim && fb != kNone;
    }
    if constexpr (CLAIM) {
      const uint32_t rot = (step >> 1) & 7u;
      uint32_t lose = injected_loss(key, inject, rot);
      uint32_t late = 0;  // the slot of an injected loss, asked for again at the end
      while (claiming) {
        const uint32_t f = fs >> 8 ? fs >> 8 : fs;
        const uint32_t c = ((uint32_t)__builtin_ctz((f * 0x101u) >> rot) + rot) & 7u;
        uint64_t expected = (fs >> 8 != 0) != (c == lose) ? kTomb : kEmpty;
        if (cas64(&t.bk[fb].s[c].key, expected, key)) {
          r.pos = (uint64_t)fb * kSlots + c;
          claiming = false;
        } else if (expected == key) {
          r.found = true;
          claiming = false;
        } else {  // taken by another key
          if (c == lose) {
            late = fs & kFreeSlot << c;
            lose = kSlots;
          }
          fs &= ~(kFreeSlot << c);
          if (!fs) {
            fs = late;
            late = 0;
          }
          if (!fs) {  // the bucket is full now
            claiming = false;
            b = next_bucket32(t, fb, step);
            left = fleft - 1;
            fb = kNone;
            look = left != 0;
          }
        }
      }
    }
  }
  return r;
}

}  // namespace ct
