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

constexpr uint32_t kBitsMatch = 0xFFu;      // bits of probe_round's answer: slots holding the key
constexpr int kEmptyShift = 8;              //   slots holding kEmpty
constexpr int kTombShift = 16;              //   slots holding kTomb (FREE rounds only)

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

// NJ bucket reads of this lane's group: items j * 8 + g for j < NJ (items past the last re-read it).
template <bool FREE, bool VAL, int NJ>
__device__ __forceinline__ uint32_t probe_lines(const Bucket* bk, WaveLds* w, uint32_t n, uint32_t g,
                                                int sub) {
  u64x2 sl[NJ];
  const char* base = reinterpret_cast<const char*>(bk) + sub * (int)sizeof(Slot);
  uint32_t r[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    r[j] = NJ == 8 ? (uint32_t)j * 8u + g : min((uint32_t)j * 8u + g, n - 1u);
    sl[j] = *reinterpret_cast<const u64x2*>(base + w->off[r[j]]);
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

// One round: every lane with `look` set has its bucket `b` compared with `key`.  Returns the slot
// bits (kBitsMatch, kEmptyShift, kTombShift) of its bucket, and with VAL the matching slot's value
// in *val.  Called by all 64 lanes of the wave together; `mask` is the ballot of `look`, not zero.
template <bool FREE, bool VAL>
__device__ __forceinline__ uint32_t probe_round(const TableView& t, WaveLds* w, uint64_t mask, bool look,
                                                uint64_t key, uint32_t b, uint64_t* val) {
  const int lane = wave_lane();
  const int sub = lane & 7;
  const uint32_t g = (uint32_t)lane >> 3;
  const uint32_t n = (uint32_t)__builtin_popcountll(mask);
  // more than half the lanes look: item = lane, in an order that leaves each answer on its owner
  // after the transpose; otherwise the looking lanes are packed
  const bool packed = n <= 32;
  const uint32_t rank = packed ? __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                           __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0))
                               : (uint32_t)sub * 8u + g;
  __builtin_amdgcn_wave_barrier();  // the items of the round before have been read
  if (look || !packed) {
    w->off[rank] = (uint64_t)b * sizeof(Bucket);
    w->key[rank] = key;
  }
  __builtin_amdgcn_wave_barrier();
  uint32_t x;
  if (n > 32) x = probe_lines<FREE, VAL, 8>(t.bk, w, n, g, sub);
  else if (n > 16) x = probe_lines<FREE, VAL, 4>(t.bk, w, n, g, sub);
  else if (n > 8) x = probe_lines<FREE, VAL, 2>(t.bk, w, n, g, sub);
  else x = probe_lines<FREE, VAL, 1>(t.bk, w, n, g, sub);
  __builtin_amdgcn_wave_barrier();
  x = transpose8(x, sub);             // lane (g, s) now answers item s * 8 + g
  if (packed) x = (uint32_t)__shfl((int)x, (int)(((rank & 7u) << 3) | (rank >> 3)), 64);
  if (VAL) *val = w->val[rank];
  return x;
}

// Bucket after b on a key's probe path.  Both terms are below 2^31.
__device__ __forceinline__ uint32_t next_bucket32(const TableView& t, uint32_t b, uint32_t step) {
  const uint32_t nb = (uint32_t)t.nb;
  const uint32_t nx = b + step;
  return nx >= nb ? nx - nb : nx;
}

}  // namespace ct
