// Rank order of (score, index) pairs as integers, and a bitonic sort over the
// 32 lanes of each wavefront half.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"

namespace pisa {

// Rank order (key desc, pack asc) as one ascending 64-bit integer: the high
// word maps the float key to an unsigned value that decreases as the key
// grows (total order, -inf last), the low word is the non-negative pack.
__device__ __forceinline__ uint32_t desc_bits(float key) {
  const uint32_t u = __float_as_uint(key + 0.0f);  // -0 ranks as +0
  const uint32_t m = static_cast<uint32_t>(static_cast<int32_t>(u) >> 31);
  return u ^ (~m & 0x7FFFFFFFu);
}
__device__ __forceinline__ float desc_bits_inv(uint32_t d) {
  const uint32_t m = static_cast<uint32_t>(static_cast<int32_t>(d) >> 31);
  return __uint_as_float(d ^ (~m & 0x7FFFFFFFu));
}

// The order word of a candidate: forced ones before every score, whatever the
// scores are (+inf and NaN among them), empty slots last.
__device__ __forceinline__ uint32_t rank_word(bool valid, bool forced, float score) {
  return !valid ? 0xFFFFFFFFu : (forced ? 0u : max(desc_bits(score), 1u));
}

// Does (word a, index ia) rank before (word b, index ib)?  On desc_bits words
// this is a total order, NaN included: of n candidates with distinct indices
// exactly k have fewer than k others before them.  Comparing the floats
// themselves, every NaN would rank first, and a list that counts on at most K
// survivors would be overrun.
__device__ __forceinline__ bool word_before(uint32_t a, int ia, uint32_t b, int ib) {
  return a < b || (a == b && ia < ib);
}

// The lanes of a wavefront whose entry e (= lane & 31 for the 32-lane
// sorts) keeps the smaller of itself and its partner in the bitonic step
// (K2, J), as a lane mask known at compile time.
template <int K2, int J>
constexpr uint64_t sort32_want_small() {
  uint64_t m = 0;
  for (int l = 0; l < 64; ++l) {
    const int e = l & 31;
    if (((e & K2) == 0) == ((e & J) == 0)) m |= uint64_t(1) << l;
  }
  return m;
}

// One compare-exchange stage of the bitonic network, without branches: the
// lane keeps the smaller of (itself, partner) where the stage wants the
// smaller, else the larger.  hl = lane & 31 (the stage's direction comes
// from a constant lane mask).
template <int K2, int J>
__device__ __forceinline__ void sort32_step(uint32_t& hi, uint32_t& lo, int hl) {
  (void)hl;
  const uint32_t ohi = static_cast<uint32_t>(xor32_i<J>(static_cast<int>(hi)));
  const uint32_t olo = static_cast<uint32_t>(xor32_i<J>(static_cast<int>(lo)));
  const uint64_t mine = (static_cast<uint64_t>(hi) << 32) | lo;
  const uint64_t other = (static_cast<uint64_t>(ohi) << 32) | olo;
  constexpr uint64_t kWant = sort32_want_small<K2, J>();
  const bool want_small = __builtin_amdgcn_inverse_ballot_w64(kWant);
  const bool take = (other < mine) == want_small;
  hi = take ? ohi : hi;
  lo = take ? olo : lo;
}

// Bitonic sort of the 32 lanes of each wavefront half by (hi, lo), ascending.
__device__ __forceinline__ void sort32_words(uint32_t& hi, uint32_t& lo, int hl) {
  sort32_step<2, 1>(hi, lo, hl);
  sort32_step<4, 2>(hi, lo, hl);
  sort32_step<4, 1>(hi, lo, hl);
  sort32_step<8, 4>(hi, lo, hl);
  sort32_step<8, 2>(hi, lo, hl);
  sort32_step<8, 1>(hi, lo, hl);
  sort32_step<16, 8>(hi, lo, hl);
  sort32_step<16, 4>(hi, lo, hl);
  sort32_step<16, 2>(hi, lo, hl);
  sort32_step<16, 1>(hi, lo, hl);
  sort32_step<32, 16>(hi, lo, hl);
  sort32_step<32, 8>(hi, lo, hl);
  sort32_step<32, 4>(hi, lo, hl);
  sort32_step<32, 2>(hi, lo, hl);
  sort32_step<32, 1>(hi, lo, hl);
}

// The same into rank order (key desc, pack asc); packs are non-negative.
__device__ __forceinline__ void sort32(float& key, int& pack, int hl) {
  uint32_t hi = desc_bits(key), lo = static_cast<uint32_t>(pack);
  sort32_words(hi, lo, hl);
  key = desc_bits_inv(hi);
  pack = static_cast<int>(lo);
}

}  // namespace pisa
