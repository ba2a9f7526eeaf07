// The group-by's key hash and its probe sequence.  Host and device share this
// code (the tests count probes and crowding with it).
#pragma once
#include <cstdint>

namespace agg {
namespace gb {

// The hash of a key: an xor-shift, so that the multiply after it is not linear in
// the key, and one 32-bit multiply.  Everything that places a key reads bits from
// the top of it downwards: its partition, then its sub-partition pass, then its
// LDS slot, and its home in the global table.
//
// 0x9638806D / 2^32 = 0.58680 has a continued fraction with small quotients (1, 1,
// 2, 2, 1, ...), so the multiples of it mod 1 spread evenly whatever their number,
// and the xor-shift maps every aligned block of 2^m codes onto such a block:
// dictionary codes and surrogate keys, which run densely, spread evenly by
// themselves, a wave's 64 first probes nearly all hit, and the slots of a
// workgroup's table lie in the order of their homes in the global table, which a
// flush walks almost sequentially.
//
// Without the xor-shift a set of keys with a stride whose multiple of the constant
// is near a whole number crowds into a small part of the hash (2000 keys i * 46423:
// 721 in one of 128 sections; with it at most 28).
//
// An int64 key's high word, made zero for keys that fit in 32 bits, enters through a
// multiply of its own and an xor, which the shift and the second multiply do not
// take apart again: two codes packed in one key must not meet in their difference
// or their sum.  (With low * c - high * c, a grid of 1000 x 1000 codes had 1999
// hashes, and their rows went to the global table one by one: int64 SUM of 30M
// rows 47 ms.  Now 0.49 ms, random keys 0.48; 45 x 45 codes 3.4 ms -> 0.146, random
// keys 0.137; 5 x 6 codes 0.132 -> 0.078.)  The multiplier is the prime
// next to 2^32 / golden ratio, as in Knuth's multiplicative hashing (The Art of
// Computer Programming, vol. 3, 6.4).
//
// Two quarter-rate multiplies (one for int32 keys) against the eight of a 64-bit
// finaliser: an LDS fold is bound by its instructions, not by its bytes.
__host__ __device__ inline uint32_t key_hash_of(int32_t k) {
  const uint32_t x = (uint32_t)k;
  return (x ^ (x >> 16)) * 0x9638806Du;
}
__host__ __device__ inline uint32_t key_hash_of(int64_t k) {
  const uint32_t lo = (uint32_t)k, hi = (uint32_t)((uint64_t)k >> 32) + (lo >> 31);
  return key_hash_of((int32_t)(lo ^ (hi * 0x9E3779B1u)));
}

// The hash of a key's next probe, again read from the top.  Each probe lands
// somewhere new: with a fixed step (double hashing) a key of a dense set whose
// step is the distance between two others' homes only ever meets occupied
// slots.  (Constants: the first multiplier of MurmurHash3's 32-bit finaliser by A.
// Appleby; an addend from C. Wellons' search for 32-bit mixers.)
__host__ __device__ inline uint32_t next_probe(uint32_t h) { return h * 0x85EBCA6Bu + 0x7FEB352Du; }

// Probes of an LDS table.  At half load a key finds none of 16 free once in 2^16:
// with 4096 keys in 256 tables that was a row in the global table every few runs,
// and merged tables (gb_merge_kernel) then went there too: 6M rows, float SUM of
// 4096 groups 99 us, or 156.
constexpr int kLdsProbes = 32;

}  // namespace gb
}  // namespace agg
