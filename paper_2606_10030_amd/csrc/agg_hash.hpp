// The group-by's key hash and its probe sequence.  Host and device share this
// code (the tests count probes and crowding with it).
#pragma once
#include <cstdint>

namespace agg {
namespace gb {

// The hash of a key: one 32-bit multiply by 2^32 / golden ratio (int64 keys
// add the high word times a second odd constant, the fraction of sqrt 2).
// Everything that places a key reads bits from the top of it downwards: its
// partition, then its sub-partition pass, then its LDS slot, and its home in
// the global table.  Dictionary codes and surrogate keys, which run densely,
// then spread evenly by themselves (the multiples of the golden ratio mod 1),
// so a wave's 64 first probes nearly all hit, and the slots of a workgroup's
// table lie in the order of their homes in the global table, which a flush
// walks almost sequentially.  Two quarter-rate multiplies (one for int32
// keys) against the eight of a 64-bit finaliser: an LDS fold is bound by its
// instructions, not by its bytes.
__host__ __device__ inline uint32_t key_hash_of(int32_t k) { return (uint32_t)k * 0x9638806Du; }
__host__ __device__ inline uint32_t key_hash_of(int64_t k) {
  return (uint32_t)k * 0x9638806Du + (uint32_t)((uint64_t)k >> 32) * 0x69C77F93u;
}

// The hash of a key's next probe, again read from the top.  Each probe lands
// somewhere new: with a fixed step (double hashing) a key of a dense set whose
// step is the distance between two others' homes only ever meets occupied
// slots.
__host__ __device__ inline uint32_t next_probe(uint32_t h) { return h * 0x85EBCA6Bu + 0x7FEB352Du; }

// Probes of an LDS table.  At half load a key finds none of 16 free once in 2^16:
// with 4096 keys in 256 tables that was a row in the global table every few runs,
// and merged tables (gb_merge_kernel) then went there too: 6M rows, float SUM of
// 4096 groups 99 us, or 156.
constexpr int kLdsProbes = 32;

}  // namespace gb
}  // namespace agg
