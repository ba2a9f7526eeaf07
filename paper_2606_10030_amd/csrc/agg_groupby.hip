// Group-by aggregation on gfx950: SUM / MIN / MAX / COUNT / AVG per distinct
// key, keys int32 / int64, values int32 / int64 / float32.
//
// Table: open addressing over a power-of-two number of slots, keys claimed
// with a 64-bit compare-and-swap (INT64_MIN marks an empty slot; the key
// INT64_MIN itself lives in one extra slot), every probe of a key hashed anew
// and their number bounded -- no thread ever waits on another.  Rows are first
// aggregated into a workgroup's own table in LDS (mostly one probe per row; a
// row whose key finds no LDS slot goes straight to the global table).  An LDS
// table that holds all rows of its keys writes its groups to the output; with
// many workgroups the tables are written out and merged by a second launch;
// else each is flushed into the global table, one update per (workgroup, key)
// instead of one per row, and the emission reads that out.  The emission clears
// the slots it reads, so the table is clean between calls.
//
// Two paths, chosen from the plan's max_groups:
//  * direct: workgroups stride over the rows; every workgroup's LDS table
//    holds all the groups in at most half of its slots (or, with up to twice
//    that many, in two passes over the rows, each taking the keys of one half
//    of the hash space).
//  * partitioned (more groups): rows are processed in chunks; each chunk is
//    radix-partitioned on the top bits of the key's hash (histogram, prefix
//    sums, scatter into a staging copy), so that one partition has few enough
//    distinct keys for an LDS table, and then one workgroup (or several, for
//    a partition with many rows) aggregates each partition in LDS (in several
//    passes, one per sub-partition, where the scatter's partitions are too
//    few for that).
//
// Determinism: integer SUM (mod 2^64), MIN, MAX and COUNT are exact in any
// order.  A float32 SUM is accumulated exactly: every finite float is
// m * 2^(k-149) with m < 2^24, added as whole numbers to a fixed-point one (64-bit
// windows in LDS, base-2^32 digits in the global table), so the group sum is
// exact whatever the order and is rounded once to double at the end.  The row
// order inside a partition (set by LDS atomics) therefore never shows in a
// result.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <limits>
#include <new>
#include <type_traits>

#include "agg.h"
#include "agg_device.hpp"
#include "agg_digits.hpp"
#include "agg_hash.hpp"
#include "agg_internal.hpp"

namespace agg {
namespace gb {

constexpr int64_t kEmpty = INT64_MIN;
constexpr int kThreads = 256;
constexpr int kGlobalProbes = 32;     // hashed probes of the global table, then linear ones
constexpr int kMaxPartBits = 14;      // at most 16384 (sub-)partitions
// At least 128 partitions (64 for 2^24 rows and more): with fewer than there are
// aggregation workgroups, several flush the same keys, and their device-scope
// atomics meet on the same addresses; more shorten the scatter's runs.  32 / 64
// / 128 / 256 partitions, 50 000 groups: float SUM of 1.7M rows 111 / 83 / 69 / 72
// us, int32 SUM 75 / 62 / 57 / 63, of 6M rows 106 / 90 / 83 / 83, of 60M rows
// 420 / 411 / 422 / 439; 4096 groups, float SUM of 30M rows 64 / 128: 235 / 256.
// From 2^21 rows on, though, partitions of fewer than about 64 keys only shorten the
// runs, so 32 are the least there.  32 / 64 / 128, float SUM by random int32 keys: 2500
// groups, 3M rows 73 / 79 / 81 us, 6M 90 / 100 / 106, 12M 124 / 134 / 140; 8000 groups,
// 3M 80 / 75 / 80, 12M 129 / 124 / 129; 12 000 groups, 6M 99 / 94 / 92; 4000 dense keys
// of 1M rows 55 / 57 / 46.
// With 2^17 groups and more, at least 256: then most partitions are one
// workgroup's, and their groups leave from LDS (emit_all).  Partitions of few
// keys are too uneven for that, and 16-byte rows pay more for short runs.  128
// (64) / 256 partitions, 200 000 groups: COUNT of 6M rows 108 / 96 us, float SUM
// 174 / 115, of 2^28 rows 1881 / 1812, int64 SUM 3075 / 3261; 90 000 groups:
// int32 SUM of 6M rows 95 / 89, of 2^28 rows 1575 / 1716; 10^6 groups, COUNT of
// 60M rows 474 / 321.
constexpr int kMinPartBits = 7, kMinPartBitsLarge = 6, kMinPartBitsMany = 8, kLeastPartBits = 5;
constexpr int64_t kFewKeysRows = (int64_t)1 << 21, kFewKeys = 128;  // at most, of a partition
constexpr int64_t kManyGroups = (int64_t)1 << 17;
constexpr int64_t kLargeRows = (int64_t)1 << 24;
// Rows are partitioned in chunks of up to 2^28: every chunk ends with each
// aggregation workgroup flushing the groups it holds, so fewer, larger
// chunks flush less (the staging area holds one chunk: up to 4 GiB).
constexpr int64_t kChunkRows = (int64_t)1 << 28;
constexpr int kMaxHistWg = 512;                    // histogram / scatter workgroups per chunk
constexpr int64_t kMinHistRows = 8192;             // rows per such workgroup, at least
constexpr int kTileThreads = 1024;    // scatter: rows staged in LDS per tile
constexpr int kTileMaxBits = 11;      // scatter into at most 2048 partitions
// Rows per tile of the scatter without carried rows: as many as LDS holds next
// to the per-partition counters (at most 152 KiB in all), 16 per thread at most
// (registers).  Longer tiles give longer runs per partition, so fewer partial
// cache lines.  With values, LDS holds keys and values only and the store phase
// hashes the key again; a tile of keys only (COUNT) keeps each row's partition
// in LDS.
template <int KD, int VD, bool HASV>
constexpr int tile_rows() {
  return !HASV ? (KD == AGG_I32 ? 16384 : 12288)
               : (KD == AGG_I32 ? 4 : 8) + (VD == AGG_I64 ? 8 : 4) == 8 ? 16384
               : (KD == AGG_I32 ? 4 : 8) + (VD == AGG_I64 ? 8 : 4) == 12 ? 10240 : 8192;
}
// A staged row with a value is stored as one record, the key's 32-bit words
// then the value's (8, 12 or 16 bytes, over the keys' and the values'
// staging regions together), so a partition's run in a scatter tile is one
// contiguous run instead of two.
template <int KD, int VD>
struct StagedRow {
  static constexpr int KW = KD == AGG_I32 ? 1 : 2, VW = VD == AGG_I64 ? 2 : 1;
  uint32_t w[KW + VW];
};

enum GOp { G_COUNT = 0, G_SUM_INT, G_MIN_INT, G_MAX_INT, G_SUM_F32, G_MIN_F32, G_MAX_F32 };

// LDS tables: one 1024-thread workgroup per CU with one table of up to
// 150 KiB, on both paths: 8192 slots for 4-byte keys, 4096 for 8-byte keys
// (twice that for COUNT, which keeps no value; 4096 for float sums, whose
// slots carry three 64-bit windows).  Measured against three 256-thread
// workgroups per CU with half the slots: fewer, larger tables hold 2x the
// groups at the same load and fold faster.
constexpr int kDirectThreads = 1024;
// Tables up to this many slots are emitted by the aggregation launch's last
// workgroup, larger ones by a launch of their own.  With the table clean from
// the call before and the group count written by the emission, a call of 1e5
// rows and 25 groups is one launch instead of four (22.4 -> 13.3 us).  The one
// workgroup reads past its L2 and a float slot has nine digits, so the line
// lies lower there.  1e5 rows, int32 keys, one launch against two: 25 groups
// 12.8 us (14.1); int32 SUM of 1000 groups, 2048 slots 33.6 (34.8), of 2000,
// 4096 slots 42.2 (40.8); float SUM of 25 groups 17.8 (18.9), of 300, 1024
// slots 36.1 (35.0), of 2000 72.9 (56.1).
constexpr int64_t fuse_slots_of(int g) { return (g == G_SUM_F32 ? 256 : 2048) + 1; }
// Direct path with many workgroups: a table's flush is bound by device-scope
// atomics (about 1.4e10 a second for the chip; 256 workgroups x 2000 groups x 2
// of them are 70 us), so the tables are written out instead, by sections of the
// hash, and a second launch merges each section's records in LDS.  6M rows (366
// workgroups' worth, 256): COUNT of 2000 groups 52 -> 38 us, int32 SUM of 4096 95
// -> 73, float SUM of 4096 223 -> 99, int64 SUM of 100 38 -> 27; 60M rows: COUNT of
// 300 76 -> 73, int32 SUM of 2000 133 -> 122; 2^28 rows within 2%.  The line, where
// the flush would be about 16 000 updates: 5e5 rows, 31 workgroups, COUNT of 2000
// groups 35 -> 28, int64 SUM of 300 19.0 -> 21.5.
constexpr int kSectionBits = 7, kSections = 1 << kSectionBits;
constexpr int kMergeSlots = 512;      // a section holds 128 keys at most, on average (1/128 of 16384)
constexpr int64_t kDirectRows = 16 * kDirectThreads;  // rows per workgroup, at least
constexpr int64_t kMergeMinWg = 16, kMergeMaxWg = 1024;
constexpr int64_t kMergeMinUpdates = 16'000;  // workgroups x groups
constexpr int64_t kMergeMaxRows = (int64_t)1 << 31;  // 32-bit row counts
constexpr int64_t kMergeMaxFloatRows = (int64_t)1 << 24;  // what a window of the merged table holds
constexpr int dump_words_of(int g, int kd) {  // a record: key, rows, value (float sum: windows, flags)
  return (kd == AGG_I32 ? 1 : 2) + 1 + (g == G_COUNT ? 0 : g == G_SUM_F32 ? 7 : 2);
}
constexpr int64_t dump_region_of(int g, int kd, int64_t most) { return kSections + 1 + most * dump_words_of(g, kd); }
constexpr int lds_slots_of(int g, int kd) {
  return g == G_SUM_F32 ? 4096 : (g == G_COUNT ? 2 : 1) * (kd == AGG_I32 ? 8192 : 4096);
}
// A float sum's LDS slot holds kWindows 64-bit fixed-point windows of
// kWinOctaves exponents each, placed where the column's exponents are
// (FloatWindows): a float of biased exponent base + 16 w + s adds its signed
// mantissa << s to window w, one add instead of the two digits it straddles
// in the global table, and a slot takes 24 bytes instead of the 56 of seven
// digits.  |mantissa << s| < 2^39, so 2^24 rows fit a window (kMaxTableRows).
// The flush splits each window into the global table's digits, exactly.
// One add for two, half the table, and so half the partitions: 2^28 rows, int32
// keys: 16 groups 370 -> 343 us, 1024 groups 428 -> 380, 2^16 groups 2139 ->
// 1653, 2^20 groups 2982 -> 2343.
constexpr int kWindows = 3;
constexpr int kWinOctaves = 16;
constexpr int64_t kMaxTableRows = (int64_t)1 << 23;
// A column of more than kWindows windows' exponents (48: 14 decades) takes a table
// of fewer slots with more windows each, in the same LDS: of 4-byte keys 2048 slots
// of 7 (112 exponents) or 1024 of 14, of 8-byte keys 2048 of 6 or 1024 of 12.  Keys
// that such a table does not hold in half of its slots take several passes over the
// rows, by the next bits of their hash, and the columns that spread over more
// exponents than 14 (12) windows two passes by exponent.  The few-groups table has
// room for 9 windows.  (Before, every column took passes of kWindows windows, each
// with its own reading of the rows and its own flush.  int32 keys, 60 exponents, 2^28
// rows: 5 groups 1044 -> 332 us, 300 746 -> 550, 50 000 2066 -> 1914; 200 exponents: 300
// groups 1774 -> 682, 50 000 3354 -> 2420; 10^6 rows of 200 exponents: 300 groups 96 ->
// 52, 50 000 146 -> 94.)
constexpr int kMidSlots = 2048, kAllSlots = 1024;
constexpr int mid_windows_of(int kd) { return kd == AGG_I32 ? 7 : 6; }
constexpr int kFewWindows = 9;
// Rows outside the windows go to the global table one by one.  When a table of
// kWindows has met this many (the sample was not of the column's kind), it is
// flushed, and the workgroup's other rows go to a table whose windows take the
// exponents of those rows in; if that is one of kWindows again and meets as many,
// to tables of all windows.  (2^28 rows of N(0, 1), 0.3% of them times 1e20, against
// staying: 16 groups 912 -> 335 us, 300 groups 695 -> 382; half of them from the middle
// on 695 -> 331 and 682 -> 384.)
constexpr uint32_t kFarRows = 256, kFewFarRows = 32;  // (few groups: the rows meet on the same slots, and a flush is cheap)
constexpr int64_t kTwoPassFloatRows = (int64_t)1 << 27;
// A float sum's tables: 2^lg slots of nw windows, which cover `span` exponents from
// `first` on in the first of `passes` passes over the rows, the next ones in the
// second, and so on; each of these is 2^sub_bits passes by the keys' hash.
struct FloatWindows {
  int first = 1;
  int passes = 1;
  int nw = kWindows;
  int lg = 0;
  int sub_bits = 0;
  int lo = 255, hi = 0;  // the exponents it was made for
  int moves = 0;         // times it was made anew
  __device__ __forceinline__ uint32_t base(int pass) const { return (uint32_t)(first + pass * nw * kWinOctaves); }
  // exponents of the pass (255 marks non-finite floats and is never one of them)
  __device__ __forceinline__ uint32_t span(int pass) const {
    return min((uint32_t)(nw * kWinOctaves), 255u - base(pass));
  }
  __device__ __forceinline__ bool narrow() const { return nw == kWindows; }
  __device__ __forceinline__ bool single() const { return narrow() && passes == 1; }
};
template <int G, int KD>
constexpr int lds_slots() { return lds_slots_of(G, KD); }
constexpr int kPartThreads = 1024;

struct Table {
  int64_t* key;        // cap + 1 slots; slot cap holds the key INT64_MIN
  uint64_t* cnt;
  int64_t* val;        // integer SUM / MIN / MAX; float MIN / MAX as order-preserving ints
  int64_t* dig;        // float SUM: kDigits per slot
  int32_t* flags;      // float SUM: 1 NaN, 2 +Inf, 4 -Inf seen
  // [0] overflow (more distinct keys than slots), [2..3] groups emitted (uint64), [4] finished
  // workgroups, merged runs: [5] the fold put rows into the global table, [6] float sums: the
  // windows' base, [7] the merge put rows there.  State and slots are clean between calls: each call's emission clears what it reads.
  int32_t* state;
  int64_t cap;         // slots, a power of two >= 64
  int32_t cap_log2;
};

// Radix partitioning of one chunk of rows.
struct Part {
  uint32_t* hist;      // [P][g1]: rows of partition p in scatter workgroup g, then their prefix
  uint32_t* tot;       // [P] rows per partition
  uint32_t* start;     // [P + 1] first staged row of each partition
  void* pk;            // staged keys (one chunk)
  void* pv;            // staged values (none for COUNT)
  int32_t bits;        // log2 of the number of partitions the rows are scattered into
  int32_t sub_bits;    // log2 of the aggregation passes over each of them (one per sub-partition)
  int32_t g1;          // histogram / scatter workgroups of this chunk
  int64_t rows_per_wg; // rows each of them covers
};

struct Args {
  Table t;
  Part pt;
  const void* keys;    // this launch's rows (a chunk in the partitioned path)
  const void* vals;
  int64_t n;
  agg_group* out;
  int64_t max_groups;
  int64_t* ngroups;
  int32_t is_avg;
  int32_t op;
  int32_t emit;        // direct path: the launch's last workgroup emits (fuse_slots_of)
  uint32_t* dump;      // direct path, merged: the workgroups' tables, a region each (gb_merge_kernel)
  int32_t dumps;       // workgroups that wrote one; 0: tables are flushed into the global one
  int32_t dump_max;    // records a region holds
  int32_t whole;       // partitioned path: all rows are in this launch (a table may emit its groups itself)
};

// The kernel's arguments, read again: what only the rare paths and the ends of the
// aggregation kernels need of them does not stay in scalar registers during the
// fold, which spills those.
__device__ __forceinline__ const Args& late_args() {
  typedef __attribute__((address_space(4))) const Args kernarg;
  kernarg* p = (kernarg*)__builtin_amdgcn_kernarg_segment_ptr();
  __asm__ volatile("" : "+s"(p));
  return *(const Args*)p;
}

template <int G>
constexpr int64_t val_identity() {
  return (G == G_MIN_INT || G == G_MIN_F32) ? INT64_MAX : (G == G_MAX_INT || G == G_MAX_F32) ? INT64_MIN : 0;
}

template <int G>
__device__ __forceinline__ void clear_slot(const Table& t, int64_t s) {
  t.key[s] = kEmpty;  // slot cap's key is the marker key itself
  t.cnt[s] = 0;
  t.val[s] = val_identity<G>();
  if constexpr (G == G_SUM_F32) {
    t.flags[s] = 0;
    for (int d = 0; d < kDigits; ++d) t.dig[s * kDigits + d] = 0;
  }
}

__device__ __forceinline__ int64_t ceil_div_dev(int64_t a, int64_t b) { return (a + b - 1) / b; }

template <int KD>
__device__ __forceinline__ uint32_t key_hash(typename std::conditional<KD == AGG_I32, int32_t, int64_t>::type k) {
  return key_hash_of(k);
}

// Partition of a key: the top bits of its hash.
__device__ __forceinline__ uint32_t part_of(uint32_t h, int bits) { return h >> (32 - bits); }

// Order-preserving map of non-NaN floats to int32 (and back).
__device__ __forceinline__ int32_t f32_order(float f) {
  const int32_t b = __float_as_int(f);
  return b >= 0 ? b : (b ^ 0x7FFFFFFF);
}
__device__ __forceinline__ float f32_unorder(int32_t o) { return __int_as_float(o >= 0 ? o : (o ^ 0x7FFFFFFF)); }

// The two fixed-point digits of a finite float (value = sum d[j] 2^(32j) 2^-149).
__device__ __forceinline__ void f32_digits(float x, int* k0, int64_t* lo, int64_t* hi) {
  const uint32_t bits = __float_as_uint(x);
  const uint32_t biased = (bits >> 23) & 0xFFu, frac = bits & 0x7FFFFFu;
  const uint64_t m = biased ? (frac | 0x800000u) : frac;
  const int k = biased ? (int)biased - 1 : 0;
  const uint64_t v = m << (k & 31);  // below 2^55
  // the signed product split as lo + hi * 2^32 with 0 <= lo < 2^32: one
  // 64-bit negation instead of one per digit (digits may take either sign)
  const int64_t sv = (bits >> 31) ? -(int64_t)v : (int64_t)v;
  *k0 = k >> 5;
  *lo = (int64_t)((uint64_t)sv & 0xFFFFFFFFu);
  *hi = sv >> 32;
}

// Atomics on a slot of an LDS table (workgroup scope) or of the global
// table (device scope).  The LDS forms name the LDS address space: left to
// infer it, the compiler may merge a row's LDS update with the global one of
// the fallback path into a single generic (flat) atomic, which is far slower
// on LDS than a DS atomic.
typedef __attribute__((address_space(3))) unsigned int lds_u32;
typedef __attribute__((address_space(3))) unsigned long long lds_u64;
typedef __attribute__((address_space(3))) long long lds_i64;
typedef __attribute__((address_space(3))) int lds_i32;

template <bool LDS>
__device__ __forceinline__ void at_add(unsigned int* p, unsigned int v) {
  if constexpr (LDS) __hip_atomic_fetch_add((lds_u32*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else atomicAdd(p, v);
}
template <bool LDS>
__device__ __forceinline__ void at_add(unsigned long long* p, unsigned long long v) {
  if constexpr (LDS) __hip_atomic_fetch_add((lds_u64*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else atomicAdd(p, v);
}
template <bool LDS>
__device__ __forceinline__ void at_min(long long* p, long long v) {
  if constexpr (LDS) __hip_atomic_fetch_min((lds_i64*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else atomicMin(p, v);
}
template <bool LDS>
__device__ __forceinline__ void at_max(long long* p, long long v) {
  if constexpr (LDS) __hip_atomic_fetch_max((lds_i64*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else atomicMax(p, v);
}
template <bool LDS>
__device__ __forceinline__ void at_or(int* p, int v) {
  if constexpr (LDS) __hip_atomic_fetch_or((lds_i32*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else atomicOr(p, v);
}

// Fold one row into a slot of an LDS table (LDS) or of the global table.
template <int G, bool LDS, typename CT>
__device__ __forceinline__ void apply(CT* cnt, int64_t* val, int64_t* dig, int32_t* flags, int64_t iv, float fv) {
  if constexpr (sizeof(CT) == 8) at_add<LDS>(reinterpret_cast<unsigned long long*>(cnt), 1ull);
  else at_add<LDS>(reinterpret_cast<unsigned int*>(cnt), 1u);
  if constexpr (G == G_SUM_INT) at_add<LDS>(reinterpret_cast<unsigned long long*>(val), (unsigned long long)iv);
  if constexpr (G == G_MIN_INT) at_min<LDS>(reinterpret_cast<long long*>(val), (long long)iv);
  if constexpr (G == G_MAX_INT) at_max<LDS>(reinterpret_cast<long long*>(val), (long long)iv);
  if constexpr (G == G_MIN_F32 || G == G_MAX_F32) {
    if (!__builtin_isnan(fv)) {
      if constexpr (G == G_MIN_F32) at_min<LDS>(reinterpret_cast<long long*>(val), (long long)f32_order(fv));
      else at_max<LDS>(reinterpret_cast<long long*>(val), (long long)f32_order(fv));
    }
  }
  if constexpr (G == G_SUM_F32) {
    if (!__builtin_isfinite(fv)) {
      at_or<LDS>(flags, __builtin_isnan(fv) ? 1 : (fv > 0 ? 2 : 4));
    } else {
      int k;
      int64_t lo, hi;
      f32_digits(fv, &k, &lo, &hi);
      if (lo) at_add<LDS>(reinterpret_cast<unsigned long long*>(dig + k), (unsigned long long)lo);
      if (hi) at_add<LDS>(reinterpret_cast<unsigned long long*>(dig + k + 1), (unsigned long long)hi);
    }
  }
}

// The global slot of key k with hash h, claiming an empty one; -1 when the
// table is full.  The home is the top bits of the hash (see key_hash).
__device__ __forceinline__ int64_t global_slot(const Table& t, int64_t k, uint32_t h) {
  if (k == kEmpty) return t.cap;
  const uint64_t mask = (uint64_t)t.cap - 1;
  uint64_t s = 0;
  for (int64_t p = 0; p < t.cap + kGlobalProbes; ++p) {
    if (p < kGlobalProbes) s = t.cap_log2 <= 32 ? (uint64_t)(h >> (32 - t.cap_log2)) : (uint64_t)h << (t.cap_log2 - 32);
    else s = (s + 1) & mask;  // from the last of them on, every slot in turn
    h = next_probe(h);
    const int64_t cur = t.key[s];
    if (cur == k) return (int64_t)s;
    if (cur == kEmpty) {
      const int64_t prev = (int64_t)atomicCAS(reinterpret_cast<unsigned long long*>(t.key + s),
                                              (unsigned long long)kEmpty, (unsigned long long)k);
      if (prev == kEmpty || prev == k) return (int64_t)s;
    }
  }
  __hip_atomic_store(&t.state[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // overflow
  return -1;
}

template <int G>
__device__ __forceinline__ void apply_global(const Table& t, int64_t s, int64_t iv, float fv) {
  apply<G, false>(t.cnt + s, t.val + s, t.dig + (G == G_SUM_F32 ? s * kDigits : 0), t.flags + s, iv, fv);
}

// A group's record, from its rows and its value (float sum: digits and flags).
template <int G>
__device__ __forceinline__ agg_group make_group(int64_t key, int64_t count, int64_t v, const int64_t* d, int32_t flags,
                                                int32_t is_avg) {
  agg_group g;
  g.key = key;
  g.count = count;
  g.i64 = 0;
  g.f64 = 0.0;
  if constexpr (G == G_COUNT) {
    g.i64 = count;
    g.f64 = (double)count;
  } else if constexpr (G == G_SUM_INT) {
    g.i64 = v;
    g.f64 = is_avg ? (double)v / (double)count : (double)v;
  } else if constexpr (G == G_MIN_INT || G == G_MAX_INT) {
    g.i64 = v;
    g.f64 = (double)v;
  } else if constexpr (G == G_SUM_F32) {
    const double sum = digits_to_double(d, flags);
    g.f64 = is_avg ? sum / (double)count : sum;
  } else {  // float MIN / MAX: NaN when every row of the group is NaN
    g.f64 = v == val_identity<G>() ? (double)__builtin_nanf("") : (double)f32_unorder((int32_t)v);
  }
  return g;
}

// V consecutive items of a column at base + tid * V, as one vector load (8 or
// 16 bytes) at any item alignment.  NT: non-temporal (a row is read once).
template <int V, bool NT, typename T>
__device__ __forceinline__ void load_items(T (&x)[V], const T* base, uint32_t tid) {
  typedef uint32_t vec __attribute__((ext_vector_type(V * sizeof(T) / 4), aligned(4)));
  static_assert(sizeof(vec) == sizeof(x), "a vector of whole items");
  const vec* p = reinterpret_cast<const vec*>(base) + tid;
  vec v;
  if constexpr (NT) v = __builtin_nontemporal_load(p);
  else v = *p;
  __builtin_memcpy(x, &v, sizeof(x));
}

// ---- histogram / prefix sums / scatter of the partitioned path ----

// Bound by HBM: every key is read once, in 16-byte vectors, the next tile's
// loads in flight while a tile is counted.  2^28 keys: int32 204 -> 160 us (6.7 TB/s),
// int64 383 -> 325 (6.6).
constexpr int kHistThreads = 512;
template <int KD>
__global__ void __launch_bounds__(kHistThreads) gb_hist_kernel(Args a) {
  using KT = typename std::conditional<KD == AGG_I32, int32_t, int64_t>::type;
  constexpr int NT = kHistThreads, V = 16 / (int)sizeof(KT), R = 4 * V, TR = R * NT;
  __shared__ uint32_t h[1 << kTileMaxBits];
  const int P = 1 << a.pt.bits;
  for (int e = threadIdx.x; e < P; e += NT) h[e] = 0;
  __syncthreads();
  const int64_t lo = (int64_t)blockIdx.x * a.pt.rows_per_wg;
  const int64_t hi = std::min<int64_t>(lo + a.pt.rows_per_wg, a.n);
  const KT* keys = static_cast<const KT*>(a.keys);
  struct Tile {
    KT k[R];
  };
  auto load = [&](Tile& t, int64_t base) {
#pragma unroll
    for (int q = 0; q < R; q += V) {
      KT kk[V];
      load_items<V, true>(kk, keys + base + q * NT, threadIdx.x);
#pragma unroll
      for (int c = 0; c < V; ++c) t.k[q + c] = kk[c];
    }
  };
  int64_t b = lo;
  if (b + TR <= hi) {
    Tile A;
    load(A, b);
    for (;;) {
      const bool more = b + 2 * TR <= hi;
      Tile B;
      load(B, more ? b + TR : b);  // never behind a branch: the count would wait for it
#pragma unroll
      for (int r = 0; r < R; ++r) atomicAdd(&h[part_of(key_hash<KD>(A.k[r]), a.pt.bits)], 1u);
      b += TR;
      if (!more) break;
      A = B;
    }
  }
  for (b += threadIdx.x; b < hi; b += NT) atomicAdd(&h[part_of(key_hash<KD>(keys[b]), a.pt.bits)], 1u);
  __syncthreads();
  for (int e = threadIdx.x; e < P; e += NT) a.pt.hist[(int64_t)e * a.pt.g1 + blockIdx.x] = h[e];
}

// One wave per partition: exclusive prefix of its per-workgroup counts, in
// place; then, in the last workgroup, the partition starts: the exclusive
// prefix of the totals.
__global__ void __launch_bounds__(kThreads) gb_scan_kernel(Args a) {
  __shared__ uint32_t wsum[kThreads / 64];
  const int P = 1 << a.pt.bits;
  const int lane = threadIdx.x & 63, w = threadIdx.x / 64;
  const int64_t p = (int64_t)blockIdx.x * (kThreads / 64) + w;
  auto prefix = [lane](uint32_t s) {  // inclusive, over the wave
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t y = __shfl_up(s, off, 64);
      if (lane >= off) s += y;
    }
    return s;
  };
  if (p < P) {
    uint32_t* row = a.pt.hist + p * a.pt.g1;
    const int q = (a.pt.g1 + 63) / 64;
    uint32_t s = 0;
    for (int j = 0; j < q; ++j) {
      const int idx = lane * q + j;
      if (idx < a.pt.g1) s += row[idx];
    }
    const uint32_t incl = prefix(s);
    uint32_t run = incl - s;
    for (int j = 0; j < q; ++j) {
      const int idx = lane * q + j;
      if (idx < a.pt.g1) {
        const uint32_t v = row[idx];
        row[idx] = run;
        run += v;
      }
    }
    if (lane == 63) __hip_atomic_store(a.pt.tot + p, incl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (!last_to_finish(reinterpret_cast<uint32_t*>(a.t.state + 4))) return;
  constexpr int Q = (1 << kTileMaxBits) / kThreads;  // totals per thread, at most
  uint32_t tot[Q], sum = 0;
#pragma unroll
  for (int j = 0; j < Q; ++j) {
    const int idx = (int)threadIdx.x * Q + j;
    tot[j] = idx < P ? __hip_atomic_load(a.pt.tot + idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    sum += tot[j];
  }
  const uint32_t incl = prefix(sum);
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  uint32_t run = incl - sum;
  for (int v = 0; v < w; ++v) run += wsum[v];
#pragma unroll
  for (int j = 0; j < Q; ++j) {
    const int idx = (int)threadIdx.x * Q + j;
    if (idx < P) a.pt.start[idx] = run;
    run += tot[j];
  }
  if (threadIdx.x == kThreads - 1) a.pt.start[P] = run;  // the last thread ends on the total
  if (threadIdx.x == 0) __hip_atomic_store(&a.t.state[4], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Each row lands at its partition's start + this workgroup's prefix (the
// histogram workgroup of the same rows) + its rank among the partition's
// rows of this workgroup.  Each tile of rows is counting-sorted by partition
// in LDS first, so the rows of one partition leave as one contiguous run
// (coalesced stores) instead of one scattered store per row.
template <int KD, int VD, bool HASV>
__global__ void __launch_bounds__(kTileThreads) gb_scatter_tiled_kernel(Args a) {
  using KT = typename std::conditional<KD == AGG_I32, int32_t, int64_t>::type;
  using VT = typename std::conditional<VD == AGG_I64, int64_t, uint32_t>::type;
  constexpr int TR = tile_rows<KD, VD, HASV>();
  constexpr int R = TR / kTileThreads;
  constexpr int PM = 1 << kTileMaxBits;
  __shared__ KT skey[TR];
  __shared__ VT sval[HASV ? TR : 1];
  __shared__ uint16_t spart[HASV ? 1 : TR];
  __shared__ uint32_t tcnt[PM], toff[PM], cur[PM];
  const int P = 1 << a.pt.bits;
  const int tid = threadIdx.x;
  for (int e = tid; e < P; e += kTileThreads) {
    cur[e] = a.pt.start[e] + a.pt.hist[(int64_t)e * a.pt.g1 + blockIdx.x];
    tcnt[e] = 0;
  }
  __syncthreads();
  const int64_t lo = (int64_t)blockIdx.x * a.pt.rows_per_wg;
  const int64_t hi = std::min<int64_t>(lo + a.pt.rows_per_wg, a.n);
  for (int64_t t0 = lo; t0 < hi; t0 += TR) {
    const int rows = (int)std::min<int64_t>(TR, hi - t0);
    KT k[R];
    VT v[R];
    uint32_t pp[R], rank[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {  // all loads first (rows past the tile re-load its last row)
      const int j = std::min(r * kTileThreads + tid, rows - 1);
      k[r] = static_cast<const KT*>(a.keys)[t0 + j];
      if constexpr (HASV) v[r] = static_cast<const VT*>(a.vals)[t0 + j];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (r * kTileThreads + tid < rows) {
        pp[r] = part_of(key_hash<KD>(k[r]), a.pt.bits);
        rank[r] = atomicAdd(&tcnt[pp[r]], 1u);
      }
    }
    __syncthreads();
    if (tid < 64) {  // one wave: exclusive prefix of the tile's counts
      const int q = (P + 63) / 64;
      uint32_t sum = 0;
      for (int j = 0; j < q; ++j) sum += (tid * q + j < P) ? tcnt[tid * q + j] : 0u;
      uint32_t incl = sum;
      for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off, 64);
        if (tid >= off) incl += y;
      }
      uint32_t run = incl - sum;
      for (int j = 0; j < q; ++j) {
        const int e = tid * q + j;
        if (e < P) {
          toff[e] = run;
          run += tcnt[e];
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int j = r * kTileThreads + tid;
      if (j < rows) {
        const uint32_t d = toff[pp[r]] + rank[r];
        skey[d] = k[r];
        if constexpr (HASV) sval[d] = v[r];
        else spart[d] = (uint16_t)pp[r];
      }
    }
    __syncthreads();
    for (int j = tid; j < rows; j += kTileThreads) {
      uint32_t q;
      if constexpr (HASV) q = part_of(key_hash<KD>(skey[j]), a.pt.bits);
      else q = spart[j];
      const uint32_t pos = cur[q] + (uint32_t)j - toff[q];
      if ((int64_t)pos >= a.n) continue;  // cannot happen: counts match the histogram
      if constexpr (HASV) {
        using SR = StagedRow<KD, VD>;
        SR row;
        const uint64_t kb = (uint64_t)(int64_t)skey[j], vb = (uint64_t)sval[j];
        row.w[0] = (uint32_t)kb;
        if constexpr (SR::KW == 2) row.w[1] = (uint32_t)(kb >> 32);
        row.w[SR::KW] = (uint32_t)vb;
        if constexpr (SR::VW == 2) row.w[SR::KW + 1] = (uint32_t)(vb >> 32);
        static_cast<SR*>(a.pt.pk)[pos] = row;
      } else {
        static_cast<KT*>(a.pt.pk)[pos] = skey[j];
      }
    }
    __syncthreads();
    for (int e = tid; e < P; e += kTileThreads) {
      cur[e] += tcnt[e];
      tcnt[e] = 0;
    }
    __syncthreads();
  }
}

// The same scatter, writing whole 64-byte pieces only, for up to PMAX
// partitions.  A tile's run for one partition is some tens of rows, and the
// incomplete lines at its ends leave L2 before the next tile completes them;
// a partial write costs the memory far more than its bytes (2^28 rows of 12
// bytes, 256 partitions, stores of the same volume: 1636 us with unaligned
// runs, 1382 with aligned ones).  So a partition's run ends at a multiple of U
// rows (64 bytes, or 192 for 12-byte rows), and the up to U - 1 rows past it
// stay: 1024 / P threads per partition carry them in registers and put them
// back at the head of their partition in the next tile.  2^28 rows: 12 bytes,
// 256 partitions 1774 -> 1522 us, 32 partitions 1330 -> 1268; 16 bytes, 512
// partitions 2626 -> 2186; 8 bytes, 512 partitions 1322 -> 1128.  (Loading the
// next tile during the stores changed nothing: reads and writes share the
// memory's time.)
template <int KD, int VD, bool HASV, bool WIDE>
struct CarryTile {
  static constexpr int RB = (KD == AGG_I32 ? 4 : 8) + (!HASV ? 0 : VD == AGG_I64 ? 8 : 4);  // bytes of a row
  static constexpr int U = RB == 16 ? 4 : RB == 8 ? 8 : 16;
  static constexpr int PMAX = (U == 16 ? 256 : 512) << (WIDE ? 1 : 0);
  // New rows per thread and tile: what LDS holds next to the carried rows.
  static constexpr int R = RB == 4 ? (WIDE ? 24 : 32) : RB == 8 ? (WIDE ? 10 : 14) : RB == 12 ? (WIDE ? 4 : 8) : WIDE ? 4 : 6;
  static constexpr int CR = ((U - 1) * PMAX + kTileThreads - 1) / kTileThreads;  // carried rows per thread
  static constexpr int CAP = R * kTileThreads + (U - 1) * PMAX;
};

template <int KD, int VD, bool HASV, bool WIDE>
__global__ void __launch_bounds__(kTileThreads) gb_scatter_carry_kernel(Args a) {
  using KT = typename std::conditional<KD == AGG_I32, int32_t, int64_t>::type;
  using VT = typename std::conditional<VD == AGG_I64, int64_t, uint32_t>::type;
  using SR = StagedRow<KD, VD>;
  using T = CarryTile<KD, VD, HASV, WIDE>;
  constexpr int NT = kTileThreads, R = T::R, U = T::U, TR = R * NT;
  constexpr int V = KD == AGG_I64 || (HASV && VD == AGG_I64) || R % 4 ? 2 : 4;
  static_assert(R % V == 0, "a thread's rows are whole vectors");
  __shared__ KT skey[T::CAP];
  __shared__ VT sval[HASV ? T::CAP : 1];
  // per partition: rows of the tile (the carried ones first); their first
  // place in the tile; the place where the stored ones end, and in the upper
  // bits how many are left; where place j is stored: delta + j; rows stored so far
  __shared__ uint32_t tcnt[T::PMAX], toff[T::PMAX], tend[T::PMAX], delta[T::PMAX], cur[T::PMAX], total;
  constexpr int kEndBits = 20;
  const int P = 1 << a.pt.bits;
  const uint32_t tid = threadIdx.x;
  // this thread's carried rows are rows lane, lane + step, ... of partition mine
  const uint32_t step = (uint32_t)NT >> a.pt.bits, mine = tid / step, lane = tid % step;
  for (int e = tid; e < P; e += NT) {
    cur[e] = a.pt.start[e] + a.pt.hist[(int64_t)e * a.pt.g1 + blockIdx.x];
    tcnt[e] = 0;
  }
  __syncthreads();
  const int64_t lo = (int64_t)blockIdx.x * a.pt.rows_per_wg;
  const int64_t hi = std::min<int64_t>(lo + a.pt.rows_per_wg, a.n);
  const uint32_t last_row = (uint32_t)(a.n - 1);
  KT k[R], ck[T::CR];
  VT v[R], cv[T::CR];
  uint32_t pr[R];      // a row's partition in the upper half, its rank there in the lower
  uint32_t kept = 0;   // rows carried in partition mine
#pragma unroll
  for (int c = 0; c < T::CR; ++c) {
    ck[c] = 0;
    cv[c] = 0;
  }
  auto row_at = [&](int r) -> uint32_t { return (uint32_t)(r / V * V * NT + r % V) + tid * V; };
  for (int64_t t0 = lo; t0 < hi; t0 += TR) {
    const bool full = t0 + TR <= hi;
    const uint32_t rows = full ? (uint32_t)TR : (uint32_t)(hi - t0);
    if (full) {
#pragma unroll
      for (int q = 0; q < R; q += V) {
        KT kk[V];
        load_items<V, !HASV>(kk, static_cast<const KT*>(a.keys) + t0 + q * NT, tid);
#pragma unroll
        for (int c = 0; c < V; ++c) k[q + c] = kk[c];
        if constexpr (HASV) {
          VT vv[V];
          load_items<V, false>(vv, static_cast<const VT*>(a.vals) + t0 + q * NT, tid);
#pragma unroll
          for (int c = 0; c < V; ++c) v[q + c] = vv[c];
        }
      }
    } else {  // rows past the end re-load the last row
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const uint32_t j = std::min<uint32_t>(row_at(r), rows - 1);
        k[r] = (static_cast<const KT*>(a.keys) + t0)[j];
        if constexpr (HASV) v[r] = (static_cast<const VT*>(a.vals) + t0)[j];
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (full || row_at(r) < rows) {
        const uint32_t q = part_of(key_hash<KD>(k[r]), a.pt.bits);
        pr[r] = (q << 16) | atomicAdd(&tcnt[q], 1u);
      }
    }
    __syncthreads();
    if (tid < 64) {  // one wave: exclusive prefix of the tile's counts
      const int q = (P + 63) / 64;
      uint32_t sum = 0;
      for (int j = 0; j < q; ++j) sum += ((int)tid * q + j < P) ? tcnt[tid * q + j] : 0u;
      uint32_t incl = sum;
      for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off, 64);
        if ((int)tid >= off) incl += y;
      }
      if (tid == 63) total = incl;
      uint32_t run = incl - sum;
      for (int j = 0; j < q; ++j) {
        const int e = tid * q + j;
        if (e < P) {
          const uint32_t c = tcnt[e], at = cur[e];
          // the last tile of the workgroup's rows keeps nothing
          const uint32_t keep = t0 + TR < hi ? std::min<uint32_t>(c, (at + c) % U) : 0u;
          toff[e] = run;
          delta[e] = at - run;
          tend[e] = (run + c - keep) | (keep << kEndBits);
          cur[e] = at + c - keep;
          tcnt[e] = keep;
          run += c;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (full || row_at(r) < rows) {
        const uint32_t d = toff[pr[r] >> 16] + (pr[r] & 0xFFFFu);
        skey[d] = k[r];
        if constexpr (HASV) sval[d] = v[r];
      }
    }
#pragma unroll
    for (int c = 0; c < T::CR; ++c) {
      const uint32_t i = lane + (uint32_t)c * step;
      if (i < kept) {
        const uint32_t d = toff[mine] + i;
        skey[d] = ck[c];
        if constexpr (HASV) sval[d] = cv[c];
      }
    }
    __syncthreads();
    const uint32_t places = total;
    for (uint32_t j = tid; j < places; j += NT) {
      const KT kj = skey[j];
      const uint32_t q = part_of(key_hash<KD>(kj), a.pt.bits);
      if (j >= (tend[q] & ((1u << kEndBits) - 1))) continue;  // carried over
      const uint32_t pos = std::min<uint32_t>(delta[q] + j, last_row);  // in bounds whatever the counts say
      if constexpr (HASV) {
        SR row;
        const uint64_t kb = (uint64_t)(int64_t)kj, vb = (uint64_t)sval[j];
        row.w[0] = (uint32_t)kb;
        if constexpr (SR::KW == 2) row.w[1] = (uint32_t)(kb >> 32);
        row.w[SR::KW] = (uint32_t)vb;
        if constexpr (SR::VW == 2) row.w[SR::KW + 1] = (uint32_t)(vb >> 32);
        static_cast<SR*>(a.pt.pk)[pos] = row;
      } else {
        static_cast<KT*>(a.pt.pk)[pos] = kj;
      }
    }
    const uint32_t end = tend[mine];
    kept = end >> kEndBits;
#pragma unroll
    for (int c = 0; c < T::CR; ++c) {
      const uint32_t i = lane + (uint32_t)c * step;
      if (i < kept) {
        const uint32_t d = (end & ((1u << kEndBits) - 1)) + i;
        ck[c] = skey[d];
        if constexpr (HASV) cv[c] = sval[d];
      }
    }
    // no barrier: the next tile's ranks touch only tcnt, which this phase does
    // not read, and everything else changes past the next two barriers
  }
}

// ---- aggregation into LDS tables, flushed into the global table ----

// 32-bit words of a row's key and value.
template <int KD, int VD, int G>
constexpr int row_words() {
  return (KD == AGG_I64 ? 2 : 1) + (G == G_COUNT ? 0 : VD == AGG_I64 ? 2 : 1);
}

// One workgroup's table: L hashed slots keyed in the key column's own width
// (4-byte keys fit twice the slots of 8-byte ones), plus slot L for the one
// key whose bit pattern marks an empty slot.  Each slot has REP copies of its
// accumulators; lane l of a wave updates copy l % REP, so the lanes of one
// wave instruction whose rows share a key spread over REP addresses (LDS
// atomics on one address serialise), and the flush merges the copies (exact
// integer merges: the results do not depend on REP).
// HOT: the table finds a key that most of its rows have, and gives each lane an
// entry for it (find_hot).
// WORDS: 64-bit windows of a float sum in all; its slots and windows are those of
// a FloatWindows `z` (2^z.lg slots of at most L_), all other tables have L_ slots.
template <int G, int KD, int L_, int NT, int REP = 1, bool HOT = false, int WORDS = 0>
struct LdsTable {
  using KT = typename std::conditional<KD == AGG_I32, int32_t, int64_t>::type;
  using UKT = typename std::conditional<KD == AGG_I32, unsigned int, unsigned long long>::type;
  static constexpr KT kMark = std::numeric_limits<KT>::min();  // empty hashed slot
  static constexpr int kMaxL = L_;
  // Accumulator entries: slot s, copy c at s * REP + c; then one per lane for
  // the hot slot's rows (find_hot).
  static constexpr int kHotLanes = HOT ? 64 : 0;
  static constexpr int kMaxE = (L_ + 1) * REP + kHotLanes;
  static constexpr uint32_t kNoHot = ~0u;
  static constexpr bool kDig = G == G_SUM_F32;
  static constexpr bool kFlex = kDig && WORDS != 0;  // (else kWindows)
  static constexpr bool kLeaves = kDig && !(kFlex && REP == 1);  // may leave rows to tables of more windows
  static __device__ __forceinline__ int log2l(const FloatWindows& z) {
    if constexpr (kFlex && REP == 1) return z.lg;
    else return __builtin_ctz((unsigned)L_);
  }
  static __device__ __forceinline__ int slots(const FloatWindows& z) { return 1 << log2l(z); }
  static __device__ __forceinline__ int entries(const FloatWindows& z) { return (slots(z) + 1) * REP + kHotLanes; }
  static __device__ __forceinline__ int windows(const FloatWindows& z) { return kFlex ? z.nw : kWindows; }
  static constexpr bool kVal = !kDig && G != G_COUNT;
  static_assert((REP & (REP - 1)) == 0 && REP <= 64, "copies: a power of two, at most a wave");
  static_assert(!HOT || REP == 1, "one kind of copies");
  static_assert((L_ & (L_ - 1)) == 0, "home_of takes log2(L) hash bits");
  // Rows a thread folds at a time (two batches are in registers: the next
  // one's loads are in flight): 8, or 4 where a row has four 32-bit words (8
  // ran 8% slower: spills), or three and copies of float windows (1e5 rows 19.2 ->
  // 14.1 us, 2^28 rows 512 -> 464).
  template <int VD>
  static constexpr int tile_rows_of() { return row_words<KD, VD, G>() >= (kDig && REP > 1 ? 3 : 4) ? 4 : 8; }
  KT key[kMaxL];
  uint32_t cnt[kMaxE];  // rows per table stay below 2^32 (a workgroup's share is at most 2^28 rows)
  int64_t val[kVal ? kMaxE : 1];
  int64_t win[kFlex ? WORDS : kDig ? kWindows * kMaxE : 1];  // float sum: window w of entry e at w * entries + e
  uint32_t flags[kDig ? kMaxL / 8 + 1 : 1];  // float sum: non-finite rows seen, four bits a slot
  uint16_t list[NT / 64][128];             // per wave: slots to flush
  uint32_t spilled;                        // a row went to the global table
  uint32_t far_rows, far_lo, far_hi;       // float sum: rows outside the windows, and their exponents
  uint32_t emit_base[2];                   // emit_all: the output range's first group
  uint32_t wave_groups[NT / 64];           // emit_all: groups per wave
  uint32_t hot_sh;                         // the hot slot + 1; 0: there is none

  __device__ __forceinline__ void clear(uint32_t skip, const FloatWindows& z) {
    const int L = slots(z), E = entries(z);
    // The marker key's home holds key 0 from the start: a row of the marker key
    // then never finds its key at home (it would take an empty slot for its
    // own), and goes on to slot L.  Key 0 may use the slot like any other it
    // finds itself in; with no rows it is not flushed.
    const int marker_home = (int)home_of(key_hash<KD>(kMark), skip, z);
    for (int e = threadIdx.x; e < L; e += NT) key[e] = e == marker_home ? (KT)0 : kMark;
    for (int e = threadIdx.x; e < E; e += NT) {
      cnt[e] = 0;
      if constexpr (kVal) val[e] = val_identity<G>();
      if constexpr (kDig && !kFlex)
        for (int w = 0; w < kWindows; ++w) win[w * E + e] = 0;
    }
    if constexpr (kDig) {
      if constexpr (kFlex)
        for (int i = threadIdx.x; i < windows(z) * E; i += NT) win[i] = 0;
      for (int e = threadIdx.x; e <= L / 8; e += NT) flags[e] = 0;
    }
    if (threadIdx.x == 0) {
      hot_sh = 0;
      spilled = 0;
      far_rows = 0;
      far_lo = 255;
      far_hi = 0;
    }
  }

  // The table's hot slot, if the home slots of its first batch show one to this
  // wave (or an earlier one to another wave), else kNoHot.  LDS atomics of a wave
  // on one address serialise, so a table whose rows are mostly one key's (one
  // partition of a skewed column) was bound by them: each lane adds the hot
  // slot's rows to an entry of its own instead, and merge_hot adds those to the
  // slot.  A wave proposes the slot that the most lanes share in any of its rows
  // (eight lanes or more); the table takes the first one proposed, which is
  // mostly the hottest.  Which it is, and which waves know of it, does not show
  // in the sums.  Partitioned path only: there a skewed column's few hottest
  // keys fill whole partitions, and the workgroups on those ended last (the
  // direct path spreads them over all tables, and lost more by the extra
  // instructions than it won: 4096 groups 219 -> 226 us).  60M rows, 50 000
  // keys of probability ~ 1/rank (uniform ones in brackets): int32 SUM 587 ->
  // 454 us (439 -> 444), COUNT 388 -> 330 (322 -> 328), float SUM 612 -> 522
  // (518 -> 519), int64 SUM 875 -> 764 (767 -> 761); 2^20 keys: int32 SUM 749 ->
  // 609 (615 -> 618).
  template <int R>
  __device__ __forceinline__ uint32_t find_hot(const uint32_t (&home)[R]) {
    uint32_t best = 0;  // lanes << 16 | slot
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint32_t s = (uint32_t)__builtin_amdgcn_readfirstlane((int)home[r]);
      best = max(best, (uint32_t)__popcll(__ballot(home[r] == s)) << 16 | s);
    }
    if (best < 8u << 16) return kNoHot;
    const uint32_t cand = best & 0xFFFFu;
    uint32_t prev = 0;
    if ((threadIdx.x & 63) == 0) prev = atomicCAS(&hot_sh, 0u, cand + 1);
    prev = (uint32_t)__builtin_amdgcn_readfirstlane((int)prev);
    return prev ? prev - 1 : cand;
  }
  __device__ __forceinline__ uint32_t hot_slot() const {
    const uint32_t h = (uint32_t)__builtin_amdgcn_readfirstlane((int)hot_sh);
    return h - 1;  // 0: none
  }
  // The entry that this lane's row of slot s goes to.
  static __device__ __forceinline__ int entry_of(uint32_t s, uint32_t hot, int L) {
    if constexpr (HOT) return (int)(s == hot ? L + 1 + (threadIdx.x & 63) : s);
    else return (int)(s * REP + (threadIdx.x & (REP - 1)));
  }
  // Between the fold's barrier and the flush.
  __device__ __forceinline__ void merge_hot(const FloatWindows& z) {
    if constexpr (kHotLanes != 0) {
      const int L = slots(z), E = entries(z);
      const uint32_t hot = hot_slot();
      if (hot == kNoHot) return;  // the whole workgroup
      if (threadIdx.x < 64) {
        const int e = L + 1 + threadIdx.x;
        at_add<true>(&cnt[hot], cnt[e]);
        if constexpr (kVal) {
          if constexpr (G == G_SUM_INT)
            at_add<true>(reinterpret_cast<unsigned long long*>(&val[hot]), (unsigned long long)val[e]);
          else if constexpr (G == G_MIN_INT || G == G_MIN_F32)
            atomicMin(reinterpret_cast<long long*>(&val[hot]), (long long)val[e]);
          else atomicMax(reinterpret_cast<long long*>(&val[hot]), (long long)val[e]);
        }
        if constexpr (kDig)
          for (int w = 0; w < windows(z); ++w)
            at_add<true>(reinterpret_cast<unsigned long long*>(&win[w * E + hot]), (unsigned long long)win[w * E + e]);
      }
      __syncthreads();
    }
  }

  // The home slot of a key with hash h: the log2(L) hash bits below the
  // `skip` that chose its partition and pass.
  static __device__ __forceinline__ uint32_t home_of(uint32_t h, uint32_t skip, const FloatWindows& z) {
    // (two operands in scalar registers would cost a bit-field extract a vector register)
    if constexpr (kFlex && REP == 1) return (h << skip) >> (32 - log2l(z));
    else return __builtin_amdgcn_ubfe(h, (uint32_t)(32 - log2l(z)) - skip, (uint32_t)log2l(z));
  }
  // The slot of its next probe, of hash h.
  static __device__ __forceinline__ uint32_t probe_of(uint32_t h, const FloatWindows& z) { return h >> (32 - log2l(z)); }

  // The slot of key k with hash h, claiming an empty one; -1 if there is none
  // within kLdsProbes probes.
  __device__ __forceinline__ int slot_of(KT k, uint32_t h, uint32_t skip, const FloatWindows& z) {
    if (k == kMark) return slots(z);
    uint32_t s = home_of(h, skip, z);
#pragma unroll 1
    for (int p = 0; p < kLdsProbes; ++p) {
      const KT cur = key[s];
      if (cur == k) return (int)s;
      if (cur == kMark) {
        const KT prev = (KT)atomicCAS(reinterpret_cast<UKT*>(&key[s]), (UKT)kMark, (UKT)k);
        if (prev == kMark || prev == k) return (int)s;
      }
      h = next_probe(h);
      s = probe_of(h, z);
    }
    return -1;
  }

  // Adds the float of bits fb to the windows of entry s; u = its bits << 1
  // less the pass's first exponent << 24, below the windows' span << 24; E: entries.
  __device__ __forceinline__ void add_window(int s, uint32_t fb, uint32_t u, int E) {
    const int32_t sign = (int32_t)fb >> 31;
    const int32_t m = (int32_t)(((fb & 0x7FFFFFu) | 0x800000u) ^ (uint32_t)sign) - sign;
    const uint32_t w = u >> 28, sh = __builtin_amdgcn_ubfe(u, 24, 4);
    static_assert(kWinOctaves == 16, "a window is the exponent's upper four bits");
    // m is never 0, so its sign word is the upper half of the 64-bit value
    const uint64_t v = (((uint64_t)(uint32_t)sign << 32) | (uint32_t)m) << sh;
    uint32_t at;
    if constexpr (kFlex)  // one full-rate instruction: left to itself the compiler takes a 32-bit multiply for an E it does not know
      __asm__("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(at) : "v"(w), "s"(E), "v"(s));
    else at = __umul24(w, E) + (uint32_t)s;
    at_add<true>(reinterpret_cast<unsigned long long*>(&win[at]), (unsigned long long)v);
  }

  // Folds the rows of the tiles first, first + tile_step, ... (kTile rows
  // each) below last whose key hash has the bits (hash >> sub_shift) &
  // sub_mask equal to sub; a row whose key finds no slot within kLdsProbes
  // probes goes to the global table.
  // ROWS: keys holds staged (key, value) records.  SUB: the plan has
  // sub-partition passes (0: every row belongs to the single pass and the
  // per-row test of its hash bits is left out; 2: sub_mask 0 is a single pass).
  // Returns the first row that this wave leaves to another table (kFarRows), or
  // last.
  //
  // Bound by instructions and LDS atomics, so a full tile's rows carry neither
  // bounds test nor address arithmetic (a uniform base per row and one lane
  // offset), the next tile's loads are in flight while a tile is folded, and
  // the first probes of a batch are read before the first of them is
  // resolved.  A row whose home slot holds its key takes a few straight
  // instructions; a batch with any other row (a new key, a collision, a float
  // outside the windows) reads all second probes too, and what neither probe
  // finds sets a bit for one loop after the batch, which handles one row of
  // each lane at a time.  (Random keys that fill half a table, 2^28 rows:
  // int64 SUM of 4096 groups 830 -> 721 us; with the loop right after the
  // first probes 923.)
  template <int VD, bool ROWS, int SUB>
  __device__ __forceinline__ int64_t fold_rows(const Args& a_, const void* keys, const void* vals, int64_t first,
                                               int64_t last, int64_t tile_step, uint32_t skip, uint32_t sub_shift,
                                               uint32_t sub_mask, uint32_t sub, const FloatWindows& fw, int pass) {
    constexpr int R = tile_rows_of<VD>();
    constexpr int TR = R * NT;
    constexpr bool kStaged = ROWS && G != G_COUNT;
    const int L = slots(fw), E = entries(fw);
    using IVT = typename std::conditional<VD == AGG_I64, int64_t, int32_t>::type;
    using SR = StagedRow<KD, VD == AGG_I64 ? AGG_I64 : AGG_I32>;
    struct Row {
      KT k;
      IVT iv;
      float fv;
    };
    struct Batch {  // R rows' registers
      Row x[R];
    };
    const uint32_t tid = threadIdx.x;
    uint32_t hot = kNoHot;
    bool cold = true;  // the first batch
    // a float's exponent is compared in place, as the top byte of its bits << 1
    // less the pass's first exponent (exponents below it wrap past the span);
    // no pass takes out_from and up, seen from the first one (zeros, subnormals
    // and non-finite floats among them)
    const uint32_t win_off = 0u - (fw.base(pass) << 24), win_span = fw.span(pass) << 24;
    const uint32_t out_from =
        pass == 0 ? min((uint32_t)(fw.passes * fw.nw * kWinOctaves), 255u - fw.base(0)) << 24 : UINT32_MAX;
    auto load_row = [&](Row& x, int64_t base, uint32_t lane) {  // row base + lane (base uniform)
      x.iv = 0;
      x.fv = 0.0f;
      if constexpr (ROWS && G != G_COUNT) {
        const SR row = (static_cast<const SR*>(keys) + base)[lane];
        if constexpr (SR::KW == 2) x.k = (KT)(((uint64_t)row.w[1] << 32) | row.w[0]);
        else x.k = (KT)(int32_t)row.w[0];
        if constexpr (VD == AGG_F32) x.fv = __uint_as_float(row.w[SR::KW]);
        else if constexpr (VD == AGG_I64) x.iv = (int64_t)(((uint64_t)row.w[SR::KW + 1] << 32) | row.w[SR::KW]);
        else x.iv = (int32_t)row.w[SR::KW];
      } else {
        x.k = (static_cast<const KT*>(keys) + base)[lane];
        if constexpr (G != G_COUNT) {
          if constexpr (VD == AGG_F32) x.fv = (static_cast<const float*>(vals) + base)[lane];
          else x.iv = (static_cast<const IVT*>(vals) + base)[lane];
        }
      }
    };
    // Row r of a tile sits at row_at(r) from its base.  Rows of a column: a
    // thread takes V consecutive ones, so that the wider of key and value is
    // read in 16-byte vectors and every load of a wave is contiguous; staged
    // records: one every NT, a whole record a load.
    constexpr int V = KD == AGG_I64 || (G != G_COUNT && VD == AGG_I64) ? 2 : 4;
    auto row_at = [&](int r) -> uint32_t {
      if constexpr (kStaged) return (uint32_t)(r * NT) + tid;
      else return (uint32_t)(r / V * V * NT + r % V) + tid * V;
    };
    auto load = [&](Batch& b, int64_t base) {
      if constexpr (kStaged) {
#pragma unroll
        for (int r = 0; r < R; ++r) load_row(b.x[r], base + r * NT, tid);
      } else {
#pragma unroll
        for (int q = 0; q < R; q += V) {
          KT kk[V];
          load_items<V, true>(kk, static_cast<const KT*>(keys) + base + q * NT, tid);
#pragma unroll
          for (int c = 0; c < V; ++c) {
            b.x[q + c].k = kk[c];
            b.x[q + c].iv = 0;
            b.x[q + c].fv = 0.0f;
          }
          if constexpr (G != G_COUNT) {
            IVT vv[V];
            load_items<V, true>(vv, static_cast<const IVT*>(vals) + base + q * NT, tid);
#pragma unroll
            for (int c = 0; c < V; ++c) {
              if constexpr (VD == AGG_F32) b.x[q + c].fv = __int_as_float(vv[c]);
              else b.x[q + c].iv = vv[c];
            }
          }
        }
      }
    };
    // the last, partial tile: rows past its end re-load its last row (in
    // bounds, not folded)
    auto load_tail = [&](Batch& b, int64_t base, uint32_t left) {
#pragma unroll
      for (int r = 0; r < R; ++r) load_row(b.x[r], base, std::min<uint32_t>(row_at(r), left - 1));
    };
    // true: the wave's other rows are for another table
    auto fold = [&](Batch& b, int64_t base, bool full, uint32_t left) -> bool {
      // the batch's loads are complete before its first row is folded: left
      // alone, the compiler sinks a value load into the branch that uses it,
      // and that load's whole latency then stalls the wave
#pragma unroll
      for (int r = 0; r < R; ++r) {
        __asm__ volatile("" : "+v"(b.x[r].k));
        if constexpr (G != G_COUNT) {
          if constexpr (VD == AGG_F32) __asm__ volatile("" : "+v"(b.x[r].fv));
          else __asm__ volatile("" : "+v"(b.x[r].iv));
        }
      }
      uint32_t rest = 0;  // bit R - 1 - r: row r is for the loop below
      uint32_t home[R];
      KT cur[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        home[r] = home_of(key_hash<KD>(b.x[r].k), skip, fw);
        cur[r] = key[home[r]];
      }
      // one wait for all of the batch's probes: left alone, each row's check
      // would also wait for the atomics of the rows before it
#pragma unroll
      for (int r = 0; r < R; ++r) __asm__ volatile("" : "+v"(cur[r]));
      // Nearly every batch of a wave: each row of each lane finds its key at
      // home (and its float in a window), tested for all of them at once, so
      // a row is its adds and nothing else.
      auto all_found = [&]() -> bool {
        KT differ = 0;
        uint32_t far = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          differ |= cur[r] ^ b.x[r].k;
          if constexpr (kDig) far = max(far, (__float_as_uint(b.x[r].fv) << 1) + win_off);
        }
        return full && __all(differ == 0 && (!kDig || far < win_span));
      };
      bool found = false;
      if constexpr (SUB != 1) found = (SUB == 0 || sub_mask == 0) && all_found();
      if constexpr (REP > 1) {
        // Few keys, so many rows may be of one that is not at home: the next probes
        // of the whole batch, up to three, until all are found (not in the first
        // batch, which finds the table empty).  Random int32 keys, 2^28 rows, with 128
        // slots and the loop below instead: 25 groups, int32 SUM 390 -> 315 us, COUNT
        // 327 -> 163, float SUM 516 -> 333; 32 groups 467 -> 324, 414 -> 186, 609 ->
        // 349 (a set of which a key is at its third slot: COUNT 240, at its fourth 310).
        uint32_t h[R];
#pragma unroll
        for (int r = 0; r < R; ++r) h[r] = key_hash<KD>(b.x[r].k);
#pragma unroll 1
        for (int p = 0; p < 3 && full && !found && !cold; ++p) {
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const bool hit = cur[r] == b.x[r].k;
            h[r] = next_probe(h[r]);
            home[r] = hit ? home[r] : probe_of(h[r], fw);
          }
#pragma unroll
          for (int r = 0; r < R; ++r) {  // (an empty slot is no match for the marker key)
            cur[r] = key[home[r]];
            cur[r] = b.x[r].k == kMark ? (KT)0 : cur[r];
          }
          found = all_found();
        }
      }
      if (found) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int s = entry_of(home[r], hot, L);
          if constexpr (kDig) {
            const uint32_t fb = __float_as_uint(b.x[r].fv);
            at_add<true>(&cnt[s], 1u);
            add_window(s, fb, (fb << 1) + win_off, E);
          } else {
            apply<G, true>(&cnt[s], &val[kVal ? s : 0], nullptr, nullptr, (int64_t)b.x[r].iv, b.x[r].fv);
          }
        }
        return false;
      }
      if constexpr (REP == 1) {
        // Somewhere a key is not at home: the second probes, four rows' in flight
        // at once.
#pragma unroll
        for (int q = 0; q < R; q += 4) {
          KT cur2[4];
          uint32_t second[4];
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            second[c] = probe_of(next_probe(key_hash<KD>(b.x[q + c].k)), fw);
            cur2[c] = key[second[c]];
          }
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            __asm__ volatile("" : "+v"(cur2[c]));
            const bool home_hit = cur[q + c] == b.x[q + c].k;
            home[q + c] = home_hit ? home[q + c] : second[c];
            cur[q + c] = home_hit ? cur[q + c] : cur2[c];
          }
        }
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const KT k = b.x[r].k;
        bool mine = full || row_at(r) < left;
        if constexpr (SUB) mine = mine && ((key_hash<KD>(k) >> sub_shift) & sub_mask) == sub;
        const bool hit = cur[r] == k && k != kMark && mine;
        const int s = entry_of(home[r], hot, L);
        bool miss = mine && !hit;
        if constexpr (kDig) {
          const uint32_t fb = __float_as_uint(b.x[r].fv), u = (fb << 1) + win_off;
          const bool in = u < win_span, zero = pass == 0 && b.x[r].fv == 0.0f;
          const bool done = hit && (in || zero);
          if (done) {
            at_add<true>(&cnt[s], 1u);
            if (in) add_window(s, fb, u, E);
          }
          miss = mine && !done && (in || u >= out_from);

        } else {
          if (hit) apply<G, true>(&cnt[s], &val[kVal ? s : 0], nullptr, nullptr, (int64_t)b.x[r].iv, b.x[r].fv);
        }
        rest = rest + rest + (miss ? 1u : 0u);
      }
      bool far_row = false;  // a row of this lane was outside the windows
      while (rest) {
        const int r = R - 1 - __builtin_ctz(rest);
        rest &= rest - 1;
        Row x = b.x[0];
#pragma unroll
        for (int j = 1; j < R; ++j) {  // field by field: a struct would go through scratch memory
          x.k = r == j ? b.x[j].k : x.k;
          x.iv = r == j ? b.x[j].iv : x.iv;
          x.fv = r == j ? b.x[j].fv : x.fv;
        }
        const uint32_t h = key_hash<KD>(x.k), fb = __float_as_uint(x.fv), u = (fb << 1) + win_off;
        const bool nonfinite = (fb << 1) >= 0xFF000000u;
        const bool in = !kDig || u < win_span || x.fv == 0.0f || nonfinite;  // an LDS slot can take it
        const int slot = in ? slot_of(x.k, h, skip, fw) : -1;
        if (slot >= 0) {
          const int s = entry_of((uint32_t)slot, hot, L);
          if constexpr (kDig) {
            at_add<true>(&cnt[s], 1u);
            if (u < win_span) add_window(s, fb, u, E);
            else if (nonfinite)
              at_or<true>(reinterpret_cast<int*>(&flags[slot >> 3]),
                          (__builtin_isnan(x.fv) ? 1 : (x.fv > 0 ? 2 : 4)) << (4 * (slot & 7)));
          } else {
            apply<G, true>(&cnt[s], &val[kVal ? s : 0], nullptr, nullptr, (int64_t)x.iv, x.fv);
          }
        } else {
          spilled = 1;
          if constexpr (kLeaves)
            if (!in && fb << 1 >= 1u << 24) {  // (a subnormal is outside all windows)
              at_add<true>(&far_rows, 1u);
              __hip_atomic_fetch_min((lds_u32*)&far_lo, (fb >> 23) & 0xFFu, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
              __hip_atomic_fetch_max((lds_u32*)&far_hi, (fb >> 23) & 0xFFu, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
              far_row = true;
            }
          const Table t = (kFlex && REP == 1 ? a_ : late_args()).t;
          const int64_t g = global_slot(t, (int64_t)x.k, h);
          if (g >= 0) apply_global<G>(t, g, (int64_t)x.iv, x.fv);
        }
      }
      // (read only by a wave that has just met such a row: it waits for the wave's atomics)
      return kLeaves && fw.single() && __any(far_row) && __builtin_amdgcn_readfirstlane((int)far_count()) != 0;
    };
    int64_t b = first;
    Batch A;
    if (b + TR <= last) {
      bool leaves = false;
      load(A, b);
      if constexpr (kHotLanes != 0 && SUB != 1) {
        uint32_t home[R];
#pragma unroll
        for (int r = 0; r < R; ++r) home[r] = home_of(key_hash<KD>(A.x[r].k), skip, fw);
        hot = find_hot<R>(home);
      }
      for (;;) {
        const int64_t next = b + tile_step;
        const bool more = next + TR <= last;
        Batch B;
        load(B, more ? next : b);  // never behind a branch: the fold would wait for it (the last one is not used)
        const bool leave = fold(A, b, true, 0);
        cold = false;
        b = next;
        leaves = kLeaves && leave;
        if (!more || leaves) break;
        A = B;
      }
      if (leaves) return b;
    }
    if (b < last) {  // the partial tile
      load_tail(A, b, (uint32_t)(last - b));
      fold(A, b, false, (uint32_t)(last - b));
    }
    return last;
  }
  __device__ __forceinline__ bool far_count() const {
    return __hip_atomic_load((const lds_u32*)&far_rows, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >
           (REP > 1 ? kFewFarRows : kFarRows);
  }
  // Rows of the workgroup are left for another table (between barriers).
  // In a scalar register: all that depends on the windows is else kept per lane.
  __device__ __forceinline__ bool left(const FloatWindows& z) const {
    return kLeaves && z.single() && __builtin_amdgcn_readfirstlane((int)far_count()) != 0;
  }

  // Window w of slot e.
  __device__ __forceinline__ int64_t window_of(int e, int w, int E) const {
    uint64_t v = 0;  // the copies' rows are at most kMaxTableRows in all
    for (int r = 0; r < REP; ++r) v += (uint64_t)win[w * E + e * REP + r];
    return (int64_t)v;
  }
  // Slot e's kWindows windows as a whole number of 2^(32 d - 149), d = (win_base - 1) / 32.
  __device__ __forceinline__ __int128 window_total(int e, uint32_t win_base, int E) const {
    __int128 sum = 0;
    for (int w = kWindows - 1; w >= 0; --w) sum = sum * (1 << kWinOctaves) + window_of(e, w, E);
    return sum * ((int64_t)1 << (((int)win_base - 1) & 31));
  }

  // The group of entry e, which holds all of its rows.
  __device__ __forceinline__ agg_group group_of(int e, uint32_t win_base, int32_t is_avg, const FloatWindows& z) const {
    static_assert(REP == 1, "one entry per slot");
    const int L = slots(z), E = entries(z);
    int64_t v = 0, d[kDig ? kDigits : 1] = {};
    int32_t f = 0;
    if constexpr (kVal) v = val[e];
    if constexpr (kDig) {
      f = (int32_t)((flags[e >> 3] >> (4 * (e & 7))) & 7u);
      const __int128 sum = window_total(e, win_base, E);
      const int first = ((int)win_base - 1) >> 5;
#pragma unroll
      for (int k = 0; k < kDigits; ++k) {  // digit 8 takes all there is from it on
        const int i = k - first;
        if (i < 0 || i > 3) continue;
        const __int128 up = sum >> (32 * i);
        d[k] = i == 3 || k == kDigits - 1 ? (int64_t)up : (int64_t)(uint32_t)up;
      }
    }
    return make_group<G>(e < L ? (int64_t)key[e] : (int64_t)kMark, (int64_t)cnt[e], v, d, f, is_avg);
  }

  // Lists the wave's slots with rows, 64 at a time: fn(slot, rank among the
  // wave's listed slots), or slot -1 for a lane with none.
  template <class F>
  __device__ __forceinline__ void each_listed(int off, const FloatWindows& z, F fn) {
    const int L = slots(z);
    const int lane = threadIdx.x & 63;
    volatile uint16_t* mine = list[threadIdx.x / 64];
    uint32_t pending = 0, done = 0;  // the same in all lanes
    for (int i = threadIdx.x; i < L + NT; i += NT) {
      const bool end = i >= L;  // the whole wave's last step
      const int e = (i + off) & (L - 1);
      bool has = false;
      if (!end)
        for (int r = 0; r < REP; ++r) has |= cnt[e * REP + r] != 0;
      const uint64_t used = __ballot(has);
      if (has) mine[pending + __popcll(used & ((1ull << lane) - 1))] = (uint16_t)e;
      pending += (uint32_t)__popcll(used);
      if (pending >= 64 || end) {
        const uint32_t take = min(pending, 64u);
        pending -= take;
        if ((uint32_t)lane < take) fn((int)mine[pending + lane], done + lane);
        done += take;
      }
    }
  }

  // Writes the table's groups straight to the caller's array: for a table that
  // holds all rows of its keys.  One range of the output per table, one
  // contiguous piece per 64 groups.
  __device__ __forceinline__ void emit_all(const Args& a, uint32_t win_base, const FloatWindows& z) {
    const int L = slots(z);
    const int w = threadIdx.x / 64;
    uint32_t mine = 0;
    for (int i = threadIdx.x; i < L; i += NT) mine += (uint32_t)__popcll(__ballot(cnt[i] != 0));
    const bool marker = cnt[L] != 0;
    if ((threadIdx.x & 63) == 0) wave_groups[w] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t total = marker ? 1 : 0;
      for (int v = 0; v < NT / 64; ++v) total += wave_groups[v];
      const unsigned long long at =
          total ? atomicAdd(reinterpret_cast<unsigned long long*>(a.t.state + 2), (unsigned long long)total) : 0;
      emit_base[0] = (uint32_t)at;
      emit_base[1] = (uint32_t)(at >> 32);
    }
    __syncthreads();
    int64_t base = (int64_t)((uint64_t)emit_base[1] << 32 | emit_base[0]);
    if (marker && threadIdx.x == NT - 1 && base < a.max_groups) a.out[base] = group_of(L, win_base, a.is_avg, z);
    base += marker ? 1 : 0;
    for (int v = 0; v < w; ++v) base += wave_groups[v];
    each_listed(0, z, [&](int e, uint32_t rank) {
      if (base + rank < a.max_groups) a.out[base + rank] = group_of(e, win_base, a.is_avg, z);
    });
  }

  // Adds entry e (which has rows) to the global table.
  __device__ __forceinline__ void flush_entry(const Table& t, int e, uint32_t win_base, const FloatWindows& z) {
    const int L = slots(z);
    const KT k = e < L ? key[e] : kMark;
    uint64_t c = 0;
    for (int r = 0; r < REP; ++r) c += cnt[e * REP + r];
    const int64_t g = global_slot(t, (int64_t)k, key_hash<KD>(k));
    if (g < 0) return;
    atomicAdd(reinterpret_cast<unsigned long long*>(t.cnt + g), (unsigned long long)c);
    if constexpr (kVal) {
      int64_t v = val[e * REP];
      for (int r = 1; r < REP; ++r) {
        const int64_t w = val[e * REP + r];
        if constexpr (G == G_SUM_INT) v = (int64_t)((uint64_t)v + (uint64_t)w);
        else if constexpr (G == G_MIN_INT || G == G_MIN_F32) v = w < v ? w : v;
        else v = w > v ? w : v;
      }
      if constexpr (G == G_SUM_INT) atomicAdd(reinterpret_cast<unsigned long long*>(t.val + g), (unsigned long long)v);
      if constexpr (G == G_MIN_INT || G == G_MIN_F32) atomicMin(reinterpret_cast<long long*>(t.val + g), (long long)v);
      if constexpr (G == G_MAX_INT || G == G_MAX_F32) atomicMax(reinterpret_cast<long long*>(t.val + g), (long long)v);
    }
    if constexpr (kDig) {
      const int32_t f = (int32_t)((flags[e >> 3] >> (4 * (e & 7))) & 7u);
      if (f) atomicOr(t.flags + g, f);
      // The windows, whole numbers of 2^(win_base - 150), 2^(win_base - 134), ..., as
      // 32-bit digits from digit (win_base - 1) / 32 on: unsigned ones and a signed
      // top one.  Digit 8 takes all there is from it on (floats end at 2^128,
      // which keeps that below 2^53 over 2^31 rows).
      const int E = entries(z), nw = windows(z);
      unsigned long long* dig = reinterpret_cast<unsigned long long*>(t.dig + g * kDigits);
      __int128 sum = 0;
      int w = 0, shift = ((int)win_base - 1) & 31;
#pragma unroll 1
      for (int d = ((int)win_base - 1) >> 5;; ++d) {
        for (; w < nw && shift < 32; ++w, shift += kWinOctaves) sum += (__int128)window_of(e, w, E) * ((int64_t)1 << shift);
        shift -= 32;
        const bool top = d == kDigits - 1 || (w == nw && sum == (int32_t)sum);
        const int64_t v = top ? (int64_t)sum : (int64_t)(uint32_t)sum;
        if (v) atomicAdd(dig + d, (unsigned long long)v);
        if (top) break;
        sum >>= 32;
      }
    }
  }

  // Adds a float sum's window total to the global slot g.
  static __device__ __forceinline__ void add_digits(const Table& t, int64_t g, __int128 sum, uint32_t win_base) {
    const int d = ((int)win_base - 1) >> 5;
    unsigned long long* dig = reinterpret_cast<unsigned long long*>(t.dig + g * kDigits + d);
    for (int i = 0; i < 4; ++i) {
      const bool top = i == 3 || d + i == kDigits - 1;
      const int64_t v = top ? (int64_t)(sum >> (32 * i)) : (int64_t)(uint32_t)(sum >> (32 * i));
      if (v) atomicAdd(dig + i, (unsigned long long)v);
      if (top) break;
    }
  }

  // ---- merged tables: records of key, rows and value, by section of the hash ----
  static constexpr int kKeyWords = KD == AGG_I32 ? 1 : 2;
  static constexpr int kRecWords = dump_words_of(G, KD);

  // Writes the table to its region: the sections' starts, then the records by
  // section (a counting sort).  False, with nothing written but the empty
  // sections, if the region is too small: more keys than the plan allows.
  __device__ __forceinline__ bool dump(uint32_t* region, int most, const FloatWindows& z) {
    static_assert(sizeof(list) >= 2 * kSections * 4, "the counters lie over the list");
    uint32_t* count = reinterpret_cast<uint32_t*>(&list[0][0]);
    if (threadIdx.x <= kSections) count[threadIdx.x] = 0;
    __syncthreads();
    const int L = slots(z), E = entries(z);
    auto section_of = [&](int e) { return key_hash<KD>(e < L ? key[e] : kMark) >> (32 - kSectionBits); };
    for (int e = threadIdx.x; e <= L; e += NT)
      if (cnt[e] != 0) at_add<true>(&count[section_of(e)], 1u);
    __syncthreads();
    if (threadIdx.x < 64) {  // exclusive prefix, two sections a lane
      const uint32_t c0 = count[2 * threadIdx.x], c1 = count[2 * threadIdx.x + 1];
      uint32_t incl = c0 + c1;
      for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off, 64);
        if ((int)threadIdx.x >= off) incl += y;
      }
      count[2 * threadIdx.x] = incl - c0 - c1;
      count[2 * threadIdx.x + 1] = incl - c1;
      if (threadIdx.x == 63) count[kSections] = incl;
    }
    __syncthreads();
    const bool fits = (int64_t)count[kSections] <= most;
    if (threadIdx.x <= kSections) region[threadIdx.x] = fits ? count[threadIdx.x] : 0;
    __syncthreads();
    if (!fits) return false;
    for (int e = threadIdx.x; e <= L; e += NT) {
      if (cnt[e] == 0) continue;
      const KT k = e < L ? key[e] : kMark;
      uint32_t* r = region + kSections + 1 + (int64_t)at_fetch_add(&count[section_of(e)], 1u) * kRecWords;
      r[0] = (uint32_t)k;
      if constexpr (kKeyWords == 2) r[1] = (uint32_t)((uint64_t)k >> 32);
      r[kKeyWords] = cnt[e];
      if constexpr (kVal) put64(r + kKeyWords + 1, val[e]);
      if constexpr (kDig) {
        for (int w = 0; w < kWindows; ++w) put64(r + kKeyWords + 1 + 2 * w, win[w * E + e]);
        r[kKeyWords + 1 + 2 * kWindows] = (flags[e >> 3] >> (4 * (e & 7))) & 7u;
      }
    }
    return true;
  }
  static __device__ __forceinline__ void put64(uint32_t* p, int64_t v) {
    p[0] = (uint32_t)v;
    p[1] = (uint32_t)((uint64_t)v >> 32);
  }
  static __device__ __forceinline__ int64_t get64(const uint32_t* p) { return (int64_t)((uint64_t)p[1] << 32 | p[0]); }
  static __device__ __forceinline__ uint32_t at_fetch_add(uint32_t* p, uint32_t v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }

  // The merge's: adds a record, to the global table if its key finds no slot (as
  // any other record of the key then does too).
  __device__ __forceinline__ void add_record(const Table& t, const uint32_t* r, uint32_t skip, uint32_t win_base) {
    const KT k = kKeyWords == 2 ? (KT)get64(r) : (KT)(int32_t)r[0];
    const uint32_t rows = r[kKeyWords], h = key_hash<KD>(k);
    const uint32_t* x = r + kKeyWords + 1;
    const FloatWindows z;
    const int E = entries(z), s = slot_of(k, h, skip, z);
    if (s >= 0) {
      at_add<true>(&cnt[s], rows);
      if constexpr (G == G_SUM_INT)
        at_add<true>(reinterpret_cast<unsigned long long*>(&val[s]), (unsigned long long)get64(x));
      else if constexpr (G == G_MIN_INT || G == G_MIN_F32)
        atomicMin(reinterpret_cast<long long*>(&val[s]), (long long)get64(x));
      else if constexpr (kVal)
        atomicMax(reinterpret_cast<long long*>(&val[s]), (long long)get64(x));
      if constexpr (kDig) {
        for (int w = 0; w < kWindows; ++w)
          at_add<true>(reinterpret_cast<unsigned long long*>(&win[w * E + s]), (unsigned long long)get64(x + 2 * w));
        const uint32_t f = x[2 * kWindows];
        if (f) at_or<true>(reinterpret_cast<int*>(&flags[s >> 3]), (int)(f << (4 * (s & 7))));
      }
      return;
    }
    mark_global(t, 7);
    const int64_t g = global_slot(t, (int64_t)k, h);
    if (g < 0) return;
    atomicAdd(reinterpret_cast<unsigned long long*>(t.cnt + g), (unsigned long long)rows);
    if constexpr (G == G_SUM_INT)
      atomicAdd(reinterpret_cast<unsigned long long*>(t.val + g), (unsigned long long)get64(x));
    else if constexpr (G == G_MIN_INT || G == G_MIN_F32)
      atomicMin(reinterpret_cast<long long*>(t.val + g), (long long)get64(x));
    else if constexpr (kVal) atomicMax(reinterpret_cast<long long*>(t.val + g), (long long)get64(x));
    if constexpr (kDig) {
      __int128 sum = 0;
      for (int w = kWindows - 1; w >= 0; --w) sum = sum * (1 << kWinOctaves) + get64(x + 2 * w);
      add_digits(t, g, sum * ((int64_t)1 << (((int)win_base - 1) & 31)), win_base);
      if (x[2 * kWindows]) atomicOr(t.flags + g, (int32_t)x[2 * kWindows]);
    }
  }
  // Merged runs: the global table holds rows, so the merge's last workgroup emits
  // it too.  The fold and the merge have a mark each (state[word]): what a merge
  // workgroup does must not hang on when it looks, so it goes by the fold's mark,
  // which is final before the merge starts.
  static __device__ __forceinline__ void mark_global(const Table& t, int word) {
    __hip_atomic_store(&t.state[word], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }

  // A slot's flush is a chain of device-scope accesses (read the global home,
  // claim it, add: 2 us), so a wave first lists its slots with rows, and flushes
  // 64 listed ones at a time: a table of few keys takes one such chain per wave
  // instead of one for every 64 slots.  1e5 rows, int32 keys: COUNT of 2000
  // groups 55.6 -> 31.5 us, of 50 000 159 -> 85, int32 SUM 122 -> 80.
  // Not where many workgroups have the same keys (direct path): more of them
  // would claim a key at the same moment (6M rows, 2000 groups, 256 workgroups:
  // COUNT 56.5 -> 72.4 us; 31 workgroups 54.9 -> 34.6).
  __device__ __forceinline__ void flush(const Table& t, uint32_t win_base, bool listed, const FloatWindows& z) {
    const int L = slots(z);
    // Every workgroup's table holds its keys in about the same slots (same
    // hash), so flushing all tables in slot order would have every workgroup
    // update the same global slots at the same moment, and device-scope
    // atomics on one address serialise.  Each workgroup starts its pass at
    // its own offset instead (2^28 rows, 1024 groups: COUNT 0.43 -> 0.39 ms;
    // the other cases within noise).
    const int off = (int)(blockIdx.x * 2654435761u >> 16);
    if (listed) {
      each_listed(off & (L - 1), z, [&](int e, uint32_t) { flush_entry(t, e, win_base, z); });
    } else {
      for (int i = threadIdx.x; i < L; i += NT) {
        const int e = (i + off) & (L - 1);
        uint32_t c = 0;
        for (int r = 0; r < REP; ++r) c |= cnt[e * REP + r];
        if (c != 0) flush_entry(t, e, win_base, z);
      }
    }
    if (threadIdx.x == NT - 1) {  // slot L
      uint32_t c = 0;
      for (int r = 0; r < REP; ++r) c |= cnt[L * REP + r];
      if (c != 0) flush_entry(t, L, win_base, z);
    }
  }
};

// Few groups (at most kFewGroups): with a full-size table a wave's 64 rows
// fall on about as many slots as there are groups, and the LDS atomics of
// lanes that meet on a slot serialise (measured on MI355X: a 64-bit add from a
// wave whose rows spread over 16 slots takes about 24 clocks, over 64
// addresses 6).  A small table whose slots carry kFewCopies copies of the
// accumulators (lane l updates copy l % kFewCopies) cuts the meetings by that
// factor, and is cleared and flushed in one step.  2^28 rows, int32 keys,
// full table -> this one: int64 SUM 1056 -> 478 us at 2 groups, 499 -> 478 at
// 16; COUNT 545 -> 163 and 210 -> 163; float SUM 1580 -> 348 and 620 -> 343.
// 256 slots: of 32 random keys in 128, four meet at home and one at its second
// slot too (512 cost small calls another 0.3 us to clear and flush).
constexpr int kFewGroups = 32;
constexpr int kFewCopies = 8;
constexpr int kFewSlots = 256;

// The tables for the exponents emin..emax and `groups` keys a table (FEW: the few-groups
// table).  Slots enough for the keys at up to 5/8 of them, else passes by the keys'
// hash.  MANY (partitions, and the direct path's two passes): or, if those are not
// more, passes by exponent of the full-size table, whose rows need no other test (10^6
// rows and groups, 60 exponents 236 us, by hash 276; with fewer groups the flushes
// cost more than the test: 10^6 rows, 2000 groups 118 us by exponent, 93 by hash).
template <int KD, bool FEW, bool MANY>
__device__ __forceinline__ FloatWindows place_windows(int emin, int emax, int64_t groups, int moves = 0) {
  const int n = emax - emin + 1;
  FloatWindows f;
  const int least = (n + kWinOctaves - 1) / kWinOctaves, mid = mid_windows_of(KD);
  if (FEW) {
    f.nw = least <= kWindows ? kWindows : kFewWindows;
  } else if (least > kWindows) {
    f.nw = least <= mid ? mid : 2 * mid;
    f.lg = __builtin_ctz(least <= mid ? kMidSlots : kAllSlots);
    while (groups >> f.sub_bits > (5 << f.lg) / 8) ++f.sub_bits;
    if (MANY && f.sub_bits && (least + kWindows - 1) / kWindows <= (least + f.nw - 1) / f.nw << f.sub_bits) {
      f.nw = kWindows;
      f.sub_bits = 0;
    }
  }
  const int span = f.nw * kWinOctaves;
  f.passes = (n + span - 1) / span;
  f.first = std::max(1, emax + std::min((f.passes * span - n) / 2, 8) - f.passes * span + 1);
  f.lo = emin;
  f.hi = emax;
  f.moves = moves;
  return f;
}
// The tables for the rows that a table of `fw` left.  (Scalars: see left().)
template <int KD, bool FEW, bool MANY, class Tab>
__device__ __forceinline__ FloatWindows move_windows(const Tab& tab, const FloatWindows& fw, int64_t groups) {
  const int lo = __builtin_amdgcn_readfirstlane((int)tab.far_lo), hi = __builtin_amdgcn_readfirstlane((int)tab.far_hi);
  return fw.moves ? place_windows<KD, FEW, MANY>(1, 254, groups, fw.moves + 1)
                  : place_windows<KD, FEW, MANY>(std::min(fw.lo, lo), std::max(fw.hi, hi), groups, 1);
}

// Where a launch's float-sum windows go, from one row of each of blockDim.x equal
// parts of the launch's n rows (word `at` of every `stride`): the sampled
// exponents, with most of the slack below them (sums of small parts) and up to
// 2^8 of room above.  The row's place in its part differs from part to part, so that
// no period of the column's shows it one kind of row only.  Every workgroup reads
// the same rows and gets the same answer.  (1024 rows:
// a sample is bound by page-table misses, 4096 rows took 13 to 20 us at 2^28;
// reduced by shuffles, 2 us: LDS min / max of one address by every lane took 8.)
template <int KD, bool FEW, bool MANY>
__device__ __forceinline__ FloatWindows sample_windows(const uint32_t* words, int stride, int at, int64_t n, int64_t groups) {
  __shared__ int range[2][16];
  const int64_t part = (int64_t)((uint64_t)n * threadIdx.x / blockDim.x);
  const uint32_t size = (uint32_t)((uint64_t)n / blockDim.x);  // n <= 2^31
  const int64_t row = part + (int64_t)__umulhi(next_probe(threadIdx.x), size);
  const int e = (int)((words[row * stride + at] >> 23) & 0xFFu);
  const bool placed = e != 0 && e != 255;  // zeros, subnormals and non-finite rows do not place a window
  int emin = placed ? e : 255, emax = placed ? e : 0;
  for (int off = 32; off >= 1; off >>= 1) {
    emin = std::min(emin, __shfl_xor(emin, off, 64));
    emax = std::max(emax, __shfl_xor(emax, off, 64));
  }
  if ((threadIdx.x & 63) == 0) {
    range[0][threadIdx.x / 64] = emin;
    range[1][threadIdx.x / 64] = emax;
  }
  __syncthreads();
  for (int w = 0; w < (int)blockDim.x / 64; ++w) {
    emin = std::min(emin, range[0][w]);
    emax = std::max(emax, range[1][w]);
  }
  // every wave has the same two numbers: in scalar registers from here on
  emin = __builtin_amdgcn_readfirstlane(emin);
  emax = __builtin_amdgcn_readfirstlane(emax);
  FloatWindows f = emin > emax ? place_windows<KD, FEW, MANY>(127, 127, groups) : place_windows<KD, FEW, MANY>(emin, emax, groups);
  f.lo = emin;  // none sampled: as such
  f.hi = emax;
  return f;
}

// An aggregation kernel's tables, in the same LDS: one of full size, and for a
// float sum those of fewer slots and more windows (the table of few groups is both:
// its windows' number is all that changes).  The full-size one's shape is known to
// the compiler, so that columns of few exponents pay nothing for the others (with
// one table for all, 2^28 rows, 300 groups 376 -> 433 us).
template <int KD>
constexpr int flex_words() { return 2 * mid_windows_of(KD) * (kAllSlots + 1); }
template <int G, int KD, bool FEW, bool HOT>
union AggTables {
  static_assert(mid_windows_of(KD) * (kMidSlots + 1) <= flex_words<KD>(), "the other shape needs no more");
  LdsTable<G, KD, FEW ? kFewSlots : lds_slots<G, KD>(), kDirectThreads, FEW ? kFewCopies : 1, HOT,
           FEW && G == G_SUM_F32 ? kFewWindows*(kFewSlots + 1) * kFewCopies : 0> full;
  LdsTable<G, KD, kMidSlots, kDirectThreads, 1, false, G == G_SUM_F32 && !FEW ? flex_words<KD>() : 0> flex;
};

// ---- emission: the global table's groups to the caller's array ----

template <bool COHERENT, typename T>
__device__ __forceinline__ T table_load(const T* p) {  // COHERENT: written by this launch's other workgroups
  return load_partial<COHERENT>(p);
}

// Writes the used slots of [lo, hi) as groups and clears them (and so leaves
// the table as the next call needs it: no launch clears it first).  A workgroup
// takes kEmitPer x NT slots at a time, the keys in registers; it counts the used
// ones, takes one output range with a single atomic (updates of one address
// serialise), and writes each group at its slot's rank, so that a wave's
// groups leave as one contiguous piece.
constexpr int kEmitPer = 4;  // slots per thread at a time
template <int G, bool COHERENT, int NT>
__device__ __forceinline__ void emit_slots(const Args& a, int64_t lo, int64_t hi) {
  constexpr int NW = NT / 64, CELLS = kEmitPer * NW;
  static_assert(CELLS <= 64, "one wave scans the counts");
  __shared__ uint32_t cell[CELLS];
  __shared__ unsigned long long base_sh;
  const Table& t = a.t;
  const int lane = threadIdx.x & 63, w = threadIdx.x / 64;
  for (int64_t c0 = lo; c0 < hi; c0 += kEmitPer * NT) {
    int64_t key[kEmitPer];
    uint64_t cnt[kEmitPer];
    uint32_t before[kEmitPer];
#pragma unroll
    for (int i = 0; i < kEmitPer; ++i) {
      const int64_t s = c0 + i * NT + threadIdx.x;
      key[i] = s < hi && s < t.cap ? table_load<COHERENT>(t.key + s) : kEmpty;
      // the extra slot's key marks an empty one: its rows tell
      cnt[i] = s < hi && s == t.cap ? table_load<COHERENT>(t.cnt + s) : 0;
    }
#pragma unroll
    for (int i = 0; i < kEmitPer; ++i) {
      const uint64_t m = __ballot(key[i] != kEmpty || cnt[i] != 0);
      before[i] = (uint32_t)__popcll(m & ((1ull << lane) - 1));
      if (lane == 0) cell[i * NW + w] = (uint32_t)__popcll(m);
    }
    __syncthreads();
    if (threadIdx.x < 64) {
      const uint32_t c = lane < CELLS ? cell[lane] : 0;
      uint32_t incl = c;
      for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
      }
      if (lane < CELLS) cell[lane] = incl - c;
      if (lane == 63)
        base_sh = incl ? atomicAdd(reinterpret_cast<unsigned long long*>(t.state + 2), (unsigned long long)incl) : 0;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kEmitPer; ++i) {
      const int64_t s = c0 + i * NT + threadIdx.x;
      if (key[i] == kEmpty && cnt[i] == 0) continue;
      const unsigned long long my = base_sh + cell[i * NW + w] + before[i];
      int64_t v = 0, d[G == G_SUM_F32 ? kDigits : 1] = {};
      int32_t f = 0;
      if constexpr (G == G_SUM_F32) {
#pragma unroll
        for (int k = 0; k < kDigits; ++k) d[k] = table_load<COHERENT>(t.dig + s * kDigits + k);
        f = table_load<COHERENT>(t.flags + s);
      } else if constexpr (G != G_COUNT) {
        v = table_load<COHERENT>(t.val + s);
      }
      const agg_group g = make_group<G>(key[i], (int64_t)table_load<COHERENT>(t.cnt + s), v, d, f, a.is_avg);
      clear_slot<G>(t, s);
      if ((int64_t)my < a.max_groups) a.out[my] = g;
    }
    __syncthreads();  // cell and base_sh are free again
  }
}

// By the last workgroup to emit, once its groups are written: the number of
// groups, and a clean state for the next call.
__device__ __forceinline__ void finish_emission(const Args& a) {
  if (threadIdx.x != 0) return;
  unsigned long long* emitted = reinterpret_cast<unsigned long long*>(a.t.state + 2);
  const unsigned long long e = __hip_atomic_load(emitted, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int32_t over = __hip_atomic_load(&a.t.state[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  *a.ngroups = (over || (int64_t)e > a.max_groups) ? -1 : (int64_t)e;
  __hip_atomic_store(emitted, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(&a.t.state[0], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(&a.t.state[4], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Folds a workgroup's rows from `from` on (each wave its own) of the plan's pass
// `sub` into tables of more windows.  A function of its own, so that its registers
// are not the fold's of the full-size table (within the kernels: 41 registers
// spilled instead of 7, 2^28 rows, 300 groups 353 -> 373 us, 1e5 rows 22 -> 25; as it
// is 353 -> 368 and 22 -> 23).  A function's arguments come in vector registers;
// these are the same in all lanes.
typedef __attribute__((address_space(3))) char lds_char;
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uniform(int64_t v) {
  return (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32 |
                   (uint32_t)__builtin_amdgcn_readfirstlane((int)v));
}
template <int VD, bool ROWS, class Tab>
__device__ __attribute__((noinline)) void fold_flex(lds_char* space, const Args* ap, int first, int passes, int nw, int lg,
                                                    int fsub, int64_t from, int64_t last, int64_t step,
                                                    int sub) {
  Tab& tab = *(Tab*)space;
  typedef __attribute__((address_space(4))) const Args kernarg;
  const Args& a = *(const Args*)(kernarg*)uniform((int64_t)ap);  // the kernel's own, scalar loads
  FloatWindows fw;
  fw.first = uniform(first);
  fw.passes = uniform(passes);
  fw.nw = uniform(nw);
  fw.lg = uniform(lg);
  fw.sub_bits = uniform(fsub);
  from = uniform(from);
  last = uniform(last);
  step = uniform(step);
  sub = uniform(sub);
  const int bits = ROWS ? a.pt.bits : 0, sub_bits = a.pt.sub_bits;
  const void* keys = ROWS ? a.pt.pk : a.keys;
  const void* vals = ROWS ? a.pt.pv : a.vals;
  const int pass_bits = sub_bits + fw.sub_bits;
#pragma unroll 1
  for (uint32_t i = 0; i < (uint32_t)fw.passes << fw.sub_bits; ++i) {
    const int pass = (int)(i >> fw.sub_bits);
    tab.clear((uint32_t)(bits + pass_bits), fw);
    __syncthreads();
    tab.template fold_rows<VD, ROWS, 2>(a, keys, vals, from, last, step, (uint32_t)(bits + pass_bits),
                                        pass_bits ? (uint32_t)(32 - bits - pass_bits) : 0u, (1u << pass_bits) - 1u,
                                        (uint32_t)sub << fw.sub_bits | (i & ((1u << fw.sub_bits) - 1u)), fw, pass);
    __syncthreads();
    tab.flush(a.t, fw.base(pass), ROWS || gridDim.x <= 64, fw);
    __syncthreads();
  }
}

// Direct path: every workgroup sweeps its share of the rows' tiles into one
// LDS table, in 2^sub_bits passes (each taking the keys of one sub-partition:
// the top bits of the key's hash) when the groups need more than one table.
// Bound by HBM where a row is 12 bytes or more: 2^28 rows, int32 keys, 1024
// dense keys: int64 SUM 563 -> 490 us (6.5 TB/s), COUNT 367 -> 177 (6.0),
// float SUM 923 -> 380 (5.7); the loads alone run at 6.6 TB/s.
// Two workgroups per CU, which the few-groups table would leave room for, ran
// slower: half the registers are half the rows in flight per thread (16
// groups: COUNT 177 us against 161, float SUM 367 against 345).
template <int KD, int VD, int G, bool FEW, bool SUB>
__global__ void __launch_bounds__(kDirectThreads)
gb_aggregate_kernel(Args a) {
  __shared__ AggTables<G, KD, FEW, false> tables;
  auto& tab = tables.full;
  constexpr int TR = decltype(tables.full)::template tile_rows_of<VD>() * kDirectThreads;
  const int64_t step = (int64_t)gridDim.x * TR;
  const uint32_t sub_mask = (1u << a.pt.sub_bits) - 1u;
  const uint32_t sub_shift = a.pt.sub_bits ? (uint32_t)(32 - a.pt.sub_bits) : 0u;
  FloatWindows fw;
  if constexpr (G == G_SUM_F32) {
    fw = sample_windows<KD, FEW, SUB>(static_cast<const uint32_t*>(a.vals), 1, 0, a.n, a.max_groups >> a.pt.sub_bits);
    // (-1: no workgroup writes its table out)
    if (a.dumps && blockIdx.x == 0 && threadIdx.x == 0) a.t.state[6] = fw.single() ? (int32_t)fw.base(0) : -1;
  }
  for (uint32_t sub = 0; sub <= sub_mask; ++sub) {
    int64_t from = (int64_t)blockIdx.x * TR;
    bool dumped = false, global = !fw.narrow();  // the table was written out; rows are in the global table
    for (int pass = 0; pass < (FEW || fw.narrow() ? fw.passes : 0); ++pass) {
      tab.clear((uint32_t)a.pt.sub_bits, fw);
      __syncthreads();
      const int64_t next = tab.template fold_rows<VD, false, SUB>(a, a.keys, a.vals, from, a.n, step, (uint32_t)a.pt.sub_bits,
                                                                  sub_shift, sub_mask, sub, fw, pass);
      __syncthreads();
      const bool left = tab.left(fw);
      const Args& b = late_args();
      if constexpr (!FEW)
        if (b.dumps && !left && fw.single() && !fw.moves)  // its region; its rows may be in the global table as well (spilled)
          dumped = tab.dump(b.dump + ((int64_t)blockIdx.x * (sub_mask + 1) + sub) * dump_region_of(G, KD, b.dump_max),
                            b.dump_max, fw);
      global = !dumped || tab.spilled;
      if (!dumped) tab.flush(b.t, fw.base(pass), gridDim.x <= 64, fw);
      if constexpr (G == G_SUM_F32)
        if (left) {  // (before the barrier: the next table is cleared after it)
          fw = move_windows<KD, FEW, SUB>(tab, fw, a.max_groups >> a.pt.sub_bits);
          from = next;
          pass = -1;
        }
      __syncthreads();
    }
    if constexpr (!FEW) {
      const Args& b = late_args();
      if (b.dumps) {  // one region per workgroup and hash half
        uint32_t* region = b.dump + ((int64_t)blockIdx.x * (sub_mask + 1) + sub) * dump_region_of(G, KD, b.dump_max);
        if (!dumped && threadIdx.x <= kSections) region[threadIdx.x] = 0;
        if (threadIdx.x == 0 && global) decltype(tables.full)::mark_global(b.t, 5);
      }
      if constexpr (G == G_SUM_F32)
        if (!fw.narrow())
          fold_flex<VD, false, decltype(tables.flex)>((lds_char*)&tables, &b, fw.first, fw.passes, fw.nw, fw.lg, fw.sub_bits, from, b.n, step, (int)sub);
    }
  }
  const Args& b = late_args();
  if (b.emit && last_to_finish(reinterpret_cast<uint32_t*>(b.t.state + 4))) {
    emit_slots<G, true, kDirectThreads>(b, 0, b.t.cap + 1);
    finish_emission(b);
  }
}

// Partitioned path: workgroup w takes the w-th equal share of the staged rows
// and folds it partition by partition, flushing its LDS table at each
// partition boundary (a partition's keys fit one table; the next partition's
// keys are all different).  Equal shares keep every workgroup equally busy
// whatever the partition sizes.  Where a partition holds more keys than one
// table (more partitions than the scatter takes), its rows are folded in
// several passes, each taking the rows of one sub-partition (the next bits of
// the key's hash) and flushing the table after it.
template <int KD, int VD, int G, bool SUB>
__global__ void __launch_bounds__(kPartThreads) gb_aggregate_part_kernel(Args a) {
  static_assert(kPartThreads == kDirectThreads, "one AggTable");
  __shared__ AggTables<G, KD, false, !SUB> tables;
  auto& tab = tables.full;
  constexpr int TR = decltype(tables.full)::template tile_rows_of<VD>() * kPartThreads;
  const int64_t groups = a.max_groups >> (a.pt.bits + a.pt.sub_bits);  // keys of a table
  FloatWindows fw;
  if constexpr (G == G_SUM_F32) {
    using SR = StagedRow<KD, AGG_F32>;
    fw = sample_windows<KD, false, true>(static_cast<const uint32_t*>(a.pt.pk), SR::KW + SR::VW, SR::KW, a.n, groups);
  }
  const int P = 1 << a.pt.bits;
  // The workgroup's rows: an equal share.  Where there are as many partitions as
  // workgroups, each end is moved to the nearest partition start within a quarter
  // of a share: the partitions between are wholly this workgroup's, and their
  // groups need no global table.  (2^20 groups, 256 partitions and more: COUNT
  // of 6M rows 181 -> 85 us, of 2^28 rows 1425 -> 1157; float SUM of 6M rows 362
  // -> 144.  With fewer partitions it gains nothing and makes the shares
  // uneven: 2^28 rows, 50 000 groups, COUNT 951 -> 984.)
  uint32_t* start = tab.cnt;  // the partition starts, until the table is cleared
  for (int i = threadIdx.x; i <= P; i += kPartThreads) start[i] = a.pt.start[i];
  __syncthreads();
  int p = 0;  // the last partition that starts at or before the row last asked for
  auto snap = [&](int64_t row) -> int64_t {
    int lo = 0, hi = P;
    while (lo < hi) {
      const int mid = (lo + hi + 1) / 2;
      if ((int64_t)start[mid] <= row) lo = mid;
      else hi = mid - 1;
    }
    p = lo;
    const int64_t down = row - (int64_t)start[lo], up = lo < P ? (int64_t)start[lo + 1] - row : down;
    const int64_t most = P >= (int)gridDim.x ? a.n / gridDim.x / 4 : 0;
    return down <= up ? (down <= most ? row - down : row) : (up <= most ? row + up : row);
  };
  const int64_t r1 = snap(a.n * ((int64_t)blockIdx.x + 1) / gridDim.x);
  int64_t r = snap(a.n * (int64_t)blockIdx.x / gridDim.x);
  __syncthreads();
  if (r >= r1) return;  // the whole workgroup leaves together
  const uint32_t sub_mask = (1u << a.pt.sub_bits) - 1u;
  const uint32_t sub_shift = a.pt.sub_bits ? (uint32_t)(32 - a.pt.bits - a.pt.sub_bits) : 0u;
  while (r < r1) {
    while ((int64_t)a.pt.start[p + 1] <= r) ++p;  // skip partitions that end before r
    const int64_t seg_end = std::min<int64_t>(r1, (int64_t)a.pt.start[p + 1]);
    // the workgroup has all rows of the partition's keys
    const bool whole = a.whole && r == (int64_t)a.pt.start[p] && seg_end == (int64_t)a.pt.start[p + 1];
    for (uint32_t sub = 0; sub <= sub_mask; ++sub) {
      int64_t from = r;
      bool flushed = false;  // rows of these keys are in the global table already
      for (int pass = 0; pass < (fw.narrow() ? fw.passes : 0); ++pass) {
        tab.clear((uint32_t)(a.pt.bits + a.pt.sub_bits), fw);
        __syncthreads();
        const int64_t next = tab.template fold_rows<VD, true, SUB>(a, a.pt.pk, a.pt.pv, from, seg_end, TR,
                                                                   (uint32_t)(a.pt.bits + a.pt.sub_bits), sub_shift,
                                                                   sub_mask, sub, fw, pass);
        __syncthreads();
        const bool left = tab.left(fw);
        tab.merge_hot(fw);
        if (whole && fw.single() && tab.spilled == 0 && !flushed) tab.emit_all(late_args(), fw.base(0), fw);
        else tab.flush(late_args().t, fw.base(pass), true, fw);
        if constexpr (G == G_SUM_F32)
          if (left) {  // (before the barrier: the next table is cleared after it)
            fw = move_windows<KD, false, true>(tab, fw, groups);
            flushed = true;
            from = next;
            pass = -1;
          }
        __syncthreads();
      }
      if constexpr (G == G_SUM_F32)
        if (!fw.narrow())
          fold_flex<VD, true, decltype(tables.flex)>((lds_char*)&tables, &late_args(), fw.first, fw.passes, fw.nw, fw.lg, fw.sub_bits, from, seg_end, TR, (int)sub);
    }
    r = seg_end;
  }
}

// Merges the direct path's tables: workgroup s adds the records of section s of
// every region in an LDS table and writes its groups.  If the fold left rows in
// the global table too, the tables go there instead.  A key that finds no slot
// here (a section holds far more than its share of the keys) is in no table here,
// so its records go to the global table and the others' groups leave as usual.
// The last workgroup emits what the global table holds.
template <int KD, int G>
__global__ void __launch_bounds__(kDirectThreads) gb_merge_kernel(Args a) {
  __shared__ LdsTable<G, KD, kMergeSlots, kDirectThreads> tab;
  __shared__ uint32_t first[kMergeMaxWg], upto[kMergeMaxWg];  // a region's records of the section; their running total
  __shared__ uint32_t wave_sum[kDirectThreads / 64];
  if constexpr (G == G_SUM_F32)
    if (a.t.state[6] < 0) {  // tables of more windows, all flushed: the launch emits the global table
      const int64_t slots = a.t.cap + 1, per = ceil_div_dev(slots, gridDim.x);
      emit_slots<G, false, kDirectThreads>(a, blockIdx.x * per, std::min<int64_t>((blockIdx.x + 1) * per, slots));
      if (!last_to_finish(reinterpret_cast<uint32_t*>(a.t.state + 4))) return;
      if (threadIdx.x == 0) __hip_atomic_store(&a.t.state[5], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      finish_emission(a);
      return;
    }
  const FloatWindows fw;  // (the merge's table has kWindows)
  const uint32_t section = blockIdx.x;
  const uint32_t subs = 1u << a.pt.sub_bits, sub = section >> (kSectionBits - a.pt.sub_bits);
  const int64_t region = dump_region_of(G, KD, a.dump_max);
  const int tid = threadIdx.x, lane = tid & 63, w = tid / 64;
  const uint32_t* mine = a.dump + ((int64_t)tid * subs + sub) * region;
  uint32_t n = 0;
  if (tid < a.dumps) {
    first[tid] = mine[section];
    n = mine[section + 1] - first[tid];
  }
  tab.clear((uint32_t)kSectionBits, fw);
  uint32_t incl = n;
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(incl, off, 64);
    if (lane >= off) incl += y;
  }
  if (lane == 63) wave_sum[w] = incl;
  __syncthreads();
  for (int v = 0; v < w; ++v) incl += wave_sum[v];
  upto[tid] = incl;
  __syncthreads();
  const uint32_t total = upto[kDirectThreads - 1];
  const uint32_t win_base = G == G_SUM_F32 ? (uint32_t)a.t.state[6] : 0u;
  // the same in every wave and workgroup: nothing writes this word before the last workgroup below
  const bool global = __hip_atomic_load(&a.t.state[5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
  for (uint32_t i = tid; i < total; i += kDirectThreads) {
    int lo = 0, hi = a.dumps - 1;  // the first region that ends after record i
    while (lo < hi) {
      const int mid = (lo + hi) / 2;
      if (upto[mid] > i) hi = mid;
      else lo = mid + 1;
    }
    const uint32_t at = first[lo] + i - (lo ? upto[lo - 1] : 0u);
    const uint32_t* records = a.dump + ((int64_t)lo * subs + sub) * region + kSections + 1;
    const uint32_t* r = records + (int64_t)at * decltype(tab)::kRecWords;
    tab.add_record(a.t, r, (uint32_t)kSectionBits, win_base);
  }
  __syncthreads();
  if (global) tab.flush(a.t, win_base, true, fw);
  else tab.emit_all(a, win_base, fw);
  if (!last_to_finish(reinterpret_cast<uint32_t*>(a.t.state + 4))) return;
  if (global || __hip_atomic_load(&a.t.state[7], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)
    emit_slots<G, true, kDirectThreads>(a, 0, a.t.cap + 1);
  __syncthreads();  // every wave has read the marks
  if (tid == 0) {
    __hip_atomic_store(&a.t.state[5], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&a.t.state[7], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  finish_emission(a);
}

// Clears the whole table: once, before a plan's first call.
template <int G>
__global__ void __launch_bounds__(kThreads) gb_init_kernel(Args a) {
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  for (int64_t s = (int64_t)blockIdx.x * kThreads + threadIdx.x; s <= a.t.cap; s += stride) {
    clear_slot<G>(a.t, s);
    a.t.flags[s] = 0;
  }
  if (blockIdx.x == 0 && threadIdx.x < 8) a.t.state[threadIdx.x] = 0;
}

// Each workgroup emits a contiguous slot range; the last one to finish writes
// the number of groups.
constexpr int kEmitThreads = 1024;
template <int G>
__global__ void __launch_bounds__(kEmitThreads) gb_emit_kernel(Args a) {
  const int64_t slots = a.t.cap + 1;
  const int64_t per = ceil_div_dev(slots, gridDim.x);
  const int64_t lo = (int64_t)blockIdx.x * per;
  emit_slots<G, false, kEmitThreads>(a, lo, std::min<int64_t>(lo + per, slots));
  if (last_to_finish(reinterpret_cast<uint32_t*>(a.t.state + 4))) finish_emission(a);
}

// ---- kernel tables ----

int gop_of(int32_t val_dtype, int32_t op) {
  if (op == AGG_COUNT) return G_COUNT;
  const bool f = val_dtype == AGG_F32;
  if (op == AGG_SUM || op == AGG_AVG) return f ? G_SUM_F32 : G_SUM_INT;
  if (op == AGG_MIN) return f ? G_MIN_F32 : G_MIN_INT;
  if (op == AGG_MAX) return f ? G_MAX_F32 : G_MAX_INT;
  return -1;
}

// PATH: 0 direct, 1 partitioned, 2 direct with few groups (accumulator copies),
// 3 direct in sub-partition passes (no COUNT and no float SUM: they partition instead), 4
// partitioned in sub-partition passes.  Plans without passes take kernels whose fold has no
// per-row pass test.
template <int KD, int VD, int PATH>
const void* agg_row(int g) {
#define GB_AGG(GG)                                                                                        \
  (PATH == 1 || PATH == 4                                                                                 \
       ? reinterpret_cast<const void*>(&gb_aggregate_part_kernel<KD, VD, GG, PATH == 4>)                  \
       : reinterpret_cast<const void*>(&gb_aggregate_kernel<KD, VD, GG, PATH == 2, PATH == 3>))
  if constexpr (VD == AGG_F32) {
    if constexpr (PATH != 3 || KD == AGG_I64)
      if (g == G_SUM_F32) return GB_AGG(G_SUM_F32);
    switch (g) {
      case G_MIN_F32: return GB_AGG(G_MIN_F32);
      case G_MAX_F32: return GB_AGG(G_MAX_F32);
      default: return nullptr;
    }
  } else {
    if constexpr (VD == AGG_I32 && PATH != 3)
      if (g == G_COUNT) return GB_AGG(G_COUNT);
    switch (g) {
      case G_SUM_INT: return GB_AGG(G_SUM_INT);
      case G_MIN_INT: return GB_AGG(G_MIN_INT);
      case G_MAX_INT: return GB_AGG(G_MAX_INT);
      default: return nullptr;
    }
  }
#undef GB_AGG
}

template <int KD, int PATH>
const void* agg_kernel_kd(int32_t vd, int g) {
  if (g == G_COUNT) return agg_row<KD, AGG_I32, PATH>(g);  // reads no values
  switch (vd) {
    case AGG_I32: return agg_row<KD, AGG_I32, PATH>(g);
    case AGG_I64: return agg_row<KD, AGG_I64, PATH>(g);
    case AGG_F32: return agg_row<KD, AGG_F32, PATH>(g);
    default: return nullptr;
  }
}

template <int KD>
const void* agg_kernel_path(int32_t vd, int g, int path) {
  switch (path) {
    case 1: return agg_kernel_kd<KD, 1>(vd, g);
    case 2: return agg_kernel_kd<KD, 2>(vd, g);
    case 3: return agg_kernel_kd<KD, 3>(vd, g);
    case 4: return agg_kernel_kd<KD, 4>(vd, g);
    default: return agg_kernel_kd<KD, 0>(vd, g);
  }
}

const void* agg_kernel(int32_t kd, int32_t vd, int g, int path) {
  return kd == AGG_I32 ? agg_kernel_path<AGG_I32>(vd, g, path) : agg_kernel_path<AGG_I64>(vd, g, path);
}

template <int KD, int VD, bool HASV>
const void* scatter_row(int bits) {
  if ((1 << bits) <= CarryTile<KD, VD, HASV, false>::PMAX)
    return reinterpret_cast<const void*>(&gb_scatter_carry_kernel<KD, VD, HASV, false>);
  // Twice as many partitions still gain where a row is 8 or 16 bytes (1577 ->
  // 1391 us and 2972 -> 2630 at 1024), but not at 12, whose carried rows leave
  // too little of LDS to new ones (2046 against 2066 at 512).
  using W = CarryTile<KD, VD, HASV, true>;
  if constexpr (W::RB != 12)
    if ((1 << bits) <= W::PMAX) return reinterpret_cast<const void*>(&gb_scatter_carry_kernel<KD, VD, HASV, true>);
  return reinterpret_cast<const void*>(&gb_scatter_tiled_kernel<KD, VD, HASV>);
}

template <int KD>
const void* scatter_kd(int32_t vd, bool hasv, int bits) {
  if (!hasv) return scatter_row<KD, AGG_I32, false>(bits);
  return vd == AGG_I64 ? scatter_row<KD, AGG_I64, true>(bits) : scatter_row<KD, AGG_I32, true>(bits);  // 4-byte values move as bits
}

const void* init_kernel(int g) {
  switch (g) {
    case G_COUNT: return reinterpret_cast<const void*>(&gb_init_kernel<G_COUNT>);
    case G_SUM_INT: return reinterpret_cast<const void*>(&gb_init_kernel<G_SUM_INT>);
    case G_MIN_INT: return reinterpret_cast<const void*>(&gb_init_kernel<G_MIN_INT>);
    case G_MAX_INT: return reinterpret_cast<const void*>(&gb_init_kernel<G_MAX_INT>);
    case G_SUM_F32: return reinterpret_cast<const void*>(&gb_init_kernel<G_SUM_F32>);
    case G_MIN_F32: return reinterpret_cast<const void*>(&gb_init_kernel<G_MIN_F32>);
    case G_MAX_F32: return reinterpret_cast<const void*>(&gb_init_kernel<G_MAX_F32>);
    default: return nullptr;
  }
}

const void* emit_kernel(int g) {
  switch (g) {
    case G_COUNT: return reinterpret_cast<const void*>(&gb_emit_kernel<G_COUNT>);
    case G_SUM_INT: return reinterpret_cast<const void*>(&gb_emit_kernel<G_SUM_INT>);
    case G_MIN_INT: return reinterpret_cast<const void*>(&gb_emit_kernel<G_MIN_INT>);
    case G_MAX_INT: return reinterpret_cast<const void*>(&gb_emit_kernel<G_MAX_INT>);
    case G_SUM_F32: return reinterpret_cast<const void*>(&gb_emit_kernel<G_SUM_F32>);
    case G_MIN_F32: return reinterpret_cast<const void*>(&gb_emit_kernel<G_MIN_F32>);
    case G_MAX_F32: return reinterpret_cast<const void*>(&gb_emit_kernel<G_MAX_F32>);
    default: return nullptr;
  }
}

template <int KD>
const void* merge_kernel(int g) {
  switch (g) {
    case G_COUNT: return reinterpret_cast<const void*>(&gb_merge_kernel<KD, G_COUNT>);
    case G_SUM_INT: return reinterpret_cast<const void*>(&gb_merge_kernel<KD, G_SUM_INT>);
    case G_MIN_INT: return reinterpret_cast<const void*>(&gb_merge_kernel<KD, G_MIN_INT>);
    case G_MAX_INT: return reinterpret_cast<const void*>(&gb_merge_kernel<KD, G_MAX_INT>);
    case G_SUM_F32: return reinterpret_cast<const void*>(&gb_merge_kernel<KD, G_SUM_F32>);
    case G_MIN_F32: return reinterpret_cast<const void*>(&gb_merge_kernel<KD, G_MIN_F32>);
    case G_MAX_F32: return reinterpret_cast<const void*>(&gb_merge_kernel<KD, G_MAX_F32>);
    default: return nullptr;
  }
}

int launch_lds(const void* fn, int64_t grid, int block, size_t lds, Args* args, hipStream_t stream) {
  void* kargs[] = {args};
  const hipError_t e = hipLaunchKernel(fn, dim3((unsigned)grid), dim3(block), kargs, lds, stream);
  if (e != hipSuccess) {
    record_hip_error((int32_t)e);
    (void)hipGetLastError();
    return AGG_E_HIP;
  }
  return AGG_OK;
}

}  // namespace gb
}  // namespace agg

using namespace agg;
using namespace agg::gb;

struct agg_groupby_s {
  int device = 0;
  int32_t key_dtype = 0, val_dtype = 0, op = 0;
  int gop = 0;
  int64_t max_n = 0, max_groups = 0;
  void* ws = nullptr;
  Table t{};
  Part pt{};           // bits == 0: the direct path
  int path = 0;        // 0 direct, 1 partitioned, 2 few groups, 3 / 4: 0 / 1 in sub-partition passes
  int agg_blocks = 1;  // aggregation workgroups resident per CU
  bool clean = false;  // the table and its state are as a call needs them
  uint32_t* dump = nullptr;  // direct path: regions for dump_wgs workgroups' tables
  int dump_wgs = 0, dump_max = 0;
};

extern "C" {

int agg_groupby_plan(agg_groupby_t* out, int32_t key_dtype, int32_t val_dtype, int32_t op, int64_t max_n,
                     int64_t max_groups) {
  if (!out) return AGG_E_INVALID;
  *out = nullptr;
  const int g = gop_of(val_dtype, op);
  if ((key_dtype != AGG_I32 && key_dtype != AGG_I64) || width_of(val_dtype) == 0 || g < 0) return AGG_E_INVALID;
  if (max_n < 0 || max_groups < 1 || max_groups > ((int64_t)1 << 32)) return AGG_E_INVALID;
  if (g == G_SUM_F32 && max_n > ((int64_t)1 << 31)) return AGG_E_INVALID;  // digit headroom
  if (max_n > ((int64_t)1 << 36)) return AGG_E_INVALID;
  int dev = 0;
  const int dr = current_device(&dev);
  if (dr != AGG_OK) return dr;
  int64_t cap = 64;
  while (cap < 2 * max_groups) cap <<= 1;
  const int64_t slots = cap + 1;
  const bool dig = g == G_SUM_F32;
  // LDS tables are filled at most half (every probe hashed anew, a half-full
  // table still probes fast; measured, linear probing slowed sharply past a
  // quarter): the direct path up to half of its table, or in two passes over
  // the rows up to a whole table's worth, partitions sized for half of
  // theirs.  (Measured on 2^28 rows: two direct passes take 0.65x the
  // partitioned path's time for int64 SUM, about the same for float sums,
  // but 1.09x for COUNT, which moves the fewest bytes when partitioned; each
  // pass costs about one direct run, so four would lose.)
  int bits = 0, direct_sub_bits = 0;
  const int64_t half_table = lds_slots_of(g, key_dtype) / 2;
  // Float sums of int32 keys, or of fewer rows, partition too: 4096 groups, 3e7 rows
  // 335 us in two passes, 239 partitioned; 5e5 rows 61 and 53; 2^28 rows, int32 keys,
  // 1411 and 1640, but with 60 exponents 2311 and 1660.  int64 keys, 2^28 rows, whose
  // staged rows are 12 bytes: 1480 in two passes, 2490 partitioned; with 60 exponents
  // 2600 and 2480 (and 5670 and 3950 with 200).
  const bool two_passes = g != G_COUNT && !(g == G_SUM_F32 && (key_dtype == AGG_I32 || max_n < kTwoPassFloatRows));
  if (max_groups > half_table && max_groups <= 2 * half_table && two_passes) {
    direct_sub_bits = 1;
  } else if (max_groups > half_table) {
    auto bits_for = [max_groups](int64_t per_part) {
      int b = 0;
      while (b < kMaxPartBits && (per_part << b) < max_groups) ++b;
      return b;
    };
    bits = bits_for(half_table);
    const bool large = max_n >= kLargeRows;
    const bool wide = width_of(key_dtype) + (op == AGG_COUNT ? 0 : width_of(val_dtype)) >= 16;
    const int few_keys = max_n < kFewKeysRows ? kMinPartBits : std::max(kLeastPartBits, bits_for(kFewKeys));
    bits = std::max(bits, max_groups >= kManyGroups && !(large && wide) ? kMinPartBitsMany
                          : large                                      ? kMinPartBitsLarge
                                                                       : std::min(few_keys, kMinPartBits));
  }
  // The scatter takes at most 2^kTileMaxBits partitions (its per-partition
  // counters live in LDS, and more would shorten the coalesced runs); past
  // that each partition is folded in 2^sub_bits passes.
  const int sub_bits = bits ? std::max(0, bits - kTileMaxBits) : direct_sub_bits;
  bits -= bits ? sub_bits : 0;
  const int64_t P = bits ? (int64_t)1 << bits : 0;
  const int64_t crow = bits ? std::max<int64_t>(1, std::min<int64_t>(max_n, kChunkRows)) : 0;
  const int kw = width_of(key_dtype), vw = op == AGG_COUNT ? 0 : width_of(val_dtype);
  auto up = [](int64_t x) { return (x + 255) & ~(int64_t)255; };
  const int64_t b_key = up(slots * 8), b_cnt = up(slots * 8), b_val = up(slots * 8);
  const int64_t b_dig = dig ? up(slots * 8 * kDigits) : 256, b_flags = up(slots * 4), b_state = 256;
  const int64_t b_hist = up(P * kMaxHistWg * 4), b_tot = up(P * 4 + 4), b_start = up(P * 4 + 4),
                b_pk = up(crow * kw), b_pv = up(crow * vw);
  // Regions for one table per workgroup and hash half, if a run can have enough
  // of them to merge: room for the groups (for a half of them, half and a quarter
  // more; a table with more than that is flushed as usual).  A run has at most a
  // workgroup per CU and per kDirectRows rows (10^6 rows of 2000 groups: 62 regions,
  // 1.0 MB of COUNT, for 256 of them 4.2), and too few updates are never merged.
  int64_t wgs = bits || max_groups <= kFewGroups ? 0 : std::min<int64_t>(device_cu(dev), ceil_div(max_n, kDirectRows));
  if (wgs <= kMergeMinWg || wgs * max_groups < kMergeMinUpdates) wgs = 0;
  const int64_t dump_max = sub_bits ? max_groups / 2 + max_groups / 8 + 64 : max_groups + 1;
  const int64_t b_dump = up(wgs * (dump_region_of(g, key_dtype, dump_max) << sub_bits) * 4);
  const int64_t total = b_key + b_cnt + b_val + b_dig + b_flags + b_state + b_hist + b_tot + b_start +
                        b_pk + b_pv + b_dump;
  agg_groupby_s* p = new (std::nothrow) agg_groupby_s();
  if (!p) return AGG_E_NOMEM;
  const int arc = device_alloc(&p->ws, (size_t)total);
  if (arc != AGG_OK) {
    delete p;
    return arc;
  }
  char* c = static_cast<char*>(p->ws);
  auto take = [&c](int64_t bytes) {
    char* r = c;
    c += bytes;
    return r;
  };
  p->t.key = reinterpret_cast<int64_t*>(take(b_key));
  p->t.cnt = reinterpret_cast<uint64_t*>(take(b_cnt));
  p->t.val = reinterpret_cast<int64_t*>(take(b_val));
  p->t.dig = reinterpret_cast<int64_t*>(take(b_dig));
  p->t.flags = reinterpret_cast<int32_t*>(take(b_flags));
  p->t.state = reinterpret_cast<int32_t*>(take(b_state));
  p->t.cap = cap;
  p->t.cap_log2 = __builtin_ctzll((unsigned long long)cap);
  p->pt.hist = reinterpret_cast<uint32_t*>(take(b_hist));
  p->pt.tot = reinterpret_cast<uint32_t*>(take(b_tot));
  p->pt.start = reinterpret_cast<uint32_t*>(take(b_start));
  p->pt.pk = take(b_pk);
  p->pt.pv = vw ? take(b_pv) : nullptr;  // right after pk: staged (key, value) records span both
  p->dump = wgs ? reinterpret_cast<uint32_t*>(take(b_dump)) : nullptr;
  p->dump_wgs = (int)wgs;
  p->dump_max = (int)dump_max;
  p->pt.bits = bits;
  p->pt.sub_bits = sub_bits;
  p->device = dev;
  p->key_dtype = key_dtype;
  p->val_dtype = val_dtype;
  p->op = op;
  p->gop = g;
  p->max_n = max_n;
  p->max_groups = max_groups;
  // aggregation grids are sized to what the chip holds at once (no second, mostly idle wave of workgroups)
  int nb = 0;
  p->path = bits ? (sub_bits ? 4 : 1) : sub_bits ? 3 : max_groups <= kFewGroups ? 2 : 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, agg_kernel(key_dtype, val_dtype, g, p->path),
                                                   bits ? kPartThreads : kDirectThreads, 0) !=
          hipSuccess ||
      nb < 1) {
    (void)hipGetLastError();
    nb = 1;
  }
  p->agg_blocks = nb;
  *out = p;
  return AGG_OK;
}

int agg_groupby_run(agg_groupby_t p, const void* keys, const void* vals, int64_t n, agg_group* groups,
                    int64_t* ngroups, void* stream_v) {
  if (!p || !groups || !ngroups || n < 0 || n > p->max_n || (n > 0 && (!keys || !vals))) return AGG_E_INVALID;
  const int kw = width_of(p->key_dtype), vw = width_of(p->val_dtype);
  if (n > 0 && (reinterpret_cast<uintptr_t>(keys) % (uintptr_t)kw || reinterpret_cast<uintptr_t>(vals) % (uintptr_t)vw))
    return AGG_E_INVALID;
  if (n > 0) {
    int rc = check_pointer(keys, n * kw, AGG_SRC_DEVICE, p->device);
    if (rc == AGG_OK && p->op != AGG_COUNT) rc = check_pointer(vals, n * vw, AGG_SRC_DEVICE, p->device);
    if (rc != AGG_OK) return rc;
  }
  int rc = check_out_pointer(groups, p->max_groups * (int64_t)sizeof(agg_group), p->device);
  if (rc == AGG_OK) rc = check_out_pointer(ngroups, sizeof(int64_t), p->device);
  if (rc != AGG_OK) return rc;
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  const int cu = device_cu(p->device);
  Args a{};
  a.t = p->t;
  a.pt = p->pt;
  a.keys = keys;
  a.vals = vals;
  a.n = n;
  a.out = groups;
  a.max_groups = p->max_groups;
  a.ngroups = ngroups;
  a.is_avg = p->op == AGG_AVG;
  a.op = p->op;
  // The table is clean between calls (each clears what it emits); a plan's
  // first call clears it, and so does one after a launch that failed.  A call
  // recorded into a graph with the clearing in it leaves it to the replays.
  const bool first = !p->clean;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (first && hipStreamIsCapturing(stream, &cap) != hipSuccess) {
    (void)hipGetLastError();
    cap = hipStreamCaptureStatusActive;
  }
  p->clean = false;
  const int64_t slots = p->t.cap + 1;
  if (first) {
    const int64_t grid = std::min<int64_t>(ceil_div(slots, kThreads), (int64_t)cu * 8);
    rc = launch(init_kernel(p->gop), (int)grid, kThreads, &a, stream);
    if (rc != AGG_OK) return rc;
  }
  if (n > 0 && p->pt.bits == 0) {
    // Two tiles per workgroup at least, so that its table's flush serves more
    // rows (1e6 rows, int32 keys and values: 1000 groups 37.4 us, 38.5 with one
    // tile; float SUM 53.1, 64.6).  The few-groups table's flush is nothing, so
    // one tile (25 groups 15.1 us either way).
    const int64_t wg_rows = p->path == 2 ? kDirectRows / 2 : kDirectRows;
    const int64_t grid = std::max<int64_t>(ceil_div(n, kMaxTableRows),
                                           std::min<int64_t>(ceil_div(n, wg_rows), (int64_t)cu * p->agg_blocks));
    // (a float sum's windows take the rows of one table, merged or not)
    const bool merge = grid > kMergeMinWg && grid <= p->dump_wgs && grid * p->max_groups >= kMergeMinUpdates &&
                       n <= (p->gop == G_SUM_F32 ? kMergeMaxFloatRows : kMergeMaxRows);
    a.dump = p->dump;
    a.dump_max = p->dump_max;
    a.dumps = merge ? (int)grid : 0;
    a.emit = merge || slots <= fuse_slots_of(p->gop);
    Args fold = a;
    fold.emit = !merge && a.emit;
    rc = launch(agg_kernel(p->key_dtype, p->val_dtype, p->gop, p->path), (int)grid, kDirectThreads, &fold, stream);
    if (rc == AGG_OK && merge)
      rc = launch(p->key_dtype == AGG_I32 ? merge_kernel<AGG_I32>(p->gop) : merge_kernel<AGG_I64>(p->gop), kSections,
                  kDirectThreads, &a, stream);
    if (rc != AGG_OK) return rc;
  } else if (n > 0) {
    const int64_t P = (int64_t)1 << p->pt.bits;
    const bool hasv = p->op != AGG_COUNT;
    const void* hist = p->key_dtype == AGG_I32 ? reinterpret_cast<const void*>(&gb_hist_kernel<AGG_I32>)
                                               : reinterpret_cast<const void*>(&gb_hist_kernel<AGG_I64>);
    const void* scat = p->key_dtype == AGG_I32 ? scatter_kd<AGG_I32>(p->val_dtype, hasv, p->pt.bits)
                                               : scatter_kd<AGG_I64>(p->val_dtype, hasv, p->pt.bits);
    const void* aggk = agg_kernel(p->key_dtype, p->val_dtype, p->gop, p->path);
    for (int64_t c0 = 0; c0 < n; c0 += kChunkRows) {
      const int64_t m = std::min<int64_t>(kChunkRows, n - c0);
      a.keys = static_cast<const char*>(keys) + c0 * kw;
      a.vals = static_cast<const char*>(vals) + c0 * vw;
      a.n = m;
      a.whole = m == n;
      a.pt.g1 = (int)std::min<int64_t>(kMaxHistWg, ceil_div(m, kMinHistRows));
      a.pt.rows_per_wg = ceil_div(m, a.pt.g1);
      if ((rc = launch_lds(hist, a.pt.g1, kHistThreads, 0, &a, stream)) != AGG_OK) return rc;
      if ((rc = launch_lds(reinterpret_cast<const void*>(&gb_scan_kernel), ceil_div(P, kThreads / 64), kThreads, 0, &a,
                           stream)) != AGG_OK)
        return rc;
      if ((rc = launch_lds(scat, a.pt.g1, kTileThreads, 0, &a, stream)) != AGG_OK)
        return rc;
      // a workgroup for each tile of rows, or for each partition if those are
      // more: every partition costs its workgroup a table to clear and flush
      // (1e5 rows, 50 000 groups: int32 SUM 80 us with 12 workgroups, 53 with 32)
      const int64_t awg = std::max(ceil_div(m, kPartThreads * 8), std::min(P, ceil_div(m, 64)));
      const int64_t agrid =
          std::max<int64_t>(ceil_div(m, kMaxTableRows), std::min<int64_t>(awg, (int64_t)cu * p->agg_blocks));
      if ((rc = launch_lds(aggk, agrid, kPartThreads, 0, &a, stream)) != AGG_OK) return rc;
    }
    a.keys = keys;
    a.vals = vals;
    a.n = n;
  }
  if (!a.emit) {
    const int64_t grid = std::max<int64_t>(1, std::min<int64_t>(ceil_div(slots, kEmitThreads), (int64_t)cu * 2));
    if ((rc = launch(emit_kernel(p->gop), (int)grid, kEmitThreads, &a, stream)) != AGG_OK) return rc;
  }
  p->clean = !(first && cap != hipStreamCaptureStatusNone);
  return AGG_OK;
}

int agg_groupby_destroy(agg_groupby_t p) {
  if (!p) return AGG_E_INVALID;
  (void)hipDeviceSynchronize();
  if (p->ws) (void)hipFree(p->ws);
  delete p;
  return AGG_OK;
}

}  // extern "C"
