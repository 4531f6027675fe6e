// Hive hash table on MI355X (gfx950): kernels and the C ABI of include/hive.h.
//
// A batch runs as stream-ordered phases (launches):
//   dedupe  (optional) by hash ranges in LDS: per key, the last insert and the
//           first delete of the batch stand; the others become no-ops, so
//           repeated keys cannot leave two copies (the paper does not say what
//           happens to repeats inside one batch);
//   P1      every operation: hash, match-and-elect over the first and then
//           the second candidate bucket (Section III-F), then replace
//           (Algorithm 1), lookup, delete (Algorithm 4) or claim-then-commit
//           of a free slot (Section III-E, Algorithm 2).  No entry moves in
//           P1, so lookups and deletes never miss a key in flight;
//   P3      inserts whose two buckets were full: bounded cuckoo eviction
//           (Algorithm 3), and after max_evictions displacements the item in
//           hand goes to the stash, or the pending list when the stash is
//           full (Section IV-A step 4; the stash here is an open-addressed
//           table rather than the paper's ring, so a search stops at the
//           first EMPTY slot of its key's probe run instead of scanning).
//
// gfx950 mapping of the warp protocols: with S = 16 a bucket is one 128-byte
// line probed by a 16-lane group, so one wave-wide load probes 4 buckets.
// Each wave owns 64 operations: lanes hash their own operation, the groups
// then issue all 16 bucket loads of the wave before consuming any (memory
// parallelism), ballot the key matches and the empty slots, and hand the
// per-operation result back through LDS.  The free mask of a bucket is the
// ballot of its EMPTY slots; claiming a slot and publishing the entry is one
// 64-bit CAS(EMPTY -> entry), issued lane-per-operation so a wave has 64
// CAS in flight.  A failed CAS returns the word it found, which corrects a
// stale view of the bucket (each XCD has its own L2).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstddef>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <thread>
#include <type_traits>
#include <vector>

#include "hash_fns.hpp"
#include "hive.h"
#include "hive_device.hpp"

static_assert(hive::PAIR_BITHASH == HIVE_PAIR_BITHASH && hive::PAIR_CRC == HIVE_PAIR_CRC &&
                  hive::PAIR_MURMUR == HIVE_PAIR_MURMUR && hive::PAIR_TRIPLE == HIVE_PAIR_TRIPLE,
              "hash pair numbering");

namespace hive {

constexpr int WAVES = 4;  // waves per block
constexpr int BLOCK = 64 * WAVES;
#ifndef EVICT_SLOTS_PER_LANE
#define EVICT_SLOTS_PER_LANE 16  // 16-slot buckets: slots per lane of an eviction group (2, 4, 8, 16)
#endif
constexpr int EVICT_GRID = 2048;  // most blocks of the eviction phase (all resident at once)
constexpr int RESIZE_GRID = 1024; // most blocks of resize_kernel (they stride over buckets and stash words)
constexpr int MERGE_GRID = 512;   // blocks of merge_kernel, two per compute unit
constexpr int MERGE_BLOCK = 512;  // (a larger one has no room beside a resident executor)
constexpr uint64_t MERGE_RUN = 64;  // pairs of a run, at least
constexpr int MERGE_LOADS = 4;      // pairs in flight per group of lanes
// Most blocks of a probe launch: larger batches stride over tiles, about
// eight tiles per block at 2^26 operations (bulk step +4% against one tile
// per block, measured over 2,048 .. 65,536 blocks: the launch pays less
// block setup, such as the coherent read of the control line)
constexpr uint64_t OPS_GRID = 32768;
constexpr int DRAIN_WORDS = 8;  // stash words per thread and trip of the drain
#ifndef OPS_WAVES_PER_EU
#define OPS_WAVES_PER_EU 4  // occupancy target of the probe kernel (waves per SIMD)
#endif

template <int S>
struct Traits {
  static_assert(S == 16 || S == 32 || S == 64, "slots per bucket must be 16, 32 or 64");
  static constexpr int G = 64 / S;  // buckets probed by one wave-wide load
  static constexpr int CH = 16;     // loads in flight per chunk of a probe round
  static constexpr int OPS_PER_CHUNK = CH * G;
  using Mask = typename std::conditional<(S <= 32), uint32_t, uint64_t>::type;
  static constexpr uint64_t FULL = (S == 64) ? ~0ull : ((1ull << S) - 1ull);
};

__device__ __forceinline__ int ctz_mask(uint32_t m) { return __builtin_ctz(m); }
__device__ __forceinline__ int ctz_mask(uint64_t m) { return __builtin_ctzll(m); }
__device__ __forceinline__ int popc_mask(uint32_t m) { return __builtin_popcount(m); }
__device__ __forceinline__ int popc_mask(uint64_t m) { return __builtin_popcountll(m); }

// The EMPTY slot (a set bit of m, not zero) that key k tries to claim first:
// the first one at or after a slot picked by the key, cyclically.  Claims of
// one bucket that run side by side all see the same EMPTY slots; with the
// lowest slot as every key's first choice, c keys of one bucket took up to c
// rounds of failing CASes, while keys that start at slots of their own mostly
// commit with their first.  Measured, lowest slot against this: the build,
// lookups and deletes of 2^16 keys in 2^13 buckets 160 -> 151 us; 4.0 M
// entries exported in bucket order and re-inserted 1,667 -> 1,315 us; a
// key-only set's 2^22 inserts and lookups 551 -> 469 us; growing a linear
// table to 12.6 M keys and back 6,271 -> 6,157 us.
template <int S, typename Mask>
__device__ __forceinline__ int claim_slot(Mask m, uint32_t k) {
  static_assert((S & (S - 1)) == 0, "a power of two");
  const int r = (int)((k * 0x9E3779B1u) >> (32 - __builtin_ctz(S)));
  const Mask from = m & (Mask)(~(Mask)0 << r);
  return ctz_mask(from ? from : m);
}

__device__ __forceinline__ uint64_t read_lane64(uint64_t x, int lane) {
  uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, lane);
  uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), lane);
  return ((uint64_t)hi << 32) | lo;
}

// Value of lane `src` of the wave, for a 64-bit word.
__device__ __forceinline__ uint64_t shfl64(uint64_t x, int src) {
  const int lo = __builtin_amdgcn_ds_bpermute(src << 2, (int)(uint32_t)x);
  const int hi = __builtin_amdgcn_ds_bpermute(src << 2, (int)(uint32_t)(x >> 32));
  return ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
}

// Sum over the 64 lanes of a wave (every lane active); every lane gets it.
__device__ __forceinline__ uint64_t wave_sum64(uint64_t x) {
  const int lane = threadIdx.x & 63;
  for (int o = 32; o > 0; o >>= 1) x += shfl64(x, lane ^ o);
  return x;
}

// Worklist segments.  The eviction worklist is NSHARD segments of seg_cap
// entries; tile t (256 operations, or 256 stash entries of a drain) appends
// to segment t % NSHARD through that shard's wl_count, so appends spread
// over NSHARD counters.  A segment receives at most 256 entries from each of
// ceil(tiles / NSHARD) tiles, which bounds seg_cap.
__device__ __forceinline__ uint64_t wl_append(const Ctl *c, uint64_t tile, uint64_t n) {
  return add64(&shard_of(c, tile % NSHARD)->wl_count, n);
}

// Exclusive prefix of the segment fills, pre[0..NSHARD] (pre[NSHARD] is the
// total); the whole block calls it, wave 0 loads and scans.
__device__ __forceinline__ void wl_prefix(const Ctl *c, uint64_t *pre) {
  if (threadIdx.x < NSHARD) {
    const int lane = threadIdx.x;
    uint64_t x = ld_ctl(&shard_of(c, lane)->wl_count);
    for (int o = 1; o < NSHARD; o <<= 1) {
      const uint64_t y = shfl64(x, lane >= o ? lane - o : lane);
      if (lane >= o) x += y;
    }
    pre[lane + 1] = x;
    if (lane == 0) pre[0] = 0;
  }
  __syncthreads();
}

// Position in the worklist of item k < pre[NSHARD] (items numbered segment
// by segment): the last segment whose prefix is <= k holds it.
__device__ __forceinline__ uint64_t wl_slot(const uint64_t *pre, uint64_t k, uint64_t seg_cap) {
  int s = 0;
  for (int step = NSHARD / 2; step > 0; step >>= 1)
    if (pre[s + step] <= k) s += step;
  return (uint64_t)s * seg_cap + (k - pre[s]);
}

// Fold the shards into the totals of Ctl line 1 (one full wave; nothing else
// may update this table's shards meanwhile).  With wl_done the worklist's
// items are counted and its segments emptied.  `inserts`: operations of the
// batch that may have inserted (Ctl::inserted).  Returns the worklist size.
__device__ __forceinline__ uint64_t fold_shards_wave(Ctl *c, bool wl_done, uint64_t inserts = 0) {
  const int lane = threadIdx.x & 63;
  Shard *sh = shard_of(c, lane);
  // the last pair: stash placements made without a reservation join the
  // stash count here, after the launch (or executor phase) that made them
  constexpr int NF = 7;
  uint64_t *src[NF] = {&sh->live,          &sh->evictions,       &sh->full_chains,     &sh->invalid_keys,
                       &sh->stash_inserts, &sh->pending_inserts, &sh->stash_unreserved};
  uint64_t *dst[NF] = {&c->live,          &c->evictions,       &c->full_chains, &c->invalid_keys,
                       &c->stash_inserts, &c->pending_inserts, &c->stash_count};
  uint64_t v[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) v[f] = ld_ctl(src[f]);
  const uint64_t wl = ld_ctl(&sh->wl_count);
#pragma unroll
  for (int f = 0; f < NF; ++f)
    if (v[f]) __hip_atomic_store(src[f], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (wl_done && wl) __hip_atomic_store(&sh->wl_count, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
  for (int f = 0; f < NF; ++f) v[f] = wave_sum64(v[f]);
  const uint64_t total_wl = wave_sum64(wl);
  if (lane == 0) {
#pragma unroll
    for (int f = 0; f < NF; ++f)
      if (v[f]) add64(dst[f], v[f]);
    if (wl_done && total_wl) add64(&c->evict_items, total_wl);
    if (inserts) add64(&c->inserted, inserts);
  }
  return total_wl;
}

// After a batch without inserts, and while phases are timed (one wave of 64
// threads).
__global__ __launch_bounds__(64) void finish_kernel(Ctl *c, uint64_t inserts) {
  (void)fold_shards_wave(c, true, inserts);
}

// ---------------------------------------------------------------------------
// Spill filter and first-candidate placement (FIXED tables of two candidates
// that are probed one after the other).
//
// A probe is bound by the 128-byte lines it reads, and a key that is absent,
// or sits in its second candidate, costs two.  So a new key goes to its first
// candidate while that has at least `first_min` EMPTY slots (only then to the
// emptier of both), and every bucket b has 2^shift filter bits of its own:
// whenever a key whose first candidate is b is put anywhere else (its second
// candidate, the stash, the pending list), the bit that the key picks is set.
// A search that finds nothing in the first candidate and whose bit is clear is
// over: one line, and the filter's.  While no entry was ever deleted, a first
// candidate with first_min EMPTY slots always had them, so none of its keys is
// elsewhere and the bits are not even read.
//
// It serves a table's first fill.  Bits are only cleared with the table: under
// inserts and deletes more and more are set, and a search whose bit is set
// takes three accesses where it would take two (2^24 keys at 90% load, lookups
// with no hits, before and after six turnovers of the contents 109 and 174 us,
// without a filter 165 throughout); and new keys for a loaded table mostly go
// to their second candidate, each with an atomic on its bit and after a second
// dependent round.  So a batch that starts when FILTER_START_PCT of the slots'
// number was inserted, or ends beyond FILTER_END_PCT, is `plain`: placed by
// two-choice, both candidates in one round, and the filter is dropped until the
// table is cleared.  (One batch of 2^21 keys to 97 / 99% load: two-choice 200 /
// 240 us and 94 / 3,858 stash entries, packed 217 / 267 us and 624 / 7,301.
// Wider buckets gain at any load: 2^25 keys in 32 slots to 99%, 3,237 us, packed
// 2,638.)  The host counts along (hive_table::inserted) and launches what
// suits; the device's own count and flag decide what the bits are worth, for
// replays of captured launches and for the executor.
// Slices of new keys into a 2^26-key table, 0-55-65-75-85-90-95-97%, without a
// filter: 2,083, 428, 426, 440, 251, 320, 261 us, so: 1,609, 423, 427, 436, 244,
// 288, 212; with the filter kept up throughout: 1,539, 373, 410, 452, 273, 412,
// 392 (the last two with the buckets of chains in scratch memory).  A limit of
// 75% was slower between 55 and 75% (2^22 keys: 65 and 73 us a slice against 49
// and 51).  One batch to 95% of 2^26 keys 3,610 / 3,229 us, lookups at 50% hits
// after it 2,080 / 1,920; 2^24 lookups in a table of 2^24 keys 504 / 424 us.
//
// first_min, a share of the slots: less leaves more keys in their first
// candidate, and costs chains and stash entries once the table is nearly full,
// since buckets that few keys have first stay emptier than two-choice would
// leave them.  2^21 keys built to 95% load in 16-slot buckets, two-choice /
// 7 / 6 / 5 sixteenths: stash entries 3 / 32 / 59 / 139; the build, two sets of
// lookups and a delete of 2^26 keys 9,950 / 9,340 / 9,210 / 9,090 us.  (A fixed
// 5 slots is less than a sixth of a 32-slot bucket: 637 stash entries of 2^21
// keys in a key-only set where two-choice has none.)
// Two-choice alone, and no filter, where chains or the stash have little room:
// tables with an eviction bound under FIRST_MIN_CHAIN, and those whose stash
// holds less than the default 1% of the slots (a stash sized for two-choice
// placement may not hold the entries above).
// shift: 8 bits a bucket while the filter stays within FILTER_BYTES, beyond which
// fewer bits in fewer lines are ahead (2^24 lookups without hits at 53 / 90% load:
// 458 / 615 us with 8 bits in 5.20 M buckets, 441 / 591 with 4 in 5.28 M; its lines
// mostly miss the L2s, which bucket lines stream through); at 95% load
// a missing key finds its bit set with probability 0.74 / 0.59 / 0.41 / 0.25
// for 1 / 2 / 4 / 8 bits.
// LINEAR tables have none: their unsplit buckets are full, so that most bits
// would be set, and splits would have to hand them on (growth to 12.6 M keys
// and back 3,500 us without, 3,840 with; mixed batches the same either way).
// ---------------------------------------------------------------------------
constexpr uint32_t FIRST_MIN_16THS = 7;
constexpr uint64_t FILTER_START_PCT = 55;
constexpr uint64_t FILTER_END_PCT = 96;  // 16-slot buckets
constexpr uint32_t FIRST_MIN_CHAIN = 4;
constexpr uint64_t FILTER_BYTES = 5ull << 20;

struct Spill {
  uint32_t *bits;  // null: the table has no filter
  uint32_t shift;
  uint32_t first_min;
  uint64_t start, end;  // a batch keeps it up that starts below and ends within these numbers of inserts
};

// The filter as a batch meets it: `plain`, when the batch places by two-choice
// alone and sets no bits; `dropped`, when a plain batch ran since the table was
// empty and the bits mean nothing any more.  Both stay as they are while the
// batch's launches run (Ctl::inserted moves at their end), but for `dropped`,
// which its probe launch sets when it is plain.
struct SpillState {
  bool plain, dropped;
};
__device__ __forceinline__ SpillState spill_state(const Spill &f, const Ctl *c, uint64_t n) {
  SpillState s;
  const uint64_t inserted = ld_ctl(&c->inserted);
  s.dropped = ld_ctl32(&c->dropped) != 0;
  s.plain = s.dropped || inserted >= f.start || inserted + n > f.end;
  return s;
}

// No filter, two-choice placement.
__host__ __device__ __forceinline__ Spill spill_none(uint32_t S) { return Spill{nullptr, 0, S + 1, 0, 0}; }

// The filter that a placement phase keeps up.
__device__ __forceinline__ Spill spill_placing(const Spill &f, const Ctl *c, uint64_t n, uint32_t S) {
  return f.bits && !spill_state(f, c, n).plain ? f : spill_none(S);
}

__device__ __forceinline__ uint64_t spill_bit(const Spill &f, uint32_t c1, uint32_t k) {
  return ((uint64_t)c1 << f.shift) | (((k * 0x9E3779B1u) >> 29) & ((1u << f.shift) - 1u));
}

// Whether key k, whose first candidate is c1, may be elsewhere.
__device__ __forceinline__ bool spill_test(const Spill &f, uint32_t c1, uint32_t k) {
  const uint64_t t = spill_bit(f, c1, k);
  return (f.bits[t >> 5] >> (t & 31)) & 1u;
}

// Key k, whose first candidate is c1, is being put elsewhere.
__device__ __forceinline__ void spill_mark(const Spill &f, uint32_t c1, uint32_t k) {
  if (!f.bits) return;
  const uint64_t t = spill_bit(f, c1, k);
  or32(&f.bits[t >> 5], 1u << (t & 31));
}

struct OpsArgs {
  uint64_t *buckets;
  Spill spill;
  uint32_t *hint;
  uint64_t *stash;
  uint64_t *pending;
  Ctl *ctl;
  uint64_t *wl;        // eviction worklist: NSHARD segments of wl_seg_cap entries
  uint64_t wl_seg_cap;
  const uint64_t *dd;  // dedupe set, or null
  uint64_t dd_mask;
  const uint8_t *ops;
  const uint32_t *keys;
  const uint32_t *vals;
  uint32_t *vals_out;
  uint8_t *flags_out;
  uint64_t n;
  uint64_t stash_cap;
  uint64_t pending_cap;
  const uint8_t *win;  // dedupe winner flag per operation (plain launches), or null
};

// ---------------------------------------------------------------------------
// Dedupe: per key, the largest index among inserts (last occurrence wins) and
// the smallest among deletes (the first occurrence reports the deletion).
// Entries are (key << 32 | index); EMPTY never collides since key
// 0xFFFFFFFF is reserved.
// ---------------------------------------------------------------------------
// Record entry e = (k << 32 | index) of an operation of type `op` in the
// set.  Plain loads come first: a key already present costs no CAS, and an
// index that cannot win costs no max/min atomic (a stale load is only ever
// an older value, which would already beat the index, so the skip is safe).
// Settle record e of key k whose claim of slot s found `cur` (not EMPTY):
// the same key keeps the larger insert index or the smaller delete index;
// another key sends the record on along the probe sequence.
__device__ __forceinline__ void dedupe_settle(uint64_t *dd, uint64_t mask, uint32_t op, uint32_t k, uint64_t e,
                                              uint64_t s, uint64_t cur) {
  for (uint64_t probe = 0; probe <= mask; ++probe) {
    if ((uint32_t)(cur >> 32) == k) {
      if (op == OP_INSERT) {
        if (cur < e) __hip_atomic_fetch_max(&dd[s], e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else if (cur > e) {
        __hip_atomic_fetch_min(&dd[s], e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      return;
    }
    s = (s + 1) & mask;
    cur = dd[s];
    if (cur == EMPTY) {
      cur = cas64(&dd[s], EMPTY, e);
      if (cur == EMPTY) return;
    }
  }
}

__device__ __forceinline__ void dedupe_record(uint64_t *dd, uint64_t mask, uint32_t op, uint32_t k, uint64_t e) {
  const uint64_t s = mix32(k) & mask;
  uint64_t cur = dd[s];
  if (cur == EMPTY) {
    cur = cas64(&dd[s], EMPTY, e);
    if (cur == EMPTY) return;
  }
  dedupe_settle(dd, mask, op, k, e, s, cur);
}

__device__ __forceinline__ void dedupe_insert(uint64_t *dd, uint64_t mask, uint32_t op, const uint32_t *keys,
                                              uint64_t i) {
  const uint32_t k = keys[i];
  if (valid_key(k)) dedupe_record(dd, mask, op, k, ((uint64_t)k << 32) | (uint32_t)i);
}

// Thread t records operation n-1-t if it is an insert and operation t if it
// is a delete: blocks start roughly in order, so inserts arrive in falling
// index order (the winner, the last, comes first) and deletes in rising
// order (the first comes first), and repeated hot keys mostly skip their
// atomics.
__device__ __forceinline__ void dedupe_thread(uint64_t *dd, uint64_t mask, uint32_t mode, const uint8_t *ops,
                                              const uint32_t *keys, uint64_t n, uint64_t t) {
  if (t >= n) return;
  const uint64_t ii = n - 1 - t;
  if (mode == OP_INSERT || (mode == OP_MIXED && ops[ii] == OP_INSERT)) dedupe_insert(dd, mask, OP_INSERT, keys, ii);
  if (mode == OP_DELETE || (mode == OP_MIXED && ops[t] == OP_DELETE)) dedupe_insert(dd, mask, OP_DELETE, keys, t);
}

// ---------------------------------------------------------------------------
// Dedupe of batches of up to DDS_MAX operations in one launch.
//
// Block p owns the keys of hash range p, reads the whole batch's keys (they
// stay in the L2: tens of KB read by every block, coalesced), keeps its own
// operations as records in LDS, collapses them in an LDS table (largest index
// of an insert, smallest of a delete) and writes the flags of its operations:
// no staging, no atomics outside LDS.  Bound by the launch and a few dependent
// round trips: 7 us at 64 operations, 11 us at 2^14.  Every block reads every
// key, so the time grows with blocks x keys: at 2^15 operations the two
// launches of ddr_chunk_kernel and ddr_resolve_kernel take about as long (19
// us), at 2^16 they are ahead (18 us against 23, and 55 on Zipf(0.99) keys).
// Five launches (collect, two of prefix sums, scatter, resolve) took 35 us
// from 2^12 operations on and 46 us at 2^14.
//
// A block whose range holds more distinct keys than its table takes splits
// the range: it works through sub-ranges, halving the width whenever one
// overflows and doubling it after one that fits.  The hash is a bijection of
// the 32-bit keys, so a sub-range of at most DDS_CAP values always fits and
// the loop ends.  Operations beyond the record list (a hot key's) go to the
// table directly, and the flags then take a second reading of the keys.
// ---------------------------------------------------------------------------
// Most LDS of a block that finds room beside a resident executor's blocks of 25
// KiB.  (Measured with blocks that wait out a time: next to one of them on a
// compute unit blocks of 16 waves run with 80 KiB and wait with 81.25, though
// 135 are free; next to two, blocks of any size do.)
constexpr uint32_t BESIDE_LDS = 80 * 1024;
constexpr int DDS_BLOCK = 1024;
constexpr uint64_t DDS_MAX = 1ull << 14;
constexpr uint32_t DDS_PER = 512;     // operations per range aimed at
constexpr int DDS_TAB = 4096;         // table entries (32 KiB)
constexpr int DDS_LIST = 6080;        // records held (with the table 80 KiB at most, see BESIDE_LDS)
// the executor's blocks
constexpr uint64_t DDS_EXEC_MAX = 1ull << 14;
constexpr int DDS_EXEC_TAB = 2048;
constexpr int DDS_EXEC_LIST = 1024;
constexpr int DDS_LOADS = 8;          // keys in flight per thread
// and of a mixed batch, whose types are in flight too: with 8 the kernel takes 42
// registers, and 16 waves of more than 40 have no room beside a resident executor
constexpr int DDS_MIXED_LOADS = 7;
static_assert(DDS_MAX < (1ull << 31), "an index shares a word with the type bit");

struct DdsArgs {
  const uint8_t *ops;
  const uint32_t *keys;
  uint8_t *win;
  uint32_t n, mode, bits;  // 2^bits ranges
};

// Range hash of a key: a bijection, whose top bits pick the range; its low bits
// pick the slot in a range's table.  (The key times an odd constant put some
// arithmetic progressions of keys into one range: 12,000 such keys took 460 us
// in the one-launch form, 64 spread out.)
__device__ __forceinline__ uint32_t dds_hash(uint32_t k) { return mix32(k); }

__device__ __forceinline__ uint32_t dds_range(uint32_t k, uint32_t bits) {
  return bits ? dds_hash(k) >> (32 - bits) : 0u;
}

template <int TAB, int LIST>
struct DdsShared {
  uint64_t tab[TAB];
  uint64_t list[LIST];
  uint32_t count, claims;
};

// Record e (key << 32 | type << 31 | index) into the table.
template <int TAB>
__device__ __forceinline__ void dds_settle(uint64_t *tab, uint64_t e, bool keep_last, uint32_t *claims) {
  const uint32_t k = (uint32_t)(e >> 32);
  for (uint32_t s = mix32(k) & (TAB - 1);; s = (s + 1) & (TAB - 1)) {
    uint64_t cur = *(volatile uint64_t *)&tab[s];
    if (cur == EMPTY) {
      cur = atomicCAS((unsigned long long *)&tab[s], (unsigned long long)EMPTY, (unsigned long long)e);
      if (cur == EMPTY) {
        if (claims) atomicAdd(claims, 1u);
        return;
      }
    }
    if ((uint32_t)(cur >> 32) == k) {
      // only an update that can change the word (a hot
      // key's later occurrences mostly lose, and atomics on one word serialize)
      if (keep_last) {
        if (cur < e) atomicMax((unsigned long long *)&tab[s], (unsigned long long)e);
      } else if (cur > e) {
        atomicMin((unsigned long long *)&tab[s], (unsigned long long)e);
      }
      return;
    }
  }
}

// Whether record e is the one its key's table word kept.
template <int TAB>
__device__ __forceinline__ bool dds_kept(const uint64_t *tab, uint64_t e) {
  const uint32_t k = (uint32_t)(e >> 32);
  uint32_t s = mix32(k) & (TAB - 1);
  while ((uint32_t)(tab[s] >> 32) != k) s = (s + 1) & (TAB - 1);
  return tab[s] == e;
}

// Operations base + j * NT + thread of the batch as records, EMPTY
// where there is none to record or its key is outside [lo, lo + width).
template <int NT, int U>
__device__ __forceinline__ void dds_read(const DdsArgs &d, uint32_t base, uint32_t lo, uint64_t width, uint64_t *e) {
  uint32_t k[U], o[U];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const uint32_t i = base + j * NT + threadIdx.x;
    k[j] = i < d.n ? d.keys[i] : 0u;
    o[j] = (d.mode == OP_MIXED && i < d.n) ? d.ops[i] : d.mode;
  }
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const uint32_t i = base + j * NT + threadIdx.x;
    // a mixed batch's deletes carry the type bit: the key sets of the types are
    // disjoint by contract, so one table takes both
    const uint32_t ty = (d.mode == OP_MIXED && o[j] == OP_DELETE) ? 1u : 0u;
    const bool rec = (o[j] == OP_INSERT || o[j] == OP_DELETE) && valid_key(k[j]) &&
                     dds_hash(k[j]) - lo <= (uint32_t)(width - 1);
    e[j] = rec ? ((uint64_t)k[j] << 32) | (ty << 31) | i : EMPTY;
  }
}

// Range `range` of the batch, by a block of NT threads (every one calls it).
template <int NT, int U, int TAB, int LIST>
__device__ __forceinline__ void dds_range_of(const DdsArgs &d, uint32_t range, DdsShared<TAB, LIST> &sh) {
  constexpr uint32_t CAP = TAB * 5 / 8;
  static_assert(CAP + NT < TAB, "one claim per thread past the limit still leaves EMPTY words");
  uint64_t *tab = sh.tab, *list = sh.list;
  const int lane = threadIdx.x & 63;
  // inserts keep the last occurrence (type 0 of a mixed batch), deletes the first
  const auto keep_last = [&](uint64_t e) { return d.mode == OP_MIXED ? ((uint32_t)e >> 31) == 0 : d.mode == OP_INSERT; };
  const uint64_t whole = 1ull << (32 - d.bits), first = (uint64_t)range * whole, last = first + whole;
  uint64_t lo = first, width = whole;
  while (lo < last) {
    width = min(width, last - lo);
    for (int j = threadIdx.x; j < TAB; j += NT) tab[j] = EMPTY;
    if (threadIdx.x == 0) sh.count = sh.claims = 0;
    __syncthreads();
    for (uint32_t base = 0; base < d.n; base += U * NT) {
      uint64_t e[U], m[U];
      dds_read<NT, U>(d, base, (uint32_t)lo, width, e);
      uint32_t c = 0;
#pragma unroll
      for (int j = 0; j < U; ++j) {
        m[j] = ballot(e[j] != EMPTY);
        c += (uint32_t)__popcll(m[j]);
      }
      if (c == 0) continue;
      uint32_t at = 0;
      if (lane == 0) at = atomicAdd(&sh.count, c);
      at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
      for (int j = 0; j < U; ++j) {
        if (e[j] != EMPTY) {
          const uint32_t pos = at + rank_below(m[j]);
          if (pos < LIST)
            list[pos] = e[j];
          else if (*(volatile uint32_t *)&sh.claims <= CAP)
            dds_settle<TAB>(tab, e[j], keep_last(e[j]), &sh.claims);
        }
        at += (uint32_t)__popcll(m[j]);
      }
    }
    __syncthreads();
    const uint32_t held = min(sh.count, (uint32_t)LIST);
    const bool spilled = sh.count > LIST;
    for (uint32_t t = threadIdx.x; t < held; t += NT)
      if (*(volatile uint32_t *)&sh.claims <= CAP) dds_settle<TAB>(tab, list[t], keep_last(list[t]), &sh.claims);
    __syncthreads();
    const uint32_t claims = sh.claims;
    const bool over = claims > CAP;  // the same in the whole block
    if (!over) {
      for (uint32_t t = threadIdx.x; t < held; t += NT) {
        const uint64_t e = list[t];
        d.win[(uint32_t)e & 0x7FFFFFFFu] = dds_kept<TAB>(tab, e);
      }
      if (spilled) {
        for (uint32_t base = 0; base < d.n; base += U * NT) {
          uint64_t e[U];
          dds_read<NT, U>(d, base, (uint32_t)lo, width, e);
#pragma unroll
          for (int j = 0; j < U; ++j)
            if (e[j] != EMPTY) d.win[(uint32_t)e[j] & 0x7FFFFFFFu] = dds_kept<TAB>(tab, e[j]);
        }
      }
    }
    __syncthreads();  // the table, the list and the counts are free
    if (over) {
      width = (width + 1) / 2;
    } else {
      lo += width;
      if (claims <= CAP / 2) width *= 2;
    }
  }
}

template <uint32_t MODE>
__global__ __launch_bounds__(DDS_BLOCK) void dds_kernel(DdsArgs d) {
  __shared__ DdsShared<DDS_TAB, DDS_LIST> sh;
  d.mode = MODE;  // known when the reads are compiled
  dds_range_of<DDS_BLOCK, MODE == OP_MIXED ? DDS_MIXED_LOADS : DDS_LOADS>(d, blockIdx.x, sh);
}

// ---------------------------------------------------------------------------
// Dedupe of larger batches in two launches, with no global atomics.
//
// Device-scope atomics on random words run at about 26 G/s on this GPU
// however many are in flight (measured: 3.1 M CAS into a 64 MiB set take
// 119 us at one or at eight per thread), so a set in HBM costs at least one
// such atomic per distinct key of a chunk.  Instead:
//   1. chunk: a block collapses the repeats of its chunk in an LDS table (a
//      Zipf(0.99) hot key is about 5% of the operations), sorts the distinct
//      records by hash range in LDS (a counting sort) and writes them, range
//      after range, with the ranges' bounds; the flags of its operations
//      become 1 for the chunk's winners and 0 for the rest;
//   2. resolve: a block per range reads the range's run of every chunk and
//      settles the records in an LDS table.  Whichever of two records of one
//      key loses is known when they meet, and its flag is cleared then, so
//      there is no second pass over the records.
// P1 then reads one flag byte per operation, coalesced.  The records are
// written once and read once, in runs.  (Staging them by chunk, prefix sums
// over chunks in two launches and a scatter to whole partitions before a
// resolve of two passes took five launches, and partitions of more distinct
// keys than their tables a set in HBM.)  Time at 2^16, 2^18 and 2^20 inserts
// of 2^20 keys: 18, 21 and 39 us (five launches: 49, 51 and 62 us); at 2^22, 2^24,
// 2^26 and 2^28 distinct keys: 0.12, 0.56, 5.3 and 29.7 ms (0.49, 1.80, 7.9 and
// 34.2).  Slower is only a batch of 2^25 operations and more whose keys repeat
// dozens of times: 2^26 and 2^28 on 2^20 keys 2.91 and 10.7 ms (2.54 and 8.9); whole
// inserts of them are not (3.69 and 13.8 ms for 3.99 and 14.4), deletes are (3.62
// and 13.2 for 3.30 and 11.7).  Bound by LDS atomics
// and the latency between the phases of a block.
//
// Inserts and deletes of a mixed batch share the ranges; bit 31 of a record
// is the type, so a mixed batch of 2^31 operations and more runs once per
// type (`only`).  A range with more distinct keys than the table takes is
// worked through in sub-ranges, as in dds_kernel; beyond 2^24 operations that
// is the ordinary course.  Runs get short with many ranges (one record from 2^24 on), but
// the runs of neighbouring ranges share cache lines, and the neighbours run
// on one XCD at about the same time.
// ---------------------------------------------------------------------------
constexpr int DDR_BLOCK = 1024;
constexpr int DDR_BINS = 512;       // most hash ranges of batches of up to 2^20 operations,
constexpr int DDR_BINS_MID = 1024;  // of up to DDR_MORE
constexpr int DDR_BINS_BIG = 4096;  // and beyond
constexpr uint64_t DDR_MORE = 1ull << 22;

struct DdrArgs {
  const uint8_t *ops;
  const uint32_t *keys;
  uint8_t *win;
  uint64_t *rec;     // chunk c's records from c * chunk on, sorted by range
  uint32_t *bounds;  // [chunk][range]: first record of the range's run | its end << 16
  uint64_t *set, *used;         // ddr_set's words (2 n), and how many of them are taken
  uint32_t n, mode, bits, nch;  // 2^bits ranges, nch chunks
  uint32_t only;                // OP_NONE, or the one type of a mixed batch to record
};

// Whether index words carry the type in bit 31, and the mask of their index.
__device__ __forceinline__ bool ddr_typed(const DdrArgs &d) { return d.mode == OP_MIXED && d.only == OP_NONE; }
__device__ __forceinline__ uint32_t ddr_index(const DdrArgs &d, uint64_t e) {
  return (uint32_t)e & (ddr_typed(d) ? 0x7FFFFFFFu : ~0u);
}
// The last occurrence of an insert wins, the first of a delete.
__device__ __forceinline__ bool ddr_keep_last(const DdrArgs &d, uint64_t e) {
  return ddr_typed(d) ? ((uint32_t)e >> 31) == 0 : (d.only == OP_NONE ? d.mode : d.only) == OP_INSERT;
}

// Slot of key k in a chunk's or range's table (not by the hash's top bits: those of a range
// share them), and the next one.
template <uint32_t TAB>
__device__ __forceinline__ uint32_t ddr_slot(uint32_t k) {
  if constexpr ((TAB & (TAB - 1)) == 0) return dds_hash(k) & (TAB - 1);
  else return (dds_hash(k) & 0xFFFFu) * TAB >> 16;
}
template <uint32_t TAB>
__device__ __forceinline__ uint32_t ddr_next(uint32_t s) {
  if constexpr ((TAB & (TAB - 1)) == 0) return (s + 1) & (TAB - 1);
  else return s + 1 < TAB ? s + 1 : 0;
}

template <int PER, int BINS>
__global__ __launch_bounds__(DDR_BLOCK) void ddr_chunk_kernel(DdrArgs d) {
  constexpr int Q = BINS > DDR_BLOCK ? BINS / DDR_BLOCK : 1;  // ranges per thread of the prefix sums
  constexpr int SCAN = BINS / Q;                              // threads that take part
  constexpr uint32_t CH = (uint32_t)DDR_BLOCK * PER, MOST = (BESIDE_LDS - BINS * 4 - 128) / 8,
                     TAB = 2 * CH < MOST ? 2 * CH : MOST;
  static_assert(TAB >= CH + CH / 4, "at most 80% full");
  static_assert(CH < 65536, "run bounds are 16 bits");
  __shared__ uint64_t tab[TAB];
  __shared__ uint32_t cnt[BINS], part[SCAN / 64];
  const uint64_t base = (uint64_t)blockIdx.x * CH;
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
  const uint32_t nb = 1u << d.bits;
  if (blockIdx.x == 0 && tid == 0) *d.used = 0;
  uint32_t kk[PER];
  int ty[PER];  // 0, or 1 for a mixed batch's deletes; -1: not recorded
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const uint64_t i = base + j * DDR_BLOCK + tid;
    ty[j] = -1;
    kk[j] = 0;
    if (i < d.n) {
      kk[j] = d.keys[i];
      if (d.mode != OP_MIXED) {
        ty[j] = 0;
      } else {
        const uint32_t o = d.ops[i];
        if (d.only != OP_NONE) ty[j] = o == d.only ? 0 : -1;
        else ty[j] = o == OP_INSERT ? 0 : (o == OP_DELETE ? 1 : -1);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < PER; ++j)
    if (ty[j] >= 0) d.win[base + j * DDR_BLOCK + tid] = 0;
  for (uint32_t j = tid; j < TAB; j += DDR_BLOCK) tab[j] = EMPTY;
  for (int j = tid; j < BINS; j += DDR_BLOCK) cnt[j] = 0;
  __syncthreads();
  uint32_t slot[PER];  // the table slot this operation claimed, TAB when none
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    slot[j] = TAB;
    const uint32_t k = kk[j];
    if (ty[j] < 0 || !valid_key(k)) continue;
    const uint64_t e = ((uint64_t)k << 32) | ((uint32_t)ty[j] << 31) | (uint32_t)(base + j * DDR_BLOCK + tid);
    const bool keep_last = ddr_keep_last(d, e);
    for (uint32_t s = ddr_slot<TAB>(k);; s = ddr_next<TAB>(s)) {
      uint64_t cur = tab[s];
      if (cur == EMPTY) {
        cur = atomicCAS((unsigned long long *)&tab[s], (unsigned long long)EMPTY, (unsigned long long)e);
        if (cur == EMPTY) {
          slot[j] = s;
          break;
        }
      }
      if ((uint32_t)(cur >> 32) == k) {
        // only an update that can change the word (a hot key's later
        // occurrences mostly lose, and atomics on one word serialize)
        if (keep_last) {
          if (cur < e) atomicMax((unsigned long long *)&tab[s], (unsigned long long)e);
        } else if (cur > e) {
          atomicMin((unsigned long long *)&tab[s], (unsigned long long)e);
        }
        break;
      }
    }
  }
  __syncthreads();
  // claimants take their key's record, as the collapse left it, and its rank
  // in its range
  uint64_t rec[PER];
  uint32_t rank[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    rec[j] = slot[j] < TAB ? tab[slot[j]] : EMPTY;
    if (rec[j] != EMPTY) rank[j] = atomicAdd(&cnt[dds_range((uint32_t)(rec[j] >> 32), d.bits)], 1u);
  }
  __syncthreads();  // counts complete; the table may be overwritten
  uint32_t own[Q], mine = 0, incl = 0;
  if (tid < SCAN) {
#pragma unroll
    for (int q = 0; q < Q; ++q) mine += own[q] = cnt[tid * Q + q];
    incl = mine;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(incl, o, 64);
      if (lane >= o) incl += y;
    }
    if (lane == 63) part[wv] = incl;
  }
  __syncthreads();
  if (tid < SCAN) {
    uint32_t start = incl - mine;
    for (int w = 0; w < wv; ++w) start += part[w];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const uint32_t x = tid * Q + q;
      cnt[x] = start;
      if (x < nb) d.bounds[(uint64_t)blockIdx.x * nb + x] = start | ((start + own[q]) << 16);
      start += own[q];
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < PER; ++j)
    if (rec[j] != EMPTY) {
      tab[cnt[dds_range((uint32_t)(rec[j] >> 32), d.bits)] + rank[j]] = rec[j];
      d.win[ddr_index(d, rec[j])] = 1;  // within this chunk's flags, cleared before a barrier
    }
  uint32_t total = 0;
#pragma unroll
  for (int w = 0; w < SCAN / 64; ++w) total += part[w];
  __syncthreads();
  for (uint32_t t = tid; t < total; t += DDR_BLOCK) d.rec[base + t] = tab[t];
}

// The records of chunk c in the block's range: c's run, read by the LANES lanes
// of one group, `body` on each (false: stop).
template <int LANES, uint32_t CH, typename F>
__device__ __forceinline__ void ddr_run(const DdrArgs &d, uint32_t c, uint32_t b, F body) {
  constexpr int LOADS = LANES <= 2 ? 4 : 2;  // reads in flight
  const uint32_t be = d.bounds[((uint64_t)c << d.bits) + b], end = be >> 16;
  const uint64_t *run = d.rec + (uint64_t)c * CH;
  for (uint32_t t0 = (be & 0xFFFFu) + threadIdx.x % LANES; t0 < end; t0 += LANES * LOADS) {
    uint64_t es[LOADS];
#pragma unroll
    for (int u = 0; u < LOADS; ++u) es[u] = t0 + u * LANES < end ? run[t0 + u * LANES] : EMPTY;
#pragma unroll
    for (int u = 0; u < LOADS; ++u)
      if (es[u] != EMPTY && !body(es[u])) return;
  }
}

// Whether record e is in [lo, lo + width) of its range's hash values.
__device__ __forceinline__ bool ddr_in(uint64_t e, uint64_t lo, uint64_t width) {
  return (uint64_t)(dds_hash((uint32_t)(e >> 32)) - (uint32_t)lo) < width;
}

// Of two records of one key, whether e beats cur.
__device__ __forceinline__ bool ddr_beats(const DdrArgs &d, uint64_t e, uint64_t cur) {
  return ddr_keep_last(d, e) ? cur < e : cur > e;
}

// The records from lo on of range b settled in an open-addressed set in HBM, of
// twice as many words as records (all ranges together: at most 2 n).
template <int LANES, uint32_t CH>
__device__ __forceinline__ void ddr_set(const DdrArgs &d, uint32_t b, uint64_t lo, uint64_t last) {
  __shared__ unsigned long long s_n, s_at;
  if (threadIdx.x == 0) s_n = 0;
  __syncthreads();
  uint64_t mine = 0;
  for (uint32_t c = threadIdx.x / LANES; c < d.nch; c += DDR_BLOCK / LANES)
    ddr_run<LANES, CH>(d, c, b, [&](uint64_t e) {
      mine += ddr_in(e, lo, last - lo) ? 1 : 0;
      return true;
    });
  if (mine) atomicAdd(&s_n, (unsigned long long)mine);
  __syncthreads();
  const uint64_t m = 2 * s_n;
  if (threadIdx.x == 0) s_at = add64(d.used, m);
  __syncthreads();
  uint64_t *set = d.set + s_at;
  for (uint64_t t = threadIdx.x; t < m; t += DDR_BLOCK)
    __hip_atomic_store(&set[t], EMPTY, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  for (uint32_t c = threadIdx.x / LANES; c < d.nch; c += DDR_BLOCK / LANES)
    ddr_run<LANES, CH>(d, c, b, [&](uint64_t e) {
      if (!ddr_in(e, lo, last - lo)) return true;
      const uint32_t k = (uint32_t)(e >> 32);
      // (not by the range hash: a range's keys share its top bits)
      for (uint64_t s = __umul64hi((uint64_t)(k * 0x9E3779B1u) << 32, m);; s = s + 1 == m ? 0 : s + 1) {
        uint64_t cur = load_fresh(&set[s]);
        if (cur == EMPTY) {
          cur = cas64(&set[s], EMPTY, e);
          if (cur == EMPTY) return true;
        }
        if ((uint32_t)(cur >> 32) != k) continue;
        if (ddr_beats(d, e, cur))
          cur = ddr_keep_last(d, e)
                    ? __hip_atomic_fetch_max(&set[s], e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                    : __hip_atomic_fetch_min(&set[s], e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        d.win[ddr_index(d, ddr_beats(d, e, cur) ? cur : e)] = 0;
        return true;
      }
    });
}

// The table is sized for the records of a range: up to about 2,048 of the
// smaller batches, 4,096 beyond 2^20 operations.  LANES lanes read one chunk's run
// together: eight where runs are eight records or more; beyond 2^23
// operations runs are short and there are thousands of chunks, and the
// dependent reads of bounds and records take the time; lanes that read
// neighbouring chunks clear flags that share cache lines (with chunks and tables
// twice as large, eight, four, two and one lanes: 2^26 distinct keys 4.31, 3.11,
// 2.87 and 2.80 ms, 2^26 operations on 2^20 keys 3.19, 3.02, 2.95 and 3.08).
//
// A pass reads the whole range, so a range of many sub-ranges would take time
// quadratic in its records (2^20 operations on 2^16 keys of one range: 34 ms).
// Once more than DDR_PASSES passes are ahead, the rest of the range goes to
// ddr_set, whose atomics take about the time of that many passes (the same
// batch 4.1 ms, in one block; beyond 2^29 distinct keys every range).
// With DDR_BINS_BIG all ranges grow alike, and the line lies where their passes
// take as long as the set
// (2^28 distinct keys: 85 ms in passes alone, 30 so).
constexpr uint64_t DDR_PASSES = 24;
constexpr uint64_t DDR_PASSES_BIG = 6;
template <int PER, int BINS, int LANES>
__global__ __launch_bounds__(DDR_BLOCK) void ddr_resolve_kernel(DdrArgs d) {
  constexpr uint32_t CH = (uint32_t)DDR_BLOCK * PER;
  constexpr uint32_t TAB = BINS > DDR_BINS ? (BESIDE_LDS - 256) / 8 : 4096;
  constexpr uint32_t CAP = TAB * 3 / 4;
  static_assert(CAP + DDR_BLOCK < TAB + 1, "at most one claim per thread past the limit");
  __shared__ uint64_t tab[TAB];
  __shared__ uint32_t s_claims;
  const uint32_t nb = 1u << d.bits;
  // neighbouring ranges on one XCD (blocks go to the XCDs in turn): their
  // bounds share cache lines
  const uint32_t b = nb >= 8 ? (blockIdx.x & 7) * (nb >> 3) + (blockIdx.x >> 3) : blockIdx.x;
  const uint64_t whole = 1ull << (32 - d.bits), first = (uint64_t)b * whole, last = first + whole;
  uint64_t lo = first, width = whole;
  if constexpr (BINS == DDR_BINS_BIG) {
    // The first width: the whole range where keys repeat, by a sample of up to
    // 1,024 records of as many chunks (of 4,096 keys, 88% of the sample are
    // distinct, of 7,656 94%); else so that the records it may hold fit.
    const uint64_t per = (uint64_t)d.n >> d.bits;  // records, at most about that many
    if (per > CAP) {
      __shared__ uint32_t s_sample, s_distinct;
      for (uint32_t j = threadIdx.x; j < TAB; j += DDR_BLOCK) tab[j] = EMPTY;
      if (threadIdx.x == 0) s_sample = s_distinct = 0;
      __syncthreads();
      bool have = false, fresh = false;
      if (threadIdx.x < d.nch)
        ddr_run<1, CH>(d, (uint32_t)((uint64_t)threadIdx.x * d.nch / min(d.nch, (uint32_t)DDR_BLOCK)), b, [&](uint64_t e) {
          have = true;
          for (uint32_t s = ddr_slot<TAB>((uint32_t)(e >> 32));; s = ddr_next<TAB>(s)) {
            const uint64_t cur =
                atomicCAS((unsigned long long *)&tab[s], (unsigned long long)EMPTY, (unsigned long long)(e | 0xFFFFFFFFu));
            if (cur == EMPTY) fresh = true;
            if (cur == EMPTY || (uint32_t)(cur >> 32) == (uint32_t)(e >> 32)) return false;
          }
        });
      const uint64_t hm = ballot(have), fm = ballot(fresh);
      if ((threadIdx.x & 63) == 0) {
        atomicAdd(&s_sample, (uint32_t)__popcll(hm));
        atomicAdd(&s_distinct, (uint32_t)__popcll(fm));
      }
      __syncthreads();
      if ((uint64_t)s_distinct * 8 > (uint64_t)s_sample * 7)
        for (uint64_t r = per; r > CAP; r /= 2) width = (width + 1) / 2;
    }
  }
  // chunks from the end that holds the winners: most later records of a key
  // lose to what the table holds, by a load instead of an atomic
  const bool backwards = ddr_typed(d) || (d.only == OP_NONE ? d.mode : d.only) == OP_INSERT;
  while (lo < last) {
    width = min(width, last - lo);
    for (uint32_t j = threadIdx.x; j < TAB; j += DDR_BLOCK) tab[j] = EMPTY;
    if (threadIdx.x == 0) s_claims = 0;
    __syncthreads();
    for (uint32_t c0 = threadIdx.x / LANES; c0 < d.nch; c0 += DDR_BLOCK / LANES) {
      if (*(volatile uint32_t *)&s_claims > CAP) break;
      ddr_run<LANES, CH>(d, backwards ? d.nch - 1 - c0 : c0, b, [&](uint64_t e) {
        if (!ddr_in(e, lo, width)) return true;
        if (*(volatile uint32_t *)&s_claims > CAP) return false;
        const uint32_t k = (uint32_t)(e >> 32);
        const bool keep_last = ddr_keep_last(d, e);
        for (uint32_t s = ddr_slot<TAB>(k);; s = ddr_next<TAB>(s)) {
          uint64_t cur = *(volatile uint64_t *)&tab[s];
          if (cur == EMPTY) {
            cur = atomicCAS((unsigned long long *)&tab[s], (unsigned long long)EMPTY, (unsigned long long)e);
            if (cur == EMPTY) {
              atomicAdd(&s_claims, 1u);
              return true;
            }
          }
          if ((uint32_t)(cur >> 32) != k) continue;
          // two records of one key: the loser's flag goes (a record met
          // again after its range was split loses to the same records)
          if (keep_last ? cur < e : cur > e)
            cur = keep_last ? atomicMax((unsigned long long *)&tab[s], (unsigned long long)e)
                            : atomicMin((unsigned long long *)&tab[s], (unsigned long long)e);
          const uint64_t loser = (keep_last ? cur < e : cur > e) ? cur : e;
          d.win[ddr_index(d, loser)] = 0;
          return true;
        }
      });
    }
    __syncthreads();
    const uint32_t claims = s_claims;
    const bool over = claims > CAP;  // the same in the whole block
    __syncthreads();
    if (over) {
      width = (width + 1) / 2;
    } else {
      lo += width;
      // as wide as fills half the table at this density, two at least
      if (claims <= CAP / 2) width *= claims ? max(2u, CAP / 2 / claims) : CAP;
    }
    if (lo < last && (last - lo) / width > (BINS == DDR_BINS_BIG ? DDR_PASSES_BIG : DDR_PASSES)) {
      ddr_set<LANES, CH>(d, b, lo, last);
      return;
    }
  }
}

__device__ __forceinline__ bool dedupe_winner(const uint64_t *dd, uint64_t mask, uint32_t k, uint32_t i) {
  uint64_t s = mix32(k) & mask;
  for (uint64_t probe = 0; probe <= mask; ++probe) {
    const uint64_t cur = dd[s];
    if ((uint32_t)(cur >> 32) == k) return (uint32_t)cur == i;
    if (cur == EMPTY) return true;
    s = (s + 1) & mask;
  }
  return true;
}

// ---------------------------------------------------------------------------
// P1 helpers
// ---------------------------------------------------------------------------

// One probe round of match-and-elect.  Operations t < count of the round
// have their key and bucket in keys[t], bkts[t] and their owning lane in
// list[t] (t itself when list is null).  Each 16-lane group loads one bucket
// per wave-wide load and publishes, through LDS and indexed by the owning
// lane, the match mask, the empty-slot mask and the word of the lowest
// matching slot.  All loads of a chunk are issued before any is consumed.
// bkts[] holds 64 entries: entries from `count` on repeat the round's last
// bucket (the caller pads them), so idle group slots re-load a line that is
// loaded anyway, their result is ignored, and the loads need neither
// control flow nor clamped indices.
// PIPE: wave-wide loads in flight per chunk (the probe's pipelining depth).
template <int S, int PIPE = Traits<S>::CH>
__device__ __forceinline__ void probe_round(const uint64_t *__restrict__ buckets, const uint32_t *keys,
                                            const uint32_t *bkts, const uint8_t *list, int count,
                                            typename Traits<S>::Mask *m_out, typename Traits<S>::Mask *e_out,
                                            uint64_t *w_out, int g, int sl) {
  using T = Traits<S>;
  using Mask = typename T::Mask;
  for (int base = 0; base < count; base += PIPE * T::G) {
    uint64_t w[PIPE];
#pragma unroll
    for (int j = 0; j < PIPE; ++j) w[j] = buckets[(uint64_t)bkts[base + j * T::G + g] * S + sl];
    // keep the operands of the consume loop from being read (and held in
    // registers) while the loads are in flight
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < PIPE; ++j) {
      const int t = base + j * T::G + g;
      const bool mine = t < count;
      const uint32_t ko = keys[t];
      const uint64_t mm = ballot(mine && ko != 0u && key_of(w[j]) == ko);
      const uint64_t ee = ballot(w[j] == EMPTY);
      const Mask gm = (Mask)((mm >> (g * S)) & T::FULL);
      const Mask ge = (Mask)((ee >> (g * S)) & T::FULL);
      if (mine) {
        const int o = list ? list[t] : t;
        if (sl == 0) {
          m_out[o] = gm;
          e_out[o] = ge;
        }
        if (gm != 0 && sl == ctz_mask(gm)) w_out[o] = w[j];
      }
    }
  }
}

// Both probe rounds of an insert batch at once (S = 16): PIPE loads for the
// first candidates and PIPE for the second are in flight together (with
// PIPE = 16 one chunk covers the wave's 64 operations).
template <int S, int PIPE = Traits<S>::CH>
__device__ __forceinline__ void probe_round_pair(const uint64_t *__restrict__ buckets, const uint32_t *keys1,
                                                 const uint32_t *bkts1, typename Traits<S>::Mask *m1_out,
                                                 typename Traits<S>::Mask *e1_out, uint64_t *w1_out,
                                                 const uint32_t *keys2, const uint32_t *bkts2, const uint8_t *list2,
                                                 int count2, typename Traits<S>::Mask *m2_out,
                                                 typename Traits<S>::Mask *e2_out, uint64_t *w2_out, int g, int sl) {
  using T = Traits<S>;
  using Mask = typename T::Mask;
  static_assert(S == 16, "the fused round is built for 16-slot buckets");
  for (int base = 0; base < 64; base += PIPE * T::G) {
    uint64_t wa[PIPE], wb[PIPE];
#pragma unroll
    for (int j = 0; j < PIPE; ++j) wa[j] = buckets[(uint64_t)bkts1[base + j * T::G + g] * S + sl];
#pragma unroll
    for (int j = 0; j < PIPE; ++j) wb[j] = buckets[(uint64_t)bkts2[base + j * T::G + g] * S + sl];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < PIPE; ++j) {
      const int t = base + j * T::G + g;
      const uint32_t ko = keys1[t];
      const uint64_t mm = ballot(ko != 0u && key_of(wa[j]) == ko);
      const uint64_t ee = ballot(wa[j] == EMPTY);
      const Mask gm = (Mask)((mm >> (g * S)) & T::FULL);
      if (sl == 0) {
        m1_out[t] = gm;
        e1_out[t] = (Mask)((ee >> (g * S)) & T::FULL);
      }
      if (gm != 0 && sl == ctz_mask(gm)) w1_out[t] = wa[j];
    }
#pragma unroll
    for (int j = 0; j < PIPE; ++j) {
      const int t = base + j * T::G + g;
      const bool mine = t < count2;
      const uint32_t ko = mine ? keys2[t] : 0u;
      const uint64_t mm = ballot(mine && ko != 0u && key_of(wb[j]) == ko);
      const uint64_t ee = ballot(wb[j] == EMPTY);
      const Mask gm = (Mask)((mm >> (g * S)) & T::FULL);
      if (mine) {
        const int o = list2[t];
        if (sl == 0) {
          m2_out[o] = gm;
          e2_out[o] = (Mask)((ee >> (g * S)) & T::FULL);
        }
        if (gm != 0 && sl == ctz_mask(gm)) w2_out[o] = wb[j];
      }
    }
  }
}

__device__ __forceinline__ bool hinted(const uint32_t *hint, uint32_t c1, uint32_t c2) {
  return ((hint[c1 >> 5] >> (c1 & 31)) & 1u) | ((hint[c2 >> 5] >> (c2 & 31)) & 1u);
}

// Lane-wise search of the stash and the pending list.  The stash is an
// open-addressed table (linear probing from mix32(key)); a search ends at
// the key or at an EMPTY word (tombstones keep probe runs intact).
__device__ __forceinline__ uint64_t *overflow_find(uint64_t *stash, uint64_t stash_cap, uint64_t n_stash,
                                                   uint64_t *pending, uint64_t n_pend, uint32_t k, uint64_t *word,
                                                   bool fresh) {
  if (n_stash) {
    const uint64_t mask = stash_slots_for(stash_cap) - 1;
    for (uint64_t i = 0, p = mix32(k) & mask; i <= mask; ++i, p = (p + 1) & mask) {
      const uint64_t x = fresh ? load_fresh(stash + p) : stash[p];
      if (x == EMPTY) break;
      if (key_of(x) == k) {
        *word = x;
        return stash + p;
      }
    }
  }
  for (uint64_t p = 0; p < n_pend; ++p) {
    const uint64_t x = fresh ? load_fresh(pending + p) : pending[p];
    if (key_of(x) == k) {
      *word = x;
      return pending + p;
    }
  }
  return nullptr;
}

// The second-candidate round's operand list: the operations that need it,
// compacted in lane order (key, bucket, owning lane), and the rest of the 64
// entries padded with the last listed bucket (with lane 0's first bucket when
// the list is empty).
__device__ __forceinline__ void compact_second(bool need2, uint64_t need2_mask, int n2, uint32_t k, uint32_t c2,
                                               uint32_t c1, int lane, uint32_t *k2, uint32_t *b2, uint8_t *list) {
  const uint32_t pad = n2 > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)c2, 63 - __builtin_clzll(need2_mask))
                              : (uint32_t)__builtin_amdgcn_readlane((int)c1, 0);
  if (need2) {
    const uint32_t r = rank_below(need2_mask);
    k2[r] = k;
    b2[r] = c2;
    list[r] = (uint8_t)lane;
  }
  if (lane >= n2) b2[lane] = pad;
}

// ---------------------------------------------------------------------------
// P1: hash, probe, and replace / lookup / delete / claim.
// ---------------------------------------------------------------------------
// LDS of one block of the probe phase (per wave: 64 operations).
// D: candidate buckets per key (a round of results per candidate).
template <int S, int D = 2>
struct OpsShared {
  using Mask = typename Traits<S>::Mask;
  uint32_t key[WAVES][64];
  uint32_t b1[WAVES][64];
  uint32_t k2[WAVES][64];  // rounds 2 (and 3), compacted: key, bucket, owner
  uint32_t b2[WAVES][64];
  uint8_t list[WAVES][64];
  Mask m[D][WAVES][64];
  Mask e[D][WAVES][64];
  uint64_t w[D][WAVES][64];
};

// The table state a probe tile needs, read once per launch (or per chunk of
// the persistent executor).
struct OpsView {
  Geo geo;
  uint64_t n_stash, n_pend;
  bool removed;  // an entry may have been deleted since the table was empty
  SpillState spill;
};

__device__ __forceinline__ OpsView read_view(const Ctl *c, uint64_t stash_cap, uint64_t pending_cap,
                                             const Spill &spill, uint64_t n) {
  OpsView v;
  v.geo = read_geo(c);
  v.n_stash = min(ld_ctl(&c->stash_count), stash_cap);
  v.n_pend = min(ld_ctl(&c->pending_count), pending_cap);
  v.removed = ld_ctl32(&c->removed) != 0;
  v.spill = spill_state(spill, c, n);
  return v;
}

// A wave's key-count change and reserved-key count, added to shard
// unit % NSHARD by its first lane.
__device__ __forceinline__ void ops_counts_add(Ctl *c, uint64_t unit, int64_t live_acc, uint64_t bad_acc) {
  if ((threadIdx.x & 63) == 0) {
    Shard *shd = shard_of(c, unit % NSHARD);
    if (live_acc != 0) add64(&shd->live, (uint64_t)live_acc);
    if (bad_acc) add64(&shd->invalid_keys, bad_acc);
  }
}

// Entries may be deleted by this launch: later ones read the filter even where
// a first candidate has room.
__device__ __forceinline__ void set_removed(Ctl *c) {
  __hip_atomic_store(&c->removed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The end of a probe launch or phase, by one thread: what it did to the filter
// (`filter`: it was given one).  Deletes are noted without one, too: replayed
// launches may have cleared the table and filled it with a filter again since
// the host dropped it.
template <uint32_t MODE>
__device__ __forceinline__ void ops_done(Ctl *c, const OpsView &view, bool filter) {
  if ((MODE == OP_MIXED || MODE == OP_DELETE) && !view.removed) set_removed(c);
  if ((MODE == OP_MIXED || MODE == OP_INSERT) && (!filter || view.spill.plain) && !view.spill.dropped)
    __hip_atomic_store(&c->dropped, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// P1 for one tile of WAVES x 64 operations [tile * 256, tile * 256 + 256).
// BOTH: probe both candidates in one round for every operation (inserts of
// new keys always need both; for lookups and deletes it trades bytes for one
// memory round trip fewer).
// PAIR: the table's candidate hashes (HashPair); BitHash1/2 by default.
// With three candidates (PAIR_TRIPLE) the third is probed in a third round
// by the operations that found their key in neither of the first two.
// FILTER: the table has a spill filter (FILTER_ASK: it may have one; the
// executor, whose worker holds one copy of each kind of tile).
enum : int { FILTER_NONE = 0, FILTER_USE = 1, FILTER_ASK = 2 };
template <int S, uint32_t MODE, bool BOTH, int PAIR = PAIR_BITHASH, int PIPE = Traits<S>::CH,
          int FILTER = FILTER_NONE>
__device__ __forceinline__ void ops_tile(const OpsArgs &a, const OpsView &view, uint64_t tile,
                                         OpsShared<S, PairArity<PAIR>::D> &sh, int64_t &live_acc,
                                         uint64_t &bad_acc) {
  using T = Traits<S>;
  using Mask = typename T::Mask;
  constexpr bool D3 = PairArity<PAIR>::D == 3;
  auto &s_key = sh.key;
  auto &s_b1 = sh.b1;
  auto &s_k2 = sh.k2;
  auto &s_b2 = sh.b2;
  auto &s_list = sh.list;
  auto &s_m = sh.m;
  auto &s_e = sh.e;
  auto &s_w = sh.w;

  const int wv = (threadIdx.x >> 6) % WAVES, lane = threadIdx.x & 63;
  const int g = lane / S, sl = lane % S;
  const uint64_t i = (tile * WAVES + wv) * 64 + lane;
  const bool active = i < a.n;
  const Geo &geo = view.geo;
  const uint64_t n_stash = view.n_stash, n_pend = view.n_pend;
  const bool overflow_used = (n_stash | n_pend) != 0;

  uint32_t op = OP_NONE, k = 0, v = 0, won = 0;
  if (active) {
    // the batch's inputs and outputs are touched once: non-temporal, so they
    // do not displace bucket lines from the caches (bulk step +0.7%)
    op = (MODE == OP_MIXED) ? (uint32_t)__builtin_nontemporal_load(&a.ops[i]) : MODE;
    k = __builtin_nontemporal_load(&a.keys[i]);
    if (MODE != OP_LOOKUP && a.win) won = __builtin_nontemporal_load(&a.win[i]);  // not written for lookups, nor used
    if (op == OP_INSERT) v = __builtin_nontemporal_load(&a.vals[i]);
  }
  const bool valid = active && op <= OP_LOOKUP && valid_key(k);
  bool work = valid;
  if (work && op != OP_LOOKUP) {
    if (a.win)
      work = won != 0;
    else if (a.dd)
      work = dedupe_winner(a.dd, a.dd_mask, k, (uint32_t)i);
  }
  uint32_t c1 = 0, c2 = 0, c3 = 0;
  if (work) {
    c1 = address(geo, HashPair<PAIR>::h1(k));
    c2 = address(geo, HashPair<PAIR>::h2(k));
    if constexpr (D3) c3 = address(geo, HashPair<PAIR>::h3(k));
  }
  s_key[wv][lane] = work ? k : 0u;
  s_b1[wv][lane] = c1;
  wave_lds_sync();

  // The second candidate is probed after a miss in the first, with a filter
  // by keys that may be there and by new keys whose first candidate is nearly
  // full alone.  Without one inserts of new keys always need both (absence
  // and two-choice placement) and take them in one round, as everything does
  // with BOTH.
  constexpr bool kFused = (BOTH || (MODE == OP_INSERT && FILTER != FILTER_USE)) && (S == 16);
  // spilled: the key may be outside its first candidate; marked: its filter
  // bit is known to be set
  bool spilled = true, marked = false;
  // a plain batch, or one after it, goes without the filter
  const bool filtered = (MODE == OP_LOOKUP || MODE == OP_DELETE) ? !view.spill.dropped : !view.spill.plain;
  const uint32_t first_min = FILTER == FILTER_NONE || filtered ? a.spill.first_min : (uint32_t)S + 1;
  Mask m1;
  bool need2;
  if constexpr (kFused) {
    need2 = work && c2 != c1;
    const uint64_t need2_mask = ballot(need2);
    const int n2 = __popcll(need2_mask);
    compact_second(need2, need2_mask, n2, k, c2, c1, lane, s_k2[wv], s_b2[wv], s_list[wv]);
    wave_lds_sync();
    probe_round_pair<S, PIPE>(a.buckets, s_key[wv], s_b1[wv], s_m[0][wv], s_e[0][wv], s_w[0][wv], s_k2[wv],
                              s_b2[wv], s_list[wv], n2, s_m[1][wv], s_e[1][wv], s_w[1][wv], g, sl);
    wave_lds_sync();
    m1 = s_m[0][wv][lane];
  } else {
    // round 1: first candidate of every operation
    probe_round<S, PIPE>(a.buckets, s_key[wv], s_b1[wv], nullptr, 64, s_m[0][wv], s_e[0][wv], s_w[0][wv], g, sl);
    wave_lds_sync();
    m1 = s_m[0][wv][lane];
    need2 = work && m1 == 0 && c2 != c1;
    if constexpr (FILTER != FILTER_NONE && !D3) {
      if ((FILTER == FILTER_USE || a.spill.bits) && filtered) {
        // the filter is read by the lanes that missed alone, and after the
        // round: read with it, by every lane, it cost more line reads than
        // it saved (2^26 lookups at 50% hits 2.21 ms, against 2.05 so and
        // 2.22 without a filter)
        const bool near_full = (uint32_t)popc_mask(s_e[0][wv][lane]) < first_min;
        // An insert that finds its first candidate near full reads the
        // second whatever the filter says, and skips the filter's own line
        // unless the overflow may hold the key; it may then set a bit that
        // is set.  The line and its wait before the second round cost more
        // than those atomics: a build of 2^26 keys to 95% takes 3.36 ms
        // against 3.74, 7.1 M new keys at 55-65% load 0.38 ms against 0.42
        const bool both = op == OP_INSERT && near_full;
        marked = work && m1 == 0 &&
                 (both ? overflow_used : near_full || MODE == OP_MIXED || MODE == OP_DELETE || view.removed) &&
                 spill_test(a.spill, c1, k);
        spilled = marked;
        need2 = need2 && (spilled || both);
      }
    }
    const uint64_t need2_mask = ballot(need2);
    const int n2 = __popcll(need2_mask);
    compact_second(need2, need2_mask, n2, k, c2, c1, lane, s_k2[wv], s_b2[wv], s_list[wv]);
    wave_lds_sync();
    // round 2: second candidate of the operations that missed in the first
    if (n2 > 0)
      probe_round<S, PIPE>(a.buckets, s_k2[wv], s_b2[wv], s_list[wv], n2, s_m[1][wv], s_e[1][wv], s_w[1][wv], g,
                           sl);
    wave_lds_sync();
  }
  const Mask e1 = s_e[0][wv][lane];
  // with the fused round a match in the first candidate makes the second's
  // result irrelevant; otherwise the second round ran only without one
  const Mask m2 = (need2 && m1 == 0) ? s_m[1][wv][lane] : (Mask)0;
  const Mask e2 = need2 ? s_e[1][wv][lane] : (Mask)0;
  Mask m3 = 0, e3 = 0;
  bool need3 = false;
  if constexpr (D3) {
    // round 3: the third candidate of the operations without a match so far
    need3 = work && m1 == 0 && m2 == 0 && c3 != c1 && c3 != c2;
    const uint64_t need3_mask = ballot(need3);
    const int n3 = __popcll(need3_mask);
    compact_second(need3, need3_mask, n3, k, c3, c1, lane, s_k2[wv], s_b2[wv], s_list[wv]);
    wave_lds_sync();
    if (n3 > 0)
      probe_round<S, PIPE>(a.buckets, s_k2[wv], s_b2[wv], s_list[wv], n3, s_m[2][wv], s_e[2][wv], s_w[2][wv], g,
                           sl);
    wave_lds_sync();
    if (need3) {
      m3 = s_m[2][wv][lane];
      e3 = s_e[2][wv][lane];
    }
  }

  uint32_t out_v = NO_VALUE;
  uint8_t out_f = 0;
  int dl = 0;
  bool to_wl = false;
  const uint64_t kv = pack(k, v);
  if (work) {
    uint64_t *slot = nullptr, word = 0;
    bool in_bucket = false;
    if (m1) {
      slot = a.buckets + (uint64_t)c1 * S + ctz_mask(m1);
      word = s_w[0][wv][lane];
      in_bucket = true;
    } else if (m2) {
      slot = a.buckets + (uint64_t)c2 * S + ctz_mask(m2);
      word = s_w[1][wv][lane];
      in_bucket = true;
    } else if (D3 && m3) {
      slot = a.buckets + (uint64_t)c3 * S + ctz_mask(m3);
      word = s_w[D3 ? 2 : 0][wv][lane];
      in_bucket = true;
    } else if (overflow_used && spilled && (hinted(a.hint, c1, c2) || (D3 && hinted(a.hint, c3, c3)))) {
      slot = overflow_find(a.stash, a.stash_cap, n_stash, a.pending, n_pend, k, &word, false);
    }
    if (op == OP_LOOKUP) {
      if (slot) {
        out_v = value_of(word);
        out_f = 1;
      }
    } else if (slot && in_bucket) {
      // replace (Algorithm 1) or delete (Algorithm 4).  The paper publishes
      // both with one CAS from the word seen; here the word of key k can
      // change only through this operation (no entry moves in this phase,
      // claims only fill EMPTY slots, and a batch gives each key one such
      // operation), so that CAS cannot fail and one 64-bit store does the
      // same: the whole entry is replaced at once and nothing waits for an
      // atomic's return.  The store is an agent-scope atomic one: claims of
      // other XCDs change the same bucket lines in this phase, and a plain
      // store leaves the line dirty in this XCD's L2, whose write-back
      // carries this XCD's stale copy of the neighbouring slots and
      // overwrote such claims (keys inserted by a mixed batch went missing).
      __hip_atomic_store(slot, (op == OP_INSERT) ? kv : EMPTY, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (op == OP_DELETE) {
        out_f = 1;
        dl = -1;
      }
    } else if (slot) {
      // stash or pending entry: the same single-word update, by CAS (rare)
      const uint64_t desired = (op == OP_INSERT) ? kv : TOMB;
      bool done = false;
      for (int attempt = 0; attempt < 4 && slot; ++attempt) {
        if (cas64(slot, word, desired) == word) {
          done = true;
          break;
        }
        atomicOr(&a.ctl->error, ERR_CAS_RETRY);
        slot = overflow_find(a.stash, a.stash_cap, n_stash, a.pending, n_pend, k, &word, true);
      }
      if (op == OP_DELETE && done) {
        out_f = 1;
        dl = -1;
      }
    } else if (op == OP_INSERT) {
      // claim-then-commit (Algorithm 2) in the first candidate while it has
      // room to spare, else in the candidate with more empty slots, ties to
      // the first hash: bucketed two-choice placement (three-choice with
      // three candidates); within a bucket the slots are tried from one
      // picked by the key (claim_slot).  A first candidate that filled up
      // meanwhile, with the second not probed, leaves the key to step 3,
      // which looks at both again
      dl = 1;
      Mask f_first = e1, f_second = (c2 != c1) ? e2 : (Mask)0;
      uint32_t b_first = c1, b_second = c2;
      if (popc_mask(f_second) > popc_mask(f_first) && (D3 || (uint32_t)popc_mask(f_first) < first_min)) {
        const Mask tm = f_first;
        f_first = f_second;
        f_second = tm;
        b_first = c2;
        b_second = c1;
      }
      Mask f_third = 0;
      uint32_t b_third = c3;
      if constexpr (D3) {
        f_third = need3 ? e3 : (Mask)0;
        if (popc_mask(f_third) > popc_mask(f_second)) {
          const Mask tm = f_second;
          f_second = f_third;
          f_third = tm;
          b_third = b_second;
          b_second = c3;
          if (popc_mask(f_second) > popc_mask(f_first)) {
            const Mask t2 = f_first;
            f_first = f_second;
            f_second = t2;
            const uint32_t bt = b_first;
            b_first = b_second;
            b_second = bt;
          }
        }
      }
      bool placed = false;
      while (!placed && (f_first | f_second | f_third)) {
        if (f_first == 0) {
          f_first = f_second;
          b_first = b_second;
          f_second = f_third;
          b_second = b_third;
          f_third = 0;
          continue;
        }
        const int s = claim_slot<S>(f_first, k);
        if (cas64(a.buckets + (uint64_t)b_first * S + s, EMPTY, kv) == EMPTY)
          placed = true;
        else
          f_first &= (Mask)~((Mask)1 << s);
      }
      to_wl = !placed;
      if constexpr (!D3 && FILTER != FILTER_NONE) {
        if (filtered && placed && b_first != c1 && !marked) spill_mark(a.spill, c1, k);
      }
    }
  }

  // eviction worklist: one atomic per wave, on the tile's segment counter
  const uint64_t wl_mask = ballot(to_wl);
  if (wl_mask) {
    const int leader = __builtin_ctzll(wl_mask);
    uint64_t base = 0;
    if (lane == leader) base = wl_append(a.ctl, tile, (uint64_t)__popcll(wl_mask));
    base = read_lane64(base, leader);
    if (to_wl) a.wl[(tile % NSHARD) * a.wl_seg_cap + base + rank_below(wl_mask)] = kv;
  }
  // key count and reserved keys: summed per wave in registers over the
  // wave's tiles (the caller adds them to its shard once: device atomics
  // run at about 26 G/s, and an insert batch already spends one per
  // operation; aggregating the block's waves per tile instead measured 2-4%
  // slower, its two block barriers costing more than the atomics)
  const uint64_t up = ballot(dl > 0), down = ballot(dl < 0), bad = ballot(active && !valid);
  live_acc += (int64_t)__popcll(up) - (int64_t)__popcll(down);
  bad_acc += (uint64_t)__popcll(bad);
  if (active) {
    if (MODE == OP_LOOKUP || MODE == OP_MIXED) {
      if (a.vals_out) __builtin_nontemporal_store(out_v, &a.vals_out[i]);
      if (a.flags_out) __builtin_nontemporal_store(out_f, &a.flags_out[i]);
    } else if (MODE == OP_DELETE) {
      if (a.flags_out) __builtin_nontemporal_store(out_f, &a.flags_out[i]);
    }
  }
}

// WPE: the occupancy target (waves per SIMD) the registers are allocated
// for; PIPE: loads in flight per probe chunk.  Tuned variants of the
// 16-slot BitHash kernels are picked per table (hive_config.probe_tuning).
template <int S, uint32_t MODE, bool BOTH, int PAIR = PAIR_BITHASH, int WPE = OPS_WAVES_PER_EU,
          int PIPE = Traits<S>::CH, int FILTER = FILTER_NONE>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(WPE))) void ops_kernel(OpsArgs a) {
  __shared__ OpsShared<S, PairArity<PAIR>::D> sh;
  const OpsView view = read_view(a.ctl, a.stash_cap, a.pending_cap, a.spill, a.n);
  const uint64_t ntiles = (a.n + BLOCK - 1) / BLOCK;
  int64_t live_acc = 0;
  uint64_t bad_acc = 0;
  for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x)
    ops_tile<S, MODE, BOTH, PAIR, PIPE, FILTER>(a, view, tile, sh, live_acc, bad_acc);
  ops_counts_add(a.ctl, (uint64_t)blockIdx.x * WAVES + (threadIdx.x >> 6), live_acc, bad_acc);
  if (MODE != OP_LOOKUP && blockIdx.x == 0 && threadIdx.x == 0) ops_done<MODE>(a.ctl, view, FILTER != FILTER_NONE);
}

// ---------------------------------------------------------------------------
// Dedupe and P1 of a small batch in one launch.
//
// A small batch's time is its launches and the round trips between them, so
// a block of 8 waves settles the batch's keys in an LDS table (as dds_kernel
// does) and goes on to its two tiles; beyond 512 operations there are two
// blocks, and each settles all keys.  (One block of 16 waves takes as long, but
// has no room beside a resident executor.)  Inserts of 2^6 and 2^10
// operations take 8.6 and 11.5 us against 9.9 and 12.9 in two launches, and
// the host makes one call fewer.  At 2^11 and 2^12 operations, with blocks of
// 16 waves, this was slower (15 us against 13.4, 18 against 13.5).
// ---------------------------------------------------------------------------
constexpr int SMALL_BLOCK = 2 * BLOCK;
constexpr int SMALL_PER = 2;  // operations that a thread settles
constexpr uint64_t SMALL_MAX = SMALL_PER * SMALL_BLOCK;
constexpr int SMALL_TAB = 2 * SMALL_MAX;

template <int S, uint32_t MODE, int FILTER>
__global__ __launch_bounds__(SMALL_BLOCK) void small_batch_kernel(OpsArgs a, uint8_t *win) {
  static_assert(MODE != OP_LOOKUP, "lookups need no dedupe");
  __shared__ union {
    uint64_t tab[SMALL_TAB];
    OpsShared<S> ops[SMALL_BLOCK / BLOCK];
  } sh;
  const uint32_t tid = threadIdx.x;
  for (uint32_t j = tid; j < SMALL_TAB; j += SMALL_BLOCK) sh.tab[j] = EMPTY;
  const DdsArgs d{a.ops, a.keys, win, (uint32_t)a.n, MODE, 0};
  uint64_t e[SMALL_PER];
  dds_read<SMALL_BLOCK, SMALL_PER>(d, 0, 0, 1ull << 32, e);
  const OpsView view = read_view(a.ctl, a.stash_cap, a.pending_cap, a.spill, a.n);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < SMALL_PER; ++j) {
    const bool keep_last = MODE == OP_MIXED ? ((uint32_t)e[j] >> 31) == 0 : MODE == OP_INSERT;
    if (e[j] != EMPTY) dds_settle<SMALL_TAB>(sh.tab, e[j], keep_last, nullptr);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < SMALL_PER; ++j)  // the flags of the block's own tiles
    if (e[j] != EMPTY && j == (int)blockIdx.x)
      win[(uint32_t)e[j] & 0x7FFFFFFFu] = dds_kept<SMALL_TAB>(sh.tab, e[j]);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();  // the flags are written, the table is free
  a.win = win;
  // the same in a whole wave, and known to be: fewer registers
  const uint32_t part = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid / BLOCK));
  const uint64_t tile = blockIdx.x * (SMALL_BLOCK / BLOCK) + part;
  if (tile * BLOCK < a.n) {
    int64_t live_acc = 0;
    uint64_t bad_acc = 0;
    ops_tile<S, MODE, false, PAIR_BITHASH, Traits<S>::CH, FILTER>(a, view, tile, sh.ops[part], live_acc,
                                                                 bad_acc);
    ops_counts_add(a.ctl, tile * WAVES + (tid >> 6) % WAVES, live_acc, bad_acc);
  }
  if (blockIdx.x == 0 && tid == 0) ops_done<MODE>(a.ctl, view, FILTER != FILTER_NONE);
}

// ---------------------------------------------------------------------------
// P3: bounded cuckoo eviction (Algorithm 3) and the stash (Section IV-A step 4)
// ---------------------------------------------------------------------------
struct EvictArgs {
  uint64_t *buckets;
  Spill spill;
  uint32_t *hint;
  uint64_t *stash;
  uint64_t *pending;
  Ctl *ctl;
  uint64_t *wl;
  uint64_t wl_seg_cap;
  uint64_t stash_cap;
  uint64_t pending_cap;
  uint32_t max_evictions;
  uint64_t inserts;  // operations of the batch that may have inserted
};

__device__ __forceinline__ void set_hint(uint32_t *hint, uint32_t b) { or32(&hint[b >> 5], 1u << (b & 31)); }

// Step 4: the item goes to the stash, or to the pending list when the stash
// is full.  Room is reserved by a fetch-add on the count, one per wave for
// all of its pushes (the counts may pass their capacities; every reader
// clamps them); given its reserved position c (c >= capacity: pending), the
// entry claims the first EMPTY or TOMB word of its probe run by CAS (an
// EMPTY one exists: the table has at least twice the capacity).  A TOMB word
// is reused: it already counts as used, and searches pass it, so the entry
// is found at the first free word of its run either way (no key is stashed
// twice: items here are keys absent from the table, and a word taken by
// another placement meanwhile holds a live entry).  Returns where it went:
// 0 stash (an EMPTY word), 3 stash (a TOMB word), 1 pending, 2 lost (the
// pending list was full too; latched as an error).
template <int PAIR = PAIR_BITHASH>
__device__ __forceinline__ int overflow_place(const EvictArgs &a, const Geo &geo, uint64_t kv, uint64_t c) {
  int where = -1;
  if (c < a.stash_cap) {
    const uint64_t mask = stash_slots_for(a.stash_cap) - 1;
    for (uint64_t i = 0, p = mix32(key_of(kv)) & mask; i <= mask; ++i, p = (p + 1) & mask) {
      const uint64_t cur = cas64(a.stash + p, EMPTY, kv);
      if (cur == EMPTY) {
        where = 0;
        break;
      }
      if (cur == TOMB && cas64(a.stash + p, TOMB, kv) == TOMB) {
        where = 3;
        break;
      }
    }
  }
  if (where < 0) {
    const uint64_t p = add64(&a.ctl->pending_count, 1);
    if (p < a.pending_cap) {
      __hip_atomic_store(a.pending + p, kv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      where = 1;
    } else {
      atomicOr(&a.ctl->error, ERR_PENDING_LOST);
      where = 2;
    }
  }
  const uint32_t k = key_of(kv);
  if constexpr (PairArity<PAIR>::D == 2) spill_mark(a.spill, address(geo, HashPair<PAIR>::h1(k)), k);
  set_hint(a.hint, address(geo, HashPair<PAIR>::h1(k)));
  set_hint(a.hint, address(geo, HashPair<PAIR>::h2(k)));
  if constexpr (PairArity<PAIR>::D == 3) set_hint(a.hint, address(geo, HashPair<PAIR>::h3(k)));
  return where;
}

// Entry kv was put in bucket b.
template <int PAIR>
__device__ __forceinline__ void evict_mark(const EvictArgs &a, const Geo &geo, uint64_t kv, uint32_t b) {
  if constexpr (PairArity<PAIR>::D == 2) {
    if (!a.spill.bits) return;  // without a filter the hash is not computed either
    const uint32_t c1 = address(geo, HashPair<PAIR>::h1(key_of(kv)));
    if (b != c1) spill_mark(a.spill, c1, key_of(kv));
  }
}

// Eviction group shape.  A group of L lanes works on one item and sees a
// bucket as P adjacent slots per lane (L x P = S).  A chain is a sequence of
// dependent memory round trips, so the number of chains in flight sets the
// eviction rate: for S = 16 each lane holds a whole bucket (P = 16, measured
// best against 8, 4 and 2: mixed Zipf batches at 95% load 1.2 ms against
// 1.5, 1.9 and 2.4 ms), so a wave runs 64 chains at once; wider buckets keep
// one slot per lane.
template <int S>
struct EvictShape {
  static constexpr int P = (S == 16) ? EVICT_SLOTS_PER_LANE : 1;
  static constexpr int L = S / P;
  static constexpr int G = 64 / L;  // items per wave
  static constexpr uint64_t LANES = (L == 64) ? ~0ull : ((1ull << L) - 1ull);
};

__host__ __device__ __forceinline__ int evict_groups_per_wave(uint32_t S) {
  return S == 16 ? 64 / (16 / EVICT_SLOTS_PER_LANE) : (int)(64 / S);
}

// Bits of slots s = l * P + p from per-word masks (bit l of m[p]).
template <int P, typename Mask>
__device__ __forceinline__ Mask interleave_slots(const uint64_t *m) {
  if constexpr (P == 1) {
    return (Mask)m[0];
  } else if constexpr (P == 2) {
    uint32_t a = (uint32_t)m[0], b = (uint32_t)m[1];  // 8 bits each
    a = (a | (a << 4)) & 0x0F0Fu;
    a = (a | (a << 2)) & 0x3333u;
    a = (a | (a << 1)) & 0x5555u;
    b = (b | (b << 4)) & 0x0F0Fu;
    b = (b | (b << 2)) & 0x3333u;
    b = (b | (b << 1)) & 0x5555u;
    return (Mask)(a | (b << 1));
  } else if constexpr (P == 4) {
    uint32_t r = 0;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      uint32_t x = (uint32_t)m[p];  // 4 bits
      x = (x | (x << 6)) & 0x0303u;
      x = (x | (x << 3)) & 0x1111u;
      r |= x << p;
    }
    return (Mask)r;
  } else if constexpr (P == 8) {
    uint32_t r = 0;
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      const uint32_t x = (uint32_t)m[p];  // 2 bits
      r |= ((x & 1u) | ((x & 2u) << 7)) << p;
    }
    return (Mask)r;
  } else {
    static_assert(P == 16, "two, four, eight or sixteen slots per lane");
    uint32_t r = 0;
#pragma unroll
    for (int p = 0; p < 16; ++p) r |= ((uint32_t)m[p] & 1u) << p;
    return (Mask)r;
  }
}

// One lane's fresh copy of a whole 16-slot bucket (128 bytes, 128-byte
// aligned) in eight 16-byte loads.  The compute unit's L1 is invalidated
// first, so that the bucket comes from the L2, as an agent-scope load's word
// would; the first of the eight brings the line into the L1 and the others
// find it there.  Marked as agent-scope loads (sc1) all eight went to the L2,
// whose request rate bound the eviction launches: 112 -> 91 us in the batches
// of a growing table, 270 -> 213 us after a 2^26-key build to 95%.  (Atomic
// loads are at most 8 bytes wide: sixteen scattered lines of requests.)  A
// view that is older all the same costs a failed CAS and the round it was made in:
// of its chain's bounded rounds, so that about a tenth more entries end in the
// stash at 97% load (712 for 648 of 2^26 keys).
// The block ends in its own wait for the loads, so the registers are complete
// when it returns.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void load_bucket16_fresh(const uint64_t *b, uint64_t *w) {
  u32x4 x0, x1, x2, x3, x4, x5, x6, x7;
  asm volatile(
      "buffer_inv sc0\n"
      "global_load_dwordx4 %0, %8, off\n"
      "global_load_dwordx4 %1, %8, off offset:16\n"
      "global_load_dwordx4 %2, %8, off offset:32\n"
      "global_load_dwordx4 %3, %8, off offset:48\n"
      "global_load_dwordx4 %4, %8, off offset:64\n"
      "global_load_dwordx4 %5, %8, off offset:80\n"
      "global_load_dwordx4 %6, %8, off offset:96\n"
      "global_load_dwordx4 %7, %8, off offset:112\n"
      "s_waitcnt vmcnt(0)\n"
      : "=&v"(x0), "=&v"(x1), "=&v"(x2), "=&v"(x3), "=&v"(x4), "=&v"(x5), "=&v"(x6), "=&v"(x7)
      : "v"(b)
      : "memory");
  const u32x4 xs[8] = {x0, x1, x2, x3, x4, x5, x6, x7};
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    w[2 * j] = ((uint64_t)xs[j][1] << 32) | xs[j][0];
    w[2 * j + 1] = ((uint64_t)xs[j][3] << 32) | xs[j][2];
  }
}

// Two whole buckets per lane, all sixteen loads in flight before the one
// wait (the same loads as load_bucket16_fresh).
__device__ __forceinline__ void load_bucket16x2_fresh(const uint64_t *b1, const uint64_t *b2, uint64_t *w1,
                                                      uint64_t *w2) {
  u32x4 x0, x1, x2, x3, x4, x5, x6, x7, y0, y1, y2, y3, y4, y5, y6, y7;
  asm volatile(
      "buffer_inv sc0\n"
      "global_load_dwordx4 %0, %16, off\n"
      "global_load_dwordx4 %1, %16, off offset:16\n"
      "global_load_dwordx4 %2, %16, off offset:32\n"
      "global_load_dwordx4 %3, %16, off offset:48\n"
      "global_load_dwordx4 %4, %16, off offset:64\n"
      "global_load_dwordx4 %5, %16, off offset:80\n"
      "global_load_dwordx4 %6, %16, off offset:96\n"
      "global_load_dwordx4 %7, %16, off offset:112\n"
      "global_load_dwordx4 %8, %17, off\n"
      "global_load_dwordx4 %9, %17, off offset:16\n"
      "global_load_dwordx4 %10, %17, off offset:32\n"
      "global_load_dwordx4 %11, %17, off offset:48\n"
      "global_load_dwordx4 %12, %17, off offset:64\n"
      "global_load_dwordx4 %13, %17, off offset:80\n"
      "global_load_dwordx4 %14, %17, off offset:96\n"
      "global_load_dwordx4 %15, %17, off offset:112\n"
      "s_waitcnt vmcnt(0)\n"
      : "=&v"(x0), "=&v"(x1), "=&v"(x2), "=&v"(x3), "=&v"(x4), "=&v"(x5), "=&v"(x6), "=&v"(x7), "=&v"(y0),
        "=&v"(y1), "=&v"(y2), "=&v"(y3), "=&v"(y4), "=&v"(y5), "=&v"(y6), "=&v"(y7)
      : "v"(b1), "v"(b2)
      : "memory");
  const u32x4 xs[8] = {x0, x1, x2, x3, x4, x5, x6, x7};
  const u32x4 ys[8] = {y0, y1, y2, y3, y4, y5, y6, y7};
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    w1[2 * j] = ((uint64_t)xs[j][1] << 32) | xs[j][0];
    w1[2 * j + 1] = ((uint64_t)xs[j][3] << 32) | xs[j][2];
    w2[2 * j] = ((uint64_t)ys[j][1] << 32) | ys[j][0];
    w2[2 * j + 1] = ((uint64_t)ys[j][3] << 32) | ys[j][2];
  }
}

// EMPTY-slot mask of a whole bucket held by one lane.
__device__ __forceinline__ uint32_t empty_mask16(const uint64_t *w) {
  uint32_t m = 0;
#pragma unroll
  for (int p = 0; p < 16; ++p) m |= (w[p] == EMPTY ? 1u : 0u) << p;
  return m;
}

// The group's fresh view of bucket `bkt`: words w[p] of slots sl * P + p,
// and its EMPTY-slot mask.
template <int S>
__device__ __forceinline__ typename Traits<S>::Mask load_view(const uint64_t *bkt, int g, int sl, uint64_t *w) {
  using E = EvictShape<S>;
  uint64_t m[E::P];
  if constexpr (E::L == 1 && E::P == 16) {
    load_bucket16_fresh(bkt, w);
  } else {
#pragma unroll
    for (int p = 0; p < E::P; ++p) w[p] = load_fresh(bkt + sl * E::P + p);
  }
  if constexpr (E::L == 1) {  // the lane holds the whole bucket
#pragma unroll
    for (int p = 0; p < E::P; ++p) m[p] = w[p] == EMPTY;
  } else {
#pragma unroll
    for (int p = 0; p < E::P; ++p) m[p] = (ballot(w[p] == EMPTY) >> (g * E::L)) & E::LANES;
  }
  return interleave_slots<E::P, typename Traits<S>::Mask>(m);
}

// Claim-then-commit by one group (WABC): `free_mask` holds the group's view
// of the bucket's EMPTY slots; the lowest one is claimed with one CAS by the
// lane holding it, and a failed CAS (the view was stale) drops that slot and
// tries the next.  Returns true when the entry was committed.
template <int S>
__device__ __forceinline__ bool group_claim(uint64_t *bkt, typename Traits<S>::Mask free_mask, uint64_t kv, int g,
                                            int sl) {
  using E = EvictShape<S>;
  using Mask = typename Traits<S>::Mask;
  while (free_mask) {
    const int s = ctz_mask(free_mask);
    bool won = false;
    if (sl == s / E::P) won = cas64(bkt + s, EMPTY, kv) == EMPTY;
    if ((ballot(won) >> (g * E::L)) & E::LANES) return true;
    free_mask &= (Mask)(free_mask - 1);
  }
  return false;
}

// P3: items whose two buckets were full in P1 (or stash entries re-placed
// after a split), one group per item (a group of the eviction shape: one
// lane for 16-slot buckets).  Step 2 is tried again with a fresh view of
// both buckets (two-choice), then the bounded cuckoo chain of Algorithm 3:
// each round claims a free slot of the current bucket or displaces a victim
// by CAS and carries the victim to its alternate bucket.  Returns whether
// the item was placed; if not, the caller sends the entry in hand to the
// stash (or the pending list when the stash is full).
template <int S, int PAIR = PAIR_BITHASH>
__device__ __forceinline__ bool evict_chain(const EvictArgs &a, const Geo &geo, uint64_t &kv, uint32_t max_kicks,
                                            int g, int sl, uint64_t &n_evict) {
  using T = Traits<S>;
  using Mask = typename T::Mask;
  using E = EvictShape<S>;
  const uint32_t c1 = address(geo, HashPair<PAIR>::h1(key_of(kv))), c2 = address(geo, HashPair<PAIR>::h2(key_of(kv)));
  // step 2 with fresh loads (fresh: other items of this phase change buckets)
  uint64_t w[E::P], w2v[E::P];
  // one lane holding whole buckets: both candidates in one round trip
  constexpr bool kLaneBucket = E::L == 1 && E::P == 16;
  Mask f1, f2;
  if constexpr (kLaneBucket) {
    load_bucket16x2_fresh(a.buckets + (uint64_t)c1 * S, a.buckets + (uint64_t)c2 * S, w, w2v);
    f1 = (Mask)empty_mask16(w);
    f2 = (Mask)empty_mask16(w2v) & (Mask)((c2 != c1) ? ~0ull : 0ull);
  } else {
    f1 = load_view<S>(a.buckets + (uint64_t)c1 * S, g, sl, w);
    f2 = load_view<S>(a.buckets + (uint64_t)c2 * S, g, sl, w2v) & (Mask)((c2 != c1) ? ~0ull : 0ull);
  }
  bool placed;
  if constexpr (PairArity<PAIR>::D == 3) {
    // three-choice: the emptiest candidate first, ties to the lower hash
    const uint32_t c3 = address(geo, HashPair<PAIR>::h3(key_of(kv)));
    const Mask f3 = load_view<S>(a.buckets + (uint64_t)c3 * S, g, sl, w) &
                    (Mask)((c3 != c1 && c3 != c2) ? ~0ull : 0ull);
    Mask f[3] = {f1, f2, f3};
    uint32_t c[3] = {c1, c2, c3};
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2 - x; ++y)
        if (popc_mask(f[y + 1]) > popc_mask(f[y])) {
          const Mask tf = f[y];
          f[y] = f[y + 1];
          f[y + 1] = tf;
          const uint32_t tc = c[y];
          c[y] = c[y + 1];
          c[y + 1] = tc;
        }
    placed = group_claim<S>(a.buckets + (uint64_t)c[0] * S, f[0], kv, g, sl) ||
             group_claim<S>(a.buckets + (uint64_t)c[1] * S, f[1], kv, g, sl) ||
             group_claim<S>(a.buckets + (uint64_t)c[2] * S, f[2], kv, g, sl);
  } else {
    const bool swap = popc_mask(f2) > popc_mask(f1) && (uint32_t)popc_mask(f1) < a.spill.first_min;
    const uint32_t cf = swap ? c2 : c1, cs = swap ? c1 : c2;
    const bool in_first = group_claim<S>(a.buckets + (uint64_t)cf * S, swap ? f2 : f1, kv, g, sl);
    placed = in_first || group_claim<S>(a.buckets + (uint64_t)cs * S, swap ? f1 : f2, kv, g, sl);
    if (placed && sl == 0) evict_mark<PAIR>(a, geo, kv, in_first ? cf : cs);
  }
  uint32_t b = c1;  // chains start at the first candidate
  // look-ahead chains keep the view of the bucket they move to: w holds
  // bucket b's words when `have_view` (first the view step 2 loaded; its
  // free slots were just tried)
  bool have_view = kLaneBucket && PairArity<PAIR>::D == 2;
  for (uint32_t kick = 1; kick <= max_kicks && !placed; ++kick) {
    uint64_t *bkt = a.buckets + (uint64_t)b * S;
    if (!have_view) {
      const Mask fm = load_view<S>(bkt, g, sl, w);
      if (group_claim<S>(bkt, fm, kv, g, sl)) {
        if (sl == 0) evict_mark<PAIR>(a, geo, kv, b);
        placed = true;
        break;
      }
    }
    have_view = false;
    if constexpr (kLaneBucket && PairArity<PAIR>::D == 2) {
      // Look ahead: two candidate victims at pseudo-random distinct slots;
      // both alternate buckets are loaded in one round trip, and a victim
      // whose alternate has an EMPTY slot is displaced and claims that slot
      // from the view just loaded.  At 95% load most chains then end after
      // one displacement instead of several, and far fewer run out of
      // rounds into the stash (mixed Zipf batches at 95%: 130 K stash
      // entries per 2^22 operations before, about 12 K with look-ahead);
      // with no room in either, the first is displaced and the chain goes
      // on from its alternate.  (Four candidates, loaded one after another,
      // stretched every chain that fails to four more round trips per
      // displacement.)
      constexpr int LA = 2;
      const uint32_t r = mix32(key_of(kv) ^ (kick * 0x9E3779B9u));
      int vs[LA];
      uint64_t vw[LA];
      uint32_t va[LA];
#pragma unroll
      for (int j = 0; j < LA; ++j) {
        vs[j] = (int)((r + 5u * (uint32_t)j) & 15u);
        vw[j] = w[vs[j]];
        const uint32_t a1 = address(geo, HashPair<PAIR>::h1(key_of(vw[j])));
        const uint32_t a2 = address(geo, HashPair<PAIR>::h2(key_of(vw[j])));
        va[j] = (b == a1) ? a2 : a1;
      }
      load_bucket16x2_fresh(a.buckets + (uint64_t)va[0] * S, a.buckets + (uint64_t)va[1] * S, w, w2v);
      const Mask fa = (Mask)empty_mask16(w) & (Mask)((va[0] != b) ? ~0ull : 0ull);
      const Mask fb = (Mask)empty_mask16(w2v) & (Mask)((va[1] != b) ? ~0ull : 0ull);
      const int pick = (fa == 0 && fb != 0) ? 1 : 0;
      const Mask fpick = pick ? fb : fa;
      const uint64_t victim = vw[pick];
      if (cas64(bkt + vs[pick], victim, kv) != victim) continue;  // the slot changed: count the round
      evict_mark<PAIR>(a, geo, kv, b);
      if (victim == EMPTY) {
        placed = true;  // the slot was empty after all: the CAS claimed it
        break;
      }
      ++n_evict;
      kv = victim;
      b = va[pick];
      if (fpick && group_claim<S>(a.buckets + (uint64_t)b * S, fpick, kv, g, sl)) {
        evict_mark<PAIR>(a, geo, kv, b);
        placed = true;
        break;
      }
      // no room there (or it was taken meanwhile): the next displacement
      // works from the view just loaded, one round trip fewer
      if (pick == 1) {
#pragma unroll
        for (int p = 0; p < 16; ++p) w[p] = w2v[p];
      }
      have_view = true;
      continue;
    }
    // victim: a pseudo-random slot (the paper's "first occupied" slot is
    // slot 0 of every full bucket, which lets two chains trade the same
    // pair of entries back and forth)
    const int s0 = (int)(mix32(key_of(kv) ^ (kick * 0x9E3779B9u)) & (S - 1));
    const uint64_t ws = w[s0 % E::P];  // this lane's word at the victim's position in its pair
    bool won = false;
    if (sl == s0 / E::P) won = cas64(bkt + s0, ws, kv) == ws;
    const bool ok = (ballot(won) >> (g * E::L)) & E::LANES;
    const uint64_t victim = shfl64(ws, g * E::L + s0 / E::P);
    if (!ok) continue;  // the slot changed under us: count the round, keep the item
    if (sl == 0) evict_mark<PAIR>(a, geo, kv, b);
    if (victim == EMPTY) {
      placed = true;  // the slot was empty after all: the CAS claimed it
      break;
    }
    ++n_evict;
    kv = victim;
    const uint32_t v1 = address(geo, HashPair<PAIR>::h1(key_of(kv)));
    const uint32_t v2 = address(geo, HashPair<PAIR>::h2(key_of(kv)));
    if constexpr (PairArity<PAIR>::D == 3) {
      // the victim's next candidate after b, in hash order, cyclically
      const uint32_t v3 = address(geo, HashPair<PAIR>::h3(key_of(kv)));
      b = (b == v1) ? v2 : (b == v2) ? v3 : v1;
    } else {
      b = (b == v1) ? v2 : v1;  // AltBucket: the victim's other candidate
    }
  }
  return placed;  // if not, kv is the entry in hand
}

// One item per group of the wave (`have`: the group has one, at worklist
// position `pos`); every lane of the wave calls it.  Each item takes step 2
// (two-choice claim on fresh loads) and the bounded chain of Algorithm 3;
// an entry still in hand goes to the stash.  `unreserved`: the launch cannot
// fill the stash (its count when the launch started plus the launch's items
// is within capacity), so entries take stash slots without touching the
// count, which every pushing wave would otherwise reserve from, one atomic
// each on a single address (thousands of waves queue there in a stash drain);
// their number is added per wave to the shards and folded into the count
// after the launch.  Otherwise one count reservation per wave.
//
// DEFER (phase timing of the plain path): step 4 is left to its own launch,
// stash_kernel, so that steps 3 and 4 are timed apart; the item's worklist
// word is overwritten with the entry still in hand, or EMPTY once placed.
template <int S, int PAIR = PAIR_BITHASH, bool DEFER = false>
__device__ __forceinline__ void evict_round(const EvictArgs &a, const Geo &geo, bool unreserved, bool have,
                                            uint64_t pos, int g, int sl, uint64_t &n_evict, uint64_t &n_full,
                                            uint64_t &n_side, uint64_t &n_fresh) {
  uint64_t kv = 0;
  bool placed = true;
  if (have) {
    kv = a.wl[pos];
    placed = evict_chain<S, PAIR>(a, geo, kv, a.max_evictions, g, sl, n_evict);
  }
  if constexpr (DEFER) {
    if (have && sl == 0) {
      a.wl[pos] = placed ? EMPTY : kv;
      n_full += !placed;
    }
    return;
  }
  const bool push = !placed && sl == 0;
  const uint64_t pm = ballot(push);
  if (pm) {
    const int lane = threadIdx.x & 63;
    const int leader = __builtin_ctzll(pm);
    uint64_t base = 0;
    if (!unreserved) {
      if (lane == leader) {
        const uint64_t n = (uint64_t)__popcll(pm);
        base = load_fresh(&a.ctl->stash_count) < a.stash_cap ? add64(&a.ctl->stash_count, n) : a.stash_cap;
      }
      base = read_lane64(base, leader);
    }
    if (push) {
      ++n_full;
      const int where = overflow_place<PAIR>(a, geo, kv, base + rank_below(pm));
      n_side += (where == 0 || where == 3) ? 1 : where == 1 ? (1ull << 32) : 0;
      n_fresh += where == 0;
    }
  }
}

// Chain statistics of a wave (per group, held by its lane 0) added to the
// wave's shard.  Every lane of the wave calls it.  n_side counts the lane's
// stash placements in its low half and pending ones in its high half (a
// wave places far fewer than 2^32 entries); n_fresh counts the stash
// placements that took an EMPTY word, the ones that add a used word to the
// count (when the launch reserved no room, they are added after it).
__device__ __forceinline__ void evict_counters(const EvictArgs &a, bool unreserved, uint64_t unit, uint64_t n_evict,
                                               uint64_t n_full, uint64_t n_side, uint64_t n_fresh, int sl) {
  const uint64_t e = wave_sum64(sl == 0 ? n_evict : 0), f = wave_sum64(n_full), sd = wave_sum64(n_side);
  const uint64_t fr = wave_sum64(n_fresh);
  if ((threadIdx.x & 63) == 0 && (e | f | sd)) {
    Shard *sh = shard_of(a.ctl, unit % NSHARD);
    if (e) add64(&sh->evictions, e);
    if (f) add64(&sh->full_chains, f);
    if ((uint32_t)sd) add64(&sh->stash_inserts, (uint32_t)sd);
    if (fr && unreserved) add64(&sh->stash_unreserved, fr);
    if (sd >> 32) add64(&sh->pending_inserts, sd >> 32);
  }
}

// The end of an eviction launch (every thread calls it): the block that
// finishes last folds the shards into the totals and empties the worklist;
// with no items, block 0 does (the other blocks have nothing to write).  A
// launch of its own for this took 2.9 us and a host call per batch.
__device__ __forceinline__ void evict_finish(Ctl *c, bool items, uint64_t inserts);

// P3 as a launch: every worklist item through evict_round (step 2 again,
// then the bounded chain of Algorithm 3, then the stash or the pending list),
// one item per group of the eviction shape, the grid striding over items.
// The last block empties the worklist, counts the items and folds unreserved
// stash placements into the stash count (evict_finish).  With DEFER, a launch
// of finish_kernel does, after the stash launch.
template <int S, int PAIR = PAIR_BITHASH, bool DEFER = false>
__global__ __launch_bounds__(BLOCK) void evict_kernel(EvictArgs a) {
  using E = EvictShape<S>;
  __shared__ uint64_t pre[NSHARD + 1];
  wl_prefix(a.ctl, pre);
  const uint64_t cnt = pre[NSHARD];
  if (cnt == 0) {  // same in every block
    if constexpr (!DEFER) evict_finish(a.ctl, false, a.inserts);
    return;
  }
  a.spill = spill_placing(a.spill, a.ctl, a.inserts, S);
  const Geo geo = read_geo(a.ctl);
  // the same in every block: an unreserved launch leaves the count alone
  const bool unreserved = ld_ctl(&a.ctl->stash_count) + cnt <= a.stash_cap;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int g = lane / E::L, sl = lane % E::L;
  const uint64_t groups = (uint64_t)gridDim.x * WAVES * E::G;
  uint64_t n_evict = 0, n_full = 0, n_side = 0, n_fresh = 0;
  const uint64_t first = ((uint64_t)blockIdx.x * WAVES + wv) * E::G + g;
  // a uniform trip count per wave: every lane reaches the wave-wide steps
  const uint64_t wave_first = ((uint64_t)blockIdx.x * WAVES + wv) * E::G;
  for (uint64_t base = wave_first; base < cnt; base += groups) {
    const uint64_t t = base - wave_first + first;
    evict_round<S, PAIR, DEFER>(a, geo, unreserved, t < cnt, t < cnt ? wl_slot(pre, t, a.wl_seg_cap) : 0, g, sl,
                                n_evict, n_full, n_side, n_fresh);
  }
  evict_counters(a, unreserved, (uint64_t)blockIdx.x * WAVES + wv, n_evict, n_full, n_side, n_fresh, sl);
  if constexpr (!DEFER) evict_finish(a.ctl, true, a.inserts);
}

// P3 for 16-slot buckets with two candidates, as a launch whose lanes are
// refilled as their chains end.  Each wave owns a contiguous range of the
// worklist (at least 64 items); a lane takes the range's next item whenever
// it holds none, so a wave lasts about as long as its lanes' total work
// rather than one round per 64 items, each as long as its longest chain
// (at 95% load a few percent of the chains run all their rounds, and nearly
// every group of 64 items held one).  A lane steps through one memory round
// trip at a time:
//   FRESH   both candidates loaded (step 2 again, two-choice claim);
//   LOOK    one displacement round of the look-ahead chain: two victims of
//           the bucket in hand, both alternates loaded in one round trip,
//           a victim displaced by CAS and its slot claimed from that view;
//   RELOAD  the bucket in hand loaded again after a displacement CAS found
//           its slot changed, and its free slots tried.
// The rounds, the victims and the stash placement are those of evict_chain
// and evict_round (step 4 reserves room once per wave and step, as there);
// only the order in which a wave's items run differs.  The grid should be
// resident at once: a wave's range is not shared.
template <int PAIR>
__global__ __launch_bounds__(BLOCK) void evict_lanes_kernel(EvictArgs a) {
  static_assert(PairArity<PAIR>::D == 2, "two candidate buckets");
  constexpr int S = 16;
  using Mask = typename Traits<S>::Mask;
  __shared__ uint64_t pre[NSHARD + 1];
  wl_prefix(a.ctl, pre);
  const uint64_t cnt = pre[NSHARD];
  if (cnt == 0) {  // same in every block
    evict_finish(a.ctl, false, a.inserts);
    return;
  }
  a.spill = spill_placing(a.spill, a.ctl, a.inserts, S);
  const Geo geo = read_geo(a.ctl);
  // the same in every block: an unreserved launch leaves the count alone
  const bool unreserved = ld_ctl(&a.ctl->stash_count) + cnt <= a.stash_cap;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const uint64_t nw = (uint64_t)gridDim.x * WAVES, wid = (uint64_t)blockIdx.x * WAVES + wv;
  const uint64_t q = max<uint64_t>(64, (cnt + nw - 1) / nw);
  const uint64_t end = min(cnt, (wid + 1) * q);
  uint64_t cursor = wid * q;  // the wave's next item (the same in every lane)
  const uint32_t max_kicks = a.max_evictions;
  const bool mid_round = geo.mode == ADDR_LINEAR && geo.sp != 0 && geo.sp <= geo.im;  // the same in every lane
  uint64_t n_evict = 0, n_full = 0, n_side = 0, n_fresh = 0;
  constexpr int IDLE = 0, FRESH = 1, RELOAD = 2, LOOK = 3;
  int st = IDLE;
  uint64_t kv = 0;        // the entry in hand
  uint32_t b = 0;         // the bucket it is carried into
  uint32_t kick = 0;      // displacement rounds taken
  uint64_t w[16], w2v[16];  // LOOK, RELOAD: w holds bucket b's words
  while (cursor < end || ballot(st != IDLE)) {
    // lanes without an item take the range's next ones, in lane order
    const uint64_t nm = ballot(st == IDLE);
    if (nm && cursor < end) {
      const uint64_t t = cursor + rank_below(nm);
      if (st == IDLE && t < end) {
        kv = a.wl[wl_slot(pre, t, a.wl_seg_cap)];
        st = FRESH;
        kick = 0;
      }
      cursor += (uint64_t)__popcll(nm);
    }
    // this step's two bucket loads
    uint32_t x1 = 0, x2 = 0;
    int vs0 = 0, vs1 = 0;
    uint64_t vw0 = 0, vw1 = 0;
    if (st == FRESH) {
      x1 = address(geo, HashPair<PAIR>::h1(key_of(kv)));
      x2 = address(geo, HashPair<PAIR>::h2(key_of(kv)));
    } else if (st == RELOAD) {
      x1 = b;
      x2 = b;
    } else if (st == LOOK) {
      // two candidate victims at pseudo-random distinct slots (round kick + 1)
      const uint32_t r = mix32(key_of(kv) ^ ((kick + 1) * 0x9E3779B9u));
      vs0 = (int)(r & 15u);
      vs1 = (int)((r + 5u) & 15u);
      if (mid_round) {
        // between rounds of linear hashing the buckets not yet split hold
        // about twice the load of the split ones and are full, and a chain
        // ends where a victim's alternate is a split one, which its address
        // tells without a load: of eight of the bucket's entries (every
        // second slot, from an even or odd one) prefer two such.  All 16
        // would cost twice the hashing for few more hits.  Growth to 12.6 M
        // keys in 12 batches: displacements 5.75 M -> 3.31 M, chains that ran
        // out of rounds 51 K -> 0.2 K, an eviction launch 246 -> 108 us
        const bool odd = (r & 16u) != 0;
        uint32_t good = 0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          // both words by value: `odd ? w[i] : w[j]` selects an address, which
          // put w into scratch memory, written by every load of a bucket (new
          // keys into a 2^26-key table at 90-95 and 95-97% load 313 and 273
          // us; so 285 and 203)
          const uint32_t k0 = key_of(w[2 * q]), k1 = key_of(w[2 * q + 1]), k = odd ? k1 : k0;
          const uint32_t a1 = address(geo, HashPair<PAIR>::h1(k)), a2 = address(geo, HashPair<PAIR>::h2(k));
          const uint32_t alt = b == a1 ? a2 : a1;
          good |= (alt != b && (alt < geo.sp || alt > geo.im) ? 1u : 0u) << (2 * q);
        }
        good <<= odd ? 1 : 0;
        if (good) {
          const int s0 = vs0;
          const auto next = [&](uint32_t m) {
            const uint32_t from = m & (0xFFFFu << s0);
            return ctz_mask(from ? from : m);
          };
          vs0 = next(good);
          const uint32_t rest = good & ~(1u << vs0);
          vs1 = rest ? next(rest) : (int)((vs0 + 5) & 15);
        }
      }
      vw0 = w[vs0];
      vw1 = w[vs1];
      const uint32_t a1 = address(geo, HashPair<PAIR>::h1(key_of(vw0))), a2 = address(geo, HashPair<PAIR>::h2(key_of(vw0)));
      const uint32_t b1 = address(geo, HashPair<PAIR>::h1(key_of(vw1))), b2 = address(geo, HashPair<PAIR>::h2(key_of(vw1)));
      x1 = (b == a1) ? a2 : a1;
      x2 = (b == b1) ? b2 : b1;
    }
    if (st != IDLE) load_bucket16x2_fresh(a.buckets + (uint64_t)x1 * S, a.buckets + (uint64_t)x2 * S, w, w2v);
    bool fail = false;  // the chain ran out of rounds: step 4
    if (st == FRESH) {
      const Mask f1 = (Mask)empty_mask16(w);
      const Mask f2 = (Mask)empty_mask16(w2v) & (Mask)((x2 != x1) ? ~0ull : 0ull);
      const bool swap = popc_mask(f2) > popc_mask(f1) && (uint32_t)popc_mask(f1) < a.spill.first_min;
      const uint32_t cf = swap ? x2 : x1, cs = swap ? x1 : x2;
      const bool in_first = group_claim<S>(a.buckets + (uint64_t)cf * S, swap ? f2 : f1, kv, lane, 0);
      if (in_first || group_claim<S>(a.buckets + (uint64_t)cs * S, swap ? f1 : f2, kv, lane, 0)) {
        if ((in_first ? cf : cs) != x1) spill_mark(a.spill, x1, key_of(kv));
        st = IDLE;
      } else if (max_kicks == 0) {
        fail = true;
      } else {
        b = x1;  // chains start at the first candidate, whose view w holds
        st = LOOK;
      }
    } else if (st == RELOAD) {
      const bool placed = group_claim<S>(a.buckets + (uint64_t)b * S, (Mask)empty_mask16(w), kv, lane, 0);
      if (placed) evict_mark<PAIR>(a, geo, kv, b);
      st = placed ? IDLE : LOOK;
    } else if (st == LOOK) {
      ++kick;
      const Mask fa = (Mask)empty_mask16(w) & (Mask)((x1 != b) ? ~0ull : 0ull);
      const Mask fb = (Mask)empty_mask16(w2v) & (Mask)((x2 != b) ? ~0ull : 0ull);
      const int pick = (fa == 0 && fb != 0) ? 1 : 0;
      const Mask fpick = pick ? fb : fa;
      const uint64_t victim = pick ? vw1 : vw0;
      const int vsl = pick ? vs1 : vs0;
      if (cas64(a.buckets + (uint64_t)b * S + vsl, victim, kv) != victim) {
        // the slot changed: the round is spent, the item stays in hand
        if (kick < max_kicks) st = RELOAD;
        else fail = true;
      } else if (victim == EMPTY) {
        evict_mark<PAIR>(a, geo, kv, b);
        st = IDLE;  // the slot was empty after all: the CAS claimed it
      } else {
        evict_mark<PAIR>(a, geo, kv, b);
        ++n_evict;
        kv = victim;
        b = pick ? x2 : x1;
        if (fpick && group_claim<S>(a.buckets + (uint64_t)b * S, fpick, kv, lane, 0)) {
          evict_mark<PAIR>(a, geo, kv, b);
          st = IDLE;
        } else if (kick < max_kicks) {
          // the next round works from the view just loaded
          if (pick == 1) {
#pragma unroll
            for (int p = 0; p < 16; ++p) w[p] = w2v[p];
          }
        } else {
          fail = true;
        }
      }
    }
    // step 4 for the chains that ran out of rounds
    const uint64_t pm = ballot(fail);
    if (pm) {
      const int leader = __builtin_ctzll(pm);
      uint64_t base = 0;
      if (!unreserved) {
        if (lane == leader) {
          const uint64_t n = (uint64_t)__popcll(pm);
          base = load_fresh(&a.ctl->stash_count) < a.stash_cap ? add64(&a.ctl->stash_count, n) : a.stash_cap;
        }
        base = read_lane64(base, leader);
      }
      if (fail) {
        ++n_full;
        const int where = overflow_place<PAIR>(a, geo, kv, base + rank_below(pm));
        n_side += (where == 0 || where == 3) ? 1 : where == 1 ? (1ull << 32) : 0;
        n_fresh += where == 0;
        st = IDLE;
      }
    }
  }
  evict_counters(a, unreserved, wid, n_evict, n_full, n_side, n_fresh, 0);
  evict_finish(a.ctl, true, a.inserts);
}

// Step 4 as its own launch (after evict_kernel<.., DEFER>): every worklist
// word that still holds an entry goes to the stash or the pending list, one
// entry per lane, with the same room reservation as the fused path.
template <int PAIR = PAIR_BITHASH>
__global__ __launch_bounds__(BLOCK) void stash_kernel(EvictArgs a) {
  __shared__ uint64_t pre[NSHARD + 1];
  wl_prefix(a.ctl, pre);
  const uint64_t cnt = pre[NSHARD];
  if (cnt == 0) return;
  a.spill = spill_placing(a.spill, a.ctl, a.inserts, 16);
  const Geo geo = read_geo(a.ctl);
  const bool unreserved = ld_ctl(&a.ctl->stash_count) + cnt <= a.stash_cap;
  const int lane = threadIdx.x & 63;
  const uint64_t stride = (uint64_t)gridDim.x * BLOCK;
  uint64_t n_side = 0, n_fresh = 0;
  for (uint64_t base = (uint64_t)blockIdx.x * BLOCK + (threadIdx.x & ~63u); base < cnt; base += stride) {
    const uint64_t t = base + lane;
    const uint64_t kv = t < cnt ? a.wl[wl_slot(pre, t, a.wl_seg_cap)] : EMPTY;
    const bool push = kv != EMPTY;
    const uint64_t pm = ballot(push);
    if (!pm) continue;
    const int leader = __builtin_ctzll(pm);
    uint64_t room = 0;
    if (!unreserved) {
      if (lane == leader) {
        const uint64_t n = (uint64_t)__popcll(pm);
        room = load_fresh(&a.ctl->stash_count) < a.stash_cap ? add64(&a.ctl->stash_count, n) : a.stash_cap;
      }
      room = read_lane64(room, leader);
    }
    if (push) {
      const int where = overflow_place<PAIR>(a, geo, kv, room + rank_below(pm));
      n_side += (where == 0 || where == 3) ? 1 : where == 1 ? (1ull << 32) : 0;
      n_fresh += where == 0;
    }
  }
  evict_counters(a, unreserved, (uint64_t)blockIdx.x * WAVES + (threadIdx.x >> 6), 0, 0, n_side, n_fresh, 0);
}

// ---------------------------------------------------------------------------
// Linear-hashing resize (Section IV-C), decided on the device.
//
// resize_kernel plans a call in every block (the plan is a function of the
// control block, which nobody changes before the last block has finished) and
// does all of its splits, of however many hashing rounds, in one launch: an
// entry's way through the rounds depends on the entry and its bucket alone,
// so each bucket's entries go to their last bucket at once.  merge_kernel
// does a contraction, whose pairs depend on one another, phase by phase
// within one launch.  When there is nothing to do, which is the usual batch,
// each is one idle launch; a plan, one or two passes per hashing round that
// the host could not rule out, a drain and a fold took 9 to 25 launches of
// 1 to 5 us each.
// ---------------------------------------------------------------------------
enum : uint32_t { PLAN_PRE = 0, PLAN_PRE_MIXED = 1, PLAN_POST = 2, PLAN_SPLIT = 3, PLAN_MERGE = 4, PLAN_NONE = 5 };

struct ResizeArgs {
  uint64_t *buckets;
  uint32_t *hint;
  Ctl *ctl;
  uint32_t S;
  uint32_t K;
  uint32_t lf_expand_pct;
  uint32_t lf_contract_pct;
};

// Geometry of the next segment.  Splits first finish a round (sp == im+1 is
// the same addressing as the next round with sp == 0); merges first regress
// a round when sp == 0 (again the same addressing).
__device__ __forceinline__ void plan_next(volatile Ctl *c) {
  c->seg = 0;
  if (c->resize_todo == 0) {
    c->resize_dir = 0;
    return;
  }
  if (c->resize_dir > 0) {
    if (c->sp == c->im + 1) {
      c->im = 2 * c->im + 1;
      c->sp = 0;
    }
    const uint64_t room = c->max_buckets - c->n_buckets;
    if (room == 0) {
      c->resize_todo = 0;
      c->resize_dir = 0;
      return;
    }
    c->seg = min(min(c->resize_todo, c->im + 1 - c->sp), room);
  } else {
    if (c->n_buckets <= c->initial_buckets) {
      c->resize_todo = 0;
      c->resize_dir = 0;
      return;
    }
    if (c->sp == 0) {
      c->im >>= 1;
      c->sp = c->im + 1;
    }
    c->seg = min(min(c->resize_todo, c->sp), c->n_buckets - c->initial_buckets);
    c->merge_commit = c->seg;
  }
}

// Pairs the load-factor rule asks for, in whole K-pair steps: expansion
// while (live + extra) * 100 > lf_expand * buckets * S, contraction while
// live * 100 < lf_contract * buckets * S and the table is above its initial
// size.
struct Plan {
  int64_t dir;    // +1 split, -1 merge, 0 nothing
  uint64_t todo;  // pairs
};
__device__ __forceinline__ Plan plan_policy(const ResizeArgs &a, uint64_t nb, uint64_t live, uint64_t initial,
                                            uint64_t extra, bool allow_contract) {
  const uint64_t S = a.S, K = a.K;
  const uint64_t need = live + extra;
  Plan p{0, 0};
  if (need * 100 > (uint64_t)a.lf_expand_pct * nb * S) {
    const uint64_t den = (uint64_t)a.lf_expand_pct * S;
    const uint64_t r = (need * 100 + den - 1) / den;  // fewest buckets that satisfy the rule
    const uint64_t steps = (r - nb + K - 1) / K;
    p.dir = 1;
    p.todo = steps * K;
  } else if (allow_contract && live * 100 < (uint64_t)a.lf_contract_pct * nb * S && nb > initial) {
    const uint64_t q = live * 100 / ((uint64_t)a.lf_contract_pct * S);
    const uint64_t lim = max(q, initial);
    if (nb > lim) {
      const uint64_t steps = (nb - lim + K - 1) / K;
      const uint64_t fin = (nb > steps * K && nb - steps * K > initial) ? nb - steps * K : initial;
      p.dir = -1;
      p.todo = nb - fin;
    }
  }
  return p;
}

// The pairs a call asks for.  `amount` is the insert count (PRE), or the pair
// count (SPLIT, MERGE).
__device__ __forceinline__ Plan plan_of(const ResizeArgs &a, uint32_t mode, uint64_t amount, uint64_t nb,
                                        uint64_t live, uint64_t initial) {
  switch (mode) {
    case PLAN_PRE:
    case PLAN_PRE_MIXED: return plan_policy(a, nb, live, initial, amount, false);
    case PLAN_POST: return plan_policy(a, nb, live, initial, 0, true);
    case PLAN_SPLIT: return Plan{1, amount};
    case PLAN_MERGE: return Plan{-1, amount};
    default: return Plan{0, 0};
  }
}

// Start a resize call of the persistent executor (one thread): the pairs the
// call asks for, then the first segment.
__device__ __forceinline__ void plan_start(volatile Ctl *c, const ResizeArgs &a, uint32_t mode, uint64_t amount) {
  c->resize_dir = 0;
  c->resize_todo = 0;
  c->ticket = 0;
  if (c->mode != ADDR_LINEAR) {
    c->seg = 0;
    return;
  }
  const Plan p = plan_of(a, mode, amount, c->n_buckets, c->live, c->initial_buckets);
  c->resize_dir = p.dir;
  c->resize_todo = p.todo;
  plan_next(c);
}

// Insert operations of a mixed batch, for its pre-batch plan: NSHARD blocks,
// each leaves its count in its shard (overwritten by the next batch's).
__global__ __launch_bounds__(1024) void count_inserts_kernel(Ctl *c, const uint8_t *ops, uint64_t n) {
  __shared__ uint32_t part[16];
  uint32_t mine = 0;
  const uint64_t per = (n + NSHARD - 1) / NSHARD, b = (uint64_t)blockIdx.x * per, e = min(b + per, n);
  for (uint64_t i = b + threadIdx.x; i < e; i += 8 * 1024) {
#pragma unroll
    for (int j = 0; j < 8; ++j) mine += (i + j * 1024 < e && ops[i + j * 1024] == OP_INSERT) ? 1u : 0u;
  }
  const uint64_t sum = wave_sum64(mine);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = (uint32_t)sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t total = 0;
    for (int w = 0; w < 16; ++w) total += part[w];
    __hip_atomic_store(&shard_of(c, blockIdx.x)->plan_inserts, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Ticket for "the last block of this launch": every block has finished its
// reads of the control block.  Two levels, so that no counter takes more
// than NSHARD atomics: block b counts on shard b % NSHARD, and the block
// completing a shard counts on Ctl::ticket.  The last block resets both
// levels for the next launch.
//
// No release fence before the count: the last block only rewrites control
// scalars (geometry, counts) that the other blocks read before they count
// (their loads have returned: the values bound the work they did), and the
// table words the other blocks wrote are read by later launches, which the
// kernel boundary orders.  An agent-scope release writes back the block's
// L2, one after another per XCD: with a 2,048-block grid the fences alone
// cost 26 us (43 us with dirty lines) against 7 us for the same launch
// without them.
__device__ __forceinline__ bool last_block(Ctl *c) {
  __shared__ bool last;
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint64_t grid = gridDim.x, s = blockIdx.x % NSHARD;
    const uint64_t in_shard = (grid - s + NSHARD - 1) / NSHARD;
    bool l = false;
    if (add64(&shard_of(c, s)->ticket, 1) + 1 == in_shard)
      l = add64(&c->ticket, 1) + 1 == min(grid, (uint64_t)NSHARD);
    last = l;
  }
  __syncthreads();
  if (last) {
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (threadIdx.x < NSHARD)
      __hip_atomic_store(&shard_of(c, threadIdx.x)->ticket, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (threadIdx.x == 0) __hip_atomic_store(&c->ticket, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  return last;
}

__device__ __forceinline__ void evict_finish(Ctl *c, bool items, uint64_t inserts) {
  if (items) {
    // this thread's counter updates are done before its block is counted
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (!last_block(c)) return;
  } else if (blockIdx.x != 0) {
    return;
  }
  if (threadIdx.x < 64) (void)fold_shards_wave(c, true, inserts);
}

__device__ __forceinline__ uint32_t nth_set_bit(uint64_t m, uint32_t r) {
  for (uint32_t i = 0; i < r; ++i) m &= m - 1;
  return (uint32_t)__builtin_ctzll(m);
}

// One split pair (Section IV-C-1): pair j of the segment is (src, src + 2^m)
// with src = sp + j.  An entry stays when one of its candidate hashes still
// addresses src under the next round's mask, otherwise it moves; movers are
// compacted into the partner's first slots (the partner is EMPTY).
template <int S>
__device__ __forceinline__ void split_pair(const ResizeArgs &a, uint64_t im, uint64_t sp, uint64_t j, int g, int sl) {
  using T = Traits<S>;
  const uint64_t src = sp + j, dst = src + im + 1, next = 2 * im + 1;
  const uint64_t w = a.buckets[src * S + sl];
  bool move = false;
  if (w != EMPTY) {
    const uint32_t h1 = bithash1(key_of(w)), h2 = bithash2(key_of(w));
    const bool stay = ((h1 & im) == src && (h1 & next) == src) || ((h2 & im) == src && (h2 & next) == src);
    move = !stay;
  }
  const uint64_t mm = (ballot(move) >> (g * S)) & T::FULL;
  if (move) {
    const uint32_t rank = __builtin_popcountll(mm & ((1ull << sl) - 1ull));
    a.buckets[dst * S + rank] = w;
    a.buckets[src * S + sl] = EMPTY;
  }
}

// State word of a merge phase over n pairs: kind:4 (1 test, 2 move, 0 none
// left) | runs:12 | number of the phase:48, the last one's plus one.  At most
// one run of pairs per block of merge_kernel, and of MERGE_RUN pairs at least.
// (A claim is compared by its distance to the number, so the numbers must not
// come round: 48 bits are decades of phases.)
constexpr int MERGE_NUMBER_BITS = 48;
constexpr uint64_t MERGE_NUMBER = (1ull << MERGE_NUMBER_BITS) - 1;
static_assert(MERGE_GRID < 1 << 12, "runs of a phase in 12 bits");
__device__ __forceinline__ uint64_t merge_phase(uint64_t kind, uint64_t n, uint64_t last) {
  const uint64_t number = (last + 1) & MERGE_NUMBER;
  const uint64_t runs = min((n + MERGE_RUN - 1) / MERGE_RUN, (uint64_t)MERGE_GRID);
  return n ? (kind << 60) | (runs << MERGE_NUMBER_BITS) | number : number;
}

// The word that holds the number of the last phase in which run r was claimed.
__device__ __forceinline__ uint64_t *merge_claim(const Ctl *c, uint64_t r) {
  static_assert(MERGE_GRID <= 8 * NSHARD, "eight runs a shard");
  return &shard_of(c, r % NSHARD)->merge_claim[r / NSHARD];
}

// Merge pair j of the segment, walked from the top: (lo, lo + 2^m) with
// lo = sp - 1 - j.  It fits when hi's entries fit lo's EMPTY slots
// (Section IV-C-2); the first pair that does not fit bounds the commit.
template <int S>
__device__ __forceinline__ void merge_test_pair(const ResizeArgs &a, Ctl *c, uint64_t im, uint64_t sp, uint64_t j,
                                                int g, int sl) {
  using T = Traits<S>;
  const uint64_t lo = sp - 1 - j, hi = lo + im + 1;
  const uint64_t wl = a.buckets[lo * S + sl], wh = a.buckets[hi * S + sl];
  const uint64_t fl = (ballot(wl == EMPTY) >> (g * S)) & T::FULL;
  const uint64_t lh = (ballot(wh != EMPTY) >> (g * S)) & T::FULL;
  if (sl == 0 && __builtin_popcountll(lh) > __builtin_popcountll(fl))
    __hip_atomic_fetch_min(&c->merge_commit, j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Move a merge pair that fits: the r-th live entry of hi goes to the r-th
// EMPTY slot of lo; stash entries with a candidate in hi now address lo.
template <int S>
__device__ __forceinline__ void merge_move_pair(const ResizeArgs &a, uint64_t im, uint64_t sp, uint64_t j, int g,
                                                int sl) {
  using T = Traits<S>;
  const uint64_t lo = sp - 1 - j, hi = lo + im + 1;
  const uint64_t wl = a.buckets[lo * S + sl], wh = a.buckets[hi * S + sl];
  const uint64_t fl = (ballot(wl == EMPTY) >> (g * S)) & T::FULL;
  const uint64_t lh = (ballot(wh != EMPTY) >> (g * S)) & T::FULL;
  if (wh != EMPTY) {
    const uint32_t r = __builtin_popcountll(lh & ((1ull << sl) - 1ull));
    a.buckets[lo * S + nth_set_bit(fl, r)] = wh;
    a.buckets[hi * S + sl] = EMPTY;
  }
  if (sl == 0 && ((a.hint[hi >> 5] >> (hi & 31)) & 1u)) set_hint(a.hint, (uint32_t)lo);
}

// Pairs [begin, end) of a merge phase (TEST, or move) by one block of
// merge_kernel, as the two functions above do one pair.  MERGE_LOADS pairs per
// group of lanes are in flight, and a word finds its EMPTY slot by two lane
// permutations (its rank among the live, the slot's among the EMPTY ones): 256
// blocks that waited for each pair and selected slots bit by bit took 715 us
// for 2^21 pairs in three rounds.  Loads and stores are agent-scope: the phases
// of one launch read what blocks of other XCDs wrote in the one before, and so
// need no L2 write-back and no invalidation (a fence pair per run of pairs made
// a contraction take 551 us).
template <int S, bool TEST>
__device__ __forceinline__ void merge_run(const ResizeArgs &a, Ctl *c, uint64_t im, uint64_t sp, uint64_t begin,
                                          uint64_t end) {
  using T = Traits<S>;
  constexpr int U = MERGE_LOADS;
  constexpr uint64_t STEP = (uint64_t)(MERGE_BLOCK / 64) * T::G;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int g = lane / S, sl = lane % S;
  const uint64_t below = (1ull << sl) - 1ull;
  // a uniform trip count per wave: every lane reaches the ballots
  for (uint64_t j0 = begin + (uint64_t)wv * T::G; j0 < end; j0 += U * STEP) {
    uint64_t wl[U], wh[U];
    uint32_t hint[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint64_t j = j0 + u * STEP + g, lo = sp - 1 - j, hi = lo + im + 1;
      const bool have = j < end;
      wl[u] = have ? load_fresh(a.buckets + lo * S + sl) : EMPTY;
      wh[u] = have ? load_fresh(a.buckets + hi * S + sl) : EMPTY;
      hint[u] = !TEST && have && sl == 0 ? ld_ctl32(a.hint + (hi >> 5)) >> (hi & 31) : 0u;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint64_t j = j0 + u * STEP + g, lo = sp - 1 - j, hi = lo + im + 1;
      const uint64_t fl = (ballot(wl[u] == EMPTY) >> (g * S)) & T::FULL;
      const uint64_t lh = (ballot(wh[u] != EMPTY) >> (g * S)) & T::FULL;
      const int live = __builtin_popcountll(lh);
      if constexpr (TEST) {
        if (sl == 0 && live > __builtin_popcountll(fl))
          __hip_atomic_fetch_min(&c->merge_commit, j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else {
        // live words to the group's first lanes, the others behind them
        const int rank = __builtin_popcountll(lh & below);
        const int to = (g * S + (wh[u] != EMPTY ? rank : live + sl - rank)) << 2;
        const uint32_t p0 = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)(uint32_t)wh[u]);
        const uint32_t p1 = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)(uint32_t)(wh[u] >> 32));
        const int slot = __builtin_popcountll(fl & below);  // of an EMPTY slot: its rank
        const uint64_t w = shfl64(((uint64_t)p1 << 32) | p0, g * S + min(slot, S - 1));
        if (wl[u] == EMPTY && slot < live)
          __hip_atomic_store(a.buckets + lo * S + sl, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (wh[u] != EMPTY)
          __hip_atomic_store(a.buckets + hi * S + sl, EMPTY, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (hint[u] & 1u) set_hint(a.hint, (uint32_t)lo);
      }
    }
  }
}

// Geometry after a finished segment (run by one thread once every pair of
// the segment is done), then the plan of the next segment.
__device__ __forceinline__ void split_segment_done(volatile Ctl *c, uint64_t sp, uint64_t seg) {
  c->sp = sp + seg;
  c->n_buckets += seg;
  c->resize_todo -= seg;
  c->split_happened = 1;
  plan_next(c);
}

__device__ __forceinline__ void merge_segment_done(volatile Ctl *c, uint64_t sp, uint64_t seg, uint64_t commit) {
  c->sp = sp - commit;
  c->n_buckets -= commit;
  c->resize_todo -= commit;
  if (commit < seg) c->resize_todo = 0;  // a pair did not fit: the call stops here
  plan_next(c);
}

// After splits: every stash and pending entry moves to the eviction worklist
// (the eviction phase re-places it under the new geometry) and the hint bits
// are cleared (Section III-B "Overflow Stash").  The executor's drain chunks
// make one wave-aggregated append per wave and item range; `t` indexes stash words (the whole table, which
// is reset to EMPTY on the way) then pending entries, and the 256-entry tile
// t / 256 picks the worklist segment.
__device__ __forceinline__ uint64_t drain_word(uint64_t t, uint64_t n_stash_words, uint64_t total,
                                               const uint64_t *stash, const uint64_t *pending) {
  return t < n_stash_words ? stash[t] : t < total ? pending[t - n_stash_words] : TOMB;
}

// Word w (drain_word of t) to the worklist; a used stash word is reset.
__device__ __forceinline__ void drain_append(uint64_t t, uint64_t w, uint64_t n_stash_words, uint64_t *stash,
                                             uint64_t *wl, uint64_t seg_cap, Ctl *c) {
  if (t < n_stash_words && w != EMPTY) stash[t] = EMPTY;
  const bool live = w != TOMB && w != EMPTY;
  const uint64_t m = ballot(live);
  if (m) {
    const int lane = threadIdx.x & 63;
    const int leader = __builtin_ctzll(m);
    uint64_t base = 0;
    const uint64_t tile = t / BLOCK;
    if (lane == leader) base = wl_append(c, tile, (uint64_t)__popcll(m));
    base = read_lane64(base, leader);
    if (live) wl[(tile % NSHARD) * seg_cap + base + rank_below(m)] = w;
  }
}

__device__ __forceinline__ void drain_collect(uint64_t t, uint64_t n_stash_words, uint64_t total, uint64_t *stash,
                                              const uint64_t *pending, uint64_t *wl, uint64_t seg_cap, Ctl *c) {
  drain_append(t, drain_word(t, n_stash_words, total, stash, pending), n_stash_words, stash, wl, seg_cap, c);
}

__device__ __forceinline__ void drain_done(volatile Ctl *c) {
  c->stash_count = 0;
  c->pending_count = 0;
  c->split_happened = 0;
}

struct DrainArgs {
  uint64_t *stash, *pending, *wl;
  uint64_t stash_cap, pending_cap, wl_seg_cap, hint_words;
};

// The whole grid's drain: hint bits cleared, stash words reset, live entries
// appended to the worklist.  Every thread calls it.
__device__ __forceinline__ void drain_all(const DrainArgs &d, uint32_t *hint, Ctl *c) {
  const uint64_t n_stash = min(ld_ctl(&c->stash_count), d.stash_cap) ? stash_slots_for(d.stash_cap) : 0;
  const uint64_t n_pend = min(ld_ctl(&c->pending_count), d.pending_cap);
  const uint64_t total = n_stash + n_pend;
  const uint64_t stride = (uint64_t)gridDim.x * BLOCK;
  const uint64_t tid = (uint64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (total) {
    for (uint64_t t = tid; t < d.hint_words; t += stride) hint[t] = 0u;
  }
  // A trip of a block takes DRAIN_WORDS tiles of 256 words that share one
  // worklist segment (tiles T, T + NSHARD, ...: word t is in tile t / 256,
  // which appends to segment tile % NSHARD, so segment fills stay within the
  // capacity sized from the words walked), loads all of its words at once
  // (the walk of a mostly empty stash table is bound by load latency), and
  // appends its live words with one atomic: per-wave appends queued
  // thousands of atomics on each segment counter.
  __shared__ uint32_t s_wave[WAVES];
  __shared__ uint64_t s_base;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const uint64_t tiles = (total + BLOCK - 1) / BLOCK;
  const uint64_t group = (uint64_t)NSHARD * DRAIN_WORDS;  // tiles of NSHARD trips
  const uint64_t trips = (tiles + group - 1) / group * NSHARD;
  for (uint64_t q = blockIdx.x; q < trips; q += gridDim.x) {
    const uint64_t seg = q % NSHARD, tile0 = (q / NSHARD) * group + seg;
    uint64_t w[DRAIN_WORDS];
#pragma unroll
    for (int j = 0; j < DRAIN_WORDS; ++j)
      w[j] = drain_word((tile0 + (uint64_t)j * NSHARD) * BLOCK + threadIdx.x, n_stash, total, d.stash, d.pending);
    uint32_t mine = 0;
#pragma unroll
    for (int j = 0; j < DRAIN_WORDS; ++j) {
      const uint64_t t = (tile0 + (uint64_t)j * NSHARD) * BLOCK + threadIdx.x;
      if (t < n_stash && w[j] != EMPTY) d.stash[t] = EMPTY;
      mine += (w[j] != TOMB && w[j] != EMPTY) ? 1u : 0u;
    }
    // block-wide exclusive prefix of the live counts
    uint32_t incl = mine;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(incl, o, 64);
      if (lane >= o) incl += y;
    }
    if (lane == 63) s_wave[wv] = incl;
    __syncthreads();
    uint32_t before = 0, sum = 0;
#pragma unroll
    for (int x = 0; x < WAVES; ++x) {
      before += x < wv ? s_wave[x] : 0u;
      sum += s_wave[x];
    }
    if (threadIdx.x == 0 && sum) s_base = wl_append(c, seg, sum);
    __syncthreads();
    if (sum) {
      uint64_t pos = seg * d.wl_seg_cap + s_base + before + incl - mine;
#pragma unroll
      for (int j = 0; j < DRAIN_WORDS; ++j)
        if (w[j] != TOMB && w[j] != EMPTY) d.wl[pos++] = w[j];
    }
    __syncthreads();  // s_wave and s_base of the next trip
  }
}

// One resize call: the plan, every split it asks for and the stash drain, or
// the first segment of its merges for merge_kernel.
//
// `drain`: entries of the stash and the pending list go to the worklist when
// this call or an earlier one without a drain split buckets; a later eviction
// launch places them.  Without it (a batch's growth before its probe launch,
// where the stash has to stay searchable) they stay, and a new bucket takes
// its ancestor's hint bit: the keys it may be a candidate of had the ancestor
// as theirs.
//
// A split entry's way: in each round whose range holds its bucket, it stays
// when one of its candidate hashes still addresses the bucket under the
// round's next mask, otherwise it moves to the bucket's partner (Section
// IV-C-1).  One round (the usual call) touches the buckets it splits, and so do
// two: those left of the first round and those at the second's start (a step of
// 1,024 pairs over the end of a round at 2^23 buckets took 457 us when it read
// all of them, now 15).  Movers take the first slots of their new buckets,
// which are EMPTY and which no other bucket's entries reach: a bucket b beyond
// the old count has one ancestor, b without its top bits.
template <int S>
__global__ __launch_bounds__(BLOCK) void resize_kernel(ResizeArgs a, DrainArgs d, uint32_t mode, uint64_t amount,
                                                       const uint8_t *ops, bool drain) {
  using T = Traits<S>;
  constexpr int MAX_ROUNDS = 34;
  __shared__ uint64_t r_im[MAX_ROUNDS], r_sp[MAX_ROUNDS], r_seg[MAX_ROUNDS];
  __shared__ uint64_t s_todo, s_im, s_sp, s_nb, s_ins;
  __shared__ int64_t s_dir;
  __shared__ uint32_t s_rounds, s_split_before;
  Ctl *c = a.ctl;
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
  uint64_t inserts = 0;
  if (mode == PLAN_PRE_MIXED && ops) {
    // a small batch's inserts, counted by every block
    if (tid == 0) s_ins = 0;
    __syncthreads();
    uint64_t mine = 0;
    for (uint64_t i = tid; i < amount; i += BLOCK) mine += ops[i] == OP_INSERT;
    mine = wave_sum64(mine);
    if (lane == 0 && mine) atomicAdd((unsigned long long *)&s_ins, (unsigned long long)mine);
    __syncthreads();
    inserts = s_ins;
  }
  if (tid < NSHARD) {
    // key-count changes that are still in the shards, and the count of a
    // larger batch's inserts
    const Shard *sh = shard_of(c, tid);
    const uint64_t dl = wave_sum64(ld_ctl(&sh->live));
    if (mode == PLAN_PRE_MIXED && !ops) inserts = wave_sum64(ld_ctl(&sh->plan_inserts));
    if (tid == 0) {
      const uint64_t nb = ld_ctl(&c->n_buckets), max_b = ld_ctl(&c->max_buckets);
      uint64_t im = ld_ctl(&c->im), sp = ld_ctl(&c->sp);
      const Plan p = plan_of(a, mode, mode == PLAN_PRE_MIXED ? inserts : amount, nb, ld_ctl(&c->live) + dl,
                             ld_ctl(&c->initial_buckets));
      uint64_t todo = p.dir > 0 ? min(p.todo, max_b - nb) : p.todo, left = todo;
      uint32_t rounds = 0;
      if (p.dir > 0) {
        while (left > 0) {
          if (sp == im + 1) {
            im = 2 * im + 1;
            sp = 0;
          }
          const uint64_t seg = min(left, im + 1 - sp);
          r_im[rounds] = im;
          r_sp[rounds] = sp;
          r_seg[rounds] = seg;
          ++rounds;
          sp += seg;
          left -= seg;
        }
      }
      s_dir = todo ? p.dir : 0;
      s_todo = todo;
      s_im = im;
      s_sp = sp;
      s_nb = nb;
      s_rounds = rounds;
      s_split_before = ld_ctl(&c->split_happened) != 0;
    }
  }
  __syncthreads();
  const int64_t dir = s_dir;
  const uint64_t todo = s_todo, nb = s_nb;
  const bool draining = drain && (dir > 0 || s_split_before);
  if (dir == 0 && !draining) return;  // the same in every block: nobody takes a ticket
  if (dir > 0) {
    const uint32_t rounds = s_rounds;
    const int g = lane / S, sl = lane % S;
    // [0, head) and [r_sp[0], + r_seg[0]), in one where they meet
    uint64_t head = rounds == 1 ? 0 : min(r_seg[1], nb), tail = r_seg[0];
    if (rounds > 1 && head >= r_sp[0]) {
      head = max(head, r_sp[0] + tail);
      tail = 0;
    }
    const uint64_t count = head + tail;
    const uint64_t groups = (uint64_t)gridDim.x * WAVES * T::G;
    // a uniform trip count per wave: the shuffles below take every lane
    for (uint64_t j0 = ((uint64_t)blockIdx.x * WAVES + wv) * T::G; j0 < count; j0 += groups) {
      const uint64_t at = j0 + g, src = at < head ? at : r_sp[0] + (at - head);
      const bool have = at < count;
      const uint64_t w = have ? a.buckets[src * S + sl] : EMPTY;
      uint64_t b = src;
      if (w != EMPTY) {
        const uint32_t h1 = bithash1(key_of(w)), h2 = bithash2(key_of(w));
        for (uint32_t r = 0; r < rounds; ++r) {
          const uint64_t im = r_im[r], next = 2 * im + 1;
          if (b - r_sp[r] >= r_seg[r]) continue;  // not split in this round (b below the range wraps)
          const bool stay = ((h1 & im) == b && (h1 & next) == b) || ((h2 & im) == b && (h2 & next) == b);
          if (!stay) b += im + 1;
        }
      }
      const bool move = b != src;
      const uint64_t mm = (ballot(move) >> (g * S)) & T::FULL;
      uint32_t rank = (uint32_t)__builtin_popcountll(mm & ((1ull << sl) - 1ull));
      if (rounds > 1 && ballot(move)) {
        rank = 0;
        for (int t = 0; t < S; ++t) {
          const uint32_t o = (uint32_t)__shfl((int)(uint32_t)b, g * S + t, 64);
          if (t < sl && ((mm >> t) & 1ull) && o == (uint32_t)b) ++rank;
        }
      }
      if (move) {
        a.buckets[b * S + rank] = w;
        a.buckets[src * S + sl] = EMPTY;
      }
    }
    if (!draining) {
      const uint64_t stride = (uint64_t)gridDim.x * BLOCK;
      for (uint64_t f = nb + (uint64_t)blockIdx.x * BLOCK + tid; f < nb + todo; f += stride) {
        uint64_t anc = f;
        while (anc >= nb) anc ^= 1ull << (63 - __builtin_clzll(anc));
        if ((a.hint[anc >> 5] >> (anc & 31)) & 1u) set_hint(a.hint, (uint32_t)f);
      }
    }
  }
  if (draining) drain_all(d, a.hint, c);
  if (last_block(c) && tid == 0) {
    volatile Ctl *v = c;
    if (draining) drain_done(v);
    if (dir > 0) {
      v->n_buckets = nb + todo;
      v->im = s_im;
      v->sp = s_sp;
      if (!draining) v->split_happened = 1;
    } else if (dir < 0) {
      v->resize_dir = -1;
      v->resize_todo = todo;
      plan_next(v);
      v->merge_state = merge_phase(1, v->seg, v->merge_state & MERGE_NUMBER);
    }
  }
}

// A contraction (Section IV-C-2): per hashing round, every pair of the
// segment is tested, top down, then the pairs above the first that does not
// fit are moved.  The phases run within one launch: blocks claim runs of pairs
// of the current phase, and the block that completes a phase publishes the
// next.  A block takes the run of its own number and, when it has waited a
// while, one that nobody has claimed, so that it waits only for runs that other
// running blocks have claimed and the launch ends however few blocks run at a
// time.  Claims are words of their own and completions count on two levels:
// with one counter for all claims and one for all completions, of about 64 ns
// an atomic, 131,072 pairs in three rounds (six phases of 256 runs) took 136 us,
// now 61; three rounds down from 2^20 / 2^23 more buckets 715 / 5,451 us, now
// 373 / 2,756.  (A launch per phase, with the host between rounds: 64, 290 and
// 2,609.)  A phase costs about 6 us besides its pairs, and these are bound by
// what 16 waves a compute unit keep in flight.
template <int S>
__global__ __launch_bounds__(MERGE_BLOCK) void merge_kernel(ResizeArgs a) {
  __shared__ uint64_t s_state;
  __shared__ uint32_t s_pick, s_won;
  Ctl *c = a.ctl;
  const uint32_t tid = threadIdx.x;
  uint64_t seen = ~0ull;  // the phase the block waits in, and for how long
  uint32_t polls = 0;
  for (;;) {
    if (tid == 0) {
      s_state = ld_ctl(&c->merge_state);
      s_pick = ~0u;
    }
    __syncthreads();
    const uint64_t st = s_state, nch = (st >> MERGE_NUMBER_BITS) & 0xFFFu, number = st & MERGE_NUMBER;
    if ((st >> 60) == 0) return;
    if (st != seen) {
      seen = st;
      polls = 0;
    }
    // a run whose last claim is an earlier phase's (a later one's: this block's
    // view of the state is old, and its phase complete)
    static_assert(MERGE_GRID <= MERGE_BLOCK, "a thread per run");
    const bool look = polls == 0 ? tid == blockIdx.x : polls >= 8;
    uint64_t old = 0;
    bool open = false;
    if (look && tid < nch) {
      old = load_fresh(merge_claim(c, tid));
      const uint64_t age = (number - old) & MERGE_NUMBER;
      open = age != 0 && age <= MERGE_NUMBER / 2;
      // waiting blocks start at different runs
      if (open) atomicMin(&s_pick, (uint32_t)((tid + nch - blockIdx.x % nch) % nch));
    }
    if (tid == 0) s_won = 0;
    __syncthreads();
    const uint64_t mine = ((uint64_t)s_pick + blockIdx.x % nch) % nch;
    if (s_pick != ~0u && tid == mine && open) s_won = cas64(merge_claim(c, mine), old, number) == old;
    __syncthreads();
    ++polls;
    if (!s_won) {  // other blocks are at work
      __builtin_amdgcn_s_sleep(15);
      continue;
    }
    const bool test = (st >> 60) == 1;
    const uint64_t im = ld_ctl(&c->im), sp = ld_ctl(&c->sp);
    const uint64_t pairs = test ? ld_ctl(&c->seg) : ld_ctl(&c->merge_commit);
    const uint64_t per = (pairs + nch - 1) / nch, end = min(pairs, (mine + 1) * per);
    if (test)
      merge_run<S, true>(a, c, im, sp, mine * per, end);
    else
      merge_run<S, false>(a, c, im, sp, mine * per, end);
    // every wave's stores and minima are done before the run is counted
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
      Shard *sh = shard_of(c, mine % NSHARD);
      if (add64(&sh->merge_done, 1) + 1 == (nch - mine % NSHARD + NSHARD - 1) / NSHARD) {
        __hip_atomic_store(&sh->merge_done, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // before the next phase can count on it
        if (add64(&c->merge_done, 1) + 1 == min(nch, (uint64_t)NSHARD)) {
          // merge_segment_done and plan_next in registers: loads and stores in
          // flight together, and no fence (a chain of volatile accesses and an
          // L2 write-back cost 10 us a segment)
          const uint64_t seg = ld_ctl(&c->seg), commit = ld_ctl(&c->merge_commit), initial = ld_ctl(&c->initial_buckets);
          uint64_t buckets = ld_ctl(&c->n_buckets), todo = ld_ctl(&c->resize_todo);
          const auto put = [](uint64_t *p, uint64_t v) {
            __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          };
          put(&c->merge_done, 0);
          uint64_t next;
          if (test && commit > 0) {
            next = merge_phase(2, commit, number);
          } else {
            uint64_t im2 = im, sp2 = sp - commit, seg2 = 0;
            buckets -= commit;
            todo = commit < seg ? 0 : todo - commit;  // a pair did not fit: the call stops here
            if (buckets <= initial) todo = 0;
            if (todo > 0) {
              if (sp2 == 0) {
                im2 >>= 1;
                sp2 = im2 + 1;
              }
              seg2 = min(min(todo, sp2), buckets - initial);
              put(&c->merge_commit, seg2);
            } else {
              put((uint64_t *)&c->resize_dir, 0);
            }
            put(&c->im, im2);
            put(&c->sp, sp2);
            put(&c->seg, seg2);
            put(&c->n_buckets, buckets);
            put(&c->resize_todo, todo);
            next = merge_phase(seg2 > 0 ? 1 : 0, seg2, number);
          }
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // all of it before the phase
          __hip_atomic_store(&c->merge_state, next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Dump: every live word with its place (bucket, -1 stash, -2 pending).
//
// Bound by memory (each table word read once, each live word written once)
// as long as the output positions cost little: every position comes from one
// counter, and a device atomic on one address takes about 64 ns.  A block of
// 8 waves (16 have no room beside a resident executor) therefore takes
// DUMP_LOADS words per thread and trip (64 KiB of a 64-bit table, held in
// registers), counts them by ballots and reserves
// room for the whole trip with one add; a wave's live words then go to
// consecutive positions.  One add per wave had made a 4.0 M-entry dump of
// 4.2 M slots 794 us; now about 10 us (export, re-insertion and lookups of
// the entries 1,315 -> 530 us).
// SET32: words of a key-only set (the key itself, EMPTY all ones), written as
// 64-bit words with value half 0.
// ---------------------------------------------------------------------------
constexpr int DUMP_BLOCK = 512;
constexpr int DUMP_LOADS = 16;
constexpr uint64_t DUMP_TRIP = (uint64_t)DUMP_BLOCK * DUMP_LOADS;

template <bool SET32>
__global__ __launch_bounds__(DUMP_BLOCK) __attribute__((amdgpu_waves_per_eu(6))) void dump_kernel(const void *bucket_words, uint32_t S,
                                                          const void *stash_words, const void *pending_words,
                                                          Ctl *ctl, uint64_t stash_cap, uint64_t pending_cap,
                                                          uint64_t *out, int64_t *where, uint64_t cap) {
  using Word = typename std::conditional<SET32, uint32_t, uint64_t>::type;
  constexpr int DW = DUMP_BLOCK / 64;
  constexpr int COUNTS = DUMP_LOADS * DW;
  __shared__ uint32_t off[COUNTS];  // live words of (load, wave), then their exclusive prefix
  __shared__ uint32_t part[COUNTS / 64], total_live;
  __shared__ uint64_t s_base;
  static_assert(COUNTS % 64 == 0 && COUNTS <= DUMP_BLOCK, "whole waves scan the counts");
  const Word *buckets = (const Word *)bucket_words, *stash = (const Word *)stash_words,
             *pending = (const Word *)pending_words;
  const uint64_t nb = ctl->n_buckets;
  const uint64_t n_stash = min(ctl->stash_count, stash_cap) ? stash_slots_for(stash_cap) : 0;
  const uint64_t n_pend = min(ctl->pending_count, pending_cap);
  const uint64_t n_slots = nb * S, total = n_slots + n_stash + n_pend;
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
  for (uint64_t t0 = (uint64_t)blockIdx.x * DUMP_TRIP; t0 < total; t0 += (uint64_t)gridDim.x * DUMP_TRIP) {
    Word w[DUMP_LOADS];
#pragma unroll
    for (int j = 0; j < DUMP_LOADS; ++j) {
      const uint64_t t = t0 + (uint64_t)j * DUMP_BLOCK + tid;
      w[j] = t < n_slots             ? buckets[t]
             : t < n_slots + n_stash ? stash[t - n_slots]
             : t < total             ? pending[t - n_slots - n_stash]
                                     : (Word)0;
    }
    uint64_t live[DUMP_LOADS];  // EMPTY: all ones, TOMB: 0 (no bucket word is 0)
#pragma unroll
    for (int j = 0; j < DUMP_LOADS; ++j) {
      live[j] = ballot(w[j] != (Word)~(Word)0 && w[j] != 0);
      if (lane == 0) off[j * DW + wv] = (uint32_t)__popcll(live[j]);
    }
    __syncthreads();
    uint32_t mine = 0, incl = 0;
    if (tid < COUNTS) {
      mine = incl = off[tid];
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
      }
      if (lane == 63) part[wv] = incl;
    }
    __syncthreads();
    if (tid < COUNTS) {
      uint32_t before = 0;
      for (int x = 0; x < wv; ++x) before += part[x];
      off[tid] = before + incl - mine;
      if (tid == COUNTS - 1) total_live = before + incl;
    }
    __syncthreads();
    if (tid == 0) s_base = total_live ? add64(&ctl->dump_count, total_live) : 0;
    __syncthreads();
    const uint64_t base = s_base;
#pragma unroll
    for (int j = 0; j < DUMP_LOADS; ++j) {
      if (!((live[j] >> lane) & 1ull)) continue;
      const uint64_t pos = base + off[j * DW + wv] + rank_below(live[j]);
      if (pos >= cap) continue;
      out[pos] = w[j];
      if (where) {
        const uint64_t t = t0 + (uint64_t)j * DUMP_BLOCK + tid;
        where[pos] = t < n_slots ? (int64_t)(t / S) : t < n_slots + n_stash ? -1 : -2;
      }
    }
    __syncthreads();  // off and s_base of the next trip
  }
}

// Placement census: live bucket entries in their first candidate bucket and
// in their second one (the two differ).
// SET32: buckets of 32-bit entries (the key itself; EMPTY is all ones).
template <bool SET32>
__global__ __launch_bounds__(BLOCK) void placement_kernel(const void *bucket_words, uint32_t S, Ctl *ctl) {
  __shared__ unsigned long long s_first, s_second;
  if (threadIdx.x == 0) s_first = s_second = 0;
  __syncthreads();
  unsigned long long n_first = 0, n_second = 0;
  const Geo geo = read_geo(ctl);
  const uint64_t n_slots = geo.n_buckets * S;
  const uint64_t stride = (uint64_t)gridDim.x * BLOCK;
  const uint64_t span = (n_slots + stride - 1) / stride * stride;
  for (uint64_t t = (uint64_t)blockIdx.x * BLOCK + threadIdx.x; t < span; t += stride) {
    uint64_t w = EMPTY;
    if (t < n_slots) {
      if constexpr (SET32) {
        const uint32_t x = ((const uint32_t *)bucket_words)[t];
        w = x == 0xFFFFFFFFu ? EMPTY : x;
      } else {
        w = ((const uint64_t *)bucket_words)[t];
      }
    }
    const bool live = w != EMPTY;
    const bool first = live && address(geo, bithash1(key_of(w))) == (uint32_t)(t / S);
    const uint64_t mf = ballot(first), ms = ballot(live && !first);
    if ((threadIdx.x & 63) == 0) {
      n_first += (uint64_t)__popcll(mf);
      n_second += (uint64_t)__popcll(ms);
    }
  }
  // one pair of atomics per block
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(&s_first, n_first);
    atomicAdd(&s_second, n_second);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    if (s_first) add64(&ctl->place_first, s_first);
    if (s_second) add64(&ctl->place_second, s_second);
  }
}

__global__ void ctl_zero_placement_kernel(Ctl *ctl) {
  ctl->place_first = 0;
  ctl->place_second = 0;
}

// Empties a table: every word of its buckets and stash EMPTY, hint and filter
// bits and shards cleared, the control block as at creation.  One launch: a
// small table's clear is bound by launches (five before, 2 to 3 us each).
struct ResetArgs {
  uint64_t *buckets, *stash, *shards;  // word counts even, 16-byte aligned
  uint32_t *bits;
  uint64_t n_buckets, n_stash, n_shards, n_bits;
  Ctl *ctl;
};
__global__ __launch_bounds__(BLOCK) void reset_kernel(ResetArgs a, Ctl init) {
  const uint64_t first = (uint64_t)blockIdx.x * BLOCK + threadIdx.x, stride = (uint64_t)gridDim.x * BLOCK;
  const auto fill = [&](uint64_t *p, uint64_t n, uint64_t v) {
    for (uint64_t t = first; t < n / 2; t += stride) *(ulonglong2 *)(p + 2 * t) = ulonglong2{v, v};
  };
  fill(a.buckets, a.n_buckets, EMPTY);
  fill(a.stash, a.n_stash, EMPTY);
  fill(a.shards, a.n_shards, 0);
  for (uint64_t t = first; t < a.n_bits; t += stride) a.bits[t] = 0u;
  if (first == 0) *a.ctl = init;
}

__global__ void ctl_zero_dump_kernel(Ctl *ctl) { ctl->dump_count = 0; }


// ---------------------------------------------------------------------------
// Persistent executor: one resident grid drains a queue of batches.
//
// The host appends batch descriptors to a ring in pinned host memory and
// advances a host-side tail.  Blocks of the resident grid ingest new
// descriptors into a device ring, and each batch then runs as a sequence of
// data-parallel phases (dedupe fill, dedupe, insert count, resize segments,
// stash drain, re-placement, probe tiles, eviction) split into chunks that
// any block may claim.  One 64-bit word per batch packs the phase, its chunk
// count and the number of chunks claimed, so a claim is one atomic add; the
// block that completes the last chunk of a phase runs the phase's scalar
// epilogue (geometry updates, plans) and publishes the next phase.  Batches
// on one table run in submission order (a per-table sequence number);
// batches on different tables overlap.  Completion is written to host-mapped
// memory.  Every block leaves the loop once the host has set the stop flag
// and every ingested batch is complete.
// ---------------------------------------------------------------------------
enum : uint32_t {
  PH_START = 0, PH_FILL = 1, PH_DEDUPE = 2, PH_COUNT = 3, PH_SEG_A = 4, PH_SEG_B = 5, PH_DRAIN = 6,
  PH_REPLACE = 7, PH_OPS = 8, PH_EVICT = 9, PH_DONE = 10
};
// Chunk sizes.  A claim costs a few dependent device-scope round trips, so
// streaming phases take large chunks; an eviction chunk gives each group
// one item, so a phase's chains run side by side in as many waves as the
// grid holds instead of one after another in fewer waves.
constexpr uint64_t FILL_PER_CHUNK = BLOCK * 64;   // words per fill chunk
constexpr uint64_t COUNT_PER_CHUNK = BLOCK * 16;  // operations per count chunk
constexpr uint64_t DRAIN_TILES = 16;              // stash tiles of BLOCK words per drain chunk
constexpr uint32_t DRAIN_WINDOW = 64;             // batches scanned for work

struct TableDesc {
  uint64_t *buckets;
  Spill spill;
  uint32_t *hint;
  uint64_t *stash;
  uint64_t *pending;
  Ctl *ctl;
  uint64_t *wl;
  uint64_t *dd;
  uint64_t wl_seg_cap, stash_cap, pending_cap, hint_words;
  uint32_t S, max_evictions, K, lf_expand_pct, lf_contract_pct, pre_expand, post_policy, addressing;
};

struct ReqDesc {  // written by the host
  TableDesc t;
  const uint8_t *ops;
  const uint32_t *keys;
  const uint32_t *vals;
  uint32_t *vals_out;
  uint8_t *flags_out;
  uint64_t n;
  uint32_t mode, flags;
  uint64_t seq, table_slot, ticket;
  uint64_t dd_size;  // dedupe by a set in HBM of this many words (0: not so)
  uint64_t dds;      // dedupe by hash ranges in LDS: 1 + log2 of their number (0: not so)
};
static_assert(sizeof(ReqDesc) % 8 == 0, "descriptor copied as 64-bit words");

struct ReqState {
  ReqDesc d;
  uint64_t state;  // phase:8 | chunks:28 | claimed:28
  uint64_t done;   // chunks of the current phase completed
  uint64_t aux;    // inserts counted for the pre-batch plan
  uint64_t seg_sp, seg_n, seg_im;
  int64_t seg_dir;
  uint64_t items;  // eviction items of the current eviction phase
  uint32_t resume; // phase that follows the current resize call
  uint32_t pad_;
};

struct DrainQueue {
  ReqState *req;              // device ring
  const ReqDesc *host_ring;   // pinned host ring
  const uint64_t *host_tail;  // pinned: descriptors written by the host
  const uint32_t *host_stop;  // pinned: set when no more work will come
  uint64_t *host_done;        // pinned: per ring slot, ticket + 1 once complete
  uint64_t *host_live;        // pinned: per ring slot, the table's live count after the batch
  uint64_t *table_next;       // per table slot: sequence number allowed to run
  uint64_t cap;
  uint64_t idle_ticks;        // device wall-clock ticks without queue progress before a block gives up
  uint64_t ingested;
  uint64_t head;
  uint64_t completed;
  uint32_t ingest_lock;
  uint32_t error;             // 1: a block hit the idle watchdog
  uint32_t final_seen;        // the host stopped and every submitted batch was ingested
  uint32_t pad_;
};

constexpr uint64_t M28 = (1ull << 28) - 1;

__device__ __forceinline__ uint64_t make_state(uint32_t ph, uint64_t nch) {
  return ((uint64_t)ph << 56) | ((nch & M28) << 28);
}

__device__ __forceinline__ uint64_t ld_sys(const uint64_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ ResizeArgs resize_args(const ReqDesc &d) {
  return ResizeArgs{d.t.buckets, d.t.hint, d.t.ctl, d.t.S, d.t.K, d.t.lf_expand_pct, d.t.lf_contract_pct};
}

__device__ __forceinline__ EvictArgs evict_args(const ReqDesc &d) {
  return EvictArgs{d.t.buckets, d.t.spill,      d.t.hint,        d.t.stash,        d.t.pending, d.t.ctl,
                   d.t.wl,      d.t.wl_seg_cap, d.t.stash_cap,   d.t.pending_cap,  d.t.max_evictions, 0};
}

__device__ __forceinline__ bool has_inserts(const ReqDesc &d) { return d.mode == OP_INSERT || d.mode == OP_MIXED; }

__device__ __forceinline__ uint64_t ceil_div(uint64_t a, uint64_t b) { return (a + b - 1) / b; }

// After a resize step: the next segment, the stash drain after splits, or
// the phase the resize call returns to.
__device__ __forceinline__ uint32_t seg_entry(volatile ReqState *r, const ReqDesc &d) {
  volatile Ctl *c = d.t.ctl;
  if (c->seg > 0) {
    r->seg_sp = c->sp;
    r->seg_n = c->seg;
    r->seg_im = c->im;
    r->seg_dir = c->resize_dir;
    return PH_SEG_A;
  }
  if (c->split_happened) return PH_DRAIN;
  return r->resume;
}

// Successor of a finished phase; scalar work between phases happens here.
__device__ __forceinline__ uint32_t successor(volatile ReqState *r, const ReqDesc &d, uint32_t ph) {
  volatile Ctl *c = d.t.ctl;
  const bool linear = d.t.addressing == ADDR_LINEAR;
  switch (ph) {
    case PH_START: return d.n ? PH_FILL : PH_DONE;  // an empty batch changes nothing, as in the plain path
    case PH_FILL: return PH_DEDUPE;
    case PH_DEDUPE: return PH_COUNT;
    case PH_COUNT:
      if (linear && d.t.pre_expand && has_inserts(d)) {
        plan_start(c, resize_args(d), PLAN_PRE, d.mode == OP_MIXED ? r->aux : d.n);
        r->resume = PH_OPS;
        return seg_entry(r, d);
      }
      return PH_OPS;
    case PH_SEG_A: return r->seg_dir < 0 ? PH_SEG_B : seg_entry(r, d);
    case PH_SEG_B: return seg_entry(r, d);
    case PH_DRAIN: return PH_REPLACE;
    case PH_REPLACE: return r->resume;
    case PH_OPS: return PH_EVICT;
    case PH_EVICT:
      if (linear && d.t.post_policy && d.mode != OP_LOOKUP) {
        plan_start(c, resize_args(d), PLAN_POST, 0);
        r->resume = PH_DONE;
        return seg_entry(r, d);
      }
      return PH_DONE;
    default: return PH_DONE;
  }
}

// Chunks of a phase about to start (0: nothing to do).
__device__ __forceinline__ uint64_t enter(volatile ReqState *r, const ReqDesc &d, uint32_t ph) {
  volatile Ctl *c = d.t.ctl;
  const uint64_t gpb = (uint64_t)WAVES * (64 / d.t.S);  // groups per block
  switch (ph) {
    case PH_FILL: return d.dd_size ? ceil_div(d.dd_size, FILL_PER_CHUNK) : 0;
    case PH_DEDUPE: return d.dds ? 1ull << (d.dds - 1) : d.dd_size ? ceil_div(d.n, BLOCK) : 0;
    case PH_COUNT:
      if (d.dds) return 0;  // counted with the dedupe
      r->aux = 0;
      return (d.t.addressing == ADDR_LINEAR && d.t.pre_expand && d.mode == OP_MIXED) ? ceil_div(d.n, COUNT_PER_CHUNK)
                                                                                     : 0;
    case PH_SEG_A: return ceil_div(r->seg_n, gpb);
    case PH_SEG_B: return ceil_div(c->merge_commit, gpb);
    case PH_DRAIN: {
      const uint64_t total = (min(c->stash_count, d.t.stash_cap) ? stash_slots_for(d.t.stash_cap) : 0) +
                             min(c->pending_count, d.t.pending_cap);
      return total ? max(ceil_div(total, BLOCK * DRAIN_TILES), ceil_div(d.t.hint_words, FILL_PER_CHUNK)) : 0;
    }
    case PH_REPLACE:
    case PH_EVICT:  // r->items: the worklist size, summed when the phase before it finished
      return ceil_div(r->items, (uint64_t)WAVES * evict_groups_per_wave(d.t.S));
    case PH_OPS: return ceil_div(d.n, BLOCK);
    default: return 0;
  }
}

// Scalar work at the end of a phase (also for phases with no chunks).
__device__ __forceinline__ void epilogue(volatile ReqState *r, const ReqDesc &d, uint32_t ph) {
  volatile Ctl *c = d.t.ctl;
  switch (ph) {
    case PH_SEG_A:
      if (r->seg_dir > 0) split_segment_done(c, r->seg_sp, r->seg_n);
      break;
    case PH_SEG_B: merge_segment_done(c, r->seg_sp, r->seg_n, c->merge_commit); break;
    case PH_DRAIN: drain_done(c); break;
    default: break;
  }
}

// Shard work at the end of a phase with chunks (wave 0 of the block that
// completed it): after the probe phase the key-count changes are folded and
// the worklist is sized; after a stash drain the worklist is sized; after an
// eviction phase its statistics are folded and the worklist emptied.
// own: this block ran every chunk of the phase, so no other block's writes
// need acquiring.
__device__ __forceinline__ void phase_fold(ReqState *rs, const ReqDesc &d, uint32_t ph, bool own) {
  if (!own) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  volatile ReqState *r = rs;
  Ctl *c = d.t.ctl;
  uint64_t items = 0;
  switch (ph) {
    case PH_OPS: items = fold_shards_wave(c, false); break;
    case PH_DRAIN: items = wave_sum64(ld_ctl(&shard_of(c, threadIdx.x & 63)->wl_count)); break;
    case PH_REPLACE:
    case PH_EVICT: (void)fold_shards_wave(c, true); break;
    default: return;
  }
  if ((threadIdx.x & 63) == 0) r->items = items;  // read by the same thread in advance
}

// Finish phase `ph` of r and publish the next one (one thread).  Returns the
// state word published for that phase, or 0 when the batch is done.
// own: this block ran every chunk of `ph`.  Then a next phase of at most
// SOLO_CHUNKS chunks is published already fully claimed, by this block: a
// small batch runs phase after phase in one block, without a window scan
// and without the acquires (L2 invalidations) of a handoff, since no other
// block writes its data meanwhile.  Each such phase starts with an L1
// invalidation instead (invalidate_l1: the block's own atomics of the last
// phase are not in its L1).  The release before publishing (an L2 write-back)
// stays after the phases whose plain stores later ones read with coherent
// loads (splits, merges, the stash drain); winner flags and worklist entries
// are read with plain loads, through the L2 that holds them, and buckets
// change by atomics.  The full release stays when the batch is done.
// (Chunks run one after another in a block, 6 to 8 us each with a probe's
// latency: at 8 chunks a mixed batch of 2,048 operations took 122 us, at 2
// chunks, handed to other blocks beyond, 58.)
constexpr uint64_t SOLO_CHUNKS = 2;
__device__ uint64_t advance(DrainQueue *q, ReqState *rs, const ReqDesc &d, uint32_t ph, bool own) {
  if (!own) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  volatile ReqState *r = rs;
  uint64_t nch = 0;
  // a phase whose plain stores other phases read coherently
  const bool stored = ph == PH_SEG_A || ph == PH_SEG_B || ph == PH_DRAIN;
  epilogue(r, d, ph);
  for (;;) {
    ph = successor(r, d, ph);
    if (ph == PH_DONE) break;
    nch = enter(r, d, ph);
    if (nch > 0) break;
    epilogue(r, d, ph);
  }
  r->done = 0;
  if (ph == PH_DONE) {
    if (has_inserts(d)) {
      volatile Ctl *c = d.t.ctl;
      c->inserted += d.n;
    }
    const uint64_t ticket = d.ticket;
    __hip_atomic_store(&q->host_live[ticket % q->cap], ld_ctl(&d.t.ctl->live), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
    // one fence orders the batch's outputs and updates before all of these
    // stores (a release of its own on each would write the L2 back again);
    // the ring slot is done with before the host may reuse it
    __threadfence_system();
    __hip_atomic_store(&rs->state, make_state(PH_DONE, 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&q->table_next[d.table_slot], d.seq + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __hip_atomic_store(&q->host_done[ticket % q->cap], ticket + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    add64(&q->completed, 1);
    return 0;
  }
  const bool solo = own && nch <= SOLO_CHUNKS;
  const uint64_t published = make_state(ph, nch) + (solo ? nch : 0);
  if (solo && !stored) {
    __hip_atomic_store(&rs->state, published, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else {
    __threadfence();
    __hip_atomic_store(&rs->state, published, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  }
  return published;
}

// The block that published a batch's next phase claims its first grain at
// once, without a window scan (the batch is running, so its table order is
// already satisfied).  The claim is a CAS from exactly the published state:
// if other blocks have claimed chunks meanwhile it fails and the block scans
// as usual, and a ring slot reused by a later batch cannot match, since a
// published phase is never PH_START.
__device__ bool claim_published(ReqState *r, uint64_t published, uint32_t *phase, uint64_t *chunk, uint64_t *count,
                                uint64_t *nch) {
  const uint64_t n = (published >> 28) & M28;
  const uint64_t grain = max(1ull, n / (2ull * gridDim.x));
  uint64_t expect = published;
  if (!__hip_atomic_compare_exchange_strong(&r->state, &expect, published + min(grain, n), __ATOMIC_ACQUIRE,
                                            __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    return false;
  *phase = (uint32_t)(published >> 56);
  *chunk = 0;
  *count = min(grain, n);
  *nch = n;
  return true;
}

// A value the whole wave holds, in a scalar register (the first active
// lane's copy).
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  return ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(v >> 32)) << 32) |
         __builtin_amdgcn_readfirstlane((uint32_t)v);
}

// Copy new host descriptors into the device ring, by the 64 lanes of one
// wave.  Only the block holding the ingest lock reads host memory (the tail,
// the stop flag, descriptors); every other block polls device memory.  The
// descriptors' words are copied lane-parallel (up to 64 descriptors per
// call): host reads cross the bus, and a one-thread copy of 16 descriptors
// word by word had been hundreds of dependent reads, long enough to be the
// executor's intake limit.  Lane j then publishes descriptor j.  The stop
// flag is read before the tail, so once it is seen set, the tail read after
// it is final.
__device__ void ingest(DrainQueue *q) {
  const int lane = threadIdx.x & 63;
  uint32_t got = 0;
  if (lane == 0 && __hip_atomic_load(&q->ingest_lock, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0 &&
      __hip_atomic_load(&q->final_seen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) {
    uint32_t expect = 0;
    got = __hip_atomic_compare_exchange_strong(&q->ingest_lock, &expect, 1u, __ATOMIC_ACQUIRE, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
  }
  if (!__builtin_amdgcn_readfirstlane(got)) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  const bool stop = __hip_atomic_load(q->host_stop, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_SYSTEM) != 0;
  const uint64_t tail = uniform64(ld_sys(q->host_tail));
  const uint64_t i0 = uniform64(ld_ctl(&q->ingested));
  const uint64_t n = min(tail - i0, (uint64_t)64);
  if (n == 0 && !stop) {  // nothing new: no fences
    if (lane == 0) __hip_atomic_store(&q->ingest_lock, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  constexpr uint64_t W = sizeof(ReqDesc) / 8;
  for (uint64_t k = lane; k < n * W; k += 64) {
    const uint64_t i = (i0 + k / W) % q->cap, w = k % W;
    ((uint64_t *)&q->req[i].d)[w] = ld_sys((const uint64_t *)(q->host_ring + i) + w);
  }
  ReqState *r = q->req + (i0 + lane) % q->cap;
  if ((uint64_t)lane < n) {
    volatile ReqState *vr = r;
    vr->done = 0;
    vr->aux = 0;
    vr->items = 0;
    vr->resume = PH_DONE;
  }
  __threadfence();  // every lane's descriptor words and fields before any state
  // one START chunk: the batch's first real phase is chosen when it runs,
  // i.e. after every earlier batch on its table has finished
  if ((uint64_t)lane < n)
    __hip_atomic_store(&r->state, make_state(PH_START, 1), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  __threadfence();  // the states before the new ingest count
  if (lane == 0) {
    __hip_atomic_store(&q->ingested, i0 + n, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    if (stop && i0 + n == tail) __hip_atomic_store(&q->final_seen, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&q->ingest_lock, 0u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Claim a run of chunks of runnable work, by the 64 lanes of one wave: lane
// j looks at ring entry head + j of the window (its state, then whether its
// table's previous batch is done), so a scan costs a few parallel round
// trips instead of a chain of them per entry; the oldest runnable entry is
// claimed first.  `*chunk` is the first chunk, `*count` how many (a phase of
// n chunks is claimed in grains of about n / (2 x grid) chunks, so a large
// phase costs few claims: the atomic on the request's state word is the
// same address for every block); the claiming lane writes the outputs.
// Returns, in every lane, 0 (work), 1 (none now) or 2 (exit).
static_assert(DRAIN_WINDOW == 64, "one window entry per lane");
__device__ uint32_t find_work(DrainQueue *q, uint64_t *req, uint32_t *phase, uint64_t *chunk, uint64_t *count,
                              uint64_t *nch) {
  const int lane = threadIdx.x & 63;
  ingest(q);
  uint64_t ing = ld_ctl(&q->ingested), head = ld_ctl(&q->head);  // in flight together
  ing = uniform64(ing);
  head = uniform64(head);
  // the window's states; the completed batches at the head of the ring are
  // retired (then the window has moved, and its states are read again)
  uint64_t t = head + lane, st = 0;
  for (;;) {
    // relaxed: a retired entry is only skipped; an acquire load here would
    // invalidate the XCD's L2 on every poll of every idle block
    st = t < ing ? __hip_atomic_load(&q->req[t % q->cap].state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    const uint64_t dm = ballot(t < ing && (st >> 56) == PH_DONE);
    const int lead = (dm == ~0ull) ? 64 : __builtin_ctzll(~dm);
    if (lead == 0) break;
    uint64_t h = head;
    if (lane == 0)
      __hip_atomic_compare_exchange_strong(&q->head, &h, head + lead, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
    // h: the head found; entries up to head + lead are done in any case
    head = max(uniform64(h), head + lead);
    t = head + lane;
    if (head >= ing) break;
  }
  if (head >= ing) {
    if (__hip_atomic_load(&q->final_seen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 &&
        ld_ctl(&q->ingested) == ing)
      return 2;
    return 1;
  }
  ReqState *r = q->req + t % q->cap;
  bool runnable = t < ing && (uint32_t)(st >> 56) != PH_DONE && (st & M28) < ((st >> 28) & M28);
  // the descriptor read below must see what was written before the state
  // was released; the acquire fence (an L2 invalidate) is paid only by a
  // scan that found unclaimed chunks, never by an idle poll
  if (ballot(runnable)) {
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (runnable) {
      const uint64_t slot = ld_ctl(&r->d.table_slot), seq = ld_ctl(&r->d.seq);
      runnable = ld_ctl(&q->table_next[slot]) == seq;
    }
  }
  for (uint64_t m = ballot(runnable); m; m &= m - 1) {
    const int j = __builtin_ctzll(m);
    bool won = false;
    if (lane == j) {
      const uint64_t grain = max(1ull, ((st >> 28) & M28) / (2ull * gridDim.x));
      const uint64_t old = add64(&r->state, grain);
      const uint64_t n = (old >> 28) & M28, c = old & M28;
      if ((uint32_t)(old >> 56) != PH_DONE && c < n) {
        won = true;
        *req = t;
        *phase = (uint32_t)(old >> 56);
        *chunk = c;
        *count = min(grain, n - c);
        *nch = n;
      }
    }
    if (ballot(won)) return 0;
  }
  return 1;
}

// Descriptor of the batch a block works on, read coherently into LDS.
__device__ __forceinline__ void load_desc(ReqDesc *dst, const ReqDesc *src) {
  const uint64_t *s = (const uint64_t *)src;
  uint64_t *d = (uint64_t *)dst;
  for (uint32_t w = threadIdx.x; w < sizeof(ReqDesc) / 8; w += BLOCK) d[w] = ld_ctl(s + w);
}

// A pointer the compiler knows to be global memory.  Pointers read from
// memory are generic (flat) to it; rebuilt from their address as global
// ones, their loads and stores become global instructions, which do not
// share the LDS wait counter with the tile staging.
template <typename T>
__device__ __forceinline__ T *as_global(T *p) {
  return (T *)(__attribute__((address_space(1))) T *)(uintptr_t)p;
}

// The LDS descriptor copied into scalar registers (every word goes through
// readfirstlane, so the compiler knows it is uniform), its buffers marked
// global.  Every buffer a descriptor names is device or mapped host memory.
__device__ __forceinline__ ReqDesc uniform_desc(const ReqDesc &src) {
  uint32_t w[sizeof(ReqDesc) / 4];
  __builtin_memcpy(w, &src, sizeof(ReqDesc));
#pragma unroll
  for (uint32_t i = 0; i < sizeof(ReqDesc) / 4; ++i) w[i] = __builtin_amdgcn_readfirstlane(w[i]);
  ReqDesc d;
  __builtin_memcpy(&d, w, sizeof(ReqDesc));
  d.t.buckets = as_global(d.t.buckets);
  d.t.hint = as_global(d.t.hint);
  d.t.spill.bits = as_global(d.t.spill.bits);
  d.t.stash = as_global(d.t.stash);
  d.t.pending = as_global(d.t.pending);
  d.t.ctl = as_global(d.t.ctl);
  d.t.wl = as_global(d.t.wl);
  d.t.dd = as_global(d.t.dd);
  d.ops = as_global(d.ops);
  d.keys = as_global(d.keys);
  d.vals = as_global(d.vals);
  d.vals_out = as_global(d.vals_out);
  d.flags_out = as_global(d.flags_out);
  return d;
}


template <int S>
union DrainShared {
  OpsShared<S> ops;
  DdsShared<DDS_EXEC_TAB, DDS_EXEC_LIST> dds;
};

template <int S>
__device__ __forceinline__ void run_chunk(ReqState *r, const ReqDesc &d, uint32_t ph, uint64_t c,
                                          DrainShared<S> &sh) {
  using T = Traits<S>;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int g = lane / S, sl = lane % S;
  const uint64_t gib = (uint64_t)wv * T::G + g;  // group in block
  const uint64_t gpb = (uint64_t)WAVES * T::G;
  switch (ph) {
    case PH_FILL: {
      const uint64_t b = c * FILL_PER_CHUNK, e = min(b + FILL_PER_CHUNK, d.dd_size);
      for (uint64_t t = b + threadIdx.x; t < e; t += BLOCK) d.t.dd[t] = EMPTY;
      break;
    }
    case PH_DEDUPE:
    case PH_COUNT: {
      // the inserts of a mixed batch, for its growth rule: with the first
      // range of a dedupe in LDS, else in chunks of their own
      const bool ranges = ph == PH_DEDUPE && d.dds;
      const bool counts = d.mode == OP_MIXED && d.t.addressing == ADDR_LINEAR && d.t.pre_expand;
      if (ph == PH_COUNT || (ranges && c == 0 && counts)) {
        __shared__ unsigned long long cnt;
        if (threadIdx.x == 0) cnt = 0;
        __syncthreads();
        unsigned long long mine = 0;
        const uint64_t b = ranges ? 0 : c * COUNT_PER_CHUNK, e = ranges ? d.n : min(b + COUNT_PER_CHUNK, d.n);
        for (uint64_t t = b + threadIdx.x; t < e; t += BLOCK) mine += d.ops[t] == OP_INSERT;
        mine = wave_sum64(mine);
        if (lane == 0 && mine) atomicAdd(&cnt, mine);
        __syncthreads();
        if (threadIdx.x == 0 && cnt) add64(&r->aux, cnt);
      }
      if (ranges) {
        const DdsArgs a{d.ops, d.keys, (uint8_t *)d.t.dd, (uint32_t)d.n, d.mode, (uint32_t)(d.dds - 1)};
        dds_range_of<BLOCK, DDS_LOADS>(a, (uint32_t)c, sh.dds);
      } else if (ph == PH_DEDUPE) {
        dedupe_thread(d.t.dd, d.dd_size - 1, d.mode, d.ops, d.keys, d.n, c * BLOCK + threadIdx.x);
      }
      break;
    }
    case PH_SEG_A: {
      const ResizeArgs ra = resize_args(d);
      const uint64_t j = c * gpb + gib, n = ld_ctl(&r->seg_n);
      const uint64_t im = ld_ctl(&r->seg_im), sp = ld_ctl(&r->seg_sp);
      if (j < n) {
        if ((int64_t)ld_ctl((const uint64_t *)&r->seg_dir) > 0)
          split_pair<S>(ra, im, sp, j, g, sl);
        else
          merge_test_pair<S>(ra, d.t.ctl, im, sp, j, g, sl);
      }
      break;
    }
    case PH_SEG_B: {
      const ResizeArgs ra = resize_args(d);
      const uint64_t j = c * gpb + gib, commit = ld_ctl(&d.t.ctl->merge_commit);
      if (j < commit) merge_move_pair<S>(ra, ld_ctl(&r->seg_im), ld_ctl(&r->seg_sp), j, g, sl);
      break;
    }
    case PH_DRAIN: {
      const Ctl *cc = d.t.ctl;
      const uint64_t n_stash = min(ld_ctl(&cc->stash_count), d.t.stash_cap) ? stash_slots_for(d.t.stash_cap) : 0;
      const uint64_t total = n_stash + min(ld_ctl(&cc->pending_count), d.t.pending_cap);
      const uint64_t hb = c * FILL_PER_CHUNK, he = min(hb + FILL_PER_CHUNK, d.t.hint_words);
      for (uint64_t t = hb + threadIdx.x; t < he; t += BLOCK) d.t.hint[t] = 0u;
      for (uint64_t k = 0; k < DRAIN_TILES; ++k)
        drain_collect((c * DRAIN_TILES + k) * BLOCK + threadIdx.x, n_stash, total, d.t.stash, d.t.pending, d.t.wl,
                      d.t.wl_seg_cap, d.t.ctl);
      break;
    }
    case PH_REPLACE:
    case PH_EVICT: {
      using E = EvictShape<S>;
      __shared__ uint64_t pre[NSHARD + 1];
      EvictArgs ea = evict_args(d);
      wl_prefix(d.t.ctl, pre);
      ea.spill = spill_placing(ea.spill, d.t.ctl, d.n, S);
      const Geo geo = read_geo(d.t.ctl);
      const uint64_t items = pre[NSHARD];
      const int eg = lane / E::L, esl = lane % E::L;
      const uint64_t egpb = (uint64_t)WAVES * E::G, egib = (uint64_t)wv * E::G + eg;
      uint64_t n_evict = 0, n_full = 0, n_side = 0, n_fresh = 0;
      const uint64_t t = c * egpb + egib;
      const bool unreserved = ld_ctl(&d.t.ctl->stash_count) + items <= d.t.stash_cap;
      evict_round<S>(ea, geo, unreserved, t < items, t < items ? wl_slot(pre, t, d.t.wl_seg_cap) : 0, eg, esl, n_evict,
                     n_full, n_side, n_fresh);
      evict_counters(ea, unreserved, c * WAVES + wv, n_evict, n_full, n_side, n_fresh, esl);
      break;
    }
    case PH_OPS: {
      OpsArgs a{};
      a.buckets = d.t.buckets;
      a.spill = d.t.spill;
      a.hint = d.t.hint;
      a.stash = d.t.stash;
      a.pending = d.t.pending;
      a.ctl = d.t.ctl;
      a.wl = d.t.wl;
      a.wl_seg_cap = d.t.wl_seg_cap;
      a.dd = d.dd_size ? d.t.dd : nullptr;
      a.dd_mask = d.dd_size ? d.dd_size - 1 : 0;
      a.win = d.dds ? (const uint8_t *)d.t.dd : nullptr;
      a.ops = d.ops;
      a.keys = d.keys;
      a.vals = d.vals;
      a.vals_out = d.vals_out;
      a.flags_out = d.flags_out;
      a.n = d.n;
      a.stash_cap = d.t.stash_cap;
      a.pending_cap = d.t.pending_cap;
      const OpsView view = read_view(d.t.ctl, d.t.stash_cap, d.t.pending_cap, d.t.spill, d.n);
      // one probe variant only (the second candidate after a miss): a
      // second inlined copy would cost the resident grid occupancy
      int64_t live_acc = 0;
      uint64_t bad_acc = 0;
      switch (d.mode) {
        case OP_INSERT: ops_tile<S, OP_INSERT, false, PAIR_BITHASH, Traits<S>::CH, FILTER_ASK>(a, view, c, sh.ops, live_acc, bad_acc); break;
        case OP_DELETE: ops_tile<S, OP_DELETE, false, PAIR_BITHASH, Traits<S>::CH, FILTER_ASK>(a, view, c, sh.ops, live_acc, bad_acc); break;
        case OP_LOOKUP: ops_tile<S, OP_LOOKUP, false, PAIR_BITHASH, Traits<S>::CH, FILTER_ASK>(a, view, c, sh.ops, live_acc, bad_acc); break;
        default: ops_tile<S, OP_MIXED, false, PAIR_BITHASH, Traits<S>::CH, FILTER_ASK>(a, view, c, sh.ops, live_acc, bad_acc); break;
      }
      ops_counts_add(d.t.ctl, c * WAVES + (threadIdx.x >> 6), live_acc, bad_acc);
      if (c == 0 && threadIdx.x == 0) {
        const bool filter = d.t.spill.bits != nullptr;
        if (d.mode == OP_INSERT) ops_done<OP_INSERT>(d.t.ctl, view, filter);
        else if (d.mode == OP_DELETE) ops_done<OP_DELETE>(d.t.ctl, view, filter);
        else if (d.mode == OP_MIXED) ops_done<OP_MIXED>(d.t.ctl, view, filter);
      }
      break;
    }
    default: break;  // PH_START: no data-parallel work
  }
}

__global__ void drain_reset_kernel(DrainQueue *q) { q->final_seen = 0; }

// One reading of the constant-rate device clock (clock-rate calibration).
__global__ void wall_clock_kernel(uint64_t *out) { *out = wall_clock64(); }

// Invalidate this compute unit's vector L1 cache (the L2 is untouched).
// An agent-scope acquire fence does this and also invalidates the XCD's L2
// lines of non-coherent memory types; a block that runs consecutive phases of
// one batch alone needs only the former: its own device-scope atomics
// (claims, evictions, stash placements) were performed in its XCD's L2, but
// lines its earlier plain loads brought into the L1 still hold the words
// those atomics replaced, and the next phase's plain loads (split, merge,
// stash drain, probe) would read them.
__device__ __forceinline__ void invalidate_l1() { asm volatile("buffer_inv sc0" ::: "memory"); }

// Occupancy target: 3 waves per SIMD (at most 168 VGPRs).  The 16-slot build
// spills 39 registers, mostly of the control loop; a cap of
// 128 (4 waves) spills inside the phases and runs slower.
template <int S>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(3))) void drain_worker_kernel(DrainQueue *q) {
  __shared__ DrainShared<S> sh;
  __shared__ ReqDesc desc;
  __shared__ uint64_t s_req, s_chunk, s_cnt, s_nch;
  __shared__ uint32_t s_phase, s_cmd;
  __shared__ bool s_last, s_cont, s_solo;
  // watchdog (thread 0 decides for the block): time without any progress
  // of the queue as a whole (nothing newly ingested, nothing retired), so
  // blocks that merely find no chunk while others work do not give up
  uint64_t seen_ing = ~0ull, seen_head = ~0ull;
  uint64_t idle_since = wall_clock64();
  const uint64_t idle_ticks = ld_ctl(&q->idle_ticks);
  if (threadIdx.x == 0) {
    s_cont = false;
    s_solo = false;
  }
  __syncthreads();
  for (;;) {
    // s_cont: this block claimed the next phase of its batch when it
    // published it, so it needs no scan
    if (threadIdx.x < 64 && !s_cont) {
      uint32_t cmd = find_work(q, &s_req, &s_phase, &s_chunk, &s_cnt, &s_nch);
      if (threadIdx.x == 0 && cmd == 1) {
        const uint64_t ing = ld_ctl(&q->ingested), head = ld_ctl(&q->head);
        const uint64_t now = wall_clock64();
        if (ing != seen_ing || head != seen_head) {
          seen_ing = ing;
          seen_head = head;
          idle_since = now;
        }
        if (now - idle_since > idle_ticks) {
          atomicOr(&q->error, 1u);
          cmd = 2;
        }
      }
      if (threadIdx.x == 0) s_cmd = cmd;
    }
    __syncthreads();
    const uint32_t cmd = s_cont ? 0u : s_cmd;
    if (cmd == 2) break;
    if (cmd == 1) {
      // about 7 us: every poll of an idle block reads the queue's words and
      // the states of the window, the same lines that the working blocks
      // update, and with a block per compute unit some block polls every few
      // tens of ns anyway (450 clocks: a lookup of one key 25.6 us through
      // the executor, a mixed batch of 4,096 operations 63; now 21.5 and 53)
      __builtin_amdgcn_s_sleep(127);
      __builtin_amdgcn_s_sleep(127);
      __syncthreads();
      continue;
    }
    ReqState *r = q->req + s_req % q->cap;
    // s_solo: this block also ran the batch's previous phases alone since it
    // last acquired, and its descriptor is still in LDS
    if (!s_solo) {
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      load_desc(&desc, &r->d);
      __syncthreads();
    } else {
      invalidate_l1();
    }
    const ReqDesc d = uniform_desc(desc);
    const uint32_t phase = __builtin_amdgcn_readfirstlane(s_phase);
    const uint64_t chunk = uniform64(s_chunk), cnt = uniform64(s_cnt);
    for (uint64_t k = 0; k < cnt; ++k) {
      run_chunk<S>(r, d, phase, chunk + k, sh);
      __syncthreads();
    }
    // this wave's stores and atomics are done before the block goes on
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const bool own = cnt == uniform64(s_nch);  // every chunk of the phase ran here
    if (threadIdx.x == 0) {
      if (s_solo || phase == PH_START) {
        s_last = true;  // claimed whole by this block; a start phase stores nothing
      } else {
        __threadfence();  // these chunks' writes before their completion count
        s_last = add64(&r->done, s_cnt) + s_cnt == s_nch;
      }
      s_cont = false;
      s_solo = false;
    }
    __syncthreads();
    if (s_last) {
      // the block that completed the phase: shard folds by wave 0, then the
      // scalar epilogue and the next phase by thread 0, which claims the
      // start of that phase for this block
      if (threadIdx.x < 64) phase_fold(r, desc, phase, own);
      __syncthreads();
      if (threadIdx.x == 0) {
        const uint64_t published = advance(q, r, desc, phase, own);
        const uint64_t n = (published >> 28) & M28;
        if (published != 0 && (published & M28) == n) {  // published claimed by this block
          s_phase = (uint32_t)(published >> 56);
          s_chunk = 0;
          s_cnt = n;
          s_nch = n;
          s_cont = true;
          s_solo = true;
        } else {
          s_cont = published != 0 && claim_published(r, published, &s_phase, &s_chunk, &s_cnt, &s_nch);
        }
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// 32-bit entries: a key-only set (Section III-A: with 32-bit entries a
// 32-slot bucket is one 128-byte line).  The entry is the key itself; EMPTY
// is 0xFFFFFFFF and a deleted stash or pending entry is 0 (both reserved
// keys).  The steps are those of the 64-bit table: P1 hashes, probes the
// first candidate (a 32-lane group per bucket, one 4-byte load per lane, two
// buckets per wave-wide load), the second after a miss, then looks up,
// deletes (one agent-scope atomic store of EMPTY) or inserts: a key already
// present is left as it is (there is no value to replace), a new one claims
// an EMPTY slot of its first candidate while that has room to spare, else of
// the emptier one, by a 32-bit CAS; P3 runs
// the bounded cuckoo chains one lane per item on fresh copies of whole
// buckets, then the stash or the pending list.  FIXED addressing, BitHash1/2,
// plain launches.
// ---------------------------------------------------------------------------
constexpr uint32_t EMPTY32 = 0xFFFFFFFFu;
constexpr uint32_t TOMB32 = 0u;
constexpr int SET_S = 32;        // slots per bucket
constexpr int SET_CH = 16;       // wave-wide bucket loads in flight

struct SetArgs {
  uint32_t *buckets;
  Spill spill;
  uint32_t *hint;
  uint32_t *stash;
  uint32_t *pending;
  Ctl *ctl;
  uint64_t *wl;  // eviction worklist (keys widened to 64 bits), NSHARD segments
  uint64_t wl_seg_cap;
  const uint8_t *ops;
  const uint32_t *keys;
  uint8_t *flags_out;
  uint64_t n;
  uint64_t stash_cap, pending_cap;
  uint32_t max_evictions;
  const uint8_t *win;  // dedupe winner flag per operation, or null
};

__device__ __forceinline__ uint32_t cas32(uint32_t *p, uint32_t expected, uint32_t desired) {
  __hip_atomic_compare_exchange_strong(p, &expected, desired, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
  return expected;
}

// Search of the stash (open-addressed, linear probing from mix32(key), ends
// at EMPTY) and the pending list.
__device__ __forceinline__ uint32_t *set_overflow_find(const SetArgs &a, uint64_t n_stash, uint64_t n_pend,
                                                       uint32_t k) {
  if (n_stash) {
    const uint64_t mask = stash_slots_for(a.stash_cap) - 1;
    for (uint64_t i = 0, p = mix32(k) & mask; i <= mask; ++i, p = (p + 1) & mask) {
      const uint32_t x = a.stash[p];
      if (x == EMPTY32) break;
      if (x == k) return a.stash + p;
    }
  }
  for (uint64_t p = 0; p < n_pend; ++p)
    if (a.pending[p] == k) return a.pending + p;
  return nullptr;
}

// One probe round: operations t < count have key keys[t] and bucket
// bkts[t] (owner list[t], or t itself); each 32-lane group loads one bucket
// per wave-wide load and publishes the match and EMPTY masks to the owner.
// bkts[] holds 64 entries, padded from `count` on with a bucket loaded
// anyway.
__device__ __forceinline__ void set_probe_round(const uint32_t *__restrict__ buckets, const uint32_t *keys,
                                                const uint32_t *bkts, const uint8_t *list, int count,
                                                uint32_t *m_out, uint32_t *e_out, int g, int sl) {
  for (int base = 0; base < count; base += 2 * SET_CH) {
    uint32_t w[SET_CH];
#pragma unroll
    for (int j = 0; j < SET_CH; ++j) w[j] = buckets[(uint64_t)bkts[base + 2 * j + g] * SET_S + sl];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < SET_CH; ++j) {
      const int t = base + 2 * j + g;
      const bool mine = t < count;
      const uint32_t ko = keys[t];
      const uint64_t mm = ballot(mine && ko != 0u && w[j] == ko);
      const uint64_t ee = ballot(w[j] == EMPTY32);
      if (mine && sl == 0) {
        const int o = list ? list[t] : t;
        m_out[o] = (uint32_t)(mm >> (g * 32));
        e_out[o] = (uint32_t)(ee >> (g * 32));
      }
    }
  }
}

template <uint32_t MODE>
__global__ __launch_bounds__(BLOCK) void set_ops_kernel(SetArgs a) {
  __shared__ uint32_t s_key[WAVES][64], s_b1[WAVES][64], s_k2[WAVES][64], s_b2[WAVES][64];
  __shared__ uint8_t s_list[WAVES][64];
  __shared__ uint32_t s_m[2][WAVES][64], s_e[2][WAVES][64];
  const Geo geo = read_geo(a.ctl);
  const uint64_t n_stash = min(ld_ctl(&a.ctl->stash_count), a.stash_cap);
  const uint64_t n_pend = min(ld_ctl(&a.ctl->pending_count), a.pending_cap);
  const bool overflow_used = (n_stash | n_pend) != 0;
  OpsView view;
  view.removed = ld_ctl32(&a.ctl->removed) != 0;
  view.spill = spill_state(a.spill, a.ctl, a.n);
  const bool removed = view.removed, filter = a.spill.bits != nullptr;
  if (MODE == OP_LOOKUP || MODE == OP_DELETE ? view.spill.dropped : view.spill.plain) a.spill = spill_none(SET_S);
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int g = lane >> 5, sl = lane & 31;
  const uint64_t ntiles = (a.n + BLOCK - 1) / BLOCK;
  for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const uint64_t i = tile * BLOCK + threadIdx.x;
    const bool active = i < a.n;
    uint32_t op = OP_NONE, k = 0;
    if (active) {
      op = (MODE == OP_MIXED) ? (uint32_t)__builtin_nontemporal_load(&a.ops[i]) : MODE;
      k = __builtin_nontemporal_load(&a.keys[i]);
    }
    const bool valid = active && op <= OP_LOOKUP && valid_key(k);
    bool work = valid;
    if (work && op != OP_LOOKUP) {
      if (a.win) work = __builtin_nontemporal_load(&a.win[i]) != 0;
    }
    uint32_t c1 = 0, c2 = 0;
    if (work) {
      c1 = fastmod(bithash1(k), geo.magic, (uint32_t)geo.n_buckets);
      c2 = fastmod(bithash2(k), geo.magic, (uint32_t)geo.n_buckets);
    }
    s_key[wv][lane] = work ? k : 0u;
    s_b1[wv][lane] = c1;
    wave_lds_sync();
    set_probe_round(a.buckets, s_key[wv], s_b1[wv], nullptr, 64, s_m[0][wv], s_e[0][wv], g, sl);
    wave_lds_sync();
    const uint32_t m1 = s_m[0][wv][lane], e1 = s_e[0][wv][lane];
    // filter and placement as for 64-bit entries (ops_tile)
    const bool near_full = (uint32_t)__builtin_popcount(e1) < a.spill.first_min;
    const bool both = op == OP_INSERT && near_full;
    bool spilled = true, marked = false;
    if (a.spill.bits) {
      marked = work && m1 == 0 &&
               (both ? overflow_used : near_full || MODE == OP_MIXED || MODE == OP_DELETE || removed) &&
               spill_test(a.spill, c1, k);
      spilled = marked;
    }
    const bool need2 = work && m1 == 0 && c2 != c1 && (spilled || both);
    const uint64_t need2_mask = ballot(need2);
    const int n2 = __popcll(need2_mask);
    compact_second(need2, need2_mask, n2, k, c2, c1, lane, s_k2[wv], s_b2[wv], s_list[wv]);
    wave_lds_sync();
    if (n2 > 0) set_probe_round(a.buckets, s_k2[wv], s_b2[wv], s_list[wv], n2, s_m[1][wv], s_e[1][wv], g, sl);
    wave_lds_sync();
    const uint32_t m2 = need2 ? s_m[1][wv][lane] : 0u, e2 = need2 ? s_e[1][wv][lane] : 0u;

    uint8_t out_f = 0;
    int dl = 0;
    bool to_wl = false;
    if (work) {
      uint32_t *slot = nullptr;
      bool in_bucket = false;
      if (m1) {
        slot = a.buckets + (uint64_t)c1 * SET_S + __builtin_ctz(m1);
        in_bucket = true;
      } else if (m2) {
        slot = a.buckets + (uint64_t)c2 * SET_S + __builtin_ctz(m2);
        in_bucket = true;
      } else if (overflow_used && spilled && hinted(a.hint, c1, c2)) {
        slot = set_overflow_find(a, n_stash, n_pend, k);
      }
      if (op == OP_LOOKUP) {
        out_f = slot != nullptr;
      } else if (op == OP_DELETE) {
        if (slot && in_bucket) {
          // an atomic store: claims of other XCDs change this line in the
          // same launch (see the 64-bit table's delete)
          __hip_atomic_store(slot, EMPTY32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          out_f = 1;
          dl = -1;
        } else if (slot && cas32(slot, k, TOMB32) == k) {
          out_f = 1;
          dl = -1;
        }
      } else if (!slot) {
        // a new key: claim-then-commit in the first candidate while it has
        // room to spare, else in the emptier one first
        dl = 1;
        uint32_t f_first = e1, f_second = (c2 != c1) ? e2 : 0u, b_first = c1, b_second = c2;
        if (__builtin_popcount(f_second) > __builtin_popcount(f_first) &&
            (uint32_t)__builtin_popcount(f_first) < a.spill.first_min) {
          const uint32_t tf = f_first;
          f_first = f_second;
          f_second = tf;
          b_first = c2;
          b_second = c1;
        }
        bool placed = false;
        while (!placed && (f_first | f_second)) {
          if (f_first == 0) {
            f_first = f_second;
            f_second = 0;
            b_first = b_second;
          }
          const int s = claim_slot<SET_S>(f_first, k);
          if (cas32(a.buckets + (uint64_t)b_first * SET_S + s, EMPTY32, k) == EMPTY32)
            placed = true;
          else
            f_first &= ~(1u << s);
        }
        to_wl = !placed;
        if (placed && b_first != c1 && !marked) spill_mark(a.spill, c1, k);
      }
    }
    const uint64_t wl_mask = ballot(to_wl);
    if (wl_mask) {
      const int leader = __builtin_ctzll(wl_mask);
      uint64_t base = 0;
      if (lane == leader) base = wl_append(a.ctl, tile, (uint64_t)__popcll(wl_mask));
      base = read_lane64(base, leader);
      if (to_wl) a.wl[(tile % NSHARD) * a.wl_seg_cap + base + rank_below(wl_mask)] = k;
    }
    const uint64_t up = ballot(dl > 0), down = ballot(dl < 0), bad = ballot(active && !valid);
    if (lane == 0) {
      Shard *sh = shard_of(a.ctl, (tile * WAVES + wv) % NSHARD);
      const int64_t d = (int64_t)__popcll(up) - (int64_t)__popcll(down);
      if (d != 0) add64(&sh->live, (uint64_t)d);
      if (bad) add64(&sh->invalid_keys, (uint64_t)__popcll(bad));
    }
    if (active && MODE != OP_INSERT && a.flags_out) __builtin_nontemporal_store(out_f, &a.flags_out[i]);
  }
  if (MODE != OP_LOOKUP && blockIdx.x == 0 && threadIdx.x == 0) ops_done<MODE>(a.ctl, view, filter);
}

// A lane's fresh copy of a whole 32-slot bucket (128 bytes).
__device__ __forceinline__ uint32_t load_set_bucket(const uint32_t *bkt, uint32_t *w) {
  uint64_t x[16];
  load_bucket16_fresh((const uint64_t *)bkt, x);
  uint32_t free_mask = 0;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    w[2 * j] = (uint32_t)x[j];
    w[2 * j + 1] = (uint32_t)(x[j] >> 32);
  }
#pragma unroll
  for (int j = 0; j < SET_S; ++j) free_mask |= (uint32_t)(w[j] == EMPTY32) << j;
  return free_mask;
}

__device__ __forceinline__ bool set_claim(uint32_t *bkt, uint32_t free_mask, uint32_t k) {
  for (; free_mask; free_mask &= free_mask - 1)
    if (cas32(bkt + __builtin_ctz(free_mask), EMPTY32, k) == EMPTY32) return true;
  return false;
}

// Step 4: the first EMPTY or TOMB word of the key's stash run (given a
// reserved position c < capacity), else the pending list.  Returns 0 stash
// (EMPTY word), 3 stash (TOMB word), 1 pending, 2 lost.
__device__ __forceinline__ int set_overflow_place(const SetArgs &a, const Geo &geo, uint32_t k, uint64_t c) {
  int where = -1;
  if (c < a.stash_cap) {
    const uint64_t mask = stash_slots_for(a.stash_cap) - 1;
    for (uint64_t i = 0, p = mix32(k) & mask; i <= mask; ++i, p = (p + 1) & mask) {
      const uint32_t cur = cas32(a.stash + p, EMPTY32, k);
      if (cur == EMPTY32) {
        where = 0;
        break;
      }
      if (cur == TOMB32 && cas32(a.stash + p, TOMB32, k) == TOMB32) {
        where = 3;
        break;
      }
    }
  }
  if (where < 0) {
    const uint64_t p = add64(&a.ctl->pending_count, 1);
    if (p < a.pending_cap) {
      __hip_atomic_store(a.pending + p, k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      where = 1;
    } else {
      atomicOr(&a.ctl->error, ERR_PENDING_LOST);
      where = 2;
    }
  }
  spill_mark(a.spill, fastmod(bithash1(k), geo.magic, (uint32_t)geo.n_buckets), k);
  set_hint(a.hint, fastmod(bithash1(k), geo.magic, (uint32_t)geo.n_buckets));
  set_hint(a.hint, fastmod(bithash2(k), geo.magic, (uint32_t)geo.n_buckets));
  return where;
}

// P3 of the set: one lane per worklist item, as the 64-bit table's 16-slot
// eviction shape (Algorithm 3 with a pseudo-random victim slot).
__global__ __launch_bounds__(BLOCK) void set_evict_kernel(SetArgs a) {
  __shared__ uint64_t pre[NSHARD + 1];
  wl_prefix(a.ctl, pre);
  const uint64_t cnt = pre[NSHARD];
  if (cnt == 0) {
    evict_finish(a.ctl, false, a.n);
    return;
  }
  a.spill = spill_placing(a.spill, a.ctl, a.n, SET_S);
  const Geo geo = read_geo(a.ctl);
  const bool unreserved = ld_ctl(&a.ctl->stash_count) + cnt <= a.stash_cap;
  const int lane = threadIdx.x & 63;
  const uint64_t stride = (uint64_t)gridDim.x * BLOCK;
  const uint32_t nb = (uint32_t)geo.n_buckets;
  uint64_t n_evict = 0, n_full = 0, n_side = 0, n_fresh = 0;
  for (uint64_t base = (uint64_t)blockIdx.x * BLOCK + (threadIdx.x & ~63u); base < cnt; base += stride) {
    const uint64_t t = base + lane;
    bool placed = true;
    uint32_t k = 0;
    if (t < cnt) {
      k = (uint32_t)a.wl[wl_slot(pre, t, a.wl_seg_cap)];
      const uint32_t c1 = fastmod(bithash1(k), geo.magic, nb), c2 = fastmod(bithash2(k), geo.magic, nb);
      uint32_t w[SET_S];
      const uint32_t f1 = load_set_bucket(a.buckets + (uint64_t)c1 * SET_S, w);
      const uint32_t f2 = c2 != c1 ? load_set_bucket(a.buckets + (uint64_t)c2 * SET_S, w) : 0u;
      const bool swap = __builtin_popcount(f2) > __builtin_popcount(f1) &&
                        (uint32_t)__builtin_popcount(f1) < a.spill.first_min;
      const uint32_t cf = swap ? c2 : c1, cs = swap ? c1 : c2;
      const bool in_first = set_claim(a.buckets + (uint64_t)cf * SET_S, swap ? f2 : f1, k);
      placed = in_first || set_claim(a.buckets + (uint64_t)cs * SET_S, swap ? f1 : f2, k);
      if (placed && (in_first ? cf : cs) != c1) spill_mark(a.spill, c1, k);
      uint32_t b = c1;
      for (uint32_t kick = 1; kick <= a.max_evictions && !placed; ++kick) {
        uint32_t *bkt = a.buckets + (uint64_t)b * SET_S;
        const uint32_t fm = load_set_bucket(bkt, w), k1 = fastmod(bithash1(k), geo.magic, nb);
        if (set_claim(bkt, fm, k)) {
          if (b != k1) spill_mark(a.spill, k1, k);
          placed = true;
          break;
        }
        const int s0 = (int)(mix32(k ^ (kick * 0x9E3779B9u)) & (SET_S - 1));
        uint32_t ws = 0;
#pragma unroll
        for (int j = 0; j < SET_S; ++j)
          if (j == s0) ws = w[j];
        if (cas32(bkt + s0, ws, k) != ws) continue;  // the slot changed: count the round, keep the key
        if (b != k1) spill_mark(a.spill, k1, k);
        if (ws == EMPTY32) {
          placed = true;
          break;
        }
        ++n_evict;
        k = ws;
        const uint32_t v1 = fastmod(bithash1(k), geo.magic, nb), v2 = fastmod(bithash2(k), geo.magic, nb);
        b = (b == v1) ? v2 : v1;
      }
    }
    const bool push = !placed;
    const uint64_t pm = ballot(push);
    if (pm) {
      const int leader = __builtin_ctzll(pm);
      uint64_t room = 0;
      if (!unreserved) {
        if (lane == leader) {
          const uint64_t nn = (uint64_t)__popcll(pm);
          room = load_fresh(&a.ctl->stash_count) < a.stash_cap ? add64(&a.ctl->stash_count, nn) : a.stash_cap;
        }
        room = read_lane64(room, leader);
      }
      if (push) {
        ++n_full;
        const int where = set_overflow_place(a, geo, k, room + rank_below(pm));
        n_side += (where == 0 || where == 3) ? 1 : where == 1 ? (1ull << 32) : 0;
        n_fresh += where == 0;
      }
    }
  }
  const uint64_t e = wave_sum64(n_evict), f = wave_sum64(n_full), sd = wave_sum64(n_side), fr = wave_sum64(n_fresh);
  if (lane == 0 && (e | f | sd)) {
    Shard *sh = shard_of(a.ctl, ((uint64_t)blockIdx.x * WAVES + (threadIdx.x >> 6)) % NSHARD);
    if (e) add64(&sh->evictions, e);
    if (f) add64(&sh->full_chains, f);
    if ((uint32_t)sd) add64(&sh->stash_inserts, (uint32_t)sd);
    if (fr && unreserved) add64(&sh->stash_unreserved, fr);
    if (sd >> 32) add64(&sh->pending_inserts, sd >> 32);
  }
  evict_finish(a.ctl, true, a.n);
}

}  // namespace hive

// ===========================================================================
// Host side: the C ABI
// ===========================================================================
using namespace hive;

struct hive_table {
  hive_config cfg;
  uint32_t S;
  uint32_t entry_bytes = 8;  // 4: a key-only set of 32-bit entries
  uint64_t initial_buckets;
  uint64_t max_buckets;
  uint64_t stash_cap, pending_cap;
  uint64_t *d_buckets = nullptr;
  uint32_t *d_hint = nullptr;
  Spill spill{nullptr, 0, 0, 0, 0};  // its bits follow the hint bits, in one allocation
  // Ctl::inserted and Ctl::dropped as of the batches submitted (replays of a
  // captured graph run on without the host: the device's own decide there)
  uint64_t inserted = 0;
  bool dropped = false;
  uint64_t *d_stash = nullptr;
  uint64_t *d_pending = nullptr;
  Ctl *d_ctl = nullptr;
  uint64_t *d_wl = nullptr;
  uint64_t wl_cap = 0;      // operations per batch the worklist is sized for
  uint64_t wl_seg_cap = 0;  // entries per worklist segment (NSHARD segments)
  uint64_t *d_dd = nullptr;
  uint64_t dd_cap = 0;  // power of two
  uint64_t bytes = 0;
  hipStream_t last = nullptr;
  // phase timing (hive_phase_timing): events at phase boundaries, spans
  // [a, b) of one phase group each, waiting to be read
  struct Span {
    int kind;
    hipEvent_t a, b;
  };
  bool timing = false;
  int open_kind = -1;
  hipEvent_t open_ev = nullptr;
  std::vector<Span> spans;
  std::vector<hipEvent_t> free_events;
  std::vector<hipEvent_t> all_events;
};

struct hive_drain {
  uint32_t S = 16;
  uint64_t cap = 0;
  uint32_t max_tables = 0;
  unsigned grid[2] = {0, 0};  // blocks of a launch: [0] draining, [1] resident
  int fit_per_cu = 0;         // worker blocks that fit one CU (occupancy query)
  DrainQueue *d_q = nullptr;
  ReqState *d_req = nullptr;
  uint64_t *d_table_next = nullptr;
  ReqDesc *h_ring = nullptr;
  uint64_t *h_tail = nullptr;
  uint32_t *h_stop = nullptr;
  uint64_t *h_done = nullptr;
  uint64_t *h_live = nullptr;
  uint64_t submitted = 0;
  // per registered table: its slot in table_next and its next sequence number
  hive_table *tables[4096];
  uint64_t next_seq[4096];
  uint32_t n_tables = 0;
  hipStream_t capture = nullptr;
  hipGraph_t graph[2] = {nullptr, nullptr};
  hipGraphExec_t exec[2] = {nullptr, nullptr};
  hipStream_t running_on = nullptr;
  bool running = false;
};

#define HIP_OK(expr)                                                                        \
  do {                                                                                      \
    hipError_t e_ = (expr);                                                                 \
    if (e_ != hipSuccess) {                                                                 \
      fprintf(stderr, "hive: %s failed: %s (%s:%d)\n", #expr, hipGetErrorString(e_), __FILE__, \
              __LINE__);                                                                    \
      return HIVE_ERR_HIP;                                                                  \
    }                                                                                       \
  } while (0)

static hive_status launch_check() {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    fprintf(stderr, "hive: kernel launch failed: %s\n", hipGetErrorString(e));
    return HIVE_ERR_HIP;
  }
  return HIVE_OK;
}

static unsigned grid_for(uint64_t n, uint64_t per_block, unsigned cap) {
  uint64_t g = (n + per_block - 1) / per_block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (unsigned)g;
}

static Ctl initial_ctl(const hive_table *h) {
  Ctl c;
  memset(&c, 0, sizeof(c));
  c.n_buckets = h->initial_buckets;
  c.mode = h->cfg.addressing;
  if (h->cfg.addressing == HIVE_FIXED) {
    c.magic = fastmod_magic((uint32_t)h->initial_buckets);
  } else {
    uint64_t p = 1;
    while (p * 2 <= h->initial_buckets) p *= 2;
    c.im = p - 1;
    c.sp = h->initial_buckets - p;
  }
  c.initial_buckets = h->initial_buckets;
  c.max_buckets = h->max_buckets;
  return c;
}

static uint64_t hint_words(uint64_t buckets) { return (buckets + 31) / 32; }

// Words of the hint bits and, from a 256-byte boundary on, the filter's.
static uint64_t hint_span(const hive_table *h) { return (hint_words(h->max_buckets) + 63) / 64 * 64; }
static uint64_t bit_words(const hive_table *h, bool filter) {
  return filter ? hint_span(h) + ((h->max_buckets << h->spill.shift) + 31) / 32 : hint_words(h->max_buckets);
}

static hive_status reset_table(hive_table *h, hipStream_t st) {
  ResetArgs a{};
  a.buckets = h->d_buckets;
  a.n_buckets = h->max_buckets * h->S * h->entry_bytes / 8;
  a.stash = h->d_stash;
  a.n_stash = stash_slots_for(h->stash_cap) * h->entry_bytes / 8;
  a.shards = (uint64_t *)shard_of(h->d_ctl, 0);
  a.n_shards = NSHARD * SHARD_STRIDE / 8;
  a.bits = h->d_hint;
  a.n_bits = bit_words(h, h->spill.bits != nullptr);
  a.ctl = h->d_ctl;
  hipLaunchKernelGGL(reset_kernel, dim3(grid_for(a.n_buckets + a.n_stash + a.n_shards, BLOCK * 8ull, 65535)),
                     dim3(BLOCK), 0, st, a, initial_ctl(h));
  return launch_check();
}

static void free_table(hive_table *h) {
  if (!h) return;
  for (hipEvent_t e : h->all_events) (void)hipEventDestroy(e);
  (void)hipFree(h->d_buckets);
  (void)hipFree(h->d_hint);
  (void)hipFree(h->d_stash);
  (void)hipFree(h->d_pending);
  (void)hipFree(h->d_ctl);
  (void)hipFree(h->d_wl);
  (void)hipFree(h->d_dd);
  delete h;
}

static hive_status alloc(void **p, uint64_t bytes, uint64_t *total) {
  const hipError_t e = hipMalloc(p, bytes ? bytes : 8);
  if (e != hipSuccess) {
    fprintf(stderr, "hive: hipMalloc of %llu bytes failed: %s\n", (unsigned long long)bytes, hipGetErrorString(e));
    (void)hipGetLastError();
    *p = nullptr;
    return HIVE_ERR_OOM;
  }
  *total += bytes;
  return HIVE_OK;
}

// Per-batch scratch (worklist and dedupe set) grows on demand; growing
// synchronizes the stream because the old buffers may still be in use.
// Entries per worklist segment for batches of up to n operations (or stash
// drains of up to n entries): tile t of 256 appends to segment t % NSHARD,
// at most 256 entries from each of ceil(tiles / NSHARD) tiles.
static uint64_t wl_seg_cap_for(uint64_t n) {
  const uint64_t tiles = (n + BLOCK - 1) / BLOCK;
  return std::max<uint64_t>(1, (tiles + NSHARD - 1) / NSHARD) * BLOCK;
}

// n_wl: operations (or drained entries) that may reach the eviction worklist;
// n_dd: operations the dedupe set must hold (0: none).  The set is sized
// from the whole batch, not from its inserts: a delete batch sends nothing
// to the worklist but records every operation in the set.
static uint64_t dd_set_words(uint64_t n) {  // the executor's open-addressed dedupe set
  uint64_t want = 16;
  while (want < 2 * n) want <<= 1;
  return want;
}

// Chunk of the two-launch dedupe: about 128 chunks or more (a block each, the
// chip has 256 compute units), up to four operations per thread (eight, whose table
// takes 128 KiB of LDS, are 2 to 20% faster from 2^21 to 2^24 operations and twice
// as fast beyond, but such blocks wait beside a resident executor).
static uint64_t ddr_chunk(uint64_t n) {
  return (uint64_t)DDR_BLOCK * (n <= (1ull << 17) ? 1 : n <= (1ull << 18) ? 2 : 4);
}

// log2 of its hash ranges: of about 1,024 operations up to DDR_BINS of them, of
// about 4,096 in larger batches (half of what their table takes at most).
static uint32_t ddr_bits(uint64_t n) {
  uint32_t bits = 4;
  while ((1u << bits) < DDR_BINS && (1024ull << bits) < n) ++bits;
  while ((1u << bits) < DDR_BINS_BIG && (4096ull << bits) < n) ++bits;
  return bits;
}

// The dedupe's buffers for a batch of n operations, carved from one scratch
// allocation (each piece 256-byte aligned): records and range bounds of every
// chunk (at most DDR_BLOCK * 4 operations), a winner flag per operation and,
// beyond the one-launch form, the words of ranges that are settled in HBM.
struct DdrBuffers {
  uint64_t *rec, *used, *set;
  uint32_t *bounds;
  uint8_t *win;
};
static uint64_t ddr_layout(uint64_t *base, uint64_t n, DdrBuffers *out) {
  // a chunk is shorter where the batch is (launch_dedupe); its bounds are the
  // larger part then
  const uint64_t ch = ddr_chunk(n), nch = (n + ch - 1) / ch;
  uint64_t at = 0;
  const auto take = [&](uint64_t bytes) {
    uint64_t *p = base ? base + at : nullptr;
    at += (bytes + 255) / 256 * 32;
    return p;
  };
  DdrBuffers d;
  d.rec = take(nch * ch * 8);
  d.bounds = (uint32_t *)take((nch << ddr_bits(n)) * 4);
  d.win = (uint8_t *)take(n);
  d.used = take(n > DDS_MAX ? 8 : 0);
  d.set = take(n > DDS_MAX ? 2 * n * 8 : 0);
  if (out) *out = d;
  return at;
}

// Words of the dedupe scratch for n operations: the dedupe of plain launches
// or the executor's set.
static uint64_t dd_words_for(uint64_t n) {
  return std::max(dd_set_words(n), ddr_layout(nullptr, n, nullptr));
}

// Worklist entries a stash drain may append: the whole stash table and the
// pending list.
static uint64_t drain_words(const hive_table *h) { return stash_slots_for(h->stash_cap) + h->pending_cap; }

// Entries of a worklist that holds those of a batch of n operations and of a
// drain of d words: the fills of a segment by the two are each rounded up to
// whole tiles of their own.  (A table of 64 buckets that may grow to 4,096 takes
// 0.25 MiB for both; with four tiles per segment added to the sum, 0.6.)
static uint64_t wl_batch_and_drain(uint64_t n, uint64_t d) {
  return (wl_seg_cap_for(n) + wl_seg_cap_for(d)) * NSHARD;
}

static hive_status ensure_scratch(hive_table *h, uint64_t n, uint64_t n_dd, hipStream_t st) {
  if (n > h->wl_cap) {
    HIP_OK(hipStreamSynchronize(st));
    (void)hipFree(h->d_wl);
    h->d_wl = nullptr;
    const uint64_t cap = std::max<uint64_t>(n, 2 * h->wl_cap);
    const uint64_t seg = wl_seg_cap_for(cap);
    h->bytes -= h->wl_seg_cap * NSHARD * 8;
    h->wl_cap = 0;
    h->wl_seg_cap = 0;
    if (alloc((void **)&h->d_wl, seg * NSHARD * 8, &h->bytes) != HIVE_OK) return HIVE_ERR_OOM;
    h->wl_cap = cap;
    h->wl_seg_cap = seg;
  }
  if (n_dd > 0) {
    const uint64_t want = dd_words_for(n_dd);
    if (want > h->dd_cap) {
      HIP_OK(hipStreamSynchronize(st));
      (void)hipFree(h->d_dd);
      h->d_dd = nullptr;
      h->bytes -= h->dd_cap * 8;
      h->dd_cap = 0;
      if (alloc((void **)&h->d_dd, want * 8, &h->bytes) != HIVE_OK) return HIVE_ERR_OOM;
      h->dd_cap = want;
    }
  }
  return HIVE_OK;
}

// Probe-kernel variants a table may select per operation kind
// (hive_config.probe_tuning): occupancy target in waves per SIMD and loads
// in flight per probe chunk.  A kind's 0 leaves the choice to launch_ops_mode
// (variant 0, or 4 where it is faster), TUNING_ZERO asks for variant 0 itself.
// Variants other than 0 exist for 16-slot BitHash tables probing the second
// candidate after a miss (probe_both = 0).  The insert kernel's fused round
// holds twice the loads, so variants 1 and 2 would spill registers there and
// are refused for inserts (kInsertTunings).
struct ProbeTuning {
  int waves_per_simd, loads_in_flight;
};
static constexpr ProbeTuning kProbeTunings[] = {{OPS_WAVES_PER_EU, 16}, {6, 16}, {8, 8}, {6, 8}, {8, 4}};
static constexpr int kNumProbeTunings = sizeof(kProbeTunings) / sizeof(kProbeTunings[0]);
static constexpr uint32_t TUNING_ZERO = 15;
static constexpr uint32_t kInsertTunings = (1u << 0) | (1u << 3) | (1u << 4) | (1u << TUNING_ZERO);

// By default, a 16-slot BitHash table with a spill filter takes variant 4
// (8 waves per SIMD, 4 loads in flight).  The filter ends nearly every miss
// at its first bucket, so an operation is one dependent load or two and
// more waves hide it better than more loads per wave: lookups of 2^22 keys
// in us at 4 waves and 16 loads, then at 8 and 4: tables of 2^20 keys at
// load 0.9 34.7 and 27.6, 2^22 110.6 and 90.4, 2^26 148 and 133; deletes of
// 2^22 keys at 2^26 291 and 283, replacements 290 and 281, inserts equal.
// The exception is a lookup of more than WIDE_LOOKUP_MAX keys in buckets
// larger than the last-level cache: there memory is the bound and the 16
// loads a wave keeps in flight use it better (2^26 keys in 2^26: 2.05 ms,
// against 2.08 with 8 and 4; equal at 2^24 keys, 533 and 530 us), and the
// inserts of a plain batch, whose new keys take two dependent rounds: slices of
// 420,000 of them into 2^22 keys at 65-75 and 75-85% load 64 and 72 us with 8
// and 4, 48 and 59 with 4 and 16 (both candidates in one round 49 and 63).  Tables
// without a filter stay at variant 0: 2^22 lookups at load 0.6 127 us
// against 131, deletes within 4 % of each other, first inserts into 2^18
// buckets' worth of keys 112 against 97 but later ones 48 against 55.
static constexpr uint64_t LAST_LEVEL_CACHE = 256ull << 20;
static constexpr uint64_t WIDE_LOOKUP_MAX = 1ull << 24;

template <int S, uint32_t MODE, bool BOTH, int PAIR = PAIR_BITHASH, int V = 0>
static void launch_ops(const OpsArgs &a, uint32_t grid_cap, hipStream_t st) {
  constexpr ProbeTuning t = kProbeTunings[V];
  const uint64_t blocks = std::min<uint64_t>((a.n + BLOCK - 1) / BLOCK, grid_cap ? grid_cap : OPS_GRID);
  if constexpr (!BOTH && PairArity<PAIR>::D == 2) {
    if (a.spill.bits) {
      hipLaunchKernelGGL((ops_kernel<S, MODE, BOTH, PAIR, t.waves_per_simd, t.loads_in_flight, FILTER_USE>),
                         dim3((unsigned)blocks), dim3(BLOCK), 0, st, a);
      return;
    }
  }
  hipLaunchKernelGGL((ops_kernel<S, MODE, BOTH, PAIR, t.waves_per_simd, t.loads_in_flight>),
                     dim3((unsigned)blocks), dim3(BLOCK), 0, st, a);
}

template <int S, bool BOTH, int PAIR = PAIR_BITHASH, int V = 0>
static void launch_ops_mode_v(uint32_t mode, const OpsArgs &a, uint32_t grid_cap, hipStream_t st) {
  // inserts never take the variants hive_create refuses for them
  constexpr int VI = ((kInsertTunings >> V) & 1u) ? V : 4;
  switch (mode) {
    case OP_INSERT: launch_ops<S, OP_INSERT, BOTH, PAIR, VI>(a, grid_cap, st); break;
    case OP_DELETE: launch_ops<S, OP_DELETE, BOTH, PAIR, V>(a, grid_cap, st); break;
    case OP_LOOKUP: launch_ops<S, OP_LOOKUP, BOTH, PAIR, V>(a, grid_cap, st); break;
    default: launch_ops<S, OP_MIXED, BOTH, PAIR, V>(a, grid_cap, st); break;
  }
}

template <int S, bool BOTH, int PAIR = PAIR_BITHASH>
static void launch_ops_mode(uint32_t mode, const OpsArgs &a, const hive_config &cfg, bool plain, hipStream_t st) {
  if constexpr (S == 16 && !BOTH && PAIR == PAIR_BITHASH) {
    uint32_t v = (cfg.probe_tuning >> (4 * std::min<uint32_t>(mode, OP_MIXED))) & 15u;
    if (v == 0 && a.spill.bits && !(mode == OP_INSERT && plain) &&
        !(mode == OP_LOOKUP && a.n > WIDE_LOOKUP_MAX && cfg.max_buckets * (S * 8) > LAST_LEVEL_CACHE))
      v = 4;
    switch (v) {
      case 1: launch_ops_mode_v<S, BOTH, PAIR, 1>(mode, a, cfg.probe_grid, st); return;
      case 2: launch_ops_mode_v<S, BOTH, PAIR, 2>(mode, a, cfg.probe_grid, st); return;
      case 3: launch_ops_mode_v<S, BOTH, PAIR, 3>(mode, a, cfg.probe_grid, st); return;
      case 4: launch_ops_mode_v<S, BOTH, PAIR, 4>(mode, a, cfg.probe_grid, st); return;
      default: break;
    }
  }
  launch_ops_mode_v<S, BOTH, PAIR, 0>(mode, a, cfg.probe_grid, st);
}

// The eviction grid: one group per item up to EVICT_GRID blocks (chains are
// latency-bound, so items run side by side rather than one after another in
// a group); `max_items` bounds the worklist (the batch's inserts, or the
// stash and pending capacity for a drain).
static void phase_mark(hive_table *h, int kind, hipStream_t st);

// Grid of evict_lanes_kernel<PAIR>: a block per 256 possible items, at most
// as many blocks as are resident at once (a wave's range is not shared).
template <int PAIR>
static unsigned evict_lanes_grid(uint64_t max_items) {
  static const unsigned resident = [] {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, evict_lanes_kernel<PAIR>, BLOCK, 0) != hipSuccess ||
        cus < 1 || per_cu < 1) {
      (void)hipGetLastError();
      return (unsigned)EVICT_GRID;
    }
    return (unsigned)std::min(cus * per_cu, EVICT_GRID);
  }();
  return (unsigned)std::min<uint64_t>(grid_for(max_items, (uint64_t)BLOCK, EVICT_GRID), resident);
}

// split_steps (phase timing of a 16-slot BitHash table): steps 3 and 4 in
// two launches, the second timed as its own phase.  refill: 16-slot
// two-hash tables run evict_lanes_kernel (lanes refilled from the wave's
// range); the re-placement after a split, a few thousand items that each
// start a chain at once, keeps one item per lane (evict_kernel).
static void launch_evict(hive_table *h, const Spill &spill, uint64_t max_items, uint64_t inserts, hipStream_t st,
                         bool split_steps = false, bool refill = true) {
  EvictArgs e{h->d_buckets, spill,         h->d_hint,    h->d_stash,     h->d_pending,         h->d_ctl,
              h->d_wl,      h->wl_seg_cap, h->stash_cap, h->pending_cap, h->cfg.max_evictions, inserts};
  const dim3 grid(grid_for(max_items, (uint64_t)WAVES * evict_groups_per_wave(h->S), EVICT_GRID));
  if (split_steps && h->S == 16 && h->cfg.hash_pair == PAIR_BITHASH) {
    hipLaunchKernelGGL((evict_kernel<16, PAIR_BITHASH, true>), grid, dim3(BLOCK), 0, st, e);
    phase_mark(h, HIVE_PHASE_STASH, st);
    hipLaunchKernelGGL(stash_kernel<PAIR_BITHASH>, dim3(grid_for(max_items, BLOCK, EVICT_GRID)), dim3(BLOCK), 0, st,
                       e);
    return;
  }
  switch (h->S) {
    case 16:
      if (!refill)  // after a resize alone: LINEAR tables, whose pair is BitHash
        hipLaunchKernelGGL(evict_kernel<16>, grid, dim3(BLOCK), 0, st, e);
      else if (h->cfg.hash_pair == PAIR_CRC)
        hipLaunchKernelGGL(evict_lanes_kernel<PAIR_CRC>, dim3(evict_lanes_grid<PAIR_CRC>(max_items)), dim3(BLOCK),
                           0, st, e);
      else if (h->cfg.hash_pair == PAIR_MURMUR)
        hipLaunchKernelGGL(evict_lanes_kernel<PAIR_MURMUR>, dim3(evict_lanes_grid<PAIR_MURMUR>(max_items)),
                           dim3(BLOCK), 0, st, e);
      else if (h->cfg.hash_pair == PAIR_TRIPLE)
        hipLaunchKernelGGL((evict_kernel<16, PAIR_TRIPLE>), grid, dim3(BLOCK), 0, st, e);
      else
        hipLaunchKernelGGL(evict_lanes_kernel<PAIR_BITHASH>, dim3(evict_lanes_grid<PAIR_BITHASH>(max_items)),
                           dim3(BLOCK), 0, st, e);
      break;
    case 32: hipLaunchKernelGGL(evict_kernel<32>, grid, dim3(BLOCK), 0, st, e); break;
    default: hipLaunchKernelGGL(evict_kernel<64>, grid, dim3(BLOCK), 0, st, e); break;
  }
}

// Fold the shards into the totals (batches without inserts; an eviction
// launch folds by itself).
static void launch_finish(hive_table *h, uint64_t inserts, hipStream_t st) {
  hipLaunchKernelGGL(finish_kernel, dim3(1), dim3(64), 0, st, h->d_ctl, inserts);
}

// Phase timing: close the open span (if any) at an event recorded now on
// `st` and open one of `kind` there (kind < 0: open none).  Off unless
// hive_phase_timing enabled it; a failure to get an event turns it off.
static void phase_mark(hive_table *h, int kind, hipStream_t st) {
  if (!h->timing) return;
  hipEvent_t e = nullptr;
  if (!h->free_events.empty()) {
    e = h->free_events.back();
    h->free_events.pop_back();
  } else if (hipEventCreate(&e) == hipSuccess) {
    h->all_events.push_back(e);
  } else {
    (void)hipGetLastError();
    h->timing = false;
    return;
  }
  (void)hipEventRecord(e, st);
  if (h->open_kind >= 0) h->spans.push_back({h->open_kind, h->open_ev, e});
  h->open_kind = kind;
  h->open_ev = e;
}

// A resize call's launches up to its eviction launch: the plan with its splits
// and (drain) the stash's entries to the worklist, then the merges where the
// call may contract.
static void launch_resize(hive_table *h, uint32_t mode, uint64_t amount, const uint8_t *d_ops, bool drain,
                          hipStream_t st) {
  const ResizeArgs ra{h->d_buckets, h->d_hint, h->d_ctl, h->S, h->cfg.resize_k, h->cfg.lf_expand_pct,
                      h->cfg.lf_contract_pct};
  const DrainArgs da{h->d_stash, h->d_pending, h->d_wl, h->stash_cap, h->pending_cap, h->wl_seg_cap,
                     hint_words(h->max_buckets)};
  if (mode == PLAN_PRE_MIXED && amount > BLOCK * 16ull) {
    hipLaunchKernelGGL(count_inserts_kernel, dim3(NSHARD), dim3(1024), 0, st, h->d_ctl, d_ops, amount);
    d_ops = nullptr;  // counted
  }
  // blocks for the largest split or drain the table can ask for
  const uint64_t work = std::max(h->max_buckets * h->S, drain ? drain_words(h) : 0);
  const dim3 grid(grid_for(work, BLOCK * 4ull, RESIZE_GRID));
  const bool merges = mode == PLAN_POST || mode == PLAN_MERGE;
  switch (h->S) {
    case 16:
      hipLaunchKernelGGL(resize_kernel<16>, grid, dim3(BLOCK), 0, st, ra, da, mode, amount, d_ops, drain);
      if (merges) hipLaunchKernelGGL(merge_kernel<16>, dim3(MERGE_GRID), dim3(MERGE_BLOCK), 0, st, ra);
      break;
    case 32:
      hipLaunchKernelGGL(resize_kernel<32>, grid, dim3(BLOCK), 0, st, ra, da, mode, amount, d_ops, drain);
      if (merges) hipLaunchKernelGGL(merge_kernel<32>, dim3(MERGE_GRID), dim3(MERGE_BLOCK), 0, st, ra);
      break;
    default:
      hipLaunchKernelGGL(resize_kernel<64>, grid, dim3(BLOCK), 0, st, ra, da, mode, amount, d_ops, drain);
      if (merges) hipLaunchKernelGGL(merge_kernel<64>, dim3(MERGE_GRID), dim3(MERGE_BLOCK), 0, st, ra);
      break;
  }
}

// batch_items > 0: the call follows a batch's probe launch whose eviction
// worklist (at most batch_items entries) is still to be placed; the
// drained stash joins it and one eviction launch places both.
static hive_status resize_sequence(hive_table *h, uint32_t mode, uint64_t amount, const uint8_t *d_ops,
                                   hipStream_t st, uint64_t batch_items = 0) {
  phase_mark(h, HIVE_PHASE_RESIZE, st);
  launch_resize(h, mode, amount, d_ops, true, st);
  phase_mark(h, HIVE_PHASE_DRAIN, st);
  // live entries of a drain (and the batch's worklist)
  launch_evict(h, h->spill, batch_items + h->stash_cap + h->pending_cap, 0, st, false, batch_items > 0);
  return launch_check();
}


// ---------------------------------------------------------------------------
// Persistent executor (host side)
// ---------------------------------------------------------------------------
static void free_drain(hive_drain *d) {
  if (!d) return;
  for (int m = 0; m < 2; ++m) {
    if (d->exec[m]) (void)hipGraphExecDestroy(d->exec[m]);
    if (d->graph[m]) (void)hipGraphDestroy(d->graph[m]);
  }
  if (d->capture) (void)hipStreamDestroy(d->capture);
  (void)hipFree(d->d_q);
  (void)hipFree(d->d_req);
  (void)hipFree(d->d_table_next);
  (void)hipHostFree(d->h_ring);
  (void)hipHostFree(d->h_tail);
  (void)hipHostFree(d->h_stop);
  (void)hipHostFree(d->h_done);
  (void)hipHostFree(d->h_live);
  delete d;
}

// Ticks per microsecond of the device's constant-rate clock: two readings
// 10 ms apart on the host clock (launch latency is a small error here).
static hive_status wall_clock_rate(double *ticks_per_us) {
  uint64_t *d_t = nullptr;
  uint64_t t[2] = {0, 0};
  HIP_OK(hipMalloc((void **)&d_t, 16));
  hipLaunchKernelGGL(wall_clock_kernel, dim3(1), dim3(1), 0, 0, d_t);
  hipError_t e = hipDeviceSynchronize();
  const auto h0 = std::chrono::steady_clock::now();
  std::this_thread::sleep_for(std::chrono::milliseconds(10));
  if (e == hipSuccess) {
    hipLaunchKernelGGL(wall_clock_kernel, dim3(1), dim3(1), 0, 0, d_t + 1);
    e = hipDeviceSynchronize();
  }
  const auto h1 = std::chrono::steady_clock::now();
  if (e == hipSuccess) e = hipMemcpy(t, d_t, 16, hipMemcpyDeviceToHost);
  (void)hipFree(d_t);
  if (e != hipSuccess || t[1] <= t[0]) {
    fprintf(stderr, "hive: device clock calibration failed: %s\n", hipGetErrorString(e));
    return HIVE_ERR_HIP;
  }
  const double us = std::chrono::duration<double, std::micro>(h1 - h0).count();
  *ticks_per_us = (double)(t[1] - t[0]) / us;
  return HIVE_OK;
}

// Grid sizes.  A draining grid may fill every CU: it exits once its work is
// done.  A resident grid waits for work that the host has not submitted yet,
// and the host may first need other kernels to run (its own copies: HIP runs
// small pageable copies as kernels); with every CU's registers held by the
// polling grid such a kernel cannot start until the grid exits.  So a
// resident grid takes one block per CU fewer than fit (at least one).
template <int S>
static hive_status drain_grid(uint32_t blocks_per_cu, unsigned grid[2], int *fit_per_cu) {
  int dev = 0, cus = 0, per_cu = 0;
  HIP_OK(hipGetDevice(&dev));
  HIP_OK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  HIP_OK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, drain_worker_kernel<S>, BLOCK, 0));
  if (per_cu < 1) return HIVE_ERR_HIP;
  *fit_per_cu = per_cu;
  const unsigned want = blocks_per_cu ? blocks_per_cu : (unsigned)per_cu;
  grid[0] = (unsigned)cus * std::min<unsigned>(want, (unsigned)per_cu);
  grid[1] = (unsigned)cus * std::min<unsigned>(want, (unsigned)std::max(1, per_cu - 1));
  return HIVE_OK;
}

template <int S>
static void launch_drain_kernel(hive_drain *d, int mode, hipStream_t st) {
  hipLaunchKernelGGL(drain_worker_kernel<S>, dim3(d->grid[mode]), dim3(BLOCK), 0, st, d->d_q);
}

static void launch_drain_any(hive_drain *d, int mode, hipStream_t st) {
  switch (d->S) {
    case 16: launch_drain_kernel<16>(d, mode, st); break;
    case 32: launch_drain_kernel<32>(d, mode, st); break;
    default: launch_drain_kernel<64>(d, mode, st); break;
  }
}

template <int PER, int BINS = DDR_BINS>
static void launch_ddr(const DdrArgs &a, hipStream_t st) {
  hipLaunchKernelGGL((ddr_chunk_kernel<PER, BINS>), dim3(a.nch), dim3(DDR_BLOCK), 0, st, a);
  const dim3 ranges(1u << a.bits);
  if (BINS == DDR_BINS_BIG && a.n > 2 * DDR_MORE)
    hipLaunchKernelGGL((ddr_resolve_kernel<PER, BINS, BINS == DDR_BINS_BIG ? 2 : 8>), ranges, dim3(DDR_BLOCK), 0, st,
                       a);
  else
    hipLaunchKernelGGL((ddr_resolve_kernel<PER, BINS, 8>), ranges, dim3(DDR_BLOCK), 0, st, a);
}

template <int FILTER>
static void launch_small_filter(uint32_t mode, const OpsArgs &a, uint8_t *win, hipStream_t st) {
  const dim3 grid((unsigned)((a.n + SMALL_BLOCK - 1) / SMALL_BLOCK)), block(SMALL_BLOCK);
  switch (mode) {
    case OP_INSERT: hipLaunchKernelGGL((small_batch_kernel<16, OP_INSERT, FILTER>), grid, block, 0, st, a, win); break;
    case OP_DELETE: hipLaunchKernelGGL((small_batch_kernel<16, OP_DELETE, FILTER>), grid, block, 0, st, a, win); break;
    default: hipLaunchKernelGGL((small_batch_kernel<16, OP_MIXED, FILTER>), grid, block, 0, st, a, win); break;
  }
}

static void launch_small(uint32_t mode, const OpsArgs &a, uint8_t *win, hipStream_t st) {
  if (a.spill.bits) launch_small_filter<FILTER_USE>(mode, a, win, st);
  else launch_small_filter<FILTER_NONE>(mode, a, win, st);
}

// The dedupe of a batch (one launch, or the two of the chunked form) into the
// scratch at dd, which holds dd_words_for(n) words; *win gets the winner
// flags.
static hive_status launch_dedupe(uint64_t *dd, uint32_t mode, const uint8_t *d_ops, const uint32_t *d_keys,
                                 uint64_t n, hipStream_t st, const uint8_t **win) {
  DdrBuffers buf;
  (void)ddr_layout(dd, n, &buf);
  *win = buf.win;
  if (n <= DDS_MAX) {
    uint32_t bits = 0;
    while (((uint64_t)DDS_PER << bits) < n) ++bits;
    const DdsArgs a{d_ops, d_keys, buf.win, (uint32_t)n, mode, bits};
    const dim3 grid(1u << bits), block(DDS_BLOCK);
    switch (mode) {
      case OP_INSERT: hipLaunchKernelGGL(dds_kernel<OP_INSERT>, grid, block, 0, st, a); break;
      case OP_DELETE: hipLaunchKernelGGL(dds_kernel<OP_DELETE>, grid, block, 0, st, a); break;
      default: hipLaunchKernelGGL(dds_kernel<OP_MIXED>, grid, block, 0, st, a); break;
    }
    return launch_check();
  }
  const uint32_t bits = ddr_bits(n);
  const uint64_t ch = ddr_chunk(n);
  DdrArgs a{d_ops, d_keys, buf.win, buf.rec, buf.bounds, buf.set, buf.used, (uint32_t)n, mode, bits, (uint32_t)((n + ch - 1) / ch), OP_NONE};
  const bool by_type = mode == OP_MIXED && n >= (1ull << 31);  // indices fill the word
  for (uint32_t only : {(uint32_t)OP_INSERT, (uint32_t)OP_DELETE}) {
    if (by_type) a.only = only;
    switch (ch / DDR_BLOCK) {
      case 1: launch_ddr<1>(a, st); break;
      case 2: launch_ddr<2>(a, st); break;
      default:
        if (n > DDR_MORE) launch_ddr<4, DDR_BINS_BIG>(a, st);
        else if (n > (1ull << 20)) launch_ddr<4, DDR_BINS_MID>(a, st);
        else launch_ddr<4>(a, st);
        break;
    }
    if (!by_type) break;
  }
  return launch_check();
}

// ---------------------------------------------------------------------------
// Scratch for callers that cannot allocate (hive_mixed_batch_noalloc): the
// dedupe set of one batch lives in this array instead of the table's
// grow-on-demand buffer.  Each GPU holds its own copy for the life of the
// process; host code reaches it only through the per-device address that
// hipGetSymbolAddress returns (the array's name is a host-side stand-in).
// ---------------------------------------------------------------------------
constexpr uint64_t NOALLOC_DD_WORDS = 1ull << 24;  // 128 MiB
constexpr uint64_t NOALLOC_MAX_BATCH = 1ull << 22;  // dd_words_for(n) <= NOALLOC_DD_WORDS (checked at first use)
static __device__ __align__(256) uint64_t scratch[NOALLOC_DD_WORDS];

constexpr int NOALLOC_MAX_DEVICES = 64;
static std::mutex g_scratch_mu;
static uint64_t *g_scratch_ptr[NOALLOC_MAX_DEVICES] = {};

// The current device's copy of `scratch`, looked up once per device.
static hive_status noalloc_scratch(uint64_t **out) {
  int dev = 0;
  HIP_OK(hipGetDevice(&dev));
  if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) return HIVE_ERR_HIP;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    HIP_OK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    g_scratch_ptr[dev] = (uint64_t *)p;
  }
  *out = g_scratch_ptr[dev];
  return HIVE_OK;
}

// The filter a batch about to be enqueued is given: the table's, or none once
// it places (or an earlier batch placed) without.  Inserts take the kernel with
// the filter all the same, which leaves it alone then and probes the second
// candidate after a miss only: of 2^22 keys that are present already 199 us,
// 252 with both candidates in one round; of 2^22 new ones 288 and 292.
static Spill batch_spill(hive_table *h, uint32_t mode, uint64_t n) {
  if (mode == OP_INSERT || mode == OP_MIXED) {
    h->dropped = h->dropped || h->inserted >= h->spill.start || h->inserted + n > h->spill.end;
    h->inserted += n;
  }
  return h->dropped && mode != OP_INSERT ? spill_none(h->S) : h->spill;
}

// no_alloc: take the dedupe set from `scratch` and refuse a batch that would
// grow the table's worklist, so that the call allocates nothing; phase
// timing (which creates events) is skipped for such a call.
static hive_status run_batch(hive_t h, uint32_t mode, const uint8_t *d_ops, const uint32_t *d_keys,
                             const uint32_t *d_vals, uint64_t n, uint32_t flags, uint32_t *d_vals_out,
                             uint8_t *d_flags_out, void *stream, bool no_alloc = false) {
  if (!h || (n > 0 && !d_keys)) return HIVE_ERR_ARG;
  if (n >= 0xFFFFFFFFull) return HIVE_ERR_ARG;  // batch indices are 32-bit in the dedupe set
  if (mode == OP_INSERT && n > 0 && !d_vals && h->entry_bytes == 8) return HIVE_ERR_ARG;  // sets read no values
  if (mode == OP_MIXED && n > 0 && !d_ops) return HIVE_ERR_ARG;
  if (flags & ~(uint32_t)HIVE_UNIQUE) return HIVE_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  const bool dedupe = !(flags & HIVE_UNIQUE) && mode != OP_LOOKUP;
  const bool linear = h->cfg.addressing == HIVE_LINEAR;
  const bool inserts = mode == OP_INSERT || mode == OP_MIXED;
  // A batch with inserts on a table with a load-factor rule places its
  // eviction worklist after the rules: the stash that the splits drain (of
  // the growth before the batch, too) joins the worklist and one eviction
  // launch places both.  The worklist then holds the batch's entries and a
  // full drain.
  const uint64_t wl_post = wl_batch_and_drain(n, drain_words(h));
  const bool rules = linear && (h->cfg.post_policy || h->cfg.pre_expand);
  // (a table without the post-batch rule does not grow its worklist for this
  // alone: a call that needed no allocation before needs none)
  const bool place_last = rules && inserts && h->entry_bytes == 8 && !h->timing &&
                          (wl_post <= h->wl_cap || (!no_alloc && (n > h->wl_cap || h->cfg.post_policy)));
  // only inserts reach the eviction worklist
  const uint64_t wl_need = inserts ? (place_last ? wl_post : n) : 0;
  uint64_t *dd = nullptr;
  if (no_alloc) {
    if (wl_need > h->wl_cap) {
      fprintf(stderr, "hive: a batch of %llu operations needs a larger worklist than the table's (%llu); "
              "create the table with max_batch >= n for allocation-free calls\n",
              (unsigned long long)n, (unsigned long long)h->wl_cap);
      return HIVE_ERR_BUDGET;
    }
    if (dedupe && (n > NOALLOC_MAX_BATCH || dd_words_for(n) > NOALLOC_DD_WORDS)) {
      fprintf(stderr, "hive: allocation-free batches with dedupe hold at most %llu operations (got %llu)\n",
              (unsigned long long)NOALLOC_MAX_BATCH, (unsigned long long)n);
      return HIVE_ERR_BUDGET;
    }
    if (dedupe) {
      hive_status s = noalloc_scratch(&dd);
      if (s != HIVE_OK) return s;
    }
  }
  h->last = st;
  if (n == 0) return HIVE_OK;
  hive_status s = HIVE_OK;
  if (!no_alloc) {
    if ((s = ensure_scratch(h, wl_need, dedupe ? n : 0, st)) != HIVE_OK) return s;
    dd = h->d_dd;
  }
  // phase timing creates events on demand: off for an allocation-free call
  struct TimingOff {
    hive_table *h;
    bool was;
    ~TimingOff() { h->timing = was; }
  } timing_guard{h, h->timing};
  if (no_alloc) h->timing = false;
  OpsArgs a{};
  a.buckets = h->d_buckets;
  a.spill = batch_spill(h, mode, n);
  a.hint = h->d_hint;
  a.stash = h->d_stash;
  a.pending = h->d_pending;
  a.ctl = h->d_ctl;
  a.wl = h->d_wl;
  a.wl_seg_cap = h->wl_seg_cap;
  a.ops = d_ops;
  a.keys = d_keys;
  a.vals = d_vals;
  a.vals_out = d_vals_out;
  a.flags_out = d_flags_out;
  a.n = n;
  a.stash_cap = h->stash_cap;
  a.pending_cap = h->pending_cap;
  // small batches of 16-slot BitHash tables: dedupe and probe in one launch
  const bool small = dedupe && n <= SMALL_MAX && h->S == 16 && h->entry_bytes == 8 &&
                     h->cfg.hash_pair == PAIR_BITHASH && !h->cfg.probe_both && !h->timing;
  if (dedupe && !small) {
    phase_mark(h, HIVE_PHASE_DEDUPE, st);
    // within the buffer: ensure_scratch sized the table's from n, and the
    // allocation-free path checked n against NOALLOC_MAX_BATCH
    if ((s = launch_dedupe(dd, mode, d_ops, d_keys, n, st, &a.win)) != HIVE_OK) return s;
  }
  if (h->entry_bytes == 4) {
    SetArgs sa{(uint32_t *)h->d_buckets, a.spill, h->d_hint, (uint32_t *)h->d_stash, (uint32_t *)h->d_pending, h->d_ctl,
               h->d_wl, h->wl_seg_cap, d_ops, d_keys, d_flags_out, n, h->stash_cap, h->pending_cap,
               h->cfg.max_evictions, a.win};
    phase_mark(h, HIVE_PHASE_PROBE, st);
    const uint64_t cap = h->cfg.probe_grid ? h->cfg.probe_grid : OPS_GRID;
    const dim3 grid((unsigned)std::min<uint64_t>((n + BLOCK - 1) / BLOCK, cap));
    switch (mode) {
      case OP_INSERT: hipLaunchKernelGGL(set_ops_kernel<OP_INSERT>, grid, dim3(BLOCK), 0, st, sa); break;
      case OP_DELETE: hipLaunchKernelGGL(set_ops_kernel<OP_DELETE>, grid, dim3(BLOCK), 0, st, sa); break;
      case OP_LOOKUP: hipLaunchKernelGGL(set_ops_kernel<OP_LOOKUP>, grid, dim3(BLOCK), 0, st, sa); break;
      default: hipLaunchKernelGGL(set_ops_kernel<OP_MIXED>, grid, dim3(BLOCK), 0, st, sa); break;
    }
    if (mode == OP_INSERT || mode == OP_MIXED) {
      phase_mark(h, HIVE_PHASE_EVICT, st);
      hipLaunchKernelGGL(set_evict_kernel, dim3(grid_for(n, BLOCK, EVICT_GRID)), dim3(BLOCK), 0, st, sa);
    } else if (mode != OP_LOOKUP) {
      phase_mark(h, HIVE_PHASE_FINISH, st);
      launch_finish(h, 0, st);
    }
    phase_mark(h, -1, st);
    return launch_check();
  }
  if (linear && h->cfg.pre_expand && inserts) {
    // grow before the batch so that live + (inserts of the batch) fits
    const uint32_t pre = mode == OP_MIXED ? PLAN_PRE_MIXED : PLAN_PRE;
    if (place_last) launch_resize(h, pre, n, d_ops, false, st);
    else if ((s = resize_sequence(h, pre, n, d_ops, st)) != HIVE_OK) return s;
  }
  phase_mark(h, HIVE_PHASE_PROBE, st);
  switch (h->S) {
    case 16:
      if (small)
        launch_small(mode, a, (uint8_t *)dd, st);
      else if (h->cfg.hash_pair == PAIR_CRC)
        launch_ops_mode<16, false, PAIR_CRC>(mode, a, h->cfg, h->dropped, st);
      else if (h->cfg.hash_pair == PAIR_MURMUR)
        launch_ops_mode<16, false, PAIR_MURMUR>(mode, a, h->cfg, h->dropped, st);
      else if (h->cfg.hash_pair == PAIR_TRIPLE)
        launch_ops_mode<16, false, PAIR_TRIPLE>(mode, a, h->cfg, h->dropped, st);
      else if (h->cfg.probe_both)
        launch_ops_mode<16, true>(mode, a, h->cfg, h->dropped, st);
      else
        launch_ops_mode<16, false>(mode, a, h->cfg, h->dropped, st);
      break;
    case 32: launch_ops_mode<32, false>(mode, a, h->cfg, h->dropped, st); break;
    default: launch_ops_mode<64, false>(mode, a, h->cfg, h->dropped, st); break;
  }
  if ((s = launch_check()) != HIVE_OK) return s;
  const bool post = linear && h->cfg.post_policy && mode != OP_LOOKUP;
  if (place_last) {
    if ((s = resize_sequence(h, post ? PLAN_POST : PLAN_NONE, 0, nullptr, st, n)) != HIVE_OK) return s;
    phase_mark(h, -1, st);
    return HIVE_OK;
  }
  if (inserts) {
    phase_mark(h, HIVE_PHASE_EVICT, st);
    launch_evict(h, a.spill, n, n, st, h->timing);
  }
  // the eviction launch folds, that of the post-batch rule too
  if (h->timing ? mode != OP_LOOKUP : (mode == OP_DELETE && !post)) {
    phase_mark(h, HIVE_PHASE_FINISH, st);
    // (its own inserts: an eviction launch that is not split in two counts them)
    launch_finish(h, inserts && h->S == 16 && h->cfg.hash_pair == PAIR_BITHASH ? n : 0, st);
  }
  if ((s = launch_check()) != HIVE_OK) return s;
  if (post && (s = resize_sequence(h, PLAN_POST, 0, nullptr, st)) != HIVE_OK) return s;
  phase_mark(h, -1, st);
  return HIVE_OK;
}

extern "C" {

hive_status hive_config_default(hive_config *cfg) {
  if (!cfg) return HIVE_ERR_ARG;
  memset(cfg, 0, sizeof(*cfg));
  cfg->slots_per_bucket = 16;
  cfg->max_evictions = 8;
  cfg->addressing = HIVE_FIXED;
  cfg->resize_k = 1024;
  cfg->lf_expand_pct = 90;
  cfg->lf_contract_pct = 25;
  return HIVE_OK;
}

hive_status hive_create(const hive_config *cfg_in, uint64_t initial_buckets, void *stream, hive_t *out) {
  if (!cfg_in || !out) return HIVE_ERR_ARG;
  *out = nullptr;
  hive_config cfg = *cfg_in;
  const uint32_t S = cfg.slots_per_bucket;
  if (S != 16 && S != 32 && S != 64) return HIVE_ERR_ARG;
  if (cfg.addressing != HIVE_FIXED && cfg.addressing != HIVE_LINEAR) return HIVE_ERR_ARG;
  if (cfg.hash_pair > HIVE_PAIR_TRIPLE) return HIVE_ERR_ARG;
  if (cfg.entry_bits != 0 && cfg.entry_bits != 64 && cfg.entry_bits != 32) return HIVE_ERR_ARG;
  const bool set32 = cfg.entry_bits == 32;
  // key-only sets: 32 slots of 4 bytes (one 128-byte line), FIXED, BitHash1/2
  if (set32 && (S != 32 || cfg.addressing != HIVE_FIXED || cfg.hash_pair != HIVE_PAIR_BITHASH || cfg.probe_both))
    return HIVE_ERR_ARG;
  // only 16-slot FIXED tables on plain launches have the other hash pairs
  if (cfg.hash_pair != HIVE_PAIR_BITHASH && (S != 16 || cfg.addressing != HIVE_FIXED || cfg.probe_both))
    return HIVE_ERR_ARG;
  // probe_tuning: one variant per operation kind (insert, delete, lookup,
  // mixed), four bits each
  if ((cfg.probe_tuning >> 16) != 0 || !((kInsertTunings >> (cfg.probe_tuning & 15u)) & 1u) ||
      (cfg.probe_tuning && (S != 16 || cfg.hash_pair != HIVE_PAIR_BITHASH || cfg.probe_both || set32)))
    return HIVE_ERR_ARG;
  for (int kind = 0; kind < 4; ++kind) {
    const uint32_t v = (cfg.probe_tuning >> (4 * kind)) & 15u;
    if (v >= (uint32_t)kNumProbeTunings && v != TUNING_ZERO) return HIVE_ERR_ARG;
  }
  if (cfg.probe_grid > (1u << 20)) return HIVE_ERR_ARG;
  if (initial_buckets < 1) return HIVE_ERR_ARG;
  if (cfg.max_evictions > 1024) return HIVE_ERR_ARG;
  if (cfg.lf_expand_pct == 0 || cfg.lf_expand_pct > 100 || cfg.lf_contract_pct >= cfg.lf_expand_pct)
    return HIVE_ERR_ARG;
  if (cfg.resize_k == 0) cfg.resize_k = 1024;
  uint64_t max_b = initial_buckets;
  if (cfg.addressing == HIVE_LINEAR) {
    max_b = std::max<uint64_t>(cfg.max_buckets, initial_buckets);
    if (max_b > (1ull << 31)) return HIVE_ERR_ARG;  // 32-bit bucket indices
  } else {
    if (initial_buckets > 0xFFFFFFFFull) return HIVE_ERR_ARG;
    if (cfg.max_buckets > initial_buckets) return HIVE_ERR_ARG;  // FIXED tables do not grow
  }
  if (max_b > (1ull << 40) / S) return HIVE_ERR_ARG;
  hive_table *h = new (std::nothrow) hive_table();
  if (!h) return HIVE_ERR_OOM;
  h->S = S;
  h->entry_bytes = set32 ? 4 : 8;
  h->initial_buckets = initial_buckets;
  h->max_buckets = max_b;
  // default: 1% of the slots of the largest table (the arena)
  h->stash_cap = cfg.stash_capacity ? cfg.stash_capacity : std::max<uint64_t>(1024, max_b * S / 100);
  h->pending_cap = cfg.pending_capacity ? cfg.pending_capacity : h->stash_cap;
  cfg.stash_capacity = h->stash_cap;
  cfg.pending_capacity = h->pending_cap;
  cfg.max_buckets = max_b;
  h->cfg = cfg;
  const bool filter = cfg.addressing == HIVE_FIXED && cfg.hash_pair != HIVE_PAIR_TRIPLE && !cfg.probe_both &&
                      cfg.max_evictions >= FIRST_MIN_CHAIN && h->stash_cap >= max_b * S / 100;
  h->spill.first_min = filter ? S * FIRST_MIN_16THS / 16 : S + 1;  // S + 1: by two-choice alone
  h->spill.start = max_b * S * FILTER_START_PCT / 100;
  h->spill.end = S == 16 ? max_b * S * FILTER_END_PCT / 100 : ~0ull;
  h->spill.shift = 3;
  while (h->spill.shift > 0 && (max_b << h->spill.shift) / 8 > FILTER_BYTES) --h->spill.shift;
  hive_status s = HIVE_OK;
  if ((s = alloc((void **)&h->d_buckets, max_b * S * h->entry_bytes, &h->bytes)) != HIVE_OK ||
      (s = alloc((void **)&h->d_hint, bit_words(h, filter) * 4, &h->bytes)) != HIVE_OK ||
      (s = alloc((void **)&h->d_stash, stash_slots_for(h->stash_cap) * h->entry_bytes, &h->bytes)) != HIVE_OK ||
      (s = alloc((void **)&h->d_pending, h->pending_cap * h->entry_bytes, &h->bytes)) != HIVE_OK ||
      (s = alloc((void **)&h->d_ctl, CTL_BYTES, &h->bytes)) != HIVE_OK) {
    free_table(h);
    return s;
  }
  if (filter) h->spill.bits = h->d_hint + hint_span(h);
  hipStream_t st = (hipStream_t)stream;
  h->last = st;
  // the worklist must hold a full stash + pending drain (after a split);
  // the drain walks the whole stash table
  const uint64_t min_wl = drain_words(h);
  // a table with a load-factor rule places a batch's worklist after the
  // rules, together with the drain (see run_batch)
  // (of at least min_wl operations)
  const uint64_t batch_wl = cfg.addressing == HIVE_LINEAR && (cfg.post_policy || cfg.pre_expand)
                                ? wl_batch_and_drain(std::max(cfg.max_batch, min_wl), min_wl)
                                : cfg.max_batch;
  if ((s = ensure_scratch(h, std::max<uint64_t>(batch_wl, min_wl), cfg.max_batch, st)) != HIVE_OK) {
    free_table(h);
    return s;
  }
  if ((s = reset_table(h, st)) != HIVE_OK || hipStreamSynchronize(st) != hipSuccess) {
    free_table(h);
    return s != HIVE_OK ? s : HIVE_ERR_HIP;
  }
  *out = h;
  return HIVE_OK;
}

hive_status hive_phase_timing(hive_t h, int enable) {
  if (!h) return HIVE_ERR_ARG;
  h->timing = enable != 0;
  return HIVE_OK;
}

hive_status hive_phase_times(hive_t h, double *ms_out) {
  if (!h || !ms_out) return HIVE_ERR_ARG;
  for (int k = 0; k < HIVE_PHASE_KINDS; ++k) ms_out[k] = 0.0;
  hive_status s = HIVE_OK;
  if (!h->spans.empty() && hipEventSynchronize(h->spans.back().b) != hipSuccess) s = HIVE_ERR_HIP;
  std::vector<hipEvent_t> used;
  for (const auto &sp : h->spans) {
    float ms = 0.f;
    if (s == HIVE_OK && hipEventElapsedTime(&ms, sp.a, sp.b) == hipSuccess) ms_out[sp.kind] += ms;
    used.push_back(sp.a);
    used.push_back(sp.b);
  }
  // an event may end one span and start the next: free each once, except
  // the start of a span still open
  std::sort(used.begin(), used.end());
  used.erase(std::unique(used.begin(), used.end()), used.end());
  for (hipEvent_t e : used)
    if (!(h->open_kind >= 0 && e == h->open_ev)) h->free_events.push_back(e);
  h->spans.clear();
  if (s != HIVE_OK) (void)hipGetLastError();
  return s;
}

hive_status hive_destroy(hive_t h) {
  if (!h) return HIVE_ERR_ARG;
  hipError_t e = hipStreamSynchronize(h->last);
  free_table(h);
  return e == hipSuccess ? HIVE_OK : HIVE_ERR_HIP;
}

hive_status hive_insert_batch(hive_t h, const uint32_t *d_keys, const uint32_t *d_vals, uint64_t n, uint32_t flags,
                              void *stream) {
  return run_batch(h, OP_INSERT, nullptr, d_keys, d_vals, n, flags, nullptr, nullptr, stream);
}

hive_status hive_lookup_batch(hive_t h, const uint32_t *d_keys, uint64_t n, uint32_t *d_vals_out,
                              uint8_t *d_found_out, void *stream) {
  return run_batch(h, OP_LOOKUP, nullptr, d_keys, nullptr, n, HIVE_UNIQUE, d_vals_out, d_found_out, stream);
}

hive_status hive_delete_batch(hive_t h, const uint32_t *d_keys, uint64_t n, uint32_t flags, uint8_t *d_deleted_out,
                              void *stream) {
  return run_batch(h, OP_DELETE, nullptr, d_keys, nullptr, n, flags, nullptr, d_deleted_out, stream);
}

hive_status hive_mixed_batch(hive_t h, const uint8_t *d_ops, const uint32_t *d_keys, const uint32_t *d_vals,
                             uint64_t n, uint32_t flags, uint32_t *d_vals_out, uint8_t *d_flags_out, void *stream) {
  if (h && n > 0 && !d_vals && h->entry_bytes == 8) return HIVE_ERR_ARG;  // inserts read their values
  return run_batch(h, OP_MIXED, d_ops, d_keys, d_vals, n, flags, d_vals_out, d_flags_out, stream);
}

hive_status hive_mixed_batch_noalloc(hive_t h, const uint8_t *d_ops, const uint32_t *d_keys, const uint32_t *d_vals,
                                     uint64_t n, uint32_t flags, uint32_t *d_vals_out, uint8_t *d_flags_out,
                                     void *stream) {
  if (h && n > 0 && !d_vals && h->entry_bytes == 8) return HIVE_ERR_ARG;
  return run_batch(h, OP_MIXED, d_ops, d_keys, d_vals, n, flags, d_vals_out, d_flags_out, stream, true);
}

hive_status hive_resize(hive_t h, int64_t delta, void *stream) {
  if (!h) return HIVE_ERR_ARG;
  if (h->cfg.addressing != HIVE_LINEAR) return HIVE_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  h->last = st;
  if (delta > 0) return resize_sequence(h, PLAN_SPLIT, (uint64_t)delta, nullptr, st);
  if (delta < 0) return resize_sequence(h, PLAN_MERGE, (uint64_t)(-(delta + 1)) + 1, nullptr, st);
  return resize_sequence(h, PLAN_POST, 0, nullptr, st);
}

hive_status hive_stats(hive_t h, hive_stats_t *out, void *stream) {
  if (!h || !out) return HIVE_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  Ctl c;
  HIP_OK(hipMemcpyAsync(&c, h->d_ctl, sizeof(Ctl), hipMemcpyDeviceToHost, st));
  HIP_OK(hipStreamSynchronize(st));
  memset(out, 0, sizeof(*out));
  out->live = c.live;
  out->n_buckets = c.n_buckets;
  out->index_mask = c.im;
  out->split_ptr = c.sp;
  out->stash_count = std::min(c.stash_count, h->stash_cap);
  out->pending_count = std::min(c.pending_count, h->pending_cap);
  out->evictions = c.evictions;
  out->stash_inserts = c.stash_inserts;
  out->pending_inserts = c.pending_inserts;
  out->full_chains = c.full_chains;
  out->invalid_keys = c.invalid_keys;
  out->evict_items = c.evict_items;
  out->bytes_reserved = h->bytes;
  out->slots_per_bucket = h->S;
  out->max_buckets = h->max_buckets;
  out->error_bits = c.error;
  if (c.error & ERR_PENDING_LOST) return HIVE_ERR_LOST;
  if (c.error & ERR_ARENA_FULL) return HIVE_ERR_BUDGET;
  if (out->pending_count) return HIVE_WARN_PENDING;
  if (c.invalid_keys) return HIVE_WARN_INVALID_KEYS;
  return HIVE_OK;
}

hive_status hive_dump(hive_t h, uint64_t *d_words, int64_t *d_where, uint64_t capacity, uint64_t *n_out,
                      void *stream) {
  if (!h || !n_out || (capacity > 0 && !d_words)) return HIVE_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  h->last = st;
  hipLaunchKernelGGL(ctl_zero_dump_kernel, dim3(1), dim3(1), 0, st, h->d_ctl);
  hive_status s = launch_check();
  if (s != HIVE_OK) return s;
  // a block per trip of the largest the table can be, all resident at most
  const uint64_t words = h->max_buckets * h->S + stash_slots_for(h->stash_cap) + h->pending_cap;
  const dim3 grid(grid_for(words, DUMP_TRIP, 512));
  if (h->entry_bytes == 4)
    hipLaunchKernelGGL(dump_kernel<true>, grid, dim3(DUMP_BLOCK), 0, st, h->d_buckets, h->S, h->d_stash, h->d_pending,
                       h->d_ctl, h->stash_cap, h->pending_cap, d_words, d_where, capacity);
  else
    hipLaunchKernelGGL(dump_kernel<false>, grid, dim3(DUMP_BLOCK), 0, st, h->d_buckets, h->S, h->d_stash,
                       h->d_pending, h->d_ctl, h->stash_cap, h->pending_cap, d_words, d_where, capacity);
  if ((s = launch_check()) != HIVE_OK) return s;
  Ctl c;
  HIP_OK(hipMemcpyAsync(&c, h->d_ctl, sizeof(Ctl), hipMemcpyDeviceToHost, st));
  HIP_OK(hipStreamSynchronize(st));
  *n_out = c.dump_count;
  return HIVE_OK;
}

hive_status hive_placement(hive_t h, uint64_t *out, void *stream) {
  if (!h || !out) return HIVE_ERR_ARG;
  if (h->cfg.hash_pair != HIVE_PAIR_BITHASH) return HIVE_ERR_ARG;  // the census computes BitHash1 candidates
  hipStream_t st = (hipStream_t)stream;
  h->last = st;
  hipLaunchKernelGGL(ctl_zero_placement_kernel, dim3(1), dim3(1), 0, st, h->d_ctl);
  hive_status s = launch_check();
  if (s != HIVE_OK) return s;
  if (h->entry_bytes == 4)
    hipLaunchKernelGGL(placement_kernel<true>, dim3(2048), dim3(BLOCK), 0, st, (const void *)h->d_buckets, h->S,
                       h->d_ctl);
  else
    hipLaunchKernelGGL(placement_kernel<false>, dim3(2048), dim3(BLOCK), 0, st, (const void *)h->d_buckets, h->S,
                       h->d_ctl);
  if ((s = launch_check()) != HIVE_OK) return s;
  Ctl c;
  HIP_OK(hipMemcpyAsync(&c, h->d_ctl, sizeof(Ctl), hipMemcpyDeviceToHost, st));
  HIP_OK(hipStreamSynchronize(st));
  out[0] = c.place_first;
  out[1] = c.place_second;
  out[2] = std::min(c.stash_count, h->stash_cap) + std::min(c.pending_count, h->pending_cap);
  return HIVE_OK;
}

hive_status hive_live_async(hive_t h, uint64_t *host_dst, void *stream) {
  if (!h || !host_dst) return HIVE_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  h->last = st;
  HIP_OK(hipMemcpyAsync(host_dst, &h->d_ctl->live, 8, hipMemcpyDeviceToHost, st));
  return HIVE_OK;
}

hive_status hive_clear(hive_t h, void *stream) {
  if (!h) return HIVE_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  h->last = st;
  h->inserted = 0;
  h->dropped = false;
  return reset_table(h, st);
}

const char *hive_status_string(hive_status s) {
  switch (s) {
    case HIVE_OK: return "ok";
    case HIVE_ERR_ARG: return "invalid argument";
    case HIVE_ERR_OOM: return "device allocation failed";
    case HIVE_ERR_HIP: return "HIP runtime error";
    case HIVE_ERR_BUDGET: return "bucket arena or capacity exhausted";
    case HIVE_ERR_LOST: return "pending list overflowed: entries lost";
    case HIVE_WARN_INVALID_KEYS: return "reserved keys were ignored";
    case HIVE_WARN_PENDING: return "entries wait in the pending list";
  }
  return "unknown status";
}

uint32_t hive_bithash1(uint32_t key) { return bithash1(key); }
uint32_t hive_bithash2(uint32_t key) { return bithash2(key); }

hive_status hive_bucket_of(hive_t h, uint32_t mixed_hash, uint64_t *bucket) {
  if (!h || !bucket) return HIVE_ERR_ARG;
  Ctl c;
  HIP_OK(hipMemcpyAsync(&c, h->d_ctl, sizeof(Ctl), hipMemcpyDeviceToHost, h->last));
  HIP_OK(hipStreamSynchronize(h->last));
  Geo g{c.n_buckets, c.magic, (uint32_t)c.im, (uint32_t)c.sp, c.mode};
  *bucket = address(g, mixed_hash);
  return HIVE_OK;
}


hive_status hive_drain_create(uint32_t slots_per_bucket, uint32_t blocks_per_cu, uint64_t ring_capacity,
                              uint32_t max_tables, uint64_t idle_timeout_us, hive_drain_t *out) {
  if (!out) return HIVE_ERR_ARG;
  *out = nullptr;
  if (slots_per_bucket != 16 && slots_per_bucket != 32 && slots_per_bucket != 64) return HIVE_ERR_ARG;
  if (ring_capacity < 1 || ring_capacity > (1ull << 24)) return HIVE_ERR_ARG;
  if (max_tables < 1 || max_tables > 4096) return HIVE_ERR_ARG;
  hive_drain *d = new (std::nothrow) hive_drain();
  if (!d) return HIVE_ERR_OOM;
  d->S = slots_per_bucket;
  d->cap = ring_capacity;
  d->max_tables = max_tables;
  hive_status s = HIVE_OK;
  switch (d->S) {
    case 16: s = drain_grid<16>(blocks_per_cu, d->grid, &d->fit_per_cu); break;
    case 32: s = drain_grid<32>(blocks_per_cu, d->grid, &d->fit_per_cu); break;
    default: s = drain_grid<64>(blocks_per_cu, d->grid, &d->fit_per_cu); break;
  }
  if (s != HIVE_OK) {
    free_drain(d);
    return s;
  }
  uint64_t bytes = 0;
  if (alloc((void **)&d->d_q, sizeof(DrainQueue), &bytes) != HIVE_OK ||
      alloc((void **)&d->d_req, sizeof(ReqState) * ring_capacity, &bytes) != HIVE_OK ||
      alloc((void **)&d->d_table_next, 8ull * max_tables, &bytes) != HIVE_OK) {
    free_drain(d);
    return HIVE_ERR_OOM;
  }
  const unsigned hflags = hipHostMallocMapped | hipHostMallocCoherent;
  if (hipHostMalloc((void **)&d->h_ring, sizeof(ReqDesc) * ring_capacity, hflags) != hipSuccess ||
      hipHostMalloc((void **)&d->h_tail, 64, hflags) != hipSuccess ||
      hipHostMalloc((void **)&d->h_stop, 64, hflags) != hipSuccess ||
      hipHostMalloc((void **)&d->h_done, 8 * ring_capacity, hflags) != hipSuccess ||
      hipHostMalloc((void **)&d->h_live, 8 * ring_capacity, hflags) != hipSuccess) {
    (void)hipGetLastError();
    free_drain(d);
    return HIVE_ERR_OOM;
  }
  memset(d->h_ring, 0, sizeof(ReqDesc) * ring_capacity);
  memset(d->h_done, 0, 8 * ring_capacity);
  memset(d->h_live, 0, 8 * ring_capacity);
  *d->h_tail = 0;
  *d->h_stop = 1;
  DrainQueue q;
  memset(&q, 0, sizeof(q));
  q.req = d->d_req;
  q.cap = ring_capacity;
  q.table_next = d->d_table_next;
  {
    // the watchdog runs on the constant-rate device clock; its rate is
    // measured here against the host clock rather than taken on trust
    double ticks_per_us = 0;
    if (wall_clock_rate(&ticks_per_us) != HIVE_OK) {
      free_drain(d);
      return HIVE_ERR_HIP;
    }
    const double us = idle_timeout_us ? (double)idle_timeout_us : 30e6;
    const double ticks = us * ticks_per_us;
    q.idle_ticks = ticks >= 1.8e19 ? ~0ull : (uint64_t)ticks;
  }
  void *dp = nullptr;
  if (hipHostGetDevicePointer(&dp, d->h_ring, 0) != hipSuccess) goto fail;
  q.host_ring = (const ReqDesc *)dp;
  if (hipHostGetDevicePointer(&dp, d->h_tail, 0) != hipSuccess) goto fail;
  q.host_tail = (const uint64_t *)dp;
  if (hipHostGetDevicePointer(&dp, d->h_stop, 0) != hipSuccess) goto fail;
  q.host_stop = (const uint32_t *)dp;
  if (hipHostGetDevicePointer(&dp, d->h_done, 0) != hipSuccess) goto fail;
  q.host_done = (uint64_t *)dp;
  if (hipHostGetDevicePointer(&dp, d->h_live, 0) != hipSuccess) goto fail;
  q.host_live = (uint64_t *)dp;
  if (hipMemcpy(d->d_q, &q, sizeof(q), hipMemcpyHostToDevice) != hipSuccess) goto fail;
  if (hipMemset(d->d_req, 0, sizeof(ReqState) * ring_capacity) != hipSuccess) goto fail;
  if (hipMemset(d->d_table_next, 0, 8ull * max_tables) != hipSuccess) goto fail;
  if (hipStreamCreateWithFlags(&d->capture, hipStreamNonBlocking) != hipSuccess) goto fail;
  if (hipDeviceSynchronize() != hipSuccess) goto fail;
  *out = d;
  return HIVE_OK;
fail:
  (void)hipGetLastError();
  free_drain(d);
  return HIVE_ERR_HIP;
}

hive_status hive_drain_submit(hive_drain_t d, hive_t h, const hive_batch_desc *b, uint64_t *ticket) {
  if (!d || !h || !b || !ticket) return HIVE_ERR_ARG;
  if (h->S != d->S) return HIVE_ERR_ARG;
  // the executor runs BitHash1/2 tables of 64-bit entries only
  if (h->cfg.hash_pair != HIVE_PAIR_BITHASH || h->entry_bytes != 8) return HIVE_ERR_ARG;
  if (b->op_mode > HIVE_OP_MIXED) return HIVE_ERR_ARG;
  if (b->n > 0 && !b->d_keys) return HIVE_ERR_ARG;
  if ((b->op_mode == HIVE_OP_INSERT || b->op_mode == HIVE_OP_MIXED) && b->n > 0 && !b->d_vals) return HIVE_ERR_ARG;
  if (b->op_mode == HIVE_OP_MIXED && b->n > 0 && !b->d_ops) return HIVE_ERR_ARG;
  if (b->n >= 0xFFFFFFFFull || (b->flags & ~(uint32_t)HIVE_UNIQUE)) return HIVE_ERR_ARG;
  const uint64_t t = d->submitted;
  // the ring slot must be free: the batch `cap` tickets earlier is complete
  if (t >= d->cap && __atomic_load_n(&d->h_done[t % d->cap], __ATOMIC_ACQUIRE) != t - d->cap + 1)
    return HIVE_ERR_BUDGET;
  // table slot (tables registered on first use)
  uint32_t slot = 0;
  while (slot < d->n_tables && d->tables[slot] != h) ++slot;
  if (slot == d->n_tables) {
    if (d->n_tables >= d->max_tables) return HIVE_ERR_BUDGET;
    d->tables[slot] = h;
    d->next_seq[slot] = 0;
    d->n_tables++;
  }
  const bool dedupe = !(b->flags & HIVE_UNIQUE) && b->op_mode != HIVE_OP_LOOKUP;
  uint64_t dd_size = (dedupe && b->n > 0) ? dd_set_words(b->n) : 0;
  // scratch is never reallocated under a running executor; only inserts
  // reach the eviction worklist, while the dedupe set holds every operation
  const uint64_t wl_need = (b->op_mode == HIVE_OP_INSERT || b->op_mode == HIVE_OP_MIXED) ? b->n : 0;
  if (wl_need > h->wl_cap || dd_size > h->dd_cap) {
    if (d->running) return HIVE_ERR_ARG;
    hive_status s = ensure_scratch(h, wl_need, dd_size ? b->n : 0, h->last);
    if (s != HIVE_OK) return s;
  }
  if (wl_need > h->wl_cap || dd_size > h->dd_cap) return HIVE_ERR_OOM;  // cannot happen after a good grow
  ReqDesc r;
  memset(&r, 0, sizeof(r));
  r.t = TableDesc{h->d_buckets,    batch_spill(h, b->op_mode, b->n), h->d_hint,  h->d_stash,   h->d_pending, h->d_ctl, h->d_wl, h->d_dd,
                  h->wl_seg_cap,  h->stash_cap,
                  h->pending_cap, hint_words(h->max_buckets), h->S, h->cfg.max_evictions, h->cfg.resize_k,
                  h->cfg.lf_expand_pct, h->cfg.lf_contract_pct, h->cfg.pre_expand, h->cfg.post_policy,
                  h->cfg.addressing};
  r.ops = b->d_ops;
  r.keys = b->d_keys;
  r.vals = b->d_vals;
  r.vals_out = b->d_vals_out;
  r.flags_out = b->d_flags_out;
  r.n = b->n;
  r.mode = b->op_mode;
  r.flags = b->flags;
  r.seq = d->next_seq[slot]++;
  r.table_slot = slot;
  r.ticket = t;
  if (dd_size && b->n <= DDS_EXEC_MAX) {
    // by hash ranges in LDS; the scratch (checked above for either form) holds
    // the winner flags
    r.dds = 1;
    while (((uint64_t)DDS_PER << (r.dds - 1)) < b->n) ++r.dds;
    dd_size = 0;
  }
  r.dd_size = dd_size;
  memcpy(&d->h_ring[t % d->cap], &r, sizeof(r));
  __atomic_thread_fence(__ATOMIC_RELEASE);
  __atomic_store_n(d->h_tail, t + 1, __ATOMIC_RELEASE);
  d->submitted = t + 1;
  *ticket = t;
  return HIVE_OK;
}

hive_status hive_drain_launch(hive_drain_t d, int resident, void *stream) {
  if (!d || d->running) return HIVE_ERR_ARG;
  const int mode = resident ? 1 : 0;
  // a resident grid that fills every CU leaves no room for the process's
  // other kernels (HIP's own copy kernels included), which the host may wait
  // on before its next submission: the grid then idles until its watchdog
  // (the resident grid takes at most fit_per_cu - 1 blocks per CU)
  if (resident && d->fit_per_cu < 2) {
    fprintf(stderr, "hive: a resident executor grid needs room for a second block per compute unit "
                    "(the worker fits %d per CU)\n", d->fit_per_cu);
    return HIVE_ERR_BUDGET;
  }
  hipStream_t user = (hipStream_t)stream;
  // a resident grid runs on the executor's own non-blocking stream, after the
  // work already enqueued on `stream`, so it holds up no other stream
  hipStream_t st = resident ? d->capture : user;
  if (resident) {
    hipEvent_t ev;
    HIP_OK(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
    HIP_OK(hipEventRecord(ev, user));
    HIP_OK(hipStreamWaitEvent(st, ev, 0));
    HIP_OK(hipEventDestroy(ev));
  }
  __atomic_store_n(d->h_stop, resident ? 0u : 1u, __ATOMIC_RELEASE);
  // the grid of the previous launch has exited; clear its exit flag
  hipLaunchKernelGGL(drain_reset_kernel, dim3(1), dim3(1), 0, st, d->d_q);
  HIP_OK(hipGetLastError());
  if (!d->exec[mode]) {
    // each launch form is captured once; replays read everything dynamic
    // from the queue in memory
    HIP_OK(hipStreamBeginCapture(d->capture, hipStreamCaptureModeRelaxed));
    launch_drain_any(d, mode, d->capture);
    hipError_t e = hipGetLastError();
    hipError_t e2 = hipStreamEndCapture(d->capture, &d->graph[mode]);
    if (e != hipSuccess || e2 != hipSuccess) {
      fprintf(stderr, "hive: drain graph capture failed: %s / %s\n", hipGetErrorString(e), hipGetErrorString(e2));
      return HIVE_ERR_HIP;
    }
    HIP_OK(hipGraphInstantiate(&d->exec[mode], d->graph[mode], nullptr, nullptr, 0));
  }
  HIP_OK(hipGraphLaunch(d->exec[mode], st));
  d->running = resident != 0;
  d->running_on = st;
  return HIVE_OK;
}

hive_status hive_drain_poll(hive_drain_t d, uint64_t ticket, int *done) {
  if (!d || !done || ticket >= d->submitted) return HIVE_ERR_ARG;
  if (d->submitted - ticket > d->cap) {
    *done = 1;  // its slot has been reused, so it completed long ago
    return HIVE_OK;
  }
  *done = __atomic_load_n(&d->h_done[ticket % d->cap], __ATOMIC_ACQUIRE) == ticket + 1;
  return HIVE_OK;
}

hive_status hive_drain_result(hive_drain_t d, uint64_t ticket, int *done, uint64_t *live_after) {
  if (!d || !done || !live_after || ticket >= d->submitted || d->submitted - ticket > d->cap) return HIVE_ERR_ARG;
  *done = __atomic_load_n(&d->h_done[ticket % d->cap], __ATOMIC_ACQUIRE) == ticket + 1;
  *live_after = *done ? __atomic_load_n(&d->h_live[ticket % d->cap], __ATOMIC_RELAXED) : 0;
  return HIVE_OK;
}

hive_status hive_drain_results(hive_drain_t d, const uint64_t *tickets, uint64_t n, uint8_t *done,
                               uint64_t *live_after) {
  if (!d || (n && (!tickets || !done || !live_after))) return HIVE_ERR_ARG;
  for (uint64_t i = 0; i < n; ++i)
    if (tickets[i] >= d->submitted || d->submitted - tickets[i] > d->cap) return HIVE_ERR_ARG;
  for (uint64_t i = 0; i < n; ++i) {
    const uint64_t t = tickets[i];
    done[i] = __atomic_load_n(&d->h_done[t % d->cap], __ATOMIC_ACQUIRE) == t + 1;
    live_after[i] = done[i] ? __atomic_load_n(&d->h_live[t % d->cap], __ATOMIC_RELAXED) : 0;
  }
  return HIVE_OK;
}

hive_status hive_drain_stop(hive_drain_t d, void *stream) {
  if (!d) return HIVE_ERR_ARG;
  (void)stream;
  __atomic_store_n(d->h_stop, 1u, __ATOMIC_RELEASE);
  d->running = false;
  HIP_OK(hipStreamSynchronize(d->running_on));
  uint32_t err = 0;
  HIP_OK(hipMemcpy(&err, (char *)d->d_q + offsetof(DrainQueue, error), 4, hipMemcpyDeviceToHost));
  return err ? HIVE_ERR_HIP : HIVE_OK;
}

hive_status hive_drain_destroy(hive_drain_t d) {
  if (!d) return HIVE_ERR_ARG;
  if (d->running) {
    __atomic_store_n(d->h_stop, 1u, __ATOMIC_RELEASE);
    (void)hipStreamSynchronize(d->running_on);
  }
  (void)hipDeviceSynchronize();
  free_drain(d);
  return HIVE_OK;
}

uint64_t hive_fastmod_magic(uint32_t d) { return fastmod_magic(d); }
uint32_t hive_fastmod(uint32_t a, uint64_t magic, uint32_t d) { return fastmod(a, magic, d); }

}  // extern "C"
