// Launch interface between the host table manager and the HIP kernels.
#pragma once

#include <algorithm>
#include <atomic>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mlkv_device.h"

namespace mlkv {

constexpr int kGetTile = 256;    // keys per get_probe block at most (one per lane)
constexpr int kGetTileMin = 64;  // ... and at least, unless the batch is smaller

// Positions per get_probe block for a batch of n keys on a device of
// `cus` compute units: the blocks come in whole rounds of one per CU, with
// equal tiles, so that no CU runs a block more than another.
inline int get_tile_len(int64_t n, int cus) {
  const int64_t per_round = (int64_t)kGetTile * cus;
  const int64_t rounds = (n + per_round - 1) / per_round;
  int64_t t = (n + rounds * cus - 1) / (rounds * cus);
  if (t < kGetTileMin) t = kGetTileMin;
  if (t > kGetTile) t = kGetTile;
  return (int)t;
}
constexpr int kPutTile = 1024;   // keys per put_probe block
constexpr int kPutThreads = 1024; // threads of a put_probe block
constexpr int kMaxParts = 4096;  // partitions (MSD digits) per put call
constexpr int kRedCap = 3072;    // partition items grouped in LDS by a put_group block
constexpr int kRedHash = 4096;   // LDS hash slots for that grouping (load <= 0.75)
constexpr int kPartTarget = 1024; // put keys per partition the partition count aims for
// A key repeated this often in a put_probe tile is summed there (twice, where
// rows have at most 32 floats). A key seen twice costs a row of fp64 written and
// read in place of its two fp32 rows: from 3 repeats on, two DLRM steps (dim 64)
// take 185.0 us against 187.8, two of 1M lookups at dim 128 1241 against 1244;
// two of 131k at dim 32 take 126.5 against 125.6. From 4 on hot keys cost more:
// 189.3 at dim 64.
constexpr int kPresumMinWide = 3;

// Error code a kernel latches when a put whose probe ran ahead of a get met a
// key that was not in the table before the two calls (reported as MLKV_EINVAL).
constexpr int kErrAbsent = -5;

// Kernels of the library, for per-launch timing.
enum KernelId : int {
  K_GET_PROBE = 0,
  K_GET_ROWS = 1,
  K_PUT_PROBE = 2,
  K_PUT_REDUCE = 3,    // put_group and put_apply
  K_TIER_MARK = 4,
  K_TIER_PLAN = 5,
  K_TIER_COPY = 6,
  K_RSORT_COUNT = 7,
  K_RSORT_SCATTER = 8,
  K_RSORT_REDUCE = 9,  // rsort_group and put_apply
  K_COUNT = 10
};

// How a put finds the equal keys of its batch.
enum Dedup : int {
  kDedupHash = 0,   // hash partition of the items, grouping in LDS per partition
  kDedupRadix = 1   // stable LSD radix sort of the items by row, run-length encoding
};
constexpr int kRsTile = 4096;    // items per radix-sort block (four put tiles)
constexpr int kRsMaxBits = 9;    // bits per radix pass at most
constexpr int kRsChunk = 2048;   // sorted items per radix reduce block at most, before the cut moves to a run start
constexpr int64_t kRsMaxKeys = 1 << 20;  // keys per put call with radix dedup

// Update a put call applies to each distinct key's row.
enum PutOp : int {
  kOpAdagrad = 0,  // sum the key's gradient rows, one row-wise Adagrad step
  kOpSgd = 1,      // sum the key's gradient rows, one SGD step
  kOpAssign = 2    // the value row at the key's last position replaces the row
};


// Optional callback around each launch (phase 0 before, 1 after), on the launch stream.
struct LaunchHook {
  void (*fn)(void* ctx, int kernel, int phase, hipStream_t st) = nullptr;
  void* ctx = nullptr;
  void operator()(int kernel, int phase, hipStream_t st) const {
    if (fn) fn(ctx, kernel, phase, st);
  }
};

// A get call's new keys filed by key range as the probe kernel inserts them,
// with the cut points the last ranking by key ranges left (the keys of
// global ranks floor(j M / G), j = 1 .. G - 1, of a call that inserted M keys
// with G ranges): range q holds the keys in [cut q-1, cut q). Row assignment
// then takes each range's keys from its list instead of searching every
// tile's list. The cut points serve a call with the same G; any sorted set of
// them is correct, the last call's keep the ranges about even.
constexpr int kMaxRanges = 512;  // ranges of a get call at most (its row-assignment blocks)
struct RangeLists {
  NewKey* list = nullptr;      // [entries]: range q's keys from q * cap on; nullptr: no lists
  uint64_t entries = 0;
  uint32_t cap = 0;            // entries per range (set at launch: entries / ranges)
  uint32_t* cnt = nullptr;     // [kMaxRanges] this call's counts per range (zero before it)
  uint32_t* cnt_next = nullptr;  // [kMaxRanges] the next call's counts, cleared by this call
  uint64_t* cuts = nullptr;    // [kMaxRanges - 1] the cut points
  uint32_t* cuts_g = nullptr;  // the number of ranges the cut points are for (0: none)
};

struct GetArgs {
  Bucket* idx;
  uint32_t nb_log2;
  const uint64_t* keys;
  int64_t n;
  float* out;
  RowStore store;
  float* state;
  int D;
  uint64_t seed;
  int64_t capacity;
  NewKey* newlist;
  uint32_t* tile_cnt;
  Ctrl* ctrl;
  uint64_t epoch;
  uint64_t* xkey;   // [n] scratch: new keys of a key range too large for LDS
  uint32_t* xslot;  // [n] their index slots
  // staleness bound (nullptr clock: not tracked): per-row words of
  // (get-call epoch << kClockBits) | count, this call's epoch, the bound, and
  // the per-position blocked flags the call writes
  unsigned long long* clock;
  uint64_t cepoch;
  uint32_t bound;
  uint8_t* blocked;
  // per position: the key found present (the empty key where the position
  // held no present key); with its row below, a later put reads it. nullptr:
  // not recorded
  uint64_t* pc_key;
  uint32_t* pos_row;  // per position: its key's row, kPendingRow for a key new in the call
  // 1: a position whose key equals pc_key[i] takes pos_row[i] without probing
  // (a present key's row never changes, so any recorded pair stays true);
  // not with a staleness clock
  int pc_in;
  RangeLists rl;
  int cus;  // compute units of the device
};

// What the second get kernel copies out, and the new keys its first blocks
// assign rows to.
struct GetRowsArgs {
  float* out;  // nullptr: nothing is copied
  const uint64_t* keys;
  const uint32_t* rows;  // per position (kPendingRow: the key is new in the call)
  const uint8_t* blocked;
  int64_t n;
  uint64_t seed;
  RowStore store;
  uint32_t magic;  // ceil(2^32 / units of 16 bytes per row)
};
struct AssignArgs {
  Bucket* idx;
  const NewKey* newlist;
  const uint32_t* tile_cnt;
  int ntiles;
  int tile_size;
  float* state;
  int64_t capacity;
  Ctrl* ctrl;
  uint64_t epoch;
  uint64_t* xkey;
  uint32_t* xslot;
  unsigned long long* clock;
  uint64_t cepoch;
  RangeLists rl;
  const float* values;  // an upsert's value rows (the new rows are written from them), else nullptr
  uint32_t blocks;  // blocks that assign rows (the key ranges)
};

// The update of a put call as units, one per distinct key (see k_put_group).
// Items of a unit that one lane group adds up, at most; a block takes longer
// ones. Rows of up to 32 floats have 32 lane groups in a block and more: 13.7
// us against 15.7 with 16 (131k lookups, dim 32), 10.5 against 12.4 (dim 10);
// at dim 128 a block has 8, and 8 items are 363 us against 340 with 16 (32:
// 344; dim 64, 213k lookups: 34 us against 29).
constexpr uint32_t kLongNarrow = 8, kLongWide = 16;
constexpr uint32_t kUnitFresh = 1u << 31;   // the unit's tag is an index slot (a key new in the call)
struct PutUnits {
  uint64_t* single;  // [n] keys with one gradient (or value) row: the item
  uint4* multi;      // [n] keys with a sum of at most long_over items: {tag, items | kUnitFresh, first item, 0}
  uint4* lng;        // [n / kLongNarrow] keys with a longer one
  uint32_t* mitem;   // [n] their items (the low 31 bits)
  uint32_t long_over;
};

struct PutGroupArgs {
  const uint64_t* items;
  const uint32_t* meta;
  int ntiles;
  uint32_t parts;  // partitions
  PutUnits units;
  Ctrl* ctrl;
  uint64_t epoch;
  int64_t capacity;
  uint64_t* spill;
  uint64_t spill_words;
  // an upsert:
  const float* values;
  unsigned long long* clock;
  uint32_t magic;  // ceil(2^32 / units of 16 bytes per row)
};

struct PutApplyArgs {
  const Bucket* idx;
  const float* grads;
  const double* partials;
  PutUnits units;
  const Ctrl* ctrl;
  float* state;
  unsigned long long* clock;
  int op;
  float lr;
  float eps;
};

struct PutArgs {
  Bucket* idx;
  uint32_t nb_log2;
  const uint64_t* keys;
  const float* grads;
  int64_t n;
  RowStore store;
  float* state;
  int D;
  uint64_t seed;
  int64_t capacity;
  float lr;
  float eps;
  int op;     // PutOp
  int pb;     // 2^pb partitions
  int tlen;   // keys per put_probe tile (<= kPutTile)
  uint64_t* items;
  double* partials;  // [n][D] fp64 sums of keys repeated within a tile
  uint32_t* meta;
  NewKey* newlist;
  uint32_t* tile_cnt;
  uint64_t* spill;
  uint64_t spill_words;
  PutUnits units;
  uint64_t* xkey;   // as for a get (GetArgs)
  uint32_t* xslot;
  Ctrl* ctrl;
  uint64_t epoch;
  unsigned long long* clock;  // per-row staleness words, or nullptr when not tracked
  const uint64_t* pc_key;     // the last get's present keys and rows by position
  const uint32_t* pc_row;
  int dedup;                  // Dedup
  int cus;                    // compute units (radix reduce blocks at least)
  int rs_bits;                // radix dedup: bits of the sort key (rows below capacity, new keys' slots above)
  uint64_t* rs_buf;           // radix dedup: two n-item ping-pong buffers
  uint32_t* rs_cnt;           // radix dedup: per-tile digit counts, then the item total
  // 1: the put's probe kernel runs ahead of the kernels of a get whose epoch
  // is this one's less one, its other kernels after them (the probe inserts
  // nothing: a key absent from the table before that get fails the put; it
  // writes no new-key list or tile counts, which are the get's, and marks its
  // errors in the control block's fields for such puts)
  int ahead = 0;
};

// Which kernels of a put launch_put queues: all of them, only the probe
// kernel, or the kernels after it.
enum PutPhase : int { kPutAll = 0, kPutProbe = 1, kPutAfterProbe = 2 };

// Lookahead of a tiered table, after the get kernels have resolved its n keys.
struct TierArgs {
  Bucket* idx;
  uint32_t nb_log2;
  const uint64_t* keys;
  const uint64_t* pc_key;  // the get's present keys and rows by position
  const uint32_t* pc_row;
  int64_t n;
  uint32_t* slot_of_row;  // [capacity]
  uint32_t* row_of_slot;  // [cache_rows]
  uint8_t* dirty;         // [cache_rows]
  uint32_t* keep;         // [cache_rows]
  uint32_t tag;           // this lookahead call (never 0)
  uint32_t parity;        // ping-pong index of the miss counter
  uint32_t* miss;         // [n] scratch
  uint32_t* plan_slot;    // [n] scratch
  int64_t cache_rows;
  float* cache;
  float* host;
  int D;
  Ctrl* ctrl;
};

// Row maps: lanes that cover a row, four floats each (one float each for rows
// shorter than that), at any alignment. A map of one float per lane and a
// whole wave per row, which widths that are no multiple of four (and buffers
// off 16 bytes) took before, left most lanes idle: two steps of 106,496
// lookups at dim 10 took 849 us and take 137. Not fewer than four lanes, though
// rows of dim 4 leave three of them idle: with one, a block has 1024 lane groups
// for the in-tile sums of hot keys and a wave holds 64 sums of different
// lengths. Put of 4096 / 65k / 194k / 1M lookups at dim 4 (Zipf 1.1) with four
// lanes, two and one: 29 / 37 / 46 / 154 us, 31 / 40 / 48 / 154 and 34 / 44 / 50
// / 155; uniform keys 22 / 29 / 44 / 166, 23 / 29 / 44 / 168 and 22 / 29 / 44 / 165.
using MapD3 = RowMap<1, 4, 1>;      // dim <= 3
using MapD16 = RowMap<4, 4, 1>;     // dim <= 16
using MapD32 = RowMap<4, 8, 1>;     // dim <= 32
using MapD64 = RowMap<4, 16, 1>;    // dim <= 64
using MapD128 = RowMap<4, 32, 1>;   // dim <= 128
using MapD256 = RowMap<4, 64, 1>;   // dim <= 256
using MapD512 = RowMap<4, 64, 2>;   // dim <= 512
using MapD1024 = RowMap<4, 64, 4>;  // dim <= 1024
#define MLKV_MAPS(F) F(MapD3) F(MapD16) F(MapD32) F(MapD64) F(MapD128) F(MapD256) F(MapD512) F(MapD1024)

// The items a radix tile reads. First pass: put_probe's items, tile t being
// put tiles 4t .. 4t+3, kPutTile slots each, the first (meta >> 16) of them
// used. Later passes: the dense output of the previous pass.
struct RsSrc {
  const uint64_t* src;
  const uint32_t* meta;   // first pass only
  int ntiles;             // put tiles
  const uint32_t* total;  // later passes: items in all
};

hipError_t launch_rsort_pass(const RsSrc& src, uint32_t cap, int shift, int bits, uint32_t* cnt, int rtiles,
                             int stride, uint64_t* dst, uint32_t* total_out, hipStream_t st,
                             const LaunchHook& hook);
// Loads the code that tables of dim D run (load_tier_code: of tiered tables) on
// the current device, where a process has not done so yet. The library has a
// code object for each row map; the runtime otherwise loads one at the first
// launch from it: a first put took 0.7 ms instead of 0.1, and one under stream
// capture would load (and allocate) there.
hipError_t load_code(int D);
hipError_t load_tier_code();
// Loads the code object of `kernel` on the current device, unless `on` (a bit
// for each of the first 64 devices) says that was done.
inline hipError_t load_once(std::atomic<uint64_t>& on, const void* kernel) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0ull;
  if ((on.load(std::memory_order_relaxed) & bit) != 0) return hipSuccess;
  hipFuncAttributes f;
  e = hipFuncGetAttributes(&f, kernel);
  if (e == hipSuccess) on.fetch_or(bit, std::memory_order_relaxed);
  return e;
}
template <class M>
hipError_t load_map_code();
template <class M>
hipError_t launch_put_probe_t(const PutArgs& a, int pb, hipStream_t st, const LaunchHook& hook);
template <class M>
hipError_t launch_put_apply_t(const PutArgs& a, const PutApplyArgs& u, hipStream_t st);
hipError_t launch_get(const GetArgs& a, hipStream_t st, const LaunchHook& hook);
hipError_t launch_tier_lookahead(const TierArgs& a, hipStream_t st, const LaunchHook& hook);
hipError_t launch_put(const PutArgs& a, hipStream_t st, const LaunchHook& hook, int phase = kPutAll);
hipError_t launch_lookup(Bucket* idx, uint32_t nb_log2, const uint64_t* keys, int64_t n,
                         int64_t* rows_out, hipStream_t st);
hipError_t launch_export_slots(const Bucket* idx, uint64_t nslots, uint64_t* keys_out,
                               uint32_t* rows_out, hipStream_t st);
hipError_t launch_read_clock(const unsigned long long* clock, const unsigned long long* size_now,
                             const int64_t* ids, int64_t n, uint32_t* out, Ctrl* ctrl, hipStream_t st);
hipError_t launch_read_rows(const RowStore& store, const float* state, int D, const unsigned long long* size_now,
                            const int64_t* ids, int64_t n, float* w_out, float* st_out, Ctrl* ctrl,
                            hipStream_t st);
hipError_t launch_export_rows(const RowStore& store, int64_t nrows, int D, float* out, hipStream_t st);

}  // namespace mlkv
