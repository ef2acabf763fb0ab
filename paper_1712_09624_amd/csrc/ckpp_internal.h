// ckpp_internal.h -- host-side table object and kernel launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ckpp.h"

struct ckpp_table {
  uint32_t log2_buckets;
  uint32_t max_kicks;
  uint32_t flags;
  int device;
  uint64_t seed;
  uint8_t *d_table;     // 256 * 2^B bytes: bucket b at 256 * b (ckpp_device.h)
  uint32_t path_lanes;  // lanes of the persistent insert grid
  uint32_t *d_own_paths;    // the table's own cuckoo-path scratch (own_paths
                            // arrays), allocated on the first insert
  uint32_t own_paths;
  uint8_t *d_bulk;      // bins of dense insert batches, if the table keeps them
  uint64_t bulk_bytes;  // their size, counted against device_mem
  uint64_t device_mem;  // the device's memory in bytes
  uint32_t *d_bulk_fill;  // records of each bin, zero between batches
  uint64_t *d_stats;    // device accumulator of ckpp_stats_t
  uint32_t retry_limit; // attempts per key on contended locks (ckpp_set_retry_limit)
  ckpp_launch_t lookup_launch;
  bool launch_set;      // a caller set lookup_launch (else batches take their own shape)
  int num_cus;
};

namespace ckpp {

// Words of one cuckoo-path array: max_kicks entries in whole groups of four.
inline __host__ __device__ uint32_t path_words(uint32_t max_kicks) {
  return max_kicks ? (max_kicks + 3u) / 4u * 4u : 4u;
}

// Insert batches take their cuckoo-path scratch (arrays of path_words words,
// shared by the lanes of a wavefront) from a buffer of the table's own, kept
// for its lifetime: the stream-ordered pool's allocate/free pair costs tens
// of microseconds of host time per batch, during which the device idles, and
// hundreds where the pool has given its memory back.  The buffer takes
// 1/kOwnPathShare of the table's own memory, at most kOwnPathsMax arrays and at
// least 4/3 of that memory (the bins of a dense batch that fills the table fit)
// between kOwnPathsLow and kOwnPathsMin arrays, 2 and 8 MB at 500 kicks, so that
// many small tables hold little.  Where the device has less memory left, the
// buffer is halved down to kOwnPathsLow.  Fewer arrays slow down batches that
// overfill a table, whose keys walk: 436,000 keys beyond load 0.95 of 2^20
// buckets 350 ms with 1/8, 610 with 1/32; 1.7M of 2^22 570 and 1020.
constexpr uint32_t kOwnPathsLow = 1024;
constexpr uint32_t kOwnPathsMin = 4096;
constexpr uint32_t kOwnPathsMax = 65536;
constexpr uint64_t kOwnPathShare = 8;
inline uint32_t own_paths(uint64_t table_bytes, uint32_t max_kicks) {
  const uint64_t fill = table_bytes / (4ull * path_words(max_kicks)), least = fill * 4u / 3u;
  const uint64_t low = least < kOwnPathsLow   ? kOwnPathsLow
                       : least < kOwnPathsMin ? least
                                              : kOwnPathsMin;
  const uint64_t share = fill / kOwnPathShare;
  return (uint32_t)(share < low ? low : share < kOwnPathsMax ? share : kOwnPathsMax);
}

// hipMalloc for a buffer that an insert finds it needs, which may be while
// another stream is captured: outside the relaxed mode it would fail and break
// that capture.  (The memory belongs to no graph.)
inline hipError_t malloc_beside_capture(void **p, size_t bytes) {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  hipError_t e = hipThreadExchangeStreamCaptureMode(&mode);
  if (e != hipSuccess) return e;
  e = hipMalloc(p, bytes);
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  return e;
}

// Dense insert batches (ckpp_bulk.hip).  Status of a key that waits for the
// second stage.
constexpr uint8_t kInsertPending = 0xffu;
// The batches that take that way hold at least kMinBulkKeys keys and, per
// bucket of the table, one on 2^20 buckets and more, two on fewer.  Measured
// on MI355X, this way and key by key, in us, at the line and beside it.  From
// 2^20 buckets on it is faster from every load: one key per bucket, 2^20
// buckets 131 and 185 from empty, 165 and 223 from load 0.5, 305 and 347 from
// 0.8; 2^22 585 and 652, 715 and 776, 1175 and 1223; 2^24 2164 and 2521, 2621
// and 2909, 4273 and 4411; one and a half from 0.8 (to 0.99) 1419 and 1524,
// 3766 and 3900, 12154 and 12993; half a key, 2^22 383 and 338 from empty.
// Below, two keys per bucket: 2^12 17.8 and 22.4 from empty, 34 and 40 from
// 0.5, 76 and 83 from 0.7; 2^14 21.5 and 24.4, 41 and 46, 85 and 111; 2^16 29
// and 34, 55 and 54, 130 and 121; 2^18 70 and 69, 95 and 104, 206 and 204: 6%
// faster on average over 2^11..2^19 buckets and those loads, single points from
// 24% faster to 9% slower.  Fewer keys lose there from load 0.5 on: one and a
// half, 2^16 21 and 27 from empty, 54 and 45; one, 2^18 36 and 39, 61 and 57.
// Tables of more than 2^24 buckets would need bins of more than 2^10 buckets,
// which was not measured.
constexpr uint64_t kMinBulkKeys = 4096;
constexpr uint32_t kMaxBulkLog2Buckets = 24;
constexpr uint32_t kMaxBulkLog2Bins = 14;  // their counters in LDS: 64 KiB
constexpr uint32_t kMaxBulkBins = 1u << kMaxBulkLog2Bins;
inline uint64_t min_bulk_keys(uint32_t log2b) {
  const uint64_t n = (log2b < 20u ? 2ull : 1ull) << log2b;
  return n < kMinBulkKeys ? kMinBulkKeys : n;
}
// The bins' memory: 5/8 of the table's own, in which a full table's keys fit
// in two chunks with their slack, and no less than this.  A batch in more chunks
// reads and writes the buckets' heads once per chunk (2^24 buckets at load
// 0.9 with 0.5, 1.25 and 2.5 GiB: 21.7, 18.2 and 15.5 ms).
constexpr uint64_t kMinBulkBytes = 1ull << 20;
// Tables keep their bins while those of all tables of a device stay within
// 1/kBulkShare of its memory (4.5 GiB on MI355X).  A batch beyond that takes
// its bins from the stream-ordered pool and gives them back on its stream,
// which costs a caller that waits for every batch about 300 us for 160 MiB to
// 640 MiB and 620 us for 2.5 GiB (the pool returns its memory when the device
// is idle), so only batches that save more than that do: of 2^23 keys and two
// keys per bucket (2^21 buckets, 4 per bucket: 824 us and 1430 key by key; 2^22,
// 2: 920 and 1294; 2^23, 1: 1108 and 1231, 2: 1736 and 2472).
constexpr uint64_t kBulkShare = 64;
inline uint64_t min_pooled_bulk_keys(uint32_t log2b) {
  const uint64_t n = 2ull << log2b;
  return n < (1ull << 23) ? 1ull << 23 : n;
}

// One work item of a plan: lookups [start, start + count) of the
// concatenated key batch, all of one table, with that table's parameters
// (so a wave needs a single descriptor load per item).
struct PlanItem {
  const uint4 *tab;  // the table's buckets
  uint64_t seed;     // its hash seed
  uint64_t start;
  uint32_t count;
  uint32_t log2b;    // log2 of its bucket count
  uint32_t mode;     // kMode* of its lookups
  uint32_t table;    // index of the table in the plan
};

// Largest table: 2^29 buckets (128 GiB, 2^32 slots); bucket indices fit in
// 29 bits.
constexpr uint32_t kMaxLog2Buckets = 29;

// Attempts an insert or delete makes on contended bucket locks before it
// gives up with CKPP_RETRY: the default and largest retry limit.
constexpr uint32_t kMaxRetryLimit = 1u << 20;

constexpr uint32_t kModeCuckoopp = 0;
constexpr uint32_t kModeBoth = 1;
constexpr uint32_t kModeOptimistic = 2;
// PlanItem::mode: the lookup mode in the low byte, and this flag on a table
// with timers.
constexpr uint32_t kPlanModeMask = 0xffu;
constexpr uint32_t kPlanItemTimed = 0x100u;

// Blocks of a launch over n items, per_block items per block: at most
// blocks_per_cu per compute unit (0: no cap) and at most 2^31 - 1.
inline uint64_t capped_grid(uint64_t n, uint64_t per_block, uint32_t blocks_per_cu, int num_cus) {
  uint64_t grid = (n + per_block - 1) / per_block;
  if (blocks_per_cu) {
    const uint64_t cap = (uint64_t)blocks_per_cu * (uint64_t)num_cus;
    if (grid > cap) grid = cap;
  }
  return grid > 0x7fffffffull ? 0x7fffffffull : grid;
}

// A refreshing lookup's new expiration time lies in [now, now + 1023] mod
// 2^16, so the entry it writes is alive at `now` (Sec. 4.2).
inline bool in_window(uint32_t expiry, uint32_t now) { return ((expiry - now) & 0xffffu) < 1024u; }

// Timers of a batch on a table with timers (Sec. 4.2): the current time;
// for lookups, whether a hit sets the entry's expiration time to `expiry`.
struct TimerArgs {
  uint32_t now;
  uint32_t refresh;
  uint32_t expiry;
};

// timers: null on a table without timers.
hipError_t launch_lookup(const ckpp_table *t, const void *d_keys, uint64_t n, uint32_t mode,
                         const TimerArgs *timers, uint8_t *d_found, uint64_t *d_values,
                         hipStream_t s);
// One launch of the plan's persistent lookup kernel over its items.
// d_ctr: two u32 counters (next item, finished waves), zero before the
// launch and zero again after it.  two_buffers: some table uses the
// pessimistic mode.  timers: the launch's time, for the items flagged
// kPlanItemTimed (null: no item is).
hipError_t launch_plan(const PlanItem *d_items, uint32_t nitems, uint32_t *d_ctr, bool two_buffers,
                       const TimerArgs *timers, const ckpp_plan_launch_t &L, int num_cus,
                       const void *d_keys, uint8_t *d_found, uint64_t *d_values, hipStream_t s);
// d_expiry and timers: null on a table without timers.
hipError_t launch_insert(const ckpp_table *t, const void *d_keys, const uint64_t *d_values,
                         const uint16_t *d_expiry, const TimerArgs *timers, uint64_t n,
                         uint8_t *d_status, uint64_t *d_nfailed, hipStream_t s);
// The first stage of a dense batch: places the keys that their primary bucket
// decides, writes every key's status (kInsertPending for the others).  *taken:
// whether the batch is one for this way (else nothing was done).
hipError_t bulk_insert_primary(ckpp_table *t, const void *d_keys, const uint64_t *d_values,
                               const uint16_t *d_expiry, const TimerArgs *timers, uint64_t n,
                               uint8_t *d_status, hipStream_t s, bool *taken);
// Bins of the dense batches of a table of 2^log2b buckets (0: it takes none).
uint32_t bulk_bins(uint32_t log2b);
// Frees the table's bins (nothing runs on the table).
void bulk_free(ckpp_table *t);
hipError_t launch_delete(const ckpp_table *t, const void *d_keys, uint64_t n,
                         const TimerArgs *timers, uint8_t *d_found, hipStream_t s);
// The insert without any allocation (ckpp_insert_batch_noalloc): returns a
// CKPP_* status.
int insert_noalloc(const ckpp_table *t, const void *d_keys, const uint64_t *d_values, uint64_t n,
                   uint8_t *d_status, uint64_t *d_nfailed, hipStream_t s);
// Removes every entry expired at `now` (one pass over the table).
hipError_t launch_expire_scan(const ckpp_table *t, uint32_t now, uint64_t *d_removed,
                              hipStream_t s);
hipError_t launch_stats(const ckpp_table *t, uint64_t *d_acc, hipStream_t s);
hipError_t launch_hash(const ckpp_table *t, const void *d_keys, uint64_t n, uint64_t *d_hash,
                       hipStream_t s);
hipError_t launch_fill_zero(void *d, uint64_t bytes, hipStream_t s);
// The dependent-access latency probe (ckpp_probe_latency).
hipError_t launch_latency(void *d_buf, uint64_t bytes, uint32_t kind, uint32_t steps,
                          uint64_t seed, uint64_t *d_out, hipStream_t s);
hipError_t launch_probe(const void *d_buf, uint64_t bytes, uint32_t granule, uint64_t nreads,
                        uint32_t per_lane, uint32_t cooperative, uint32_t block, uint32_t grid,
                        uint64_t seed, uint64_t *d_sink, hipStream_t s);

// Makes a device current for the duration of a call.
class DeviceGuard {
 public:
  explicit DeviceGuard(int dev) : prev_(-1), ok_(true) {
    if (hipGetDevice(&prev_) != hipSuccess) prev_ = -1;
    if (prev_ != dev) ok_ = hipSetDevice(dev) == hipSuccess;
    else prev_ = -1;
  }
  ~DeviceGuard() {
    if (prev_ >= 0) (void)hipSetDevice(prev_);
  }
  bool ok() const { return ok_; }

 private:
  int prev_;
  bool ok_;
};

inline int dev_status(hipError_t e) {
  if (e == hipSuccess) return CKPP_OK;
  return e == hipErrorOutOfMemory ? CKPP_ENOMEM : CKPP_EDEVICE;
}

}  // namespace ckpp
