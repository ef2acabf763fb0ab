// ckpp_bulk.hip -- the first stage of a dense insert batch (gfx950): keys
// that their primary bucket alone decides, placed by blocks that own whole
// ranges of buckets.
//
// A key placed on its own costs about seven memory requests (its bucket's
// lock, head, key, value, tag, other bucket, metadata), each coherent across
// the XCDs, and the rate of requests bounds the batch.  When a batch holds
// keys for most buckets it is cheaper to bring the keys to the buckets: one
// pass writes every key into the bin of its primary bucket's range, and then
// one block per bin takes the heads of its buckets (tags, filter, metadata)
// into LDS, places the bin's keys there with LDS atomics, and writes the
// heads back.  No other block touches those buckets, so nothing is locked,
// the accesses are plain cached ones, and a bucket's stores meet in the L2
// cache.  A key that needs more than its primary (the filter passes, or no
// slot is free) is marked kInsertPending in its status, and the caller's
// second stage runs its state machine (insert_marked).
//
// Entries that are in a bucket when its block starts (the busy mask `first`)
// keep their slots throughout, so a key is compared with those entries, and
// slots are claimed by a compare-and-swap on the metadata word in LDS.  A key
// that meets its own tag in a slot taken since the start waits for the second
// stage: a batch that breaks the rule of distinct keys leaves one entry of
// each, as a batch taken key by key does.
//
// Measured on MI355X, 31.9M keys into 2^22 buckets (to load 0.95) in one call:
// 6.9 ms key by key; this way 1.1 ms for the bins (2.0 TB/s of keys, values
// and records), 1.2 ms for their blocks, 2.1 ms for the 4M keys of the second
// stage.

#include <atomic>

#include "ckpp_device.h"
#include "ckpp_internal.h"

namespace ckpp {
namespace {

constexpr uint32_t kBulkBlock = 1024;
constexpr uint32_t kMaxBinShift = 8;        // buckets of a bin, unless the bins get too many
constexpr uint32_t kMinBinShift = 5;
constexpr uint32_t kSkip = 0xffffffffu;     // a record that holds no key

// A key in its bin: 32 bytes, two quarters.
//   0: the key   1: value word | index in the chunk | (unused)
struct BulkArgs {
  uint8_t *bk;
  const uint4 *keys;
  const uint64_t *vals;
  const uint16_t *expiry;  // TIMED
  uint8_t *status;
  uint32_t n;              // keys of the chunk
  uint32_t now, log2b, shift, bins, cap;
  uint64_t seed;
  uint4 *recs;             // bins x cap records
  uint32_t *fill;          // records of each bin; zero between batches
};

// Keys into bins, kBulkBlock * KPT per block: the block counts its keys of
// every bin in LDS, takes that many records of the bin with one atomic, and
// writes its keys there.  Keys that find their bin full are marked.
template <bool TIMED, uint32_t KPT>
__global__ void __launch_bounds__(kBulkBlock) bulk_scatter(BulkArgs A) {
  __shared__ uint32_t s_bin[kMaxBulkBins];
  for (uint32_t b = threadIdx.x; b < A.bins; b += kBulkBlock) s_bin[b] = 0u;
  __syncthreads();
  const uint32_t i0 = blockIdx.x * (kBulkBlock * KPT) + threadIdx.x;
  uint32_t at[KPT];  // bin << 16 | rank among the block's keys of the bin
#pragma unroll
  for (uint32_t k = 0; k < KPT; ++k) {
    const uint32_t i = i0 + k * kBulkBlock;
    at[k] = 0u;
    if (i < A.n) {
      const uint32_t bin = key_fields(key_hash(A.keys[i], A.seed), A.log2b).p >> A.shift;
      at[k] = bin << 16 | atomicAdd(&s_bin[bin], 1u);
    }
  }
  __syncthreads();
  for (uint32_t b = threadIdx.x; b < A.bins; b += kBulkBlock) {
    const uint32_t c = s_bin[b];
    if (c) s_bin[b] = atomicAdd(&A.fill[b], c);
  }
  __syncthreads();
#pragma unroll
  for (uint32_t k = 0; k < KPT; ++k) {
    const uint32_t i = i0 + k * kBulkBlock;
    if (i >= A.n) continue;
    const uint32_t bin = at[k] >> 16, r = s_bin[bin] + (at[k] & 0xffffu);
    if (r >= A.cap) {
      A.status[i] = kInsertPending;
      continue;
    }
    const uint64_t value = A.vals[i];
    // a value too wide for a table with timers fails: the second stage says so
    const bool wide = TIMED && (value >> kTimerShift) != 0ull;
    const uint64_t word = TIMED ? value | ((uint64_t)A.expiry[i] << kTimerShift) : value;
    uint4 *rec = A.recs + 2ull * ((uint64_t)bin * A.cap + r);
    rec[0] = A.keys[i];
    rec[1] = make_uint4((uint32_t)word, (uint32_t)(word >> 32), wide ? kSkip : i, 0u);
    A.status[i] = wide ? kInsertPending : (uint8_t)CKPP_INSERTED;
  }
}

// One block per bin: places the bin's keys.  LDS: the heads of the bin's
// buckets, whose lock word (zero in memory) holds the busy mask the block
// started with.
template <bool TIMED>
__global__ void __launch_bounds__(kBulkBlock) bulk_place(BulkArgs A) {
  extern __shared__ uint4 s_head[];  // two quarters per bucket
  const uint32_t nb = 1u << A.shift, b0 = blockIdx.x << A.shift;
  uint4 *tab = reinterpret_cast<uint4 *>(A.bk);
  for (uint32_t q = threadIdx.x; q < 2u * nb; q += kBulkBlock) {
    uint4 v = tab[(uint64_t)(b0 + (q >> 1)) * kQuartersPerBucket + (q & 1u)];
    if (q & 1u) v.w = meta_busy(v.z);
    s_head[q] = v;
  }
  const uint32_t held = A.fill[blockIdx.x];
  const uint32_t count = held < A.cap ? held : A.cap;
  __syncthreads();
  if (threadIdx.x == 0u) A.fill[blockIdx.x] = 0u;
  const uint4 *recs = A.recs + 2ull * blockIdx.x * A.cap;
  for (uint32_t r = threadIdx.x; r < count; r += kBulkBlock) {
    const uint4 key = recs[2u * r], rest = recs[2u * r + 1u];
    const uint32_t i = rest.z;
    if (i == kSkip) continue;
    const uint64_t word = (uint64_t)rest.x | ((uint64_t)rest.y << 32);
    const KeyFields f = key_fields(key_hash(key, A.seed), A.log2b);
    const uint32_t lb = f.p - b0;
    uint8_t *bucket = A.bk + (uint64_t)f.p * kBucketBytes;
    const uint4 q1 = s_head[2u * lb + 1u];
    uint32_t cand = tag_eq_mask(s_head[2u * lb], f.tag) & q1.w;
    bool done = false;
    while (cand != 0u && !done) {
      const uint32_t s = (uint32_t)__builtin_ctz(cand);
      cand &= cand - 1u;
      if (key_eq(*reinterpret_cast<const uint4 *>(bucket + key_offset(s)), key)) {
        uint64_t *w = reinterpret_cast<uint64_t *>(bucket + value_offset(s));
        if (!TIMED || word_alive(*w, A.now)) A.status[i] = (uint8_t)CKPP_UPDATED;
        *w = word;
        done = true;
      }
    }
    if (done) continue;
    uint32_t fs = kSlots;
    if (!bloom_pass(q1, f.bloom_bits)) {
      uint32_t *meta = &s_head[2u * lb + 1u].z;
      uint32_t m = *meta;
      while (meta_busy(m) != 0xffu) {
        const uint32_t s = (uint32_t)__builtin_ctz(~meta_busy(m));
        const uint32_t old = atomicCAS(meta, m, m | (1u << (16u + s)));
        if (old == m) {
          fs = s;
          break;
        }
        m = old;
      }
    }
    if (fs != kSlots) {
      // its tag, and then a look at the other slots taken since the start: of
      // two copies of one key, the later to write its tag sees the other's,
      // gives its slot back and waits for the second stage, which finds the
      // key (so do different keys with one tag, one pair in 65,536)
      volatile uint32_t *head = reinterpret_cast<volatile uint32_t *>(&s_head[2u * lb]);
      reinterpret_cast<volatile uint16_t *>(head)[fs] = (uint16_t)f.tag;
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup", "local");
      const uint4 tags = make_uint4(head[0], head[1], head[2], head[3]);
      const uint32_t taken = meta_busy(head[6]) & ~q1.w & ~(1u << fs);
      if (tag_eq_mask(tags, f.tag) & taken) {
        atomicAnd(&s_head[2u * lb + 1u].z, ~(1u << (16u + fs)));
        fs = kSlots;
      }
    }
    if (fs == kSlots) {
      A.status[i] = kInsertPending;
      continue;
    }
    *reinterpret_cast<uint4 *>(bucket + key_offset(fs)) = key;
    *reinterpret_cast<uint64_t *>(bucket + value_offset(fs)) = word;
    reinterpret_cast<uint32_t *>(bucket + kOtherOffset)[fs] = f.a;
  }
  __syncthreads();
  for (uint32_t q = threadIdx.x; q < 2u * nb; q += kBulkBlock) {
    uint4 v = s_head[q];
    const uint4 h = s_head[q | 1u];
    if (meta_busy(h.z) == h.w) continue;  // nothing was placed
    if (q & 1u) v.w = 0u;
    tab[(uint64_t)(b0 + (q >> 1)) * kQuartersPerBucket + (q & 1u)] = v;
  }
}

template <bool TIMED>
hipError_t launch_bulk(const BulkArgs &A, hipStream_t s) {
  // more keys per thread mean fewer atomics on the bins and longer runs of a
  // bin's records, but fewer blocks: as many as leave every compute unit one
  // (16M keys into 2048 bins: 508 us with 8, 537 with 16, 584 with 32; into
  // 16384 bins 560 with 8, 16 and 32 not timed)
  const dim3 b(kBulkBlock);
  const auto blocks = [&](uint32_t kpt) {
    return dim3((A.n + kBulkBlock * kpt - 1u) / (kBulkBlock * kpt));
  };
  if (A.n >= 256u * 8u * kBulkBlock)
    hipLaunchKernelGGL((bulk_scatter<TIMED, 8>), blocks(8), b, 0, s, A);
  else if (A.n >= 256u * 2u * kBulkBlock)
    hipLaunchKernelGGL((bulk_scatter<TIMED, 2>), blocks(2), b, 0, s, A);
  else
    hipLaunchKernelGGL((bulk_scatter<TIMED, 1>), blocks(1), b, 0, s, A);
  const uint32_t lds = (2u * (uint32_t)sizeof(uint4)) << A.shift;
  hipLaunchKernelGGL(bulk_place<TIMED>, dim3(A.bins), b, lds, s, A);
  return hipGetLastError();
}

// Buckets per bin: enough bins for two blocks on every compute unit, and at
// most 2^8 buckets, 64 KiB of the table per block, so that the three stores
// of a key meet in the L2 cache before its lines leave it (2^11 per bin,
// 512 KiB, and 2^8: 8M keys into 2^20 buckets 1.49 and 1.36 ms, half of them
// 447 and 356 us; 31.9M into 2^22 5.09 and 4.62), but no more than
// kMaxBulkBins bins (2^24 buckets at load 0.9 in 8192 and in 16384 bins: 18.2
// and 17.5 ms).
uint32_t bin_shift(uint32_t log2b) {
  const uint32_t few = log2b > 9u ? log2b - 9u : 0u;
  const uint32_t s = few < kMinBinShift ? kMinBinShift : few > kMaxBinShift ? kMaxBinShift : few;
  return log2b > s + kMaxBulkLog2Bins ? log2b - kMaxBulkLog2Bins : s;
}

// Records of a bin for `mean` keys: a bin's count is close to Poisson, and
// four deviations leave one bin in 30,000 to overflow (its last keys are then
// marked).
uint64_t bin_cap(uint64_t mean) {
  uint64_t root = 1;
  while (root * root < mean) ++root;
  return mean + 4u * root + 16u;
}

// Bytes of bins that the tables of each device keep.
constexpr int kMaxDevices = 64;
std::atomic<uint64_t> g_kept[kMaxDevices];

// Counts `bytes` of bins for the table, if its device's share has room.
bool keep_bins(ckpp_table *t, uint64_t bytes) {
  if (t->device >= kMaxDevices) return false;
  std::atomic<uint64_t> &kept = g_kept[t->device];
  uint64_t held = kept.load();
  do {
    if (held + bytes > t->device_mem / kBulkShare) return false;
  } while (!kept.compare_exchange_weak(held, held + bytes));
  t->bulk_bytes = bytes;
  return true;
}

}  // namespace

uint32_t bulk_bins(uint32_t log2b) {
  if (log2b < kMinBinShift + 1u || log2b > kMaxBulkLog2Buckets || (8ull << log2b) < kMinBulkKeys)
    return 0u;
  return 1u << (log2b - bin_shift(log2b));
}

void bulk_free(ckpp_table *t) {
  if (t->d_bulk) (void)hipFree(t->d_bulk);
  if (t->bulk_bytes) g_kept[t->device] -= t->bulk_bytes;
  t->d_bulk = nullptr;
  t->bulk_bytes = 0;
}

hipError_t bulk_insert_primary(ckpp_table *t, const void *d_keys, const uint64_t *d_values,
                               const uint16_t *d_expiry, const TimerArgs *timers, uint64_t n,
                               uint8_t *d_status, hipStream_t s, bool *taken) {
  *taken = false;
  const uint32_t log2b = t->log2_buckets;
  BulkArgs A;
  A.bins = bulk_bins(log2b);
  if ((t->flags & CKPP_PLAIN) || !d_status || A.bins == 0u || n < min_bulk_keys(log2b) ||
      n > (8ull << log2b))
    return hipSuccess;
  A.shift = bin_shift(log2b);
  // The bins take a share of the table's memory, in which the batch runs in
  // equal chunks: the cuckoo-path scratch, which the second stage needs only
  // after them, if it is as large (on tables of up to 2^15 buckets at 500
  // kicks; with a buffer of their own the first such batch of a table of
  // 2^13 took 78 us instead of 63, its destruction 48 instead of 32), else a
  // buffer of their own, kept while there is room for it (keep_bins).
  uint64_t limit = (256ull << log2b) / 8u * 5u;
  if (limit < kMinBulkBytes) limit = kMinBulkBytes;
  const uint64_t path_bytes = (uint64_t)t->own_paths * path_words(t->max_kicks) * 4u;
  const bool shared = t->d_own_paths && path_bytes >= limit;
  if (shared) limit = path_bytes;
  uint64_t chunks = (32u * n + limit - 1u) / limit, chunk = (n + chunks - 1u) / chunks;
  while (A.bins * bin_cap((chunk + A.bins - 1u) / A.bins) * 32u > limit) {
    ++chunks;
    chunk = (n + chunks - 1u) / chunks;
  }
  A.cap = (uint32_t)bin_cap((chunk + A.bins - 1u) / A.bins);
  void *bins = shared ? static_cast<void *>(t->d_own_paths) : t->d_bulk;
  bool pooled = false;
  if (!bins) {
    // no memory is taken under capture, and without it the batch runs the
    // other way
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &capture) != hipSuccess ||
        capture != hipStreamCaptureStatusNone) {
      (void)hipGetLastError();
      return hipSuccess;
    }
    hipError_t e = hipErrorOutOfMemory;
    if (keep_bins(t, limit)) {
      e = malloc_beside_capture(&bins, limit);
      if (e == hipSuccess) t->d_bulk = static_cast<uint8_t *>(bins);
      else bulk_free(t);
    } else if (n >= min_pooled_bulk_keys(log2b)) {
      e = hipMallocAsync(&bins, 32ull * A.bins * A.cap, s);
      pooled = true;
    }
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return hipSuccess;
    }
  }
  *taken = true;
  A.fill = t->d_bulk_fill;
  A.recs = static_cast<uint4 *>(bins);
  A.bk = t->d_table;
  A.log2b = log2b;
  A.seed = t->seed;
  A.now = timers ? timers->now : 0u;
  hipError_t e = hipSuccess;
  for (uint64_t i = 0; i < n && e == hipSuccess; i += chunk) {
    A.keys = reinterpret_cast<const uint4 *>(d_keys) + i;
    A.vals = d_values + i;
    A.expiry = d_expiry ? d_expiry + i : nullptr;
    A.status = d_status + i;
    A.n = (uint32_t)(n - i < chunk ? n - i : chunk);
    e = timers ? launch_bulk<true>(A, s) : launch_bulk<false>(A, s);
  }
  if (e != hipSuccess) {
    // bins may be left filled: the next batch starts with empty ones
    (void)hipDeviceSynchronize();
    (void)hipMemset(t->d_bulk_fill, 0, A.bins * sizeof(uint32_t));
  }
  if (!pooled) return e;
  const hipError_t f = hipFreeAsync(bins, s);
  return e != hipSuccess ? e : f;
}

}  // namespace ckpp
