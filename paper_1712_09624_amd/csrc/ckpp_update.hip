// ckpp_update.hip -- batched insert and delete kernels (gfx950): one lane
// per key at a time on a persistent grid; the per-key state machines are in
// ckpp_update_dev.h.

#include <mutex>

#include "ckpp_update_dev.h"

namespace ckpp {
namespace {

// Cuckoo-path scratch of ckpp_insert_batch_noalloc: a fixed array in each
// device's memory, held for the life of the process.  Host code never uses
// its name as an address: the device address comes from
// hipGetSymbolAddress, once per device (scratch_on).
constexpr uint64_t kScratchBytes = 8ull << 20;
static __device__ __align__(256) uint32_t scratch[kScratchBytes / sizeof(uint32_t)];

// Batches of at most this many keys run one key per wavefront (its lane 0):
// a wavefront runs its lanes' updates in lockstep, so a few keys side by
// side in one wavefront take several times as long as one key alone
// (measured on MI355X: an insert 2.7 us alone, 9.1 us for 8 lanes of one
// wavefront).
constexpr uint64_t kSpreadKeys = 1024;

// The key slots of a launch: its lanes, or with `spread` its wavefronts
// (lane 0 of each; false for the other lanes, which have nothing to do).
__device__ __forceinline__ bool worker_of(bool spread, uint64_t &worker, uint64_t &nworkers) {
  const uint64_t lane = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t nlanes = (uint64_t)gridDim.x * blockDim.x;
  if (!spread) {
    worker = lane;
    nworkers = nlanes;
    return true;
  }
  worker = lane >> 6;
  nworkers = nlanes >> 6;
  return (threadIdx.x & 63u) == 0u;
}

// What an insert launch needs.  TIMED kernels: expiry[i] is key i's
// expiration time and `now` the current time (Sec. 4.2).
struct InsertArgs {
  uint8_t *bk;
  const uint4 *keys;
  const uint64_t *vals;
  const uint16_t *expiry;
  uint64_t n;
  uint64_t seed;
  uint32_t now, log2b, max_kicks, plain, spin_limit;
  uint32_t *paths;       // every wavefront's path arrays, wave_paths each
  uint32_t wave_paths;   // 1..64
  uint8_t *status;       // nullable
  unsigned long long *nfailed, *nspin;  // nullable
};

// Adds the number of the wavefront's lanes for which `p` holds to *ctr.
__device__ __forceinline__ void count_lanes(bool p, unsigned long long *ctr) {
  const uint64_t m = __builtin_amdgcn_ballot_w64(p);
  if (m != 0ull && ctr && (threadIdx.x & 63u) == (uint32_t)__builtin_ctzll(m))
    atomicAdd(ctr, (unsigned long long)__builtin_popcountll(m));
}

// Key i through the whole state machine; every lane of the wavefront calls
// this together, `ok` for those that have a key.
template <bool TIMED>
__device__ __forceinline__ void insert_key(const InsertArgs &A, uint64_t i, bool ok,
                                           const WavePath &paths) {
  InsertOutcome o{CKPP_INSERTED, false};
  if (ok) {
    o = insert_one<TIMED>(A.bk, A.keys[i], A.vals[i], A.log2b, A.seed, A.max_kicks, A.plain != 0u,
                          paths, A.spin_limit, TIMED ? A.expiry[i] : 0u, A.now);
    if (A.status) A.status[i] = (uint8_t)o.status;
  }
  count_lanes(o.status == CKPP_FAILED, A.nfailed);
  count_lanes(o.spun, A.nspin);
}

__device__ __forceinline__ WavePath wave_paths(const InsertArgs &A, unsigned long long *held) {
  const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  return WavePath{A.paths + wave * A.wave_paths * path_words(A.max_kicks), A.wave_paths,
                  held + (threadIdx.x >> 6)};
}

// One key per wavefront (its lane 0).
template <bool TIMED>
__global__ void __launch_bounds__(256) insert_spread(InsertArgs A) {
  __shared__ unsigned long long s_held[4];
  if (threadIdx.x < 4u) s_held[threadIdx.x] = 0ull;
  __syncthreads();
  uint64_t worker, nworkers;
  const bool first = worker_of(true, worker, nworkers);
  const WavePath paths = wave_paths(A, s_held);
  for (uint64_t i = worker; i < A.n; i += nworkers) insert_key<TIMED>(A, i, first, paths);
}

// One lane per key, 64 keys per wavefront at a time, in two stages.  The
// first does what the primary's lock alone decides (insert_primary): a few
// round trips, the same for every lane.  A key that needs more (its
// secondary, a cuckoo path, another try at a held lock) goes into the
// wavefront's list, and once 64 are waiting the wavefront runs their state
// machines together.  A wavefront runs its lanes in lockstep, so slow keys
// run one by one as they come would each hold up 63 lanes that are done.
// A batch of one key per lane has nothing to gather and runs the state
// machines at once.  Measured on MI355X, 32M slots built to load 0.95 in one
// call: 9.5 ms without the list, 8.8 ms with it, 7.7 ms with it on 2^17 lanes
// (two wavefronts per SIMD) instead of 2^16; 2^18 lanes: 8.0 ms.
template <bool TIMED>
__global__ void __launch_bounds__(256) insert_lanes(InsertArgs A) {
  __shared__ unsigned long long s_held[4];
  __shared__ uint64_t s_wait[4][128];
  if (threadIdx.x < 4u) s_held[threadIdx.x] = 0ull;
  __syncthreads();
  const uint32_t lane = threadIdx.x & 63u;
  const WavePath paths = wave_paths(A, s_held);
  uint64_t *wait = s_wait[threadIdx.x >> 6];
  uint32_t waiting = 0u;
  const bool plain = A.plain != 0u;
  const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  if (A.n <= stride) {
    const uint64_t i = wave * 64u + lane;
    insert_key<TIMED>(A, i, i < A.n, paths);
    return;
  }
  for (uint64_t i0 = wave * 64u; i0 < A.n; i0 += stride) {
    const uint64_t i = i0 + lane;
    bool later = i < A.n;
    if (later && !plain) {
      const uint4 key = A.keys[i];
      const uint64_t value = A.vals[i];
      const bool wide = TIMED && (value >> kTimerShift) != 0ull;  // fails: not here
      const uint64_t word = TIMED ? value | ((uint64_t)A.expiry[i] << kTimerShift) : value;
      const KeyFields f = key_fields(key_hash(key, A.seed), A.log2b);
      if (!wide && try_lock(A.bk, f.p)) {
        section_begin();
        uint32_t expired = kUnknown;
        const int r = insert_primary<TIMED>(A.bk, key, word, f, read_head(A.bk, f.p), false, A.now,
                                            expired);
        if (r == kNeedPair) {
          unlock(A.bk, f.p);
        } else {
          if (A.status) A.status[i] = (uint8_t)r;
          later = false;
        }
      }
    }
    const uint64_t m = __builtin_amdgcn_ballot_w64(later);
    if (later) wait[waiting + (uint32_t)__builtin_popcountll(m & ((1ull << lane) - 1ull))] = i;
    waiting += (uint32_t)__builtin_popcountll(m);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (waiting >= 64u) {
      waiting -= 64u;
      insert_key<TIMED>(A, wait[waiting + lane], true, paths);
    }
  }
  if (waiting) {
    const bool ok = lane < waiting;
    insert_key<TIMED>(A, ok ? wait[lane] : 0ull, ok, paths);
  }
}

// The second stage of a dense batch: the keys whose status is kInsertPending,
// gathered and run 64 at a time as in insert_lanes.  A wavefront reads `tile`
// statuses at a time (at most kTile): few of them on a small batch, so that
// its slow keys spread over every wavefront.
constexpr uint32_t kTile = 256;

template <bool TIMED>
__global__ void __launch_bounds__(256) insert_marked(InsertArgs A, uint32_t tile) {
  __shared__ unsigned long long s_held[4];
  __shared__ uint64_t s_wait[4][64 + kTile];
  if (threadIdx.x < 4u) s_held[threadIdx.x] = 0ull;
  __syncthreads();
  const uint32_t lane = threadIdx.x & 63u;
  const WavePath paths = wave_paths(A, s_held);
  uint64_t *wait = s_wait[threadIdx.x >> 6];
  uint32_t waiting = 0u;
  const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const uint64_t stride = ((uint64_t)gridDim.x * blockDim.x >> 6) * tile;
  for (uint64_t i0 = wave * tile; i0 < A.n; i0 += stride) {
    const uint64_t end = i0 + tile < A.n ? i0 + tile : A.n;
    uint8_t st[kTile / 64];
#pragma unroll
    for (uint32_t k = 0; k < kTile / 64u; ++k) {
      const uint64_t i = i0 + 64u * k + lane;
      st[k] = A.status[i < end ? i : i0];
      if (i >= end) st[k] = 0u;
    }
#pragma unroll
    for (uint32_t k = 0; k < kTile / 64u; ++k) {
      const bool later = st[k] == kInsertPending;
      const uint64_t m = __builtin_amdgcn_ballot_w64(later);
      if (later)
        wait[waiting + (uint32_t)__builtin_popcountll(m & ((1ull << lane) - 1ull))] =
            i0 + 64u * k + lane;
      waiting += (uint32_t)__builtin_popcountll(m);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    while (waiting >= 64u) {
      waiting -= 64u;
      insert_key<TIMED>(A, wait[waiting + lane], true, paths);
    }
  }
  if (waiting) {
    const bool ok = lane < waiting;
    insert_key<TIMED>(A, ok ? wait[lane] : 0ull, ok, paths);
  }
}

template <bool TIMED>
__global__ void __launch_bounds__(256)
    delete_kernel(uint8_t *bk, const uint4 *__restrict__ keys, uint64_t n, uint32_t now,
                  uint32_t log2b, uint64_t seed, uint32_t plain_flag, uint32_t spin_limit,
                  uint8_t *__restrict__ found, unsigned long long *nspin, uint32_t spread) {
  const bool plain = plain_flag != 0u;
  uint64_t worker, nworkers;
  if (!worker_of(spread != 0u, worker, nworkers)) return;
  for (uint64_t i = worker; i < n; i += nworkers) {
    bool spun = false;
    const int r = delete_one<TIMED>(bk, keys[i], log2b, seed, plain, spin_limit, &spun, now);
    if (spun && nspin) atomicAdd(nspin, 1ull);
    if (found) found[i] = (uint8_t)r;
  }
}

// Anti-revival scan (Sec. 4.2): every bucket removes its expired entries,
// with the counter and filter maintenance of a delete (expire_slots_pass:
// the table is read as a stream, 16 lanes per bucket, a wavefront reading
// four consecutive buckets, 1 KiB, per instruction).  The removed entries are summed in the block and added with one
// atomic: an atomic per lane group on the one counter, which the memory side
// performs one by one, took most of a scan that removes many.  The blocks
// are large for the same reason.  Measured on MI355X, 2^20 buckets, 336,000
// entries removed: 221 us with an atomic per group, 80 us with one per block
// of 256, 53 us with one per block of 1024; nothing removed: 44 us each way
// (6.1 TB/s); 2^24 buckets, nothing removed, 835 -> 762 us.
constexpr uint32_t kScanBlock = 1024;

__global__ void __launch_bounds__(kScanBlock)
    expire_slots_kernel(uint8_t *bk, uint64_t nb, uint32_t now, uint32_t plain_flag,
                        unsigned long long *removed) {
  __shared__ unsigned long long total;
  if (threadIdx.x == 0u) total = 0ull;
  __syncthreads();
  const uint64_t count = expire_slots_pass(
      bk, nb, now, plain_flag != 0u, (uint64_t)blockIdx.x * blockDim.x + threadIdx.x,
      (uint64_t)gridDim.x * blockDim.x);
  if (count) atomicAdd(&total, (unsigned long long)count);
  __syncthreads();
  if (threadIdx.x == 0u && total && removed) atomicAdd(removed, total);
}

}  // namespace

namespace {

// Launches an insert of A.n keys with `npaths` path arrays at A.paths (at
// least the four that the wavefronts of one block need; the callers have 512
// and more): one key per wavefront for few keys, else one lane
// per key on at most t->path_lanes lanes and npaths wavefronts.
// marked: only the keys whose status is kInsertPending.
hipError_t launch_insert_kernel(const ckpp_table *t, InsertArgs A, bool timed, bool marked,
                                uint64_t npaths, hipStream_t s) {
  const bool spread = !marked && A.n <= kSpreadKeys && A.n <= npaths;
  const uint32_t block = 256, waves = block / 64u;
  uint64_t lanes = spread ? 64u * A.n : A.n < t->path_lanes && !marked ? A.n : t->path_lanes;
  if (lanes > 64u * npaths) lanes = 64u * npaths;
  uint64_t grid = (lanes + block - 1) / block;
  if (grid * waves > npaths) grid = npaths / waves;
  const uint64_t per_wave = npaths / (grid * waves);
  A.wave_paths = per_wave < 64u ? (uint32_t)per_wave : 64u;
  const dim3 g((uint32_t)grid), b(block);
  if (marked) {
    uint32_t tile = kTile;
    while (tile > 8u && (uint64_t)tile * waves * grid > A.n) tile /= 2u;
    if (timed) hipLaunchKernelGGL(insert_marked<true>, g, b, 0, s, A, tile);
    else hipLaunchKernelGGL(insert_marked<false>, g, b, 0, s, A, tile);
  } else if (timed) {
    if (spread) hipLaunchKernelGGL(insert_spread<true>, g, b, 0, s, A);
    else hipLaunchKernelGGL(insert_lanes<true>, g, b, 0, s, A);
  } else {
    if (spread) hipLaunchKernelGGL(insert_spread<false>, g, b, 0, s, A);
    else hipLaunchKernelGGL(insert_lanes<false>, g, b, 0, s, A);
  }
  return hipGetLastError();
}

InsertArgs insert_args(const ckpp_table *t, const void *d_keys, const uint64_t *d_values,
                       const uint16_t *d_expiry, uint32_t now, uint64_t n, uint32_t *paths,
                       uint8_t *d_status, uint64_t *d_nfailed) {
  InsertArgs A;
  A.bk = t->d_table;
  A.keys = reinterpret_cast<const uint4 *>(d_keys);
  A.vals = d_values;
  A.expiry = d_expiry;
  A.n = n;
  A.seed = t->seed;
  A.now = now;
  A.log2b = t->log2_buckets;
  A.max_kicks = t->max_kicks;
  A.plain = (t->flags & CKPP_PLAIN) ? 1u : 0u;
  A.spin_limit = t->retry_limit;
  A.paths = paths;
  A.wave_paths = 1u;
  A.status = d_status;
  A.nfailed = reinterpret_cast<unsigned long long *>(d_nfailed);
  A.nspin = reinterpret_cast<unsigned long long *>(t->d_stats) + 127;
  return A;
}

}  // namespace

hipError_t launch_insert(const ckpp_table *t, const void *d_keys, const uint64_t *d_values,
                         const uint16_t *d_expiry, const TimerArgs *timers, uint64_t n,
                         uint8_t *d_status, uint64_t *d_nfailed, hipStream_t s) {
  ckpp_table *tm = const_cast<ckpp_table *>(t);
  uint32_t *paths = t->d_own_paths;
  hipError_t e = hipSuccess;
  bool pooled = false;
  if (!paths) {
    // a stream under capture cannot allocate the table's buffer: that one
    // batch takes its scratch from the stream-ordered pool
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    e = hipStreamIsCapturing(s, &capture);
    if (e != hipSuccess) return e;
    pooled = capture != hipStreamCaptureStatusNone;
    for (;;) {
      const uint64_t bytes = (uint64_t)t->own_paths * path_words(t->max_kicks) * sizeof(uint32_t);
      e = pooled ? hipMallocAsync(reinterpret_cast<void **>(&paths), bytes, s)
                 : malloc_beside_capture(reinterpret_cast<void **>(&paths), bytes);
      if (e != hipErrorOutOfMemory || pooled || t->own_paths < 2u * kOwnPathsLow) break;
      (void)hipGetLastError();
      tm->own_paths /= 2u;
    }
    if (e != hipSuccess) return e;
    if (!pooled) tm->d_own_paths = paths;
  }
  const InsertArgs A = insert_args(t, d_keys, d_values, d_expiry, timers ? timers->now : 0u, n,
                                   paths, d_status, d_nfailed);
  bool bulk = false;
  e = bulk_insert_primary(tm, d_keys, d_values, d_expiry, timers, n, d_status, s, &bulk);
  if (e == hipSuccess)
    e = launch_insert_kernel(t, A, timers != nullptr, bulk, t->own_paths, s);
  if (!pooled) return e;
  const hipError_t f = hipFreeAsync(paths, s);
  return e != hipSuccess ? e : f;
}

namespace {

constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
uint32_t *g_scratch_ptr[kMaxScratchDevices];

// Device address of `scratch` on the current device `dev`, looked up once
// per device with that device current; null if the lookup fails.
uint32_t *scratch_on(int dev) {
  if (dev < 0 || dev >= kMaxScratchDevices) return nullptr;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    g_scratch_ptr[dev] = static_cast<uint32_t *>(p);
  }
  return g_scratch_ptr[dev];
}

}  // namespace

// The insert of launch_insert with its path arrays in `scratch`, no
// allocation.
int insert_noalloc(const ckpp_table *t, const void *d_keys, const uint64_t *d_values, uint64_t n,
                   uint8_t *d_status, uint64_t *d_nfailed, hipStream_t s) {
  const uint64_t path_bytes = path_words(t->max_kicks) * sizeof(uint32_t);
  uint32_t *paths = scratch_on(t->device);
  if (!paths) return CKPP_EDEVICE;
  const InsertArgs A =
      insert_args(t, d_keys, d_values, nullptr, 0u, n, paths, d_status, d_nfailed);
  return dev_status(launch_insert_kernel(t, A, false, false, kScratchBytes / path_bytes, s));
}

hipError_t launch_delete(const ckpp_table *t, const void *d_keys, uint64_t n,
                         const TimerArgs *timers, uint8_t *d_found, hipStream_t s) {
  const bool spread = n <= kSpreadKeys;
  const uint64_t lanes = spread ? 64u * n : n < t->path_lanes ? n : t->path_lanes;
  const uint32_t block = 256;
  const uint32_t grid = (uint32_t)((lanes + block - 1) / block);
  unsigned long long *nspin = reinterpret_cast<unsigned long long *>(t->d_stats) + 127;
  const uint32_t plain = (t->flags & CKPP_PLAIN) ? 1u : 0u;
  const uint4 *keys = reinterpret_cast<const uint4 *>(d_keys);
  if (timers)
    hipLaunchKernelGGL(delete_kernel<true>, dim3(grid), dim3(block), 0, s, t->d_table, keys, n,
                       timers->now, t->log2_buckets, t->seed, plain, t->retry_limit, d_found, nspin,
                       spread ? 1u : 0u);
  else
    hipLaunchKernelGGL(delete_kernel<false>, dim3(grid), dim3(block), 0, s, t->d_table, keys, n,
                       0u, t->log2_buckets, t->seed, plain, t->retry_limit, d_found, nspin,
                       spread ? 1u : 0u);
  return hipGetLastError();
}

hipError_t launch_expire_scan(const ckpp_table *t, uint32_t now, uint64_t *d_removed,
                              hipStream_t s) {
  const uint64_t nb = 1ull << t->log2_buckets;
  const uint32_t block = kScanBlock;
  // 16 lanes per bucket; a persistent grid of 4 blocks per compute unit
  uint64_t grid = (16u * nb + block - 1) / block;
  const uint64_t cap = 4ull * (uint64_t)t->num_cus;
  if (grid > cap) grid = cap;
  hipLaunchKernelGGL(expire_slots_kernel, dim3((uint32_t)grid), dim3(block), 0, s, t->d_table, nb,
                     now, (t->flags & CKPP_PLAIN) ? 1u : 0u,
                     reinterpret_cast<unsigned long long *>(d_removed));
  return hipGetLastError();
}

}  // namespace ckpp
