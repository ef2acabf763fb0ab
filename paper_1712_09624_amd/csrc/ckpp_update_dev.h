// ckpp_update_dev.h -- per-key insert and delete (device functions shared by
// the batch kernels and the serving loop).
//
// Insert (Sec. 2 insertion procedure, Sec. 4.1 filter maintenance) and
// delete (Sec. 4.1) run as many independent lanes, one key at a time per
// lane, on a persistent grid.  Each bucket's lock word (bytes 28..31) is
// taken with a single compare-and-swap and never waited on: a lane that
// misses a lock drops every lock it holds and retries in its next loop
// iteration, so no lane ever spins on a lock that a lane of its own
// wavefront holds.  Every entry that moves is moved under the locks of both
// buckets it may live in, so every bloom-filter and moved-counter update --
// which concerns the primary bucket of the entry that moves -- happens under
// the lock of that bucket.  Inside a critical section every table word is
// read and written with device-coherent accesses, so a lock cycle flushes
// no cache (section_begin / section_end).
//
// A key's state machine:
//   DIRECT  lock p; if the key is there, replace its value (UPDATED); else,
//           if it fails p's filter (so is not in a either), take the lowest
//           free slot of p (INSERTED); else lock a too: replace the value of
//           an entry there (UPDATED), or take the lowest free slot of p,
//           else of a (set the key's two bits in p's filter, moved[p] += 1)
//           (INSERTED); else, still under those locks, try a cuckoo path of
//           one or two displacements out of p (the buckets it touches are
//           locked too), and the key takes the freed slot of p (INSERTED);
//           else WALK.
//   WALK    random walk over full buckets starting at p, reading without
//           locks, with one step of lookahead: at each bucket, if the other
//           bucket of some entry has a free slot, that entry (preferably one
//           going home to its primary) ends the path; else pick a victim --
//           preferably an entry that sits in its secondary bucket (it would
//           move back home), then one whose other bucket is not the bucket
//           just left -- and continue at the victim's other bucket, at most
//           max_kicks steps; no (bucket, slot) twice.  No path: FAILED.
//   MOVE    apply the path backwards, one displacement per iteration, each
//           under the locks of its two buckets and re-validated there; a
//           move from primary to secondary adds the entry to the source's
//           filter, a move back decrements the destination's counter and
//           resets its filter at zero (Sec. 4.1).  A stale path returns to
//           DIRECT (the moves done so far are valid moves); when the path is
//           applied, p has a free slot and the key returns to DIRECT.
// Every loop is bounded: walks by max_kicks, retries by the table's retry
// limit, whose exhaustion reports CKPP_RETRY for that key (nothing changed
// for it) and is counted separately.
//
// Timers (Sec. 4.2, tables with timers only): an entry's expiration time
// sits in the high 16 bits of its value word, so every move carries it
// along.  Only alive entries are present: an insert of a key whose entry has
// expired overwrites that entry where it stands (INSERTED), and a delete of
// it reports 0.  DIRECT takes a slot holding an expired entry as if it were
// free (lazy deletion), after a free one: the expired entry is removed first,
// with the counter update of its primary bucket when it sat in its secondary
// -- under the pair's locks when that primary is p or a, else under the
// primary's own lock, taken like the others (never waited on).  A cuckoo
// path still ends only at a bucket with a free slot.

#pragma once

#include "ckpp_device.h"
#include "ckpp_internal.h"

namespace ckpp {
namespace {

// Random draws of the path search: counter-based SplitMix64 streams keyed
// by the key's hash.  kGolden is SplitMix64's own increment (2^64 / golden
// ratio); the other two are arbitrary odd salts that separate the streams
// (the multiplier of the PCG/MMIX generator, and a second golden-ratio-like
// odd constant), with no arithmetic role beyond that.
constexpr uint64_t kGolden = 0x9e3779b97f4a7c15ull;
constexpr uint64_t kDisplaceSalt = 0x5851f42d4c957f2dull;
constexpr uint64_t kWalkSalt = 0xd1b54a32d192ed03ull;
constexpr uint32_t kMaxWalks = 64;         // path searches per key
constexpr uint32_t kNoBucket = 0xffffffffu;
// A cuckoo path entry: bucket (below 2^29) | slot << 29.
constexpr uint32_t kPathSlotShift = 29;
constexpr uint32_t kPathBucketMask = (1u << kPathSlotShift) - 1u;
static_assert(kMaxLog2Buckets <= kPathSlotShift, "path entries hold a bucket index");

__device__ __forceinline__ uint8_t *bucket_ptr(uint8_t *bk, uint32_t b) {
  return bk + (uint64_t)b * kBucketBytes;
}
__device__ __forceinline__ const uint8_t *bucket_ptr(const uint8_t *bk, uint32_t b) {
  return bk + (uint64_t)b * kBucketBytes;
}

// Table words are reached through global-memory pointers: through a generic
// pointer the compiler emits flat accesses, which also wait for the LDS
// counter.
#define CKPP_GLOBAL __attribute__((address_space(1)))
template <class T>
using Global = CKPP_GLOBAL T;

template <class T>
__device__ __forceinline__ Global<T> *global_at(uint8_t *bk, uint32_t b, uint32_t offset) {
  return (Global<T> *)(bucket_ptr(bk, b) + offset);
}

__device__ __forceinline__ Global<uint32_t> *lock_word(uint8_t *bk, uint32_t b) {
  return global_at<uint32_t>(bk, b, kLockOffset);
}

__device__ __forceinline__ bool try_lock(uint8_t *bk, uint32_t b) {
  uint32_t expected = 0u;
  return __hip_atomic_compare_exchange_strong(lock_word(bk, b), &expected, 1u, __ATOMIC_RELAXED,
                                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void unlock(uint8_t *bk, uint32_t b) {
  __hip_atomic_store(lock_word(bk, b), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Writes bucket b's metadata word and drops its lock, its neighbour, in one
// 8-byte store.
static_assert(kLockOffset == kMetaOffset + 4u && kMetaOffset % 8u == 0u, "one 8-byte word");
__device__ __forceinline__ void unlock_meta(uint8_t *bk, uint32_t b, uint32_t meta) {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __hip_atomic_store(global_at<uint64_t>(bk, b, kMetaOffset), (uint64_t)meta, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}

// Ordering of a critical section.  Every table word a lane reads or writes
// under a lock goes through a device-coherent access (Coh below: relaxed
// agent-scope atomics, performed where every XCD's accesses meet), so
// taking and dropping a lock needs no flush of the per-XCD L2 caches.
// Acquire: the section's accesses are issued after the lock's CAS has
// returned (a compiler barrier keeps them there; the GPU issues a wave's
// memory accesses in order).  Release: the unlocking store waits until
// every access of the section has completed.
__device__ __forceinline__ void section_begin() { __atomic_signal_fence(__ATOMIC_SEQ_CST); }

__device__ __forceinline__ void section_end() {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0);
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// Takes the locks of buckets x != y in ascending order, or none.  The
// order makes retries live: of two lanes that need the same pair, the one
// that takes the lower lock first can always try the higher one, whereas
// two lanes taking the two locks at once could each get one, give both
// back, and repeat in lockstep forever.  On success the caller's later
// reads see every write made under these locks by earlier holders.
__device__ __forceinline__ bool lock_two(uint8_t *bk, uint32_t x, uint32_t y) {
  const uint32_t lo = x < y ? x : y, hi = x < y ? y : x;
  if (!try_lock(bk, lo)) return false;
  if (!try_lock(bk, hi)) {
    unlock(bk, lo);
    return false;
  }
  section_begin();
  return true;
}

// Publishes the writes made under the locks, then drops both locks.
__device__ __forceinline__ void unlock_two(uint8_t *bk, uint32_t x, uint32_t y) {
  section_end();
  unlock(bk, x);
  unlock(bk, y);
}

// A table word read and written with device-coherent accesses (relaxed
// agent-scope atomics): converts to its value, assigns with a store.
template <class T>
struct Coh {
  Global<T> *p;
  __device__ __forceinline__ operator T() const {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ const Coh &operator=(T v) const {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return *this;
  }
  __device__ __forceinline__ const Coh &operator|=(T v) const { return *this = (T)(T(*this) | v); }
};

// 16 bytes at once: the same agent-scope (sc1) access as the narrower words,
// one request instead of two.  Not a C++ atomic; a lock guards the bytes, so
// nothing depends on the 16 bytes being read or written indivisibly.
template <>
struct Coh<uint4> {
  Global<u32x4> *p;
  __device__ __forceinline__ operator uint4() const {
    const u32x4 v = __builtin_amdgcn_global_load_b128(p, "agent");
    return make_uint4(v.x, v.y, v.z, v.w);
  }
  __device__ __forceinline__ const Coh &operator=(uint4 v) const {
    __builtin_amdgcn_global_store_b128(p, u32x4{v.x, v.y, v.z, v.w}, "agent");
    return *this;
  }
};

// Address of table words of type T: `*` and `[]` give coherent words; p is
// the raw address (for read-modify-write atomics).
template <class T>
struct CohPtr {
  Global<T> *p;
  __device__ __forceinline__ Coh<T> operator*() const { return Coh<T>{p}; }
  __device__ __forceinline__ Coh<T> operator[](uint32_t i) const { return Coh<T>{p + i}; }
};

struct Head {
  uint4 q0;  // tags
  uint4 q1;  // bloom lo, bloom hi, meta, lock
};

__device__ __forceinline__ Coh<uint4> quarter(uint8_t *bk, uint32_t b, uint32_t offset) {
  return {global_at<u32x4>(bk, b, offset)};
}
__device__ __forceinline__ Head read_head(uint8_t *bk, uint32_t b) {
  return Head{quarter(bk, b, 0u), quarter(bk, b, 16u)};
}

__device__ __forceinline__ CohPtr<uint32_t> meta_ptr(uint8_t *bk, uint32_t b) {
  return {global_at<uint32_t>(bk, b, kMetaOffset)};
}
__device__ __forceinline__ CohPtr<uint64_t> bloom_ptr(uint8_t *bk, uint32_t b) {
  return {global_at<uint64_t>(bk, b, 16u)};
}
__device__ __forceinline__ CohPtr<uint16_t> tag_ptr(uint8_t *bk, uint32_t b) {
  return {global_at<uint16_t>(bk, b, 0u)};
}
__device__ __forceinline__ CohPtr<uint32_t> other_ptr(uint8_t *bk, uint32_t b) {
  return {global_at<uint32_t>(bk, b, kOtherOffset)};
}
__device__ __forceinline__ Coh<uint4> key_at(uint8_t *bk, uint32_t b, uint32_t s) {
  return quarter(bk, b, key_offset(s));
}
__device__ __forceinline__ CohPtr<uint64_t> value_ptr(uint8_t *bk, uint32_t b, uint32_t s) {
  return {global_at<uint64_t>(bk, b, value_offset(s))};
}

// Slot of `key` in a bucket whose head is h (bucket locked), or -1.
__device__ __forceinline__ int find_slot(uint8_t *bk, uint32_t b, const Head &h, uint4 key,
                                         uint32_t tag) {
  uint32_t cand = tag_eq_mask(h.q0, tag) & meta_busy(h.q1.z);
  while (cand) {
    const uint32_t s = (uint32_t)__builtin_ctz(cand);
    cand &= cand - 1u;
    if (key_eq(key_at(bk, b, s), key)) return (int)s;
  }
  return -1;
}

__device__ __forceinline__ void write_entry(uint8_t *bk, uint32_t b, uint32_t s, uint4 key,
                                            uint64_t value, uint32_t tag, uint32_t other) {
  key_at(bk, b, s) = key;
  *value_ptr(bk, b, s) = value;
  tag_ptr(bk, b)[s] = (uint16_t)tag;
  other_ptr(bk, b)[s] = other;
}

// A random number below n (n <= 8) from the 64 random bits r.
__device__ __forceinline__ uint32_t random_below(uint64_t r, uint32_t n) {
  return __umulhi((uint32_t)(r >> 32), n);
}

// Index of the k-th set bit of m (k < popcount(m)).
__device__ __forceinline__ uint32_t nth_bit(uint32_t m, uint32_t k) {
  for (uint32_t i = 0; i < k; ++i) m &= m - 1u;
  return (uint32_t)__builtin_ctz(m);
}

// The paths that few keys take (displacements, the walk, a move, lazy
// removal) are kept out of line: inlined, they raise the register count and
// slow the direct path every key takes (measured: 2^24 build to load 0.95 in
// 211 ms inlined, 181 ms out of line).
constexpr int kBusy = -2;    // a lock was taken by another lane: retry
// DIRECT found a displacement path, but a bucket beyond the pair was locked
// by another lane or changed before it was locked: retry DIRECT (at most
// kDisplaceRetries times per key, then the walk).
constexpr int kDisplaceBusy = -3;
constexpr uint32_t kDisplaceRetries = 4;
constexpr int kNeedPath = -1;
constexpr uint32_t kUnknown = 0xffffffffu;  // a mask of slots that was not read
constexpr int kNeedPair = -4;  // p's lock alone does not decide the key

// Busy slots of bucket b whose entries have expired at `now`: the value words
// of its slots 0..3 and 4..7 are two quarters each.
__device__ __forceinline__ uint32_t expired_mask(uint8_t *bk, uint32_t b, uint32_t busy,
                                                 uint32_t now) {
  uint4 q[4];
#pragma unroll
  for (uint32_t i = 0; i < 4u; ++i) q[i] = quarter(bk, b, value_offset(2u * i));
  uint32_t m = 0u;
#pragma unroll
  for (uint32_t i = 0; i < 4u; ++i) {
    if (!word_alive((uint64_t)q[i].x | ((uint64_t)q[i].y << 32), now)) m |= 1u << (2u * i);
    if (!word_alive((uint64_t)q[i].z | ((uint64_t)q[i].w << 32), now)) m |= 2u << (2u * i);
  }
  return m & busy;
}

// Working copy of the metadata of the two buckets a key may live in (both
// locked), written back once the insert is decided.
struct Pair {
  uint32_t b[2];
  uint32_t meta[2];
  uint64_t bloom;  // filter of b[0] as read under the lock
};

// moved - 1, and the filter of bucket y emptied when it reaches zero
// (Sec. 4.1); y's lock is held.
__device__ __forceinline__ uint32_t moved_down(uint8_t *bk, uint32_t y, uint32_t meta) {
  uint32_t mv = meta_moved(meta);
  if (mv > 0u) {
    mv -= 1u;
    if (mv == 0u) *bloom_ptr(bk, y) = 0ull;
  }
  return make_meta(mv, meta_busy(meta), meta_sec(meta));
}

// Removes the expired entry of slot s of the pair's bucket xi (lazy
// deletion, Sec. 4.2): its busy and sec bits are cleared in the working
// copy; if it sat in its secondary bucket, the moved counter of its primary
// y drops by one -- in the working copy when y is the pair's other bucket,
// else under y's lock, taken here.  Returns false, having changed nothing,
// when y's lock is held by another lane.
__device__ __attribute__((noinline)) bool remove_expired(uint8_t *bk, Pair &P, int xi, uint32_t s, bool plain) {
  const uint32_t bit = 1u << s;
  if (!plain && (meta_sec(P.meta[xi]) & bit)) {
    const uint32_t y = other_ptr(bk, P.b[xi])[s];
    const int yi = y == P.b[0] ? 0 : (y == P.b[1] ? 1 : -1);
    if (yi >= 0) {
      P.meta[yi] = moved_down(bk, y, P.meta[yi]);
    } else {
      if (!try_lock(bk, y)) return false;
      section_begin();
      *meta_ptr(bk, y) = moved_down(bk, y, *meta_ptr(bk, y));
      section_end();
      unlock(bk, y);
    }
  }
  P.meta[xi] = make_meta(meta_moved(P.meta[xi]), meta_busy(P.meta[xi]) & ~bit,
                         meta_sec(P.meta[xi]) & ~bit);
  return true;
}

// Entries of a full bucket that may move (an entry leaving its primary
// must not overflow that primary's moved counter).
__device__ __forceinline__ uint32_t movable(uint32_t meta, bool plain) {
  uint32_t c = meta_busy(meta);
  if (!plain && meta_moved(meta) >= 0xffffu) c &= meta_sec(meta);
  return c;
}

// The metadata word of bucket b, read without its lock.
__device__ __forceinline__ uint32_t peek_meta(const uint8_t *bk, uint32_t b) {
  return __hip_atomic_load((const Global<uint32_t> *)(bucket_ptr(bk, b) + kMetaOffset),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The other buckets of bucket b's entries.
__device__ __forceinline__ void read_other(uint8_t *bk, uint32_t b, uint32_t (&other)[kSlots]) {
  const uint4 lo = quarter(bk, b, kOtherOffset), hi = quarter(bk, b, kOtherOffset + 16u);
  other[0] = lo.x;
  other[1] = lo.y;
  other[2] = lo.z;
  other[3] = lo.w;
  other[4] = hi.x;
  other[5] = hi.y;
  other[6] = hi.z;
  other[7] = hi.w;
}

// a[i] for a small array indexed by a value known only at run time, as an
// OR of masked elements: an array indexed that way (or by a chain of
// selects, which the compiler turns back into an index) would live in
// scratch memory, and each load into it would wait for the one before.
__device__ __forceinline__ uint32_t pick_slot(const uint32_t (&a)[kSlots], uint32_t i) {
  uint32_t r = 0;
#pragma unroll
  for (uint32_t s = 0; s < kSlots; ++s) r |= a[s] & (0u - (uint32_t)(s == i));
  return r;
}

// The entries of bucket b (its other[] in `other`) among `cand` whose other
// bucket has a free slot, by those buckets' metadata words, read without
// locks.  Every slot's load is issued, a non-candidate reading bucket b
// itself, so that no load waits inside a branch: one round trip.
__device__ __forceinline__ uint32_t with_room(const uint8_t *bk, uint32_t b, uint32_t cand,
                                              const uint32_t (&other)[kSlots]) {
  uint32_t om[kSlots];
#pragma unroll
  for (uint32_t s = 0; s < kSlots; ++s) om[s] = peek_meta(bk, ((cand >> s) & 1u) ? other[s] : b);
  uint32_t room = 0;
#pragma unroll
  for (uint32_t s = 0; s < kSlots; ++s)
    if (((cand >> s) & 1u) && meta_busy(om[s]) != 0xffu) room |= 1u << s;
  return room;
}

// As with_room, for a search that needs one such entry: four at a time, the
// entries that sit in their secondary first, then those of the slots in
// `half`, then the rest; stops at the first four that hold one.
__device__ __forceinline__ uint32_t some_with_room(const uint8_t *bk, uint32_t b, uint32_t cand,
                                                   uint32_t sec, uint32_t half,
                                                   const uint32_t (&other)[kSlots]) {
  uint32_t room = 0u;
  for (uint32_t left = cand; left != 0u && room == 0u;) {
    uint32_t s[4], om[4];
#pragma unroll
    for (uint32_t k = 0; k < 4u; ++k) {
      const uint32_t g = left & sec, o = left & half;
      const uint32_t from = g ? g : o ? o : left;
      s[k] = from ? (uint32_t)__builtin_ctz(from) : kSlots;
      if (from) left &= ~(from & (0u - from));
      om[k] = peek_meta(bk, from ? pick_slot(other, s[k]) : b);
    }
#pragma unroll
    for (uint32_t k = 0; k < 4u; ++k)
      if (s[k] < kSlots && meta_busy(om[k]) != 0xffu) room |= 1u << s[k];
  }
  return room;
}

// An entry.
struct Slot {
  uint4 key;
  uint64_t word;
  uint32_t tag;
};
__device__ __forceinline__ Slot read_slot(uint8_t *bk, uint32_t b, uint32_t s) {
  return Slot{key_at(bk, b, s), value_ptr(bk, b, s)[0], tag_ptr(bk, b)[s]};
}

// The filter and metadata of a locked bucket as a step changes them; the
// filter is written where it changes, the metadata with the unlock.
struct Work {
  uint32_t b;
  uint32_t moved, busy, sec;
  uint64_t bloom;
  bool filter;  // the filter has changed
};
__device__ __forceinline__ Work work_of(uint32_t b, uint4 q1) {
  return Work{b, meta_moved(q1.z), meta_busy(q1.z), meta_sec(q1.z),
              (uint64_t)q1.x | ((uint64_t)q1.y << 32), false};
}
__device__ __forceinline__ void finish_filter(uint8_t *bk, const Work &W) {
  if (W.filter) *bloom_ptr(bk, W.b) = W.bloom;
}
__device__ __forceinline__ void finish_meta(uint8_t *bk, const Work &W) {
  unlock_meta(bk, W.b, make_meta(W.moved, W.busy, W.sec));
}

// Entry e moves from slot s of X to slot fs of its other bucket Y (both
// locked), with the filter maintenance of a cuckoo move (Sec. 4.1): an entry
// leaving its primary X adds its two bits to X's filter and 1 to X's moved
// counter; an entry going home to Y takes 1 off Y's counter and empties Y's
// filter when it reaches zero.  X's slot is left busy: the caller puts
// another entry there.
__device__ __forceinline__ void move_slot(uint8_t *bk, Work &X, uint32_t s, const Slot &e,
                                          Work &Y, uint32_t fs, uint32_t log2b, uint64_t seed,
                                          bool plain) {
  const bool guest = (X.sec >> s) & 1u;  // in its secondary X: Y is its home
  write_entry(bk, Y.b, fs, e.key, e.word, e.tag, X.b);
  Y.busy |= 1u << fs;
  Y.sec = guest ? (Y.sec & ~(1u << fs)) : (Y.sec | (1u << fs));
  if (plain) return;
  if (guest) {
    if (Y.moved > 0u && --Y.moved == 0u) {
      Y.bloom = 0ull;
      Y.filter = true;
    }
  } else {
    X.bloom |= key_fields(key_hash(e.key, seed), log2b).bloom_bits;
    X.moved += 1u;
    X.filter = true;
  }
}

// Takes the lock of bucket b unless the caller holds it already (own: the
// bucket beside p whose lock is held, or kNoBucket).
__device__ __forceinline__ bool lock_extra(uint8_t *bk, uint32_t b, uint32_t own) {
  return b == own || try_lock(bk, b);
}
__device__ __forceinline__ void unlock_extra(uint8_t *bk, uint32_t b, uint32_t own) {
  if (b != own) unlock(bk, b);
}

// Cuckoo displacements done inside DIRECT, under the lock of the key's full
// primary p: the walk's lookahead from p, one level and, if no entry of p can
// move at once, two.  One step: an entry v of p whose other bucket y1 has a
// free slot (preferably one going home) moves there.  Two steps: an entry t
// of some y1 = other(v) moves on to its own other bucket y2, which has a free
// slot, and v takes its place.  The buckets beyond p (and `own`, the key's
// secondary when the caller holds its lock, else kNoBucket) are locked here
// (never waited on), the path is re-checked under the locks, the moves are
// applied last to first with the filter maintenance of Sec. 4.1, and the key
// takes v's slot in p.  Almost every key that needs a cuckoo path needs at
// most two displacements, which then cost one critical section instead of a
// walk, one locked move per displacement and a second DIRECT step.
//
// Like the direct step this is bound by its memory requests, so the entries
// looked at and the words written are as few as the step allows: the entries
// are looked at four at a time (some_with_room), p's filter and metadata are
// those read under its lock (q1), and each bucket's metadata is written once,
// with its unlock; when the secondary looks full without its lock, that lock
// is not taken.  Measured on MI355X, keys that bring 2^22 buckets from load
// 0.85 to 0.9 at 1.94 -> 2.58 G/s, from 0.9 to 0.95 at 1.37 -> 1.77 G/s (all
// eight entries looked at, metadata read and written around each move).
//
// Returns 1 when the key was placed
// (every lock is dropped); 0, with nothing changed and the caller's locks
// still held, when no such path exists (the caller falls back to the walk);
// kBusy, likewise, when a bucket beyond the caller's is locked by another
// lane or its state changed before the lock (the caller may retry DIRECT:
// another lane's move is brief, and a retry costs a few round trips where the
// walk costs tens).
__device__ __attribute__((noinline)) int displace_and_place(
    uint8_t *bk, uint32_t log2b, uint64_t seed, bool plain, uint32_t p, uint32_t a, uint32_t own,
    uint32_t tag, uint64_t h, uint4 key, uint64_t word, uint4 q1) {
  const uint32_t mp = q1.z, cand = movable(mp, plain), sec = meta_sec(mp);
  uint32_t other[kSlots];
  read_other(bk, p, other);
  uint32_t v = kSlots, y1 = kNoBucket, t = kSlots, y2 = kNoBucket;
  const uint64_t draw = mix64(h ^ kDisplaceSalt);
  const uint32_t half = draw & 1u ? 0xf0u : 0x0fu;
  const uint32_t room = some_with_room(bk, p, cand, sec, half, other);
  if (room) {
    const uint32_t pick = (room & sec) ? (room & sec) : room;
    v = nth_bit(pick, random_below(draw, (uint32_t)__builtin_popcount(pick)));
    y1 = pick_slot(other, v);
  } else {
    // second level, one candidate at a time in the order of the choice
    // (entries of p going home first), two round trips each: the metadata
    // word and other[] of the candidate's other bucket y1, then the
    // metadata words of y1's entries' other buckets, all of a round trip's
    // loads issued together.  The first candidate whose y1 has an entry that
    // can move on to a bucket with a free slot wins (an entry of y1 going
    // home preferred); at the loads of the table's working loads that is
    // nearly always the first one tried.  Searching every candidate at once
    // takes 104 loads; measured on MI355X, one wavefront's lane spends some
    // 20 us issuing them and choosing, against about 1 us for a candidate's
    // two round trips.
    for (uint32_t order = 0; order < 2 && t == kSlots; ++order) {
      for (uint32_t c = cand & (order ? ~sec : sec); c && t == kSlots; c &= c - 1u) {
        const uint32_t s = (uint32_t)__builtin_ctz(c);
        const uint32_t b1 = pick_slot(other, s);
        const uint32_t m1 = peek_meta(bk, b1);
        uint32_t o1[kSlots];
        read_other(bk, b1, o1);
        const uint32_t sc = meta_sec(m1);
        const uint32_t r = some_with_room(bk, b1, movable(m1, plain), sc, half, o1);
        if (r) {
          const uint32_t pick = (r & sc) ? (r & sc) : r;
          v = s;
          t = (uint32_t)__builtin_ctz(pick);
          y1 = b1;
          y2 = pick_slot(o1, t);
        }
      }
    }
    if (t == kSlots) return 0;
  }
  // lock the buckets beyond the caller's (both compare-and-swaps issued
  // together: a failure here is not retried but falls back to DIRECT, a few
  // times, and the walk, so it cannot repeat in lockstep), then re-check the
  // path under the locks
  const bool two = y2 != kNoBucket;
  const bool ok1 = lock_extra(bk, y1, own);
  const bool ok2 = !two || lock_extra(bk, y2, own);
  if (!(ok1 && ok2)) {
    if (ok1) unlock_extra(bk, y1, own);
    if (ok2 && two) unlock_extra(bk, y2, own);
    return kBusy;
  }
  section_begin();
  Work P = work_of(p, q1);
  Work Y1 = work_of(y1, quarter(bk, y1, 16u));
  Work Y2{kNoBucket, 0u, 0u, 0u, 0ull, false};
  const Slot ev = read_slot(bk, p, v);
  uint32_t fs = t;
  bool still;
  if (two) {
    Y2 = work_of(y2, quarter(bk, y2, 16u));
    const Slot et = read_slot(bk, y1, t);
    const uint32_t ot = other_ptr(bk, y1)[t];
    still = ((Y1.busy >> t) & 1u) && ot == y2 && Y2.busy != 0xffu &&
            (plain || Y1.moved < 0xffffu || ((Y1.sec >> t) & 1u));
    if (still)
      move_slot(bk, Y1, t, et, Y2, (uint32_t)__builtin_ctz(~Y2.busy & 0xffu), log2b, seed, plain);
  } else {
    still = Y1.busy != 0xffu;
    fs = (uint32_t)__builtin_ctz(~Y1.busy & 0xffu);
  }
  if (!still) {
    if (two) unlock_extra(bk, y2, own);
    unlock_extra(bk, y1, own);
    return kBusy;
  }
  move_slot(bk, P, v, ev, Y1, fs, log2b, seed, plain);
  // the key takes slot v of p, its primary
  write_entry(bk, p, v, key, word, tag, a);
  P.sec &= ~(1u << v);
  finish_filter(bk, P);
  finish_filter(bk, Y1);
  if (two) finish_filter(bk, Y2);
  section_end();
  finish_meta(bk, P);
  finish_meta(bk, Y1);
  if (two) finish_meta(bk, Y2);
  if (own != kNoBucket && own != y1 && own != y2) unlock(bk, own);
  return 1;
}

// Takes the locks a step of a key with buckets p and a starts with: p's
// alone, or with `pair` both, in ascending order.
__device__ __forceinline__ bool lock_start(uint8_t *bk, const KeyFields &f, bool pair) {
  if (pair) return lock_two(bk, f.p, f.a);
  if (!try_lock(bk, f.p)) return false;
  section_begin();
  return true;
}

// Adds a's lock to p's.  Not waited on, and out of the ascending order when
// a < p, so a failure drops p's lock and has the key start its later
// attempts with the ordered pair: each key tries out of order at most once,
// and the ordered attempts keep concurrent keys live (lock_two).
__device__ __forceinline__ bool lock_second(uint8_t *bk, const KeyFields &f, bool &pair) {
  if (pair) return true;
  if (try_lock(bk, f.a)) {
    section_begin();
    return true;
  }
  unlock(bk, f.p);
  pair = true;
  return false;
}

// The key's entry, in slot s of bucket b (locked), gets a new value: an
// update, or with timers an expired one overwritten in place.
template <bool TIMED>
__device__ __forceinline__ int update_entry(uint8_t *bk, uint32_t b, uint32_t s, uint64_t word,
                                            uint32_t now) {
  const Coh<uint64_t> vw = value_ptr(bk, b, s)[0];
  const int r = !TIMED || word_alive(vw, now) ? CKPP_UPDATED : CKPP_INSERTED;
  vw = word;
  return r;
}

// What p's lock alone decides (see insert_direct): hp is p's head, read
// under its lock.  Updates the key in p, or places one that is in neither
// bucket there, and drops p's lock; or returns kNeedPair, having changed
// nothing, with p still locked.  expired: set to p's expired entries where it
// looks at them.
template <bool TIMED>
__device__ __forceinline__ int insert_primary(uint8_t *bk, uint4 key, uint64_t word,
                                              const KeyFields &f, const Head &hp, bool plain,
                                              uint32_t now, uint32_t &expired) {
  const int s = find_slot(bk, f.p, hp, key, f.tag);
  if (s >= 0) {
    const int r = update_entry<TIMED>(bk, f.p, (uint32_t)s, word, now);
    section_end();
    unlock(bk, f.p);
    return r;
  }
  if (plain || bloom_pass(hp.q1, f.bloom_bits)) return kNeedPair;
  const uint32_t meta = hp.q1.z, busy = meta_busy(meta);
  uint32_t room = ~busy & 0xffu;
  if (TIMED && !room) {
    expired = expired_mask(bk, f.p, busy, now);
    room = expired & ~meta_sec(meta);
  }
  if (!room) return kNeedPair;
  const uint32_t fs = (uint32_t)__builtin_ctz(room), bit = 1u << fs;
  write_entry(bk, f.p, fs, key, word, f.tag, f.a);
  section_end();
  unlock_meta(bk, f.p, make_meta(meta_moved(meta), busy | bit, meta_sec(meta) & ~bit));
  return CKPP_INSERTED;
}

// The DIRECT step of an absent key under the locks of both its buckets (q1:
// p's filter and metadata): the lowest free slot of p, else of a; with timers
// also a slot whose entry has expired, after the free ones of its bucket;
// else displacements.  Drops the locks.  expired_p: p's expired entries, or
// kUnknown.
template <bool TIMED>
__device__ __forceinline__ int insert_pair(uint8_t *bk, uint4 key, uint64_t word,
                                           const KeyFields &f, uint64_t h, uint32_t log2b,
                                           uint64_t seed, bool plain, uint32_t now,
                                           bool retry_displace, Pair &P, uint4 q1,
                                           uint32_t expired_p) {
  int r = kNeedPath;
  for (int xi = 0; xi < 2 && r == kNeedPath; ++xi) {
    if (xi == 1 && !plain && meta_moved(P.meta[0]) >= 0xffffu) break;
    const uint32_t x = P.b[xi];
    const uint32_t busy = meta_busy(P.meta[xi]);
    uint32_t fs;
    if (busy != 0xffu) {
      fs = (uint32_t)__builtin_ctz(~busy & 0xffu);
    } else {
      const uint32_t exp = !TIMED ? 0u
                           : xi == 0 && expired_p != kUnknown ? expired_p
                                                              : expired_mask(bk, x, busy, now);
      if (!exp) continue;
      // prefer an entry whose removal needs no lock beyond the pair's
      uint32_t cheap = exp & ~meta_sec(P.meta[xi]);
      for (uint32_t e = exp & meta_sec(P.meta[xi]); e; e &= e - 1u) {
        const uint32_t v = (uint32_t)__builtin_ctz(e);
        const uint32_t y = other_ptr(bk, x)[v];
        if (y == f.p || y == f.a) cheap |= 1u << v;
      }
      fs = (uint32_t)__builtin_ctz(cheap ? cheap : exp);
      if (!remove_expired(bk, P, xi, fs, plain)) {
        r = kBusy;
        break;
      }
    }
    write_entry(bk, x, fs, key, word, f.tag, xi ? f.p : f.a);
    const uint32_t m = P.meta[xi], bit = 1u << fs;
    P.meta[xi] = make_meta(meta_moved(m), meta_busy(m) | bit,
                           xi ? (meta_sec(m) | bit) : (meta_sec(m) & ~bit));
    if (xi == 1 && !plain) {
      // a lazy removal may have emptied the filter in memory
      *bloom_ptr(bk, f.p) = (TIMED ? (uint64_t)*bloom_ptr(bk, f.p) : P.bloom) | f.bloom_bits;
      P.meta[0] = make_meta(meta_moved(P.meta[0]) + 1u, meta_busy(P.meta[0]),
                            meta_sec(P.meta[0]));
    }
    r = CKPP_INSERTED;
  }
  if (r == CKPP_INSERTED) {
    section_end();
    unlock_meta(bk, f.p, P.meta[0]);
    unlock_meta(bk, f.a, P.meta[1]);
    return r;
  }
  if (r == kNeedPath) {
    const int d = displace_and_place(bk, log2b, seed, plain, f.p, f.a, f.a, f.tag, h, key, word,
                                     q1);
    if (d == 1) return CKPP_INSERTED;
    if (d == kBusy && retry_displace) r = kDisplaceBusy;
  }
  unlock_two(bk, f.p, f.a);
  return r;
}

// The DIRECT step.  TIMED: a table with timers (word = value | expiry <<
// 48); else word is the value.
//
// p's lock alone decides most keys: an entry moves only under the locks of
// both its buckets, and leaves p for a only with its bits set in p's filter,
// so a key that is not in p and fails p's filter is in neither bucket as
// long as p stays locked.  Such a key goes to a free slot of p (with timers,
// also to a slot of an expired entry that sits in its primary, whose removal
// touches p alone).  Otherwise -- the filter passes, p is full, or the table
// keeps no filter -- a's lock is taken too.  An insert is bound by the memory
// requests of its section, each a coherent access that the caches don't
// merge: this way they are p's compare-and-swap, its head (two 16-byte
// loads), the entry's key, value, tag and other bucket, and one 8-byte store
// of the metadata with the unlock, about half of what both locks from the
// start, 8-byte accesses and separate unlocks took.  Measured on MI355X:
// 65536 keys into 2^24 buckets at load 0.9 23.8 -> 18.5 us (their deletes
// 15.6 -> 11.2 us), 32M slots built to load 0.95 in one call 14.8 -> 9.5 ms.
//
// retry_displace: a displacement path found but blocked by another lane's
// lock returns kDisplaceBusy (the caller retries DIRECT) rather than
// kNeedPath.  pair: see lock_second.
template <bool TIMED>
__device__ int insert_direct(uint8_t *bk, uint4 key, uint64_t word, const KeyFields &f,
                             uint64_t h, uint32_t log2b, uint64_t seed, bool plain, uint32_t now,
                             bool retry_displace, bool &pair) {
  if (!lock_start(bk, f, pair)) return kBusy;
  const bool both = pair;  // a's lock is held too
  const Head hp = read_head(bk, f.p);
  uint32_t expired = kUnknown;
  const int r = insert_primary<TIMED>(bk, key, word, f, hp, plain, now, expired);
  if (r != kNeedPair) {
    if (both) unlock(bk, f.a);
    return r;
  }
  const bool pass = plain || bloom_pass(hp.q1, f.bloom_bits);
  if (!TIMED && !both && !pass && meta_busy(peek_meta(bk, f.a)) == 0xffu) {
    // the key is absent, p is full and a looked full without its lock:
    // displacements need p's lock alone
    const int d = displace_and_place(bk, log2b, seed, plain, f.p, f.a, kNoBucket, f.tag, h, key,
                                     word, hp.q1);
    if (d == 1) return CKPP_INSERTED;
    unlock(bk, f.p);
    return d == kBusy && retry_displace ? kDisplaceBusy : kNeedPath;
  }
  if (!lock_second(bk, f, pair)) return kBusy;
  uint4 qa;  // a's filter and metadata; its tags matter only to a key it may hold
  if (pass) {
    const Head ha = read_head(bk, f.a);
    const int s = find_slot(bk, f.a, ha, key, f.tag);
    if (s >= 0) {
      const int u = update_entry<TIMED>(bk, f.a, (uint32_t)s, word, now);
      unlock_two(bk, f.p, f.a);
      return u;
    }
    qa = ha.q1;
  } else {
    qa = quarter(bk, f.a, 16u);
  }
  Pair P{{f.p, f.a}, {hp.q1.z, qa.z}, (uint64_t)hp.q1.x | ((uint64_t)hp.q1.y << 32)};
  return insert_pair<TIMED>(bk, key, word, f, h, log2b, seed, plain, now, retry_displace, P,
                            hp.q1, expired);
}

// A cuckoo path's entries in memory (bucket | slot << 29), in groups of
// four, group g at p + g * step words (16-byte aligned): a wavefront's path
// arrays are interleaved group by group, so that the lanes of a walk, which
// advance together, read neighbouring groups.  An array holds path_words
// words.
struct PathRef {
  uint32_t *p;
  uint32_t step;
  __device__ __forceinline__ uint32_t &operator[](uint32_t i) const {
    return p[(uint64_t)(i >> 2) * step + (i & 3u)];
  }
  __device__ __forceinline__ uint4 group(uint32_t g) const {
    return *reinterpret_cast<const uint4 *>(p + (uint64_t)g * step);
  }
};

// Slots of bucket b among the first n entries of the path.  A walk that
// finds no way out looks through its whole path at every step, which takes
// most of its time: the entries are loaded kScan groups at a time (a key
// that fails after 500 steps: 11.3 ms entry by entry, 4.2 ms this way).
constexpr uint32_t kScan = 12;

__device__ __forceinline__ uint32_t path_slots(PathRef path, uint32_t n, uint32_t b) {
  uint32_t used = 0u;
  for (uint32_t i = 0; i < n; i += 4u * kScan) {
    uint4 e[kScan];
#pragma unroll
    for (uint32_t g = 0; g < kScan; ++g) {
      const uint32_t at = i + 4u * g;
      e[g] = path.group((at < n ? at : i) >> 2);
    }
#pragma unroll
    for (uint32_t g = 0; g < kScan; ++g) {
      const uint32_t w[4] = {e[g].x, e[g].y, e[g].z, e[g].w};
#pragma unroll
      for (uint32_t k = 0; k < 4u; ++k)
        if (i + 4u * g + k < n && (w[k] & kPathBucketMask) == b)
          used |= 1u << (w[k] >> kPathSlotShift);
    }
  }
  return used;
}

// Random walk with one step of lookahead from bucket `start` (read without
// locks).  At each full bucket the other buckets of all its candidate
// entries are looked at together (their metadata words, loaded in
// parallel): if one of them has a free slot, moving that entry there ends
// the path (an entry sitting in its secondary bucket, i.e. going home,
// preferred); otherwise a victim is drawn as in a plain random walk (an
// entry going home, then one whose other bucket is not the bucket just
// left, then any) and the walk continues at its other bucket.  The same
// two memory round trips per step as a plain walk, but far fewer steps: at
// load 0.9 the longest paths shrink from tens of displacements to a few.
// path[i] holds bucket | slot << 29 of the i-th victim; *last receives the
// bucket with a free slot that ends the path.  Returns the path length, or
// -1.
__device__ __attribute__((noinline)) int walk(uint8_t *bk, uint32_t start, uint64_t rbase, uint32_t max_kicks,
                    bool plain, PathRef path, uint32_t *last) {
  uint32_t cur = start, prev = kNoBucket;
  for (uint32_t step = 0; step < max_kicks; ++step) {
    const uint32_t meta = peek_meta(bk, cur);
    uint32_t other[kSlots];
    read_other(bk, cur, other);
    const uint32_t used = path_slots(path, step, cur);
    const uint32_t sec = meta_sec(meta);
    uint32_t cand = meta_busy(meta) & ~used;
    if (!plain && meta_moved(meta) >= 0xffffu) cand &= sec;  // no owner may leave
    if (!cand) return -1;
    // lookahead: which candidates' other buckets have a free slot
    const uint32_t room = with_room(bk, cur, cand, other);
    const uint64_t r = mix64(rbase + (uint64_t)(step + 1) * kGolden);
    if (room) {
      const uint32_t pick = (room & sec) ? (room & sec) : room;
      const uint32_t v = nth_bit(pick, random_below(r, (uint32_t)__builtin_popcount(pick)));
      path[step] = cur | (v << kPathSlotShift);
      *last = pick_slot(other, v);
      return (int)step + 1;
    }
    uint32_t pref = 0;
#pragma unroll
    for (uint32_t s = 0; s < kSlots; ++s)
      if (((cand >> s) & 1u) && other[s] != prev) pref |= 1u << s;
    const uint32_t home = pref & sec;
    const uint32_t pick = home ? home : (pref ? pref : cand);
    const uint32_t v = nth_bit(pick, random_below(r, (uint32_t)__builtin_popcount(pick)));
    path[step] = cur | (v << kPathSlotShift);
    prev = cur;
    cur = pick_slot(other, v);
  }
  return -1;
}

// Under the locks of x and y: moves the entry of slot s of bucket x to a
// free slot of bucket y, its other bucket, if the state still matches the
// path (the slot is taken, its entry's other bucket is y, y has a free
// slot, and an entry leaving its primary does not overflow the moved
// counter), with the filter maintenance of Sec. 4.1.  Returns 1 when
// moved, 0 when the state no longer matches (nothing changed).
__device__ int move_checked(uint8_t *bk, uint32_t x, uint32_t s, uint32_t y, uint32_t log2b,
                            uint64_t seed, bool plain) {
  int r = 0;
  const uint32_t mx = *meta_ptr(bk, x), my = *meta_ptr(bk, y);
  const uint32_t busy_x = meta_busy(mx), busy_y = meta_busy(my);
  if (((busy_x >> s) & 1u) && other_ptr(bk, x)[s] == y && busy_y != 0xffu) {
    const uint4 key = key_at(bk, x, s);
    const uint64_t val = *value_ptr(bk, x, s);
    const KeyFields fe = key_fields(key_hash(key, seed), log2b);
    const bool from_primary = fe.p == x;
    const bool consistent = from_primary ? (fe.a == y) : (fe.a == x && fe.p == y);
    if (consistent && (plain || !from_primary || meta_moved(mx) < 0xffffu)) {
      const uint32_t fs = (uint32_t)__builtin_ctz(~busy_y & 0xffu);
      write_entry(bk, y, fs, key, val, tag_ptr(bk, x)[s], x);
      uint32_t moved_x = meta_moved(mx), moved_y = meta_moved(my);
      const uint32_t sec_y =
          from_primary ? (meta_sec(my) | (1u << fs)) : (meta_sec(my) & ~(1u << fs));
      if (!plain) {
        if (from_primary) {
          *bloom_ptr(bk, x) |= fe.bloom_bits;
          moved_x += 1u;
        } else if (moved_y > 0u) {
          moved_y -= 1u;
          if (moved_y == 0u) *bloom_ptr(bk, y) = 0ull;
        }
      }
      *meta_ptr(bk, y) = make_meta(moved_y, busy_y | (1u << fs), sec_y);
      *meta_ptr(bk, x) = make_meta(moved_x, busy_x & ~(1u << s), meta_sec(mx) & ~(1u << s));
      r = 1;
    }
  }
  return r;
}

// One displacement of the MOVE state: move_checked under the lock pair of
// x and y.  Returns 1 when done, 0 when the state no longer matches the
// path, kBusy when a lock was taken.
__device__ __attribute__((noinline)) int move_entry(uint8_t *bk, uint32_t x, uint32_t s, uint32_t y,
                          uint32_t log2b, uint64_t seed, bool plain) {
  if (x == y || !lock_two(bk, x, y)) return kBusy;
  const int r = move_checked(bk, x, s, y, log2b, seed, plain);
  unlock_two(bk, x, y);
  return r;
}

// Longest cuckoo path applied in one critical section (apply_path).
constexpr uint32_t kSectionPath = 8;

// Applies a cuckoo path of len <= kSectionPath displacements (path[0..len)
// as the walk wrote it, `last` the bucket that ends it) in one critical
// section, where the MOVE state takes a lock pair, a re-check and a release
// per displacement: every bucket of the path is locked, all the lock
// requests issued together and none waited for; then the moves run last to
// first, each with move_checked's re-check.  A lock held by another lane
// gives back every lock taken and returns kBusy with nothing moved (the
// caller then moves step by step, taking the pairs in ascending order,
// which keeps concurrent keys live).  A re-check that fails stops the moves
// and returns 0 (the moves already made stand: each is a valid move on its
// own, as in the MOVE state); 1 when every displacement is made.
//
// The lock requests are atomic ORs of 1 into the lock words (a lock is
// taken by the request that reads 0), one per entry of b[0..kSectionPath]
// whatever the path's length, so that none sits behind a branch: entries
// past the path, and repeats of a bucket, request b[0]'s or that bucket's
// lock again.  A lane's requests to one word are performed in order, so a
// repeat reads 1 when an earlier request of the lane took the lock; it can
// read 0 only when the earlier one found the lock held by another lane that
// has let it go since, and then this lane holds it through the repeat and
// gives it back with the others.
__device__ __attribute__((noinline)) int apply_path(uint8_t *bk, PathRef path,
                                                    uint32_t len, uint32_t last, uint32_t log2b,
                                                    uint64_t seed, bool plain) {
  uint32_t b[kSectionPath + 1], sl[kSectionPath];
#pragma unroll
  for (uint32_t i = 0; i < kSectionPath; ++i) {
    const uint32_t e = i < len ? path[i] : 0u;
    b[i] = i < len ? (e & kPathBucketMask) : kNoBucket;
    sl[i] = e >> kPathSlotShift;
  }
  // `last` follows the path's buckets; entries past it request b[0] again
  b[kSectionPath] = kNoBucket;
#pragma unroll
  for (uint32_t i = 0; i <= kSectionPath; ++i) {
    if (i == len) b[i] = last;
  }
  uint32_t addr[kSectionPath + 1];
  bool first[kSectionPath + 1];  // the first entry of its bucket within the path
#pragma unroll
  for (uint32_t i = 0; i <= kSectionPath; ++i) {
    bool dup = b[i] == kNoBucket;
#pragma unroll
    for (uint32_t j = 0; j < i; ++j) dup = dup || b[j] == b[i];
    first[i] = !dup;
    addr[i] = b[i] == kNoBucket ? b[0] : b[i];
  }
  bool took[kSectionPath + 1];
#pragma unroll
  for (uint32_t i = 0; i <= kSectionPath; ++i)
    took[i] = __hip_atomic_fetch_or(lock_word(bk, addr[i]), 1u, __ATOMIC_RELAXED,
                                    __HIP_MEMORY_SCOPE_AGENT) == 0u;
  bool all = true;
#pragma unroll
  for (uint32_t i = 0; i <= kSectionPath; ++i) all = all && (took[i] || !first[i]);
  if (!all) {
#pragma unroll
    for (uint32_t i = 0; i <= kSectionPath; ++i)
      if (took[i]) unlock(bk, addr[i]);
    return kBusy;
  }
  section_begin();
  int r = 1;
  for (uint32_t k = len; k > 0 && r == 1; --k) {
    const uint32_t i = k - 1u;
    uint32_t x = 0u, s = 0u, y = 0u;
#pragma unroll
    for (uint32_t j = 0; j < kSectionPath; ++j) {
      if (j == i) {
        x = b[j];
        s = sl[j];
        y = b[j + 1];
      }
    }
    r = x == y ? 0 : move_checked(bk, x, s, y, log2b, seed, plain);
  }
  section_end();
  // every bucket's lock was taken by its first request (the repeats read 1)
#pragma unroll
  for (uint32_t i = 0; i <= kSectionPath; ++i)
    if (took[i]) unlock(bk, addr[i]);
  return r;
}

// Where a key's walk writes its path: a fixed array of the lane's own.
struct LanePath {
  uint32_t *p;
  __device__ __forceinline__ bool take(PathRef &path) const {
    path = PathRef{p, 4u};
    return true;
  }
  __device__ __forceinline__ void give() const {}
};

// One of the `count` path arrays (1..64, interleaved from `base`) of a
// wavefront.  Few keys walk, so a wavefront's lanes share fewer arrays than
// it has lanes: lane l may take array l mod count, when no other lane holds
// it (its bit in `held`, a word of LDS), and keeps it until its key is done.
// A lane that finds its array held tries again in its next iteration; the
// holder, a lane of the same wavefront, goes on meanwhile.
struct WavePath {
  uint32_t *base;
  uint32_t count;
  unsigned long long *held;
  bool mine = false;
  __device__ __forceinline__ uint32_t slot() const { return (threadIdx.x & 63u) % count; }
  __device__ __forceinline__ bool take(PathRef &path) {
    const uint32_t i = slot();
    if (!mine) mine = ((atomicOr(held, 1ull << i) >> i) & 1ull) == 0ull;
    path = PathRef{base + 4u * i, 4u * count};
    return mine;
  }
  __device__ __forceinline__ void give() {
    if (mine) atomicAnd(held, ~(1ull << slot()));
    mine = false;
  }
};

// Outcome of one key's insert: its status, and whether the retry bound ran
// out (then the status is CKPP_RETRY).
struct InsertOutcome {
  int status;
  bool spun;
};

// Runs one key through the DIRECT / WALK / MOVE state machine until it is
// placed, updated or fails, for at most spin_limit iterations (then
// CKPP_RETRY: the key's value is neither stored nor changed; the moves
// applied so far only relocated other entries).  paths: where the path
// scratch (path_words words) comes from; an iteration that only waits
// for it is not counted.  TIMED: the table has timers; the entry gets
// expiration time `expiry`, and a value of 2^48 or more (the device layout's
// limit) fails at once with nothing changed.
template <bool TIMED = false, class Paths>
__device__ InsertOutcome insert_one(uint8_t *bk, uint4 key, uint64_t value, uint32_t log2b,
                                    uint64_t seed, uint32_t max_kicks, bool plain,
                                    Paths paths, uint32_t spin_limit, uint32_t expiry = 0u,
                                    uint32_t now = 0u) {
  if (TIMED && (value >> kTimerShift) != 0ull) return InsertOutcome{CKPP_FAILED, false};
  const uint64_t word = TIMED ? (value | ((uint64_t)(expiry & 0xffffu) << kTimerShift)) : value;
  const uint64_t h = key_hash(key, seed);
  const KeyFields f = key_fields(h, log2b);
  enum { DIRECT, WALK, MOVE };
  int state = DIRECT, result = -1;
  uint32_t len = 0, next = 0, last = 0, walks = 0, iters = 0, dretries = 0;
  bool spun = false;
  PathRef path{nullptr, 0u};
  // a table without filters needs both buckets for every key
  bool pair = plain;
  uint32_t path_waits = 0;
  // The lanes of a wavefront leave this loop together: code after a loop runs
  // once its last lane is out, and a lane that is done must give its path
  // array back while others may still wait for it.  The ballot keeps the
  // loop whole (a lane's own `result < 0` as the condition would let the
  // compiler move the giving back behind it).
  while (__builtin_amdgcn_ballot_w64(result < 0) != 0ull) {
    if (result < 0) {
      if (++iters > spin_limit) {
        result = CKPP_RETRY;
        spun = true;
      } else if (state == DIRECT) {
        const bool retry_displace = dretries < kDisplaceRetries;
        const int r = insert_direct<TIMED>(bk, key, word, f, h, log2b, seed, plain, now,
                                           retry_displace, pair);
        if (r >= 0)
          result = r;
        else if (r == kNeedPath)
          state = WALK;
        else if (r == kDisplaceBusy)
          ++dretries;  // DIRECT again
      } else if (state == WALK) {
        if (walks >= kMaxWalks) {
          result = CKPP_FAILED;
        } else if (!paths.take(path)) {
          --iters;
          if (++path_waits > kMaxRetryLimit) {
            result = CKPP_RETRY;
            spun = true;
          }
        } else {
          const int L = walk(bk, f.p, h ^ ((uint64_t)walks * kWalkSalt), max_kicks, plain,
                             path, &last);
          ++walks;
          if (L <= 0) {
            result = CKPP_FAILED;
          } else {
            len = (uint32_t)L;
            next = len;
            state = MOVE;
            // a short path in one critical section; step by step if a lock is
            // held (then nothing was moved)
            if (len <= kSectionPath &&
                apply_path(bk, path, len, last, log2b, seed, plain) != kBusy)
              state = DIRECT;
          }
        }
      } else {
        const uint32_t e = path[next - 1];
        const uint32_t x = e & kPathBucketMask, s = e >> kPathSlotShift;
        const uint32_t y = (next == len) ? last : (path[next] & kPathBucketMask);
        const int r = move_entry(bk, x, s, y, log2b, seed, plain);
        if (r == 1) {
          if (--next == 0) state = DIRECT;
        } else if (r == 0) {
          state = DIRECT;
        }
      }
    }
    if (result >= 0) paths.give();
  }
  return InsertOutcome{result, spun};
}

// Returns 1 if the key was removed, 0 if absent, kBusy to retry.  TIMED:
// an expired entry of the key is removed too, but reports 0 (Sec. 4.2).  As
// in insert_direct, p's lock alone decides a key that is in p or fails p's
// filter.  Removing from p writes p's metadata word alone, with the unlock,
// and on a table without timers nothing is left to wait for: what the section
// read has decided that word.  The time of an expired entry decides only the
// answer, so with timers the unlock waits for it (the next holder of the lock
// may write another entry's time there).
template <bool TIMED>
__device__ int delete_direct(uint8_t *bk, uint4 key, const KeyFields &f, bool plain,
                             uint32_t now, bool &pair) {
  if (!lock_start(bk, f, pair)) return kBusy;
  const bool both = pair;
  const Head hp = read_head(bk, f.p);
  const uint32_t mp = hp.q1.z;
  int s = find_slot(bk, f.p, hp, key, f.tag);
  if (s >= 0 || !(plain || bloom_pass(hp.q1, f.bloom_bits))) {
    int r = 0;
    uint32_t m = mp;
    if (s >= 0) {
      const uint32_t bit = 1u << s;
      r = (!TIMED || word_alive(value_ptr(bk, f.p, (uint32_t)s)[0], now)) ? 1 : 0;
      m = make_meta(meta_moved(mp), meta_busy(mp) & ~bit, meta_sec(mp) & ~bit);
      if (TIMED) section_end();
    }
    unlock_meta(bk, f.p, m);
    if (both) unlock(bk, f.a);
    return r;
  }
  if (!lock_second(bk, f, pair)) return kBusy;
  const Head ha = read_head(bk, f.a);
  s = find_slot(bk, f.a, ha, key, f.tag);
  int r = 0;
  uint32_t m = mp, ma = ha.q1.z;
  if (s >= 0) {
    const uint32_t bit = 1u << s;
    r = (!TIMED || word_alive(value_ptr(bk, f.a, (uint32_t)s)[0], now)) ? 1 : 0;
    ma = make_meta(meta_moved(ma), meta_busy(ma) & ~bit, meta_sec(ma) & ~bit);
    if (!plain && meta_moved(mp) > 0u) {
      const uint32_t moved = meta_moved(mp) - 1u;
      if (moved == 0u) *bloom_ptr(bk, f.p) = 0ull;
      m = make_meta(moved, meta_busy(mp), meta_sec(mp));
    }
  }
  section_end();
  unlock_meta(bk, f.p, m);
  unlock_meta(bk, f.a, ma);
  return r;
}


// Deletes one key: 1 if it was removed, 0 if absent, CKPP_RETRY (nothing
// removed; the key may still be present) when its bucket locks stayed taken
// by other lanes for spin_limit attempts; *spun is set in that case.
template <bool TIMED = false>
__device__ int delete_one(uint8_t *bk, uint4 key, uint32_t log2b, uint64_t seed, bool plain,
                          uint32_t spin_limit, bool *spun, uint32_t now = 0u) {
  const KeyFields f = key_fields(key_hash(key, seed), log2b);
  int r = kBusy;
  uint32_t iters = 0;
  bool pair = plain;
  while (r == kBusy && iters < spin_limit) {
    ++iters;
    r = delete_direct<TIMED>(bk, key, f, plain, now, pair);
  }
  *spun = r == kBusy;
  return r == kBusy ? CKPP_RETRY : r;
}

// Anti-revival scan (Sec. 4.2) over buckets [0, nb) by the lanes gtid of a
// grid of gthreads (whole wavefronts): 16 neighbouring lanes read one bucket's
// 256 bytes, one 16-byte quarter each, and share the metadata word (lane
// 1), the value words (lanes 6, 7, 12, 13: the time in the high 16 bits)
// and the other buckets (lanes 14, 15) through cross-lane reads.  Lane 0 of
// the group clears the bucket's expired slots (busy and sec bits) with an
// atomic AND; the moved counter of the primary bucket of a removed entry
// that sat in its secondary drops by one through an atomic subtraction on
// that bucket's meta word (the counter is its low 16 bits and is at least 1
// while the entry is counted there), done by the lane that holds the
// entry's other bucket, so no lock is needed.  The subtraction that takes a
// counter from 1 to 0 empties that bucket's filter (Sec. 4.1: the filter is
// reset when its counter returns to zero): while the scan runs nothing
// raises a counter, so zero is final.  The caller runs nothing else on the
// table meanwhile.  U: the buckets a group reads before it examines the
// first (loads in flight per lane, for grids with few waves).  Returns the
// entries this lane removed.
template <uint32_t U = 1>
__device__ __forceinline__ uint64_t expire_slots_pass(uint8_t *bk, uint64_t nb, uint32_t now,
                                                      bool plain, uint64_t gtid,
                                                      uint64_t gthreads) {
  const uint32_t lane = threadIdx.x & 63u, r = lane & 15u, g0 = lane & 48u;
  const uint64_t groups = gthreads / 16u;
  uint64_t count = 0;
  for (uint64_t b0 = gtid / 16u; b0 < nb; b0 += U * groups) {
    // every load is issued before the first is used: indexes past the end
    // read the last bucket instead (no branch around a load, which would
    // wait for it inside the branch), and those buckets are skipped below
    uint4 qs[U];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      const uint64_t b = b0 + u * groups;
      qs[u] = reinterpret_cast<const uint4 *>(bucket_ptr(bk, (uint32_t)(b < nb ? b : nb - 1u)))[r];
    }
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      const uint64_t b = b0 + u * groups;
      if (b >= nb) break;
      const uint4 q = qs[u];
      const uint32_t meta = (uint32_t)__shfl((int)q.z, (int)(g0 + 1u));
      // expired bits of this lane's two value words (lanes 6, 7, 12, 13)
      uint32_t mine = 0u;
      const uint32_t s0 = r == 6u ? 0u : r == 7u ? 2u : r == 12u ? 4u : 6u;
      if (r == 6u || r == 7u || r == 12u || r == 13u) {
        if ((((q.y >> 16) - now) & 0xffffu) >= kMaxDelay) mine |= 1u << s0;
        if ((((q.w >> 16) - now) & 0xffffu) >= kMaxDelay) mine |= 2u << s0;
      }
      const uint32_t exp = meta_busy(meta) &
                           ((uint32_t)__shfl((int)mine, (int)(g0 + 6u)) |
                            (uint32_t)__shfl((int)mine, (int)(g0 + 7u)) |
                            (uint32_t)__shfl((int)mine, (int)(g0 + 12u)) |
                            (uint32_t)__shfl((int)mine, (int)(g0 + 13u)));
      if (!exp) continue;
      if (r == 0u) {
        __hip_atomic_fetch_and(meta_ptr(bk, (uint32_t)b).p, ~((exp << 16) | (exp << 24)),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        count += (uint64_t)__builtin_popcount(exp);
      }
      if (!plain && (r == 14u || r == 15u)) {
        const uint32_t base = r == 14u ? 0u : 4u;
        const uint32_t oth[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
          const uint32_t y = oth[k];
          // y < nb: always, on a table that keeps its invariants
          if (((exp & meta_sec(meta)) >> (base + k)) & 1u && y < nb) {
            const uint32_t old = __hip_atomic_fetch_sub(meta_ptr(bk, y).p, 1u, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT);
            if (meta_moved(old) == 1u) *bloom_ptr(bk, y) = 0ull;
          }
        }
      }
    }
  }
  return count;
}

}  // namespace
}  // namespace ckpp
