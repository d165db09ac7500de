// Device-side pieces shared by the ID map and the Match process: open-addressing tables of 64-bit
// global IDs (linear probing) and a workgroup-wide exclusive prefix sum.
//
// A slot holds 32 bits, -1 while empty: the POSITION in the input of an ID that hashed there, through which
// the key is read from the input itself, and in the bits above it as much of the ID's hash as fits (9 bits for
// 3 M input IDs), so that walking past other IDs reads their keys hardly ever.  What bounds the kernels around the table is the number of
// accesses at random addresses, each a line of its own over the fabric, whatever is in it: measured on
// tables of 7 to 72 MB, 50-65 G loads/s, 56-77 G stores/s, but 25 G read-modify-writes/s (compare-and-swap,
// minimum or or, 4 or 8 bytes, with or without result).  So a fresh ID costs one compare-and-swap and
// nothing else (a table of keys needs a second access for the value, and 2 to 4 times the fill).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fastgl {

constexpr int kScanBlock = 1024;             // threads (= positions) per block of the counting / ranking passes
constexpr int64_t kMaxIds = (int64_t)1 << 30;
constexpr int32_t kNoSlot = 0x7FFFFFFF;      // no table has this many slots

constexpr int32_t kEmptySlot = -1;

// Bytes per slot that a caller's workspace must have room for: part of the interface (what it refuses as too
// small), four times what a slot of positions takes.
constexpr int64_t kSlotRoom = 16;

// Bits of a position below n in a slot; the other 31 - bits hold a piece of the hash (never the sign bit).
inline int position_bits(int64_t n)
{
    int b = 1;
    while (b < 30 && ((int64_t)1 << b) < n) ++b;
    return b;
}

constexpr int kFillVec = 4;                  // 32-bit words per thread of a table fill; tables have room for whole ones

// Entry of the overlap table for many mini-batches: a key and the 64-bit mask of the mini-batches holding it.
struct __attribute__((aligned(16))) MaskSlot {
    int64_t key;              // -1 while empty
    unsigned long long mask;
};

// Entries that the workspace has room for, for n DISTINCT keys (Match, overlap counts): 2n (at least 1024), so a table
// of that many is never more than half full and a probe sequence always ends at an empty slot.
inline int64_t table_slots(int64_t n)
{
    const int64_t cap = 2 * n;
    return cap < 1024 ? 1024 : cap;
}

// The same for the n input IDs of the ID map, most of which repeat (a sampled hop holds every hub many times): 1.5 n.
inline int64_t idmap_slots(int64_t n)
{
    const int64_t cap = n + n / 2;
    return cap < 1024 ? 1024 : cap;
}

// Slots of a table of positions of n IDs whose workspace has room for `room` entries of kSlotRoom bytes: four per ID,
// which is at most what the room holds in 32-bit slots, so that a look nearly always ends at its first slot.  An ID's
// chain of dependent accesses (slot, key, next slot) is what a small table's launches wait for, a wavefront for the
// longest of 64: us with 1.5 / 3 / 4 / 6 slots per ID, ordered maps of three hops of 34 seeds 137 / 108 / 105 / 104, of
// two hops of 5 017 seeds 124 / 113 / 113 / 114, of the headline's three hops 339 / 334 / 334 / 337; with 2 / 3 / 4 / 8,
// windows of mini-batches of 34 seeds 133 / 126 / 121 / 120, of 8 000 1 580 / 1 550 / 1 545 / 1 554.
inline int64_t position_slots(int64_t n, int64_t room)
{
    static_assert(4 * (int64_t)sizeof(int32_t) <= kSlotRoom, "four slots to an entry's room");
    const int64_t cap = n <= kMaxIds / 4 ? 4 * n : 0;        // slot numbers stay below 2^30
    return cap > room ? cap : room;
}

// Hashes of an ID, both one to one.  A multiplication alone spreads IDs that lie close together, or in steps of most
// numbers, more evenly than chance (ID maps of the headline's hops 275 us, 281 with near_hash), but keeps multiples of some
// numbers (Fibonacci numbers, with this odd one) together.
constexpr uint64_t kOdd = 0x9E3779B97F4A7C15ull;
__device__ __forceinline__ uint64_t id_hash(int64_t gid) { return (uint64_t)gid * kOdd; }

// For windows of mini-batches: the low bits first take what a hash of the others says, so that every run of 2^kNearBits
// IDs is dealt evenly, on its own.  Overlaps of 4 x 16 385 multiples of 14 930 352, us: one table 117 000 with id_hash, buckets 458 000;
// 27 with this.  4 x 1.15 M IDs below 2.4 M: 85 with either, 102 with the second multiplication over all bits.
constexpr int kNearBits = 22;
__device__ __forceinline__ uint64_t near_hash(int64_t gid)
{
    uint64_t far = ((uint64_t)gid >> kNearBits) * kOdd;
    far ^= far >> 32;
    return ((uint64_t)gid ^ far * kOdd >> (64 - kNearBits)) * kOdd;
}

// Slot of a hash in a table of `cap` slots (any size below 2^31, not only powers of two): its upper
// half scaled to [0, cap).
__device__ __forceinline__ uint32_t hash_slot(uint64_t hash, uint32_t cap)
{
    return (uint32_t)((hash >> 32) * cap >> 32);
}

__device__ __forceinline__ uint32_t next_slot(uint32_t slot, uint32_t cap) { return slot + 1 == cap ? 0u : slot + 1; }

// A table of positions and what a look-up needs to know of it.
struct PositionTable {
    int32_t *slot;            // [cap]
    uint32_t cap;
    int32_t bits;             // position_bits of the input

    __device__ __forceinline__ int32_t position(int32_t word) const { return word & ((1 << bits) - 1); }
    // the lower half of the hash, whose upper half chose the slot
    __device__ __forceinline__ int32_t tag(uint64_t hash) const { return (int32_t)(((uint32_t)hash >> (1 + bits)) << bits); }
    __device__ __forceinline__ bool same_tag(int32_t word, int32_t t) const { return (word ^ t) >> bits == 0; }
};

// Slot whose key is gid after the call; `holder` = the position it was seen to hold (p: this call
// put it there).  key_at(position) = the ID at an input position; hash: of gid, the same function for a whole
// table.  `look`: the slot is first read by a load that may come from this XCD's L2: the KEY of a slot never changes once it has one (a smaller position of the same
// ID may replace the one it holds), so an old reading can only show the empty marker, and the compare-and-swap
// settles that.  Without (IDs that are not expected in the table yet) the compare-and-swap comes first.
// Ends because the table always keeps empty slots.
template <class KeyAt>
__device__ __forceinline__ uint32_t claim_slot(const PositionTable &t, int64_t gid, uint64_t hash, int32_t p,
                                               const KeyAt &key_at, int32_t &holder, bool look)
{
    uint32_t slot = hash_slot(hash, t.cap);
    const int32_t tag = t.tag(hash);
    for (;;) {
        int32_t w = kEmptySlot;
        if (look) w = __hip_atomic_load(&t.slot[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (w == kEmptySlot) {
            w = atomicCAS(&t.slot[slot], kEmptySlot, tag | p);
            if (w == kEmptySlot) {
                holder = p;
                return slot;
            }
        }
        if (t.same_tag(w, tag)) {
            holder = t.position(w);
            if (key_at(holder) == gid) return slot;
        }
        slot = next_slot(slot, t.cap);
    }
}

// Position that holds gid in a table by id_hash that is no longer written, or kEmptySlot.  Ends at the first empty slot.
template <class KeyAt>
__device__ __forceinline__ int32_t find_position(const PositionTable &t, int64_t gid, const KeyAt &key_at)
{
    uint32_t slot = hash_slot(id_hash(gid), t.cap);
    const int32_t tag = t.tag(id_hash(gid));
    for (;;) {
        const int32_t w = t.slot[slot];
        if (w == kEmptySlot) return kEmptySlot;
        if (t.same_tag(w, tag) && key_at(t.position(w)) == gid) return t.position(w);
        slot = next_slot(slot, t.cap);
    }
}

// The four words of a fill thread; words behind `cap` belong to the table's rounded-up room.
__device__ __forceinline__ void fill_words(const PositionTable &t, int64_t thread)
{
    if (thread * kFillVec < (int64_t)t.cap) reinterpret_cast<int4 *>(t.slot)[thread] = make_int4(-1, -1, -1, -1);
}

// Entry of the table of MaskSlots that holds gid after the call.
__device__ __forceinline__ uint32_t insert_key(MaskSlot *table, uint32_t cap, int64_t gid)
{
    uint32_t slot = hash_slot(id_hash(gid), cap);
    for (;;) {
        int64_t k = __hip_atomic_load(&table[slot].key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (k == -1) {
            k = (int64_t)atomicCAS((unsigned long long *)&table[slot].key, (unsigned long long)-1ll, (unsigned long long)gid);
            if (k == -1) return slot;
        }
        if (k == gid) return slot;
        slot = next_slot(slot, cap);
    }
}

// Exclusive prefix sum of v over the workgroup (blockDim.x a multiple of 64, at most kScanBlock),
// `base` added to every result; returns the workgroup's total to every thread.
__device__ __forceinline__ int block_exclusive_scan(int v, int base, int &out_excl)
{
    __shared__ int wave_sum[kScanBlock / 64];
    __shared__ int total_s;
    const int lane = threadIdx.x & 63, wv = threadIdx.x / 64;
    int incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_up(incl, d);
        if (lane >= d) incl += t;
    }
    if (lane == 63) wave_sum[wv] = incl;
    __syncthreads();
    if (wv == 0) {
        const int nw = blockDim.x / 64;
        const int w = lane < nw ? wave_sum[lane] : 0;
        int wi = w;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int t = __shfl_up(wi, d);
            if (lane >= d) wi += t;
        }
        if (lane < nw) wave_sum[lane] = wi - w;
        if (lane == nw - 1) total_s = wi;
    }
    __syncthreads();
    out_excl = base + wave_sum[wv] + incl - v;
    const int total = total_s;
    __syncthreads();
    return total;
}

// Sum of block_cnt[0 .. b) to every thread of a workgroup of kScanBlock.  Up to kSumBlocks blocks every workgroup
// of a ranking pass adds up the counts before its own (at most 16 KB, from L2); a launch of one workgroup that
// scans them costs 5 us, more than the kernel that counted a small hop.  Beyond that, scan_block_counts.
constexpr int kSumBlocks = 4096;

template <int THREADS = kScanBlock>
__device__ __forceinline__ int sum_before(const int32_t *block_cnt, int b)
{
    __shared__ int wave_sum_b[THREADS / 64];
    int s = 0;
#pragma unroll
    for (int k = 0; k < kSumBlocks / THREADS; ++k) {
        const int i = k * THREADS + threadIdx.x;
        if (i < b) s += block_cnt[i];
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d);
    if ((threadIdx.x & 63) == 0) wave_sum_b[threadIdx.x / 64] = s;
    __syncthreads();
    int total = 0;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) total += wave_sum_b[w];
    return total;
}

// Block counts -> exclusive block offsets in place, by ONE workgroup of kScanBlock threads; returns
// the grand total to every thread.
__device__ __forceinline__ int scan_block_counts(int32_t *block_cnt, int nblocks)
{
    int running = 0;
    for (int b0 = 0; b0 < nblocks; b0 += kScanBlock) {
        const int b = b0 + threadIdx.x;
        const int v = b < nblocks ? block_cnt[b] : 0;
        int excl;
        const int total = block_exclusive_scan(v, running, excl);
        if (b < nblocks) block_cnt[b] = excl;
        running += total;
    }
    return running;
}

}  // namespace fastgl
