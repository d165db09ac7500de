// Match process and Greedy Reorder Strategy (paper Section 4.1, Algorithm 1).  See
// include/fastgl_match.h for the contract.
//
// Match = set intersection through the ID map's kind of table (hash_table.h: a slot holds a position, here
// the row of the last feature matrix): the last mini-batch's IDs are inserted, the new mini-batch's IDs probe
// it; the misses are compacted in position order (count per block, rank) into the load lists.
//
// The pairwise overlaps of n mini-batches: many IDs of up to kMarkBatches mini-batches go through buckets that fit LDS
// (overlap.hip); otherwise ONE table over all their IDs.  Up to kMarkBatches mini-batches a slot has a byte per mini-batch
// beside it that every holder of the ID sets with a plain store (twice the rate of an atomic or), and the pairs are counted
// by reading those marks once, in order; beyond that, entries carry a 64-bit mask, and every ID adds its mask to its
// mini-batch's row of the count matrix (LDS histogram per workgroup, one atomic per workgroup and column).
//
// Match of two mini-batches of 1.15 M nodes, us, 16-byte entries -> positions: 130 -> 95 (insert 80 -> 46).
#include <vector>

#include "fastgl_match.h"
#include "hash_table.h"
#include "internal.h"

namespace fastgl {
namespace {

struct MatchArgs {
    const int64_t *prev_gid, *new_gid;
    int64_t n_prev, n_new;
    PositionTable table;      // rows of the last mini-batch
    int32_t *block_cnt;
    int nblocks;
    int32_t *src_row, *load_pos;
    int64_t *load_gid;
    int32_t *result;
};

struct GidAt {
    const int64_t *gid;
    __device__ __forceinline__ int64_t operator()(int64_t p) const { return gid[p]; }
};

__global__ __launch_bounds__(256) void k_match_fill(MatchArgs a)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < 2) a.result[i] = 0;
    fill_words(a.table, i);
}

// The IDs are distinct, so the compare-and-swap comes without a look at the slot.
__global__ __launch_bounds__(256) void k_match_insert_prev(MatchArgs a)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= a.n_prev) return;
    const int64_t gid = a.prev_gid[j];
    int32_t q = kEmptySlot;
    if (gid >= 0) claim_slot(a.table, gid, id_hash(gid), (int32_t)j, GidAt{a.prev_gid}, q, false);
    if (q != (int32_t)j) atomicAdd(&a.result[1], 1);          // negative or repeated ID
}

// Probe; hits get their row, misses -1 for now; misses are counted per block.
__global__ __launch_bounds__(kScanBlock) void k_match_probe(MatchArgs a)
{
    const int64_t i = (int64_t)blockIdx.x * kScanBlock + threadIdx.x;
    bool miss = false;
    if (i < a.n_new) {
        const int64_t gid = a.new_gid[i];
        int32_t row = -1;
        if (gid >= 0)
            row = find_position(a.table, gid, GidAt{a.prev_gid});
        else
            atomicAdd(&a.result[1], 1);
        a.src_row[i] = row;
        miss = row < 0;
    }
    const int c = __syncthreads_count(miss);
    if (threadIdx.x == 0) a.block_cnt[blockIdx.x] = c;
}

// More than kSumBlocks blocks only.
__global__ __launch_bounds__(kScanBlock) void k_match_scan(MatchArgs a)
{
    const int total = scan_block_counts(a.block_cnt, a.nblocks);
    if (threadIdx.x == 0) a.result[0] = total;
}

// SUM: the block counts are not scanned yet.  Four positions per thread, loaded before the counts: bound by latency, 1.15 M
// positions, 40 % misses, one position per thread 11.6 us, so 9.8.
constexpr int kRankThreads = kScanBlock / 4;
template <bool SUM>
__global__ __launch_bounds__(kRankThreads) void k_match_rank(MatchArgs a)
{
    const int64_t i0 = ((int64_t)blockIdx.x * kRankThreads + threadIdx.x) * 4;
    bool miss[4];
    int64_t gid[4];
    int c = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t i = i0 + u < a.n_new ? i0 + u : a.n_new - 1;          // past the end: the last one again
        miss[u] = a.src_row[i] < 0;
        gid[u] = a.new_gid[i];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        miss[u] = miss[u] && i0 + u < a.n_new;
        c += miss[u];
    }
    const int base = SUM ? sum_before<kRankThreads>(a.block_cnt, blockIdx.x) : a.block_cnt[blockIdx.x];
    int k;
    const int mine = block_exclusive_scan(c, base, k);
    if (SUM && threadIdx.x == 0 && (int)blockIdx.x == a.nblocks - 1) a.result[0] = base + mine;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (!miss[u]) continue;
        a.src_row[i0 + u] = -1 - k;
        a.load_pos[k] = (int32_t)(i0 + u);
        a.load_gid[k] = gid[u];
        ++k;
    }
}

// Row copy: one thread moves one VEC-byte piece; consecutive threads take consecutive pieces of a row.  The last piece of a
// row ends with it, so that rows of any length and alignment move 16 bytes per thread.  Bound by HBM.  STREAM: loads past the
// caches, as the stores go anyway: a row is read once, and what the loads leave behind pushes out what is still to be written.
// us, 400-byte rows, 60 % from the last matrix, cached loads / past the caches: 80 MB 41 / 41, 132 MB 68 / 69, 192 MB 91 / 74,
// 260 MB 122 / 99, 460 MB 195 / 173 (4.7 -> 5.3 TB/s);  460 MB right after the gather of its loaded rows 179 / 170.  The
// table gather gains nothing by it: alone behind a fill 119 / 127 at 192 MB, 235 / 238 at 460.  Windows of two mini-batches over and over,
// assembly and the two gathers, which find more of the table: 183 MB 71 + 128 / 75 + 121, 208 MB 79 + 143 / 84 + 136, 250 MB 97 + 164 / 98
// + 160, 294 MB 119 + 187 / 115 + 186.
constexpr int64_t kStreamBytes = (int64_t)160 << 20;

template <int ELEM, int VEC, bool STREAM>
__global__ __launch_bounds__(256) void k_assemble_rows(const char *__restrict__ X_prev, const char *__restrict__ X_load,
                                                       const int32_t *__restrict__ src_row, int64_t n_new,
                                                       int64_t row_bytes, int pieces, uint64_t pieces_inv, char *__restrict__ X_new)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t i = pieces > 1 ? (int64_t)__umul64hi((uint64_t)t, pieces_inv) : t;     // t / pieces: t * pieces < 2^64
    if (i >= n_new) return;
    const int64_t at = (t - i * pieces) * VEC, off = at < row_bytes - VEC ? at : row_bytes - VEC;
    const int32_t r = src_row[i];
    const char *src = r >= 0 ? X_prev + (int64_t)r * row_bytes : X_load + (int64_t)(-1 - r) * row_bytes;
    char *dst = X_new + i * row_bytes + off;
    using u32x4 = typename Words<ELEM>::x4;
    if constexpr (VEC == 16) {
        const u32x4 *from = reinterpret_cast<const u32x4 *>(src + off);
        __builtin_nontemporal_store(STREAM ? __builtin_nontemporal_load(from) : *from, reinterpret_cast<u32x4 *>(dst));
    } else if (VEC == 4)
        *reinterpret_cast<uint32_t *>(dst) = *reinterpret_cast<const uint32_t *>(src + off);
    else
        *reinterpret_cast<uint16_t *>(dst) = *reinterpret_cast<const uint16_t *>(src + off);
}

static_assert(sizeof(MaskSlot) <= kSlotRoom, "an entry fits its slot's room");
constexpr int kMarkBatches = 8;
// Windows of this many IDs go through buckets: five launches, against two and a fill that all the random accesses of few IDs
// hide behind.  us, one table / buckets, IDs that lie close together, IDs below 4 times a mini-batch's number, and of 40 bits:
//   2 mini-batches   66 000 15 / 25, 19 / 25, 23 / 25;  260 000 25 / 28, 29 / 29, 36 / 29;  400 000 31 / 32, 36 / 36, 42 / 33;  800 000 48 / 37, 56 / 40, 62 / 38
//   4                66 000 16 / 25, 16 / 25, 21 / 25;  260 000 27 / 28, 28 / 29, 34 / 28;  400 000 32 / 31, 35 / 32, 39 / 32;  800 000 51 / 36, 55 / 38, 57 / 36
//   8                66 000 26 / 33, 26 / 34, 29 / 34;  190 000 36 / 36, 36 / 36, 40 / 35;  400 000 46 / 39, 51 / 39, 52 / 39
// A program's window of two mini-batches, matches and assembly with it: 67 000 IDs 80 / 87, 264 000 102 / 105, 439 000 122 / 123,
// 502 000 150 / 146;  of three 503 000 166 / 160, 752 000 234 / 218.  Called alone with 1.15 M IDs a mini-batch: 4 of them 235 / 87 and, of
// 40 bits, 226 / 102, 8 519 / 199.  Beyond the upper line buckets of IDs that do not repeat outgrow their tables.
constexpr int64_t kBucketIds = (int64_t)7 << 16, kBucketIdsMany = (int64_t)3 << 16, kMostBucketIds = (int64_t)12 << 20;
constexpr int kCountBlocks = 256;            // workgroups that read the marks: one per compute unit

struct OverlapArgs {
    const int64_t *gid;
    int64_t offsets[FASTGL_MAX_REORDER_BATCHES + 1];
    int n;
    int64_t total;
    int64_t cap;
    unsigned long long *counts;
    int32_t *violations;
    PositionTable table;         // up to kMarkBatches
    unsigned char *marks;        // [cap][4 or 8] 1 where the mini-batch holds the ID, unless it is the slot's holder
    MaskSlot *masks;             // more: [cap]
    int32_t *slot_of;            // [total]
};

// Slots, and everything that is added up.  `violations` starts at the number of IDs: the count takes off every
// (ID, mini-batch) that it finds marked, which leaves the negative and the repeated ones.
template <typename MARK>
__global__ __launch_bounds__(256) void k_marks_fill(OverlapArgs a)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) *a.violations = (int32_t)a.total;
    if (i < (int64_t)a.n * a.n) a.counts[i] = 0;
    fill_words(a.table, i);
    if (i * kFillVec < a.cap) {
        int4 *m = reinterpret_cast<int4 *>(a.marks) + i * (sizeof(MARK) / 4);
#pragma unroll
        for (int k = 0; k < (int)sizeof(MARK) / 4; ++k) m[k] = make_int4(0, 0, 0, 0);
    }
}

// blockIdx.y = mini-batch, blockIdx.x walks its IDs.  The first mini-batch's come first and find their slots empty.
template <typename MARK>
__global__ __launch_bounds__(256) void k_marks_insert(OverlapArgs a)
{
    const int b = blockIdx.y;
    const int64_t p = a.offsets[b] + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= a.offsets[b + 1]) return;
    const int64_t gid = a.gid[p];
    if (gid < 0) return;
    int32_t q;
    const uint32_t slot = claim_slot(a.table, gid, near_hash(gid), (int32_t)p, GidAt{a.gid}, q, b > 0);
    if (q != (int32_t)p) a.marks[(size_t)slot * sizeof(MARK) + b] = 1;
}

// counts[i][j] = slots that both i and j hold: marked, or the slot's position is theirs.  A thread takes 16 bytes
// of marks at a time, with their slots; both arrays are rounded up to whole ones, filled like the rest.
template <typename MARK>
__global__ __launch_bounds__(kScanBlock) void k_marks_count(OverlapArgs a)
{
    constexpr int NB = sizeof(MARK), PER = 16 / NB, PAIRS = NB * (NB + 1) / 2;
    __shared__ int sum[PAIRS];
    if (threadIdx.x < PAIRS) sum[threadIdx.x] = 0;
    __syncthreads();
    int c[PAIRS];
#pragma unroll
    for (int k = 0; k < PAIRS; ++k) c[k] = 0;
    const int64_t pieces = (a.cap + PER - 1) / PER, step = (int64_t)gridDim.x * kScanBlock;
    for (int64_t i = (int64_t)blockIdx.x * kScanBlock + threadIdx.x; i < pieces; i += step) {
        const uint4 v = reinterpret_cast<const uint4 *>(a.marks)[i];
        uint32_t w[4] = {v.x, v.y, v.z, v.w};
        int32_t held[PER];
        if constexpr (PER == 4) {
            const int4 h = reinterpret_cast<const int4 *>(a.table.slot)[i];
            held[0] = h.x; held[1] = h.y; held[2] = h.z; held[3] = h.w;
        } else {
            const int2 h = reinterpret_cast<const int2 *>(a.table.slot)[i];
            held[0] = h.x; held[1] = h.y;
        }
#pragma unroll
        for (int s = 0; s < PER; ++s) {
            if (held[s] == kEmptySlot) continue;
            const int32_t p = a.table.position(held[s]);
            int b = 0;
            for (int x = 1; x < a.n; ++x) b += p >= a.offsets[x];
#pragma unroll
            for (int x = 0; x < NB; ++x) w[(s * NB + x) >> 2] |= b == x ? 1u << (8 * (x & 3)) : 0u;
            int k = 0;
#pragma unroll
            for (int x = 0; x < NB; ++x)
#pragma unroll
                for (int y = x; y < NB; ++y, ++k) {
                    const int at = s * NB;
                    c[k] += (w[(at + x) >> 2] >> (8 * (x & 3))) & (w[(at + y) >> 2] >> (8 * (y & 3))) & 1;
                }
        }
    }
#pragma unroll
    for (int k = 0; k < PAIRS; ++k) {
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) c[k] += __shfl_xor(c[k], d);
        if ((threadIdx.x & 63) == 0 && c[k]) atomicAdd(&sum[k], c[k]);
    }
    __syncthreads();
    if ((int)threadIdx.x < a.n * a.n) {
        const int i = threadIdx.x / a.n, j = threadIdx.x % a.n, x = i < j ? i : j, y = i < j ? j : i;
        const int v = sum[x * NB - x * (x - 1) / 2 + y - x];
        if (v) atomicAdd(&a.counts[threadIdx.x], (unsigned long long)v);
        if (v && i == j) atomicAdd(a.violations, -v);
    }
}

__global__ __launch_bounds__(256) void k_masks_fill(OverlapArgs a)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) *a.violations = 0;
    if (i < (int64_t)a.n * a.n) a.counts[i] = 0;
    if (i >= a.cap) return;
    MaskSlot e;
    e.key = -1;
    e.mask = 0;
    a.masks[i] = e;
}

// blockIdx.y = mini-batch, blockIdx.x walks its IDs.
__global__ __launch_bounds__(256) void k_overlap_insert(OverlapArgs a)
{
    const int b = blockIdx.y;
    const int64_t p = a.offsets[b] + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= a.offsets[b + 1]) return;
    const int64_t gid = a.gid[p];
    if (gid < 0) {
        a.slot_of[p] = kNoSlot;
        atomicAdd(a.violations, 1);
        return;
    }
    const uint32_t slot = insert_key(a.masks, (uint32_t)a.cap, gid);
    a.slot_of[p] = (int32_t)slot;
    const unsigned long long old = atomicOr(&a.masks[slot].mask, 1ull << b);
    if (old & (1ull << b)) atomicAdd(a.violations, 1);           // the mini-batch repeats this ID
}

__global__ __launch_bounds__(256) void k_overlap_count(OverlapArgs a)
{
    __shared__ int hist[FASTGL_MAX_REORDER_BATCHES];
    const int b = blockIdx.y;
    if (threadIdx.x < FASTGL_MAX_REORDER_BATCHES) hist[threadIdx.x] = 0;
    __syncthreads();
    const int64_t p = a.offsets[b] + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < a.offsets[b + 1]) {
        const int32_t slot = a.slot_of[p];
        unsigned long long m = slot != kNoSlot ? a.masks[slot].mask : 0ull;
        while (m) {
            const int j = __ffsll((long long)m) - 1;
            m &= m - 1;
            atomicAdd(&hist[j], 1);
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < a.n && hist[threadIdx.x])
        atomicAdd(&a.counts[(int64_t)b * a.n + threadIdx.x], (unsigned long long)hist[threadIdx.x]);
}

struct MatchLayout {
    size_t table, block_cnt, total;
};

MatchLayout match_layout(int64_t n_prev, int64_t n_new)
{
    MatchLayout L;
    size_t off = 0;
    L.table = off; off += align_up((size_t)(table_slots(n_prev) * kSlotRoom), 256);
    L.block_cnt = off; off += align_up((size_t)(ceil_div(n_new, kScanBlock) + 1) * 4, 256);
    L.total = off;
    return L;
}

struct OverlapLayout {
    size_t table, slot_of, total;
};

OverlapLayout overlap_layout(int64_t total_ids)
{
    OverlapLayout L;
    size_t off = 0;
    L.table = off; off += align_up((size_t)(table_slots(total_ids) * kSlotRoom), 256);
    L.slot_of = off; off += align_up((size_t)(total_ids > 0 ? total_ids : 1) * 4, 256);
    L.total = off;
    return L;
}

dim3 grid_for(int64_t items, int per) { return dim3((unsigned)(items > 0 ? ceil_div(items, per) : 1)); }

fastgl_status check_ws(void *workspace, size_t have, size_t need)
{
    if (!workspace || ((uintptr_t)workspace & 255)) {
        set_error("workspace must be a 256-byte aligned device buffer");
        return FASTGL_ERR_INVALID_ARG;
    }
    if (have < need) {
        set_error("workspace too small: %zu < %zu bytes", have, need);
        return FASTGL_ERR_WORKSPACE;
    }
    return FASTGL_OK;
}

}  // namespace
}  // namespace fastgl

using namespace fastgl;

extern "C" {

size_t fastgl_match_workspace_bytes(int64_t n_prev, int64_t n_new)
{
    if (n_prev < 0 || n_new < 0 || n_prev >= kMaxIds || n_new >= kMaxIds) return 0;
    return match_layout(n_prev, n_new).total;
}

fastgl_status fastgl_match(const int64_t *prev_gid, int64_t n_prev, const int64_t *new_gid, int64_t n_new,
                           int32_t *src_row, int32_t *load_pos, int64_t *load_gid, int32_t *result,
                           void *workspace, size_t workspace_bytes, void *stream)
{
    if (n_prev < 0 || n_new < 0) {
        set_error("negative size (n_prev=%lld n_new=%lld)", (long long)n_prev, (long long)n_new);
        return FASTGL_ERR_INVALID_ARG;
    }
    if (n_prev >= kMaxIds || n_new >= kMaxIds) {
        set_error("n_prev and n_new must stay below 2^30");
        return FASTGL_ERR_UNSUPPORTED;
    }
    if ((n_prev > 0 && !prev_gid) || (n_new > 0 && (!new_gid || !src_row || !load_pos || !load_gid)) || !result) {
        set_error("NULL array (prev_gid, new_gid, src_row, load_pos, load_gid or result)");
        return FASTGL_ERR_INVALID_ARG;
    }
    if ((((uintptr_t)prev_gid | (uintptr_t)new_gid | (uintptr_t)load_gid) & 7) ||
        (((uintptr_t)src_row | (uintptr_t)load_pos | (uintptr_t)result) & 3)) {
        set_error("ID arrays must be 8-byte aligned, src_row, load_pos and result 4-byte aligned");
        return FASTGL_ERR_INVALID_ARG;
    }
    const MatchLayout L = match_layout(n_prev, n_new);
    fastgl_status st = check_ws(workspace, workspace_bytes, L.total);
    if (st != FASTGL_OK) return st;
    MatchArgs a = {};
    a.prev_gid = prev_gid; a.new_gid = new_gid; a.n_prev = n_prev; a.n_new = n_new;
    const int64_t cap = position_slots(n_prev, table_slots(n_prev));
    a.table = PositionTable{(int32_t *)((char *)workspace + L.table), (uint32_t)cap, position_bits(n_prev)};
    a.block_cnt = (int32_t *)((char *)workspace + L.block_cnt);
    a.nblocks = (int)ceil_div(n_new, kScanBlock);
    a.src_row = src_row; a.load_pos = load_pos; a.load_gid = load_gid; a.result = result;
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(k_match_fill, grid_for(cap, 256 * kFillVec), dim3(256), 0, s, a);
    FASTGL_LAUNCH_CHECK("fastgl_match (fill)");
    if (n_prev > 0) {
        hipLaunchKernelGGL(k_match_insert_prev, grid_for(n_prev, 256), dim3(256), 0, s, a);
        FASTGL_LAUNCH_CHECK("fastgl_match (insert)");
    }
    if (n_new > 0) {
        hipLaunchKernelGGL(k_match_probe, dim3((unsigned)a.nblocks), dim3(kScanBlock), 0, s, a);
        FASTGL_LAUNCH_CHECK("fastgl_match (probe)");
        if (a.nblocks <= kSumBlocks) {
            hipLaunchKernelGGL(k_match_rank<true>, dim3((unsigned)a.nblocks), dim3(kRankThreads), 0, s, a);
        } else {
            hipLaunchKernelGGL(k_match_scan, dim3(1), dim3(kScanBlock), 0, s, a);
            FASTGL_LAUNCH_CHECK("fastgl_match (scan)");
            hipLaunchKernelGGL(k_match_rank<false>, dim3((unsigned)a.nblocks), dim3(kRankThreads), 0, s, a);
        }
        FASTGL_LAUNCH_CHECK("fastgl_match (rank)");
    }
    return FASTGL_OK;
}

fastgl_status fastgl_assemble_rows(const void *X_prev, int64_t n_prev, const void *X_load, int64_t n_load,
                                   const int32_t *src_row, int64_t n_new, int64_t feat, fastgl_dtype dtype,
                                   void *X_new, void *stream)
{
    if (n_prev < 0 || n_load < 0 || n_new < 0 || feat <= 0) {
        set_error("bad size (n_prev=%lld n_load=%lld n_new=%lld feat=%lld)", (long long)n_prev, (long long)n_load,
                  (long long)n_new, (long long)feat);
        return FASTGL_ERR_INVALID_ARG;
    }
    if ((int)dtype < 0 || (int)dtype > 1) {
        set_error("unknown dtype %d", (int)dtype);
        return FASTGL_ERR_INVALID_ARG;
    }
    if (n_new == 0) return FASTGL_OK;
    if (!src_row || !X_new || (n_prev > 0 && !X_prev) || (n_load > 0 && !X_load)) {
        set_error("NULL array (src_row, X_new, X_prev or X_load)");
        return FASTGL_ERR_INVALID_ARG;
    }
    const int64_t elem = dtype == FASTGL_F32 ? 4 : 2;
    if ((((uintptr_t)X_prev | (uintptr_t)X_load | (uintptr_t)X_new) & (uintptr_t)(elem - 1)) || ((uintptr_t)src_row & 3)) {
        set_error("misaligned buffer");
        return FASTGL_ERR_INVALID_ARG;
    }
    if (n_new >= kMaxIds || feat > ((int64_t)1 << 24)) {
        set_error("assemble too large");
        return FASTGL_ERR_UNSUPPORTED;
    }
    const int64_t row_bytes = feat * elem;
    const int vec = row_bytes >= 16 ? 16 : (int)elem;
    const int64_t pieces = ceil_div(row_bytes, (int64_t)vec);
    const int64_t threads = n_new * pieces;
    if (ceil_div(threads, 256) >= INT32_MAX) {
        set_error("assemble too large");
        return FASTGL_ERR_UNSUPPORTED;
    }
    const dim3 g = grid_for(threads, 256);
    hipStream_t s = (hipStream_t)stream;
    const char *xp = (const char *)X_prev, *xl = (const char *)X_load;
    const uint64_t inv = pieces > 1 ? UINT64_MAX / (uint64_t)pieces + 1 : 0;       // ceil(2^64 / pieces)
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, g, dim3(256), 0, s, xp, xl, src_row, n_new, row_bytes, (int)pieces, inv, (char *)X_new);
    };
    const bool past = n_new * row_bytes >= kStreamBytes;
    if (dtype == FASTGL_F32) {
        if (vec == 16) past ? go(k_assemble_rows<4, 16, true>) : go(k_assemble_rows<4, 16, false>);
        else go(k_assemble_rows<4, 4, false>);
    } else {
        if (vec == 16) past ? go(k_assemble_rows<2, 16, true>) : go(k_assemble_rows<2, 16, false>);
        else go(k_assemble_rows<2, 2, false>);
    }
    FASTGL_LAUNCH_CHECK("fastgl_assemble_rows");
    return FASTGL_OK;
}

size_t fastgl_overlap_workspace_bytes(int64_t total_ids)
{
    if (total_ids < 0 || total_ids >= kMaxIds) return 0;
    return overlap_layout(total_ids).total;
}

fastgl_status fastgl_overlap_counts(const int64_t *gid, const int64_t *offsets_host, int n, int64_t *counts,
                                    int32_t *violations, void *workspace, size_t workspace_bytes, void *stream)
{
    if (n < 0 || n > FASTGL_MAX_REORDER_BATCHES) {
        set_error("n must be in [0, %d]", FASTGL_MAX_REORDER_BATCHES);
        return FASTGL_ERR_INVALID_ARG;
    }
    if (!offsets_host || !violations || (n > 0 && !counts)) {
        set_error("NULL array (offsets_host, counts or violations)");
        return FASTGL_ERR_INVALID_ARG;
    }
    int64_t longest = 0;
    for (int b = 0; b < n; ++b) {
        if (offsets_host[b] < 0 || offsets_host[b + 1] < offsets_host[b]) {
            set_error("offsets_host must start at >= 0 and not decrease");
            return FASTGL_ERR_INVALID_ARG;
        }
        if (offsets_host[b + 1] - offsets_host[b] > longest) longest = offsets_host[b + 1] - offsets_host[b];
    }
    if (n > 0 && offsets_host[0] != 0) {
        set_error("offsets_host[0] must be 0");
        return FASTGL_ERR_INVALID_ARG;
    }
    const int64_t total = n > 0 ? offsets_host[n] : 0;
    if (total >= kMaxIds) {
        set_error("total number of IDs must stay below 2^30");
        return FASTGL_ERR_UNSUPPORTED;
    }
    if ((total > 0 && !gid) || ((uintptr_t)gid & 7) || ((uintptr_t)counts & 7) || ((uintptr_t)violations & 3)) {
        set_error("gid is NULL or an array is misaligned");
        return FASTGL_ERR_INVALID_ARG;
    }
    const OverlapLayout L = overlap_layout(total);
    fastgl_status st = check_ws(workspace, workspace_bytes, L.total);
    if (st != FASTGL_OK) return st;
    OverlapArgs a = {};
    a.gid = gid; a.n = n; a.total = total;
    for (int b = 0; b <= n; ++b) a.offsets[b] = offsets_host[b];
    a.counts = (unsigned long long *)counts;
    a.violations = violations;
    a.cap = table_slots(total);
    hipStream_t s = (hipStream_t)stream;
    const dim3 g((unsigned)ceil_div(longest, 256), (unsigned)n);
    char *ws = (char *)workspace;
    if (n <= kMarkBatches && total >= (n <= 4 ? kBucketIds : kBucketIdsMany) && total <= kMostBucketIds)
        return launch_overlap_buckets(gid, offsets_host, n, counts, violations, ws, workspace_bytes, s);
    if (n > kMarkBatches) {
        a.masks = (MaskSlot *)(ws + L.table);
        a.slot_of = (int32_t *)(ws + L.slot_of);
        hipLaunchKernelGGL(k_masks_fill, grid_for(a.cap > n * n ? a.cap : n * n, 256), dim3(256), 0, s, a);
        FASTGL_LAUNCH_CHECK("fastgl_overlap_counts (fill)");
        if (longest == 0) return FASTGL_OK;
        hipLaunchKernelGGL(k_overlap_insert, g, dim3(256), 0, s, a);
        FASTGL_LAUNCH_CHECK("fastgl_overlap_counts (insert)");
        hipLaunchKernelGGL(k_overlap_count, g, dim3(256), 0, s, a);
        FASTGL_LAUNCH_CHECK("fastgl_overlap_counts (count)");
        return FASTGL_OK;
    }
    // the slots' positions, then their marks: at most 4 + 8 of the 16 bytes a slot has room for
    a.table = PositionTable{(int32_t *)(ws + L.table), (uint32_t)a.cap, position_bits(total)};
    a.marks = (unsigned char *)(ws + L.table + align_up((size_t)a.cap * 4, 256));
    const bool four = n <= 4;
    const dim3 gf = grid_for(a.cap, 256 * kFillVec);
    if (four) hipLaunchKernelGGL(k_marks_fill<uint32_t>, gf, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(k_marks_fill<uint64_t>, gf, dim3(256), 0, s, a);
    FASTGL_LAUNCH_CHECK("fastgl_overlap_counts (fill)");
    if (longest == 0) return FASTGL_OK;
    if (four) hipLaunchKernelGGL(k_marks_insert<uint32_t>, g, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(k_marks_insert<uint64_t>, g, dim3(256), 0, s, a);
    FASTGL_LAUNCH_CHECK("fastgl_overlap_counts (insert)");
    if (four) hipLaunchKernelGGL(k_marks_count<uint32_t>, dim3(kCountBlocks), dim3(kScanBlock), 0, s, a);
    else hipLaunchKernelGGL(k_marks_count<uint64_t>, dim3(kCountBlocks), dim3(kScanBlock), 0, s, a);
    FASTGL_LAUNCH_CHECK("fastgl_overlap_counts (count)");
    return FASTGL_OK;
}

fastgl_status fastgl_greedy_reorder(const int64_t *overlap_host, const int64_t *size_host, int64_t n,
                                    int32_t *order_host)
{
    if (n < 0 || n > ((int64_t)1 << 15)) {
        set_error("n must be in [0, 32768]");
        return FASTGL_ERR_INVALID_ARG;
    }
    if (n > 0 && (!overlap_host || !size_host || !order_host)) {
        set_error("NULL host array");
        return FASTGL_ERR_INVALID_ARG;
    }
    if (n == 0) return FASTGL_OK;
    // Walk the list: `last` is the mini-batch appended last, `todo` the ones still to place.
    std::vector<int32_t> todo;
    for (int64_t k = 1; k < n; ++k) todo.push_back((int32_t)k);
    int32_t last = 0;
    int64_t filled = 0;
    order_host[filled++] = 0;
    while (!todo.empty()) {
        size_t best = 0;
        double best_deg = -1.0;
        for (size_t t = 0; t < todo.size(); ++t) {        // ascending index, strict improvement: ties stay low
            const int32_t k = todo[t];
            const int64_t small = size_host[last] < size_host[k] ? size_host[last] : size_host[k];
            const double deg = small > 0 ? (double)overlap_host[(int64_t)last * n + k] / (double)small : 0.0;
            if (deg > best_deg) {
                best_deg = deg;
                best = t;
            }
        }
        last = todo[best];
        todo.erase(todo.begin() + (long)best);
        order_host[filled++] = last;
    }
    return FASTGL_OK;
}

}  // extern "C"
