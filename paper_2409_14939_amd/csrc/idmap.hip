// ID map of the sample phase (paper Section 2.2; Section 4.3, Algorithm 2): global IDs of one
// sampled hop -> consecutive local IDs.  See include/fastgl_idmap.h for the contract.
//
// Table: open addressing with linear probing, 32-bit slots that hold input positions (hash_table.h),
// four slots per input ID (most of which repeat).
//
// FUSED mode is Algorithm 2: destinations claim their slots first, then every neighbour entry; the claimant of
// a slot takes the next local ID from a counter (one atomic add per workgroup, the threads that claimed a slot
// share it), a second kernel translates.
// ORDERED mode replaces the counter by "smallest position seen at this slot" (an atomic minimum, needed only
// where a later position got there first), then a prefix count over the positions that are first occurrences
// gives every distinct ID its rank in order of first appearance.
//
// A neighbour entry whose slot holds a destination, or that claimed the slot itself, has its local ID at
// once; only the others are left to the translation (about half of a sampled hop's).  In FUSED mode they
// remember the claimant's position and copy the local ID it wrote; in ORDERED mode the slot, where the ranking
// pass has replaced the position of a first neighbour entry by its local ID (a destination's position is its
// local ID).
//
// Bound by random accesses.  Products-shaped hop of 0.51 M destinations and 2.56 M neighbours, us, 16-byte
// entries {key, smallest position, local ID} -> positions -> marks of the displaced:  ordered 265 -> 166 -> 139 (insert 134 -> 108
// -> 96, count 51 -> 23 -> 5, rank 22 -> 18, translate 43 -> 11);  fused 153 -> 124 (destinations 35 -> 22, translate 35 -> 11).
#include "fastgl_idmap.h"
#include "hash_table.h"
#include "internal.h"

namespace fastgl {
namespace {

constexpr int32_t kFirstBit = (int32_t)0x80000000u;

struct IdmapArgs {
    const int64_t *dst_gid, *nbr_gid;
    int64_t n_dst, n_nbr, n;
    PositionTable table;      // positions of input IDs; ORDERED: a first neighbour entry's local ID after ranking
    int32_t *ref;             // ORDERED: [n] slot of every input position, bit 31 set on (candidates for) first
                              // occurrences; FUSED: [n_nbr] neighbour entry that claimed the ID;
                              // kNoSlot: nothing to translate
    unsigned char *displaced; // ORDERED: [n] 1 where a smaller position of the same ID came after this one
    int32_t *block_cnt;       // [blocks + 1]
    int32_t *local_nbr;
    int64_t *unique_gid;
    int32_t *result;          // [0] U, [1] violations
    int nblocks;
    int fused;
};

__device__ __forceinline__ int64_t id_at(const IdmapArgs &a, int64_t p)
{
    return p < a.n_dst ? a.dst_gid[p] : a.nbr_gid[p - a.n_dst];
}

struct IdAt {
    const IdmapArgs &a;
    __device__ __forceinline__ int64_t operator()(int64_t p) const { return id_at(a, p); }
};

__global__ __launch_bounds__(256) void k_idmap_fill(IdmapArgs a)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) {
        a.result[0] = a.fused ? (int32_t)a.n_dst : 0;
        a.result[1] = 0;
    }
    fill_words(a.table, i);
    if (!a.fused && i * 16 < a.n) reinterpret_cast<int4 *>(a.displaced)[i] = make_int4(0, 0, 0, 0);
}

// ORDERED pass 1: claim slots, keep the smallest position per slot.  Destinations find their slots empty and do not look.
// A position that was its ID's smallest when it came is marked by the smaller one that comes after it, so that nobody has to
// read the slots a second time to see which are left.  (Counting them per block here, up when they come and down when they
// are displaced, is slower than the pass below: the atomics meet in a few lines, 96 -> 105 us, with one small hop 14 -> 27.)
__global__ __launch_bounds__(256) void k_idmap_insert_min(IdmapArgs a)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= a.n) return;
    const int64_t gid = id_at(a, p);
    int32_t ref = kNoSlot;
    if (gid < 0) {
        if (p >= a.n_dst) a.local_nbr[p - a.n_dst] = -1;
        atomicAdd(&a.result[1], 1);
    } else {
        int32_t q;
        const uint32_t slot = claim_slot(a.table, gid, id_hash(gid), (int32_t)p, IdAt{a}, q, p >= a.n_dst);
        if (q > (int32_t)p) {
            q = a.table.position(atomicMin(&a.table.slot[slot], a.table.tag(id_hash(gid)) | (int32_t)p));
            if (q > (int32_t)p) a.displaced[q] = 1;
        }
        if (q >= (int32_t)p)
            ref = (int32_t)slot | kFirstBit;
        else if (q < a.n_dst && p >= a.n_dst)
            a.local_nbr[p - a.n_dst] = q;
        else
            ref = (int32_t)slot;
    }
    a.ref[p] = ref;
}

// ORDERED pass 2: how many positions of every block of kScanBlock are first occurrences, and which are not after all.
// Four positions per thread; the arrays have room for whole fours.
constexpr int kCountThreads = kScanBlock / 4;
__global__ __launch_bounds__(kCountThreads) void k_idmap_count(IdmapArgs a)
{
    __shared__ int wave_sum[kCountThreads / 64];
    const int64_t p = ((int64_t)blockIdx.x * kCountThreads + threadIdx.x) * 4;
    int c = 0;
    if (p < a.n) {
        const int4 r = *reinterpret_cast<const int4 *>(a.ref + p);
        const uint32_t d = *reinterpret_cast<const uint32_t *>(a.displaced + p);
        const int32_t ref[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (p + i >= a.n || ref[i] >= 0) continue;        // bit 31
            if (d >> (8 * i) & 0xFF) a.ref[p + i] = ref[i] & kNoSlot;
            else ++c;
        }
    }
#pragma unroll
    for (int k = 32; k > 0; k >>= 1) c += __shfl_xor(c, k);
    if ((threadIdx.x & 63) == 0) wave_sum[threadIdx.x / 64] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        int total = 0;
#pragma unroll
        for (int w = 0; w < kCountThreads / 64; ++w) total += wave_sum[w];
        a.block_cnt[blockIdx.x] = total;
    }
}

// More than kSumBlocks blocks only: block counts -> block offsets, in place, with the total behind them.
// One workgroup.
__global__ __launch_bounds__(kScanBlock) void k_idmap_scan(IdmapArgs a)
{
    const int total = scan_block_counts(a.block_cnt, a.nblocks);
    if (threadIdx.x == 0) a.result[0] = total;
}

// ORDERED pass 3: rank of every first occurrence = its local ID.  SUM: the block counts are not scanned yet.
template <bool SUM>
__global__ __launch_bounds__(kCountThreads) void k_idmap_rank(IdmapArgs a)
{
    const int64_t p0 = ((int64_t)blockIdx.x * kCountThreads + threadIdx.x) * 4;
    int32_t ref[4] = {kNoSlot, kNoSlot, kNoSlot, kNoSlot};
    int64_t gid[4];
    if (p0 < a.n) {
        const int4 r = *reinterpret_cast<const int4 *>(a.ref + p0);
        ref[0] = r.x; ref[1] = r.y; ref[2] = r.z; ref[3] = r.w;
    }
    int c = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (p0 + i >= a.n) ref[i] = kNoSlot;
        if (ref[i] < 0) {                          // bit 31
            gid[i] = id_at(a, p0 + i);
            ++c;
        }
    }
    const int base = SUM ? sum_before<kCountThreads>(a.block_cnt, blockIdx.x) : a.block_cnt[blockIdx.x];
    int rank;
    const int mine = block_exclusive_scan(c, base, rank);
    if (SUM && threadIdx.x == 0 && (int)blockIdx.x == a.nblocks - 1) a.result[0] = base + mine;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t p = p0 + i;
        const bool first = ref[i] < 0;
        if (first) {
            a.unique_gid[rank] = gid[i];
            if (p >= a.n_dst) {
                a.table.slot[ref[i] & kNoSlot] = rank;
                a.local_nbr[p - a.n_dst] = rank;
            }
        }
        if (p < a.n_dst && (!first || rank != (int)p)) atomicAdd(&a.result[1], 1);   // repeated destination
        rank += first;
    }
}

// ORDERED pass 4: the entries that neither are first occurrences nor met a destination.
__global__ __launch_bounds__(256) void k_idmap_translate(IdmapArgs a)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= a.n_nbr) return;
    const int32_t ref = a.ref[a.n_dst + e];
    if (ref >= 0 && ref != kNoSlot) a.local_nbr[e] = a.table.position(a.table.slot[ref]);
}

// FUSED pass 1a: destination i takes local ID i.
__global__ __launch_bounds__(256) void k_idmap_fused_dst(IdmapArgs a)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= a.n_dst) return;
    const int64_t gid = a.dst_gid[p];
    int32_t q = kEmptySlot;
    if (gid >= 0) claim_slot(a.table, gid, id_hash(gid), (int32_t)p, IdAt{a}, q, false);
    if (q == (int32_t)p)
        a.unique_gid[p] = gid;
    else
        atomicAdd(&a.result[1], 1);               // negative or repeated destination
}

// FUSED pass 1b (Algorithm 2): whoever claims a slot takes the next local ID.  The claimants of a
// workgroup share one atomic add on the counter (a prefix count inside the workgroup hands out the
// IDs of the range it returns).
__global__ __launch_bounds__(kScanBlock) void k_idmap_fused_nbr(IdmapArgs a)
{
    __shared__ int range_base;
    const int64_t e = (int64_t)blockIdx.x * kScanBlock + threadIdx.x;
    const bool active = e < a.n_nbr;
    const int64_t gid = active ? a.nbr_gid[e] : -1;
    const int32_t p = (int32_t)(a.n_dst + e);
    int32_t q = kEmptySlot;
    if (gid >= 0) claim_slot(a.table, gid, id_hash(gid), p, IdAt{a}, q, true);
    const bool fresh = gid >= 0 && q == p;
    if (active) {
        a.ref[e] = q >= (int32_t)a.n_dst && !fresh ? q - (int32_t)a.n_dst : kNoSlot;
        if (q < (int32_t)a.n_dst) a.local_nbr[e] = q;            // a destination's local ID; a rejected ID's -1
        if (gid < 0) atomicAdd(&a.result[1], 1);
    }
    int mine;
    const int claimed = block_exclusive_scan(fresh ? 1 : 0, 0, mine);
    if (claimed == 0) return;
    if (threadIdx.x == 0) range_base = atomicAdd(&a.result[0], claimed);
    __syncthreads();
    if (fresh) {
        const int l = range_base + mine;
        a.local_nbr[e] = l;
        a.unique_gid[l] = gid;
    }
}

// FUSED pass 2: the entries whose ID another neighbour entry claimed.  A claimant's own entry is not
// written here, so that reading it is safe.
__global__ __launch_bounds__(256) void k_idmap_fused_translate(IdmapArgs a)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= a.n_nbr) return;
    const int32_t ref = a.ref[e];
    if (ref != kNoSlot) a.local_nbr[e] = a.local_nbr[ref];
}

struct Layout {
    size_t table, ref, block_cnt, total;
};

Layout layout(int64_t n)
{
    const int64_t cap = idmap_slots(n);
    Layout L;
    size_t off = 0;
    L.table = off; off += align_up((size_t)(cap * kSlotRoom), 256);
    L.ref = off; off += align_up((size_t)(n > 0 ? n : 1) * 4, 256);      // room for whole fours
    L.block_cnt = off; off += align_up((size_t)(ceil_div(n, kScanBlock) + 1) * 4, 256);
    L.total = off;
    return L;
}

}  // namespace
}  // namespace fastgl

using namespace fastgl;

extern "C" {

int64_t fastgl_idmap_table_slots(int64_t n_ids)
{
    if (n_ids < 0 || n_ids >= kMaxIds) return 0;
    return idmap_slots(n_ids);
}

size_t fastgl_idmap_workspace_bytes(int64_t n_dst, int64_t n_nbr)
{
    if (n_dst < 0 || n_nbr < 0 || n_dst + n_nbr >= kMaxIds) return 0;
    return layout(n_dst + n_nbr).total;
}

fastgl_status fastgl_idmap(const int64_t *dst_gid, int64_t n_dst, const int64_t *nbr_gid, int64_t n_nbr,
                           fastgl_idmap_mode mode, int32_t *local_nbr, int64_t *unique_gid, int32_t *result,
                           void *workspace, size_t workspace_bytes, void *stream)
{
    if (n_dst < 0 || n_nbr < 0) {
        set_error("negative size (n_dst=%lld n_nbr=%lld)", (long long)n_dst, (long long)n_nbr);
        return FASTGL_ERR_INVALID_ARG;
    }
    if (n_dst + n_nbr >= kMaxIds) {
        set_error("n_dst + n_nbr must stay below 2^30");
        return FASTGL_ERR_UNSUPPORTED;
    }
    if ((int)mode != FASTGL_IDMAP_ORDERED && (int)mode != FASTGL_IDMAP_FUSED) {
        set_error("unknown ID-map mode %d", (int)mode);
        return FASTGL_ERR_INVALID_ARG;
    }
    const int64_t n = n_dst + n_nbr;
    if ((n_dst > 0 && !dst_gid) || (n_nbr > 0 && (!nbr_gid || !local_nbr)) || (n > 0 && !unique_gid) || !result) {
        set_error("NULL array (dst_gid, nbr_gid, local_nbr, unique_gid or result)");
        return FASTGL_ERR_INVALID_ARG;
    }
    if ((((uintptr_t)dst_gid | (uintptr_t)nbr_gid | (uintptr_t)unique_gid) & 7) ||
        (((uintptr_t)local_nbr | (uintptr_t)result) & 3)) {
        set_error("ID arrays must be 8-byte aligned, local_nbr and result 4-byte aligned");
        return FASTGL_ERR_INVALID_ARG;
    }
    if (!workspace || ((uintptr_t)workspace & 255)) {
        set_error("workspace must be a 256-byte aligned device buffer");
        return FASTGL_ERR_INVALID_ARG;
    }
    const Layout L = layout(n);
    if (workspace_bytes < L.total) {
        set_error("workspace too small: %zu < %zu bytes", workspace_bytes, L.total);
        return FASTGL_ERR_WORKSPACE;
    }
    char *ws = (char *)workspace;
    IdmapArgs a = {};
    a.dst_gid = dst_gid; a.nbr_gid = nbr_gid;
    a.n_dst = n_dst; a.n_nbr = n_nbr; a.n = n;
    const int64_t cap = position_slots(n, idmap_slots(n));
    a.table = PositionTable{(int32_t *)(ws + L.table), (uint32_t)cap, position_bits(n)};
    // behind the slots, which leave a third of the table's room and more
    const size_t displaced = align_up((size_t)ceil_div(cap, kFillVec) * kFillVec * sizeof(int32_t), 256);
    if (L.table + displaced + align_up((size_t)n, 16) > L.ref) {
        set_error("ID map: no room behind %lld slots", (long long)cap);      // not reached
        return FASTGL_ERR_UNSUPPORTED;
    }
    a.displaced = (unsigned char *)(ws + L.table + displaced);
    a.ref = (int32_t *)(ws + L.ref);
    a.block_cnt = (int32_t *)(ws + L.block_cnt);
    a.local_nbr = local_nbr; a.unique_gid = unique_gid; a.result = result;
    a.nblocks = (int)ceil_div(n, kScanBlock);
    a.fused = mode == FASTGL_IDMAP_FUSED;
    hipStream_t s = (hipStream_t)stream;
    auto grid = [](int64_t items, int per) { return dim3((unsigned)(items > 0 ? ceil_div(items, per) : 1)); };

    hipLaunchKernelGGL(k_idmap_fill, grid(cap, 256 * kFillVec), dim3(256), 0, s, a);
    FASTGL_LAUNCH_CHECK("fastgl_idmap (fill)");
    if (a.fused) {
        if (n_dst > 0) {
            hipLaunchKernelGGL(k_idmap_fused_dst, grid(n_dst, 256), dim3(256), 0, s, a);
            FASTGL_LAUNCH_CHECK("fastgl_idmap (destinations)");
        }
        if (n_nbr > 0) {
            hipLaunchKernelGGL(k_idmap_fused_nbr, grid(n_nbr, kScanBlock), dim3(kScanBlock), 0, s, a);
            FASTGL_LAUNCH_CHECK("fastgl_idmap (fused map)");
        }
        if (n_nbr > 0) {
            hipLaunchKernelGGL(k_idmap_fused_translate, grid(n_nbr, 256), dim3(256), 0, s, a);
            FASTGL_LAUNCH_CHECK("fastgl_idmap (translate)");
        }
    } else if (n > 0) {
        const dim3 blocks((unsigned)a.nblocks);
        hipLaunchKernelGGL(k_idmap_insert_min, grid(n, 256), dim3(256), 0, s, a);
        FASTGL_LAUNCH_CHECK("fastgl_idmap (insert)");
        hipLaunchKernelGGL(k_idmap_count, blocks, dim3(kCountThreads), 0, s, a);
        FASTGL_LAUNCH_CHECK("fastgl_idmap (count)");
        if (a.nblocks <= kSumBlocks) {
            hipLaunchKernelGGL(k_idmap_rank<true>, blocks, dim3(kCountThreads), 0, s, a);
        } else {
            hipLaunchKernelGGL(k_idmap_scan, dim3(1), dim3(kScanBlock), 0, s, a);
            FASTGL_LAUNCH_CHECK("fastgl_idmap (scan)");
            hipLaunchKernelGGL(k_idmap_rank<false>, blocks, dim3(kCountThreads), 0, s, a);
        }
        FASTGL_LAUNCH_CHECK("fastgl_idmap (rank)");
        if (n_nbr > 0) {
            hipLaunchKernelGGL(k_idmap_translate, grid(n_nbr, 256), dim3(256), 0, s, a);
            FASTGL_LAUNCH_CHECK("fastgl_idmap (translate)");
        }
    }
    return FASTGL_OK;
}

}  // extern "C"
