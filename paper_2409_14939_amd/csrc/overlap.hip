// Pairwise overlaps of a window of mini-batches (paper Section 4.1: N_o of every pair), many IDs: through buckets of IDs
// whose tables fit LDS.  See include/fastgl_match.h for the contract, match.hip for windows of few IDs or many mini-batches.
//
// In one table in memory every ID costs a compare-and-swap or a marking store at a random address (25 and 56-77 G/s), and that is
// the whole cost.  Here the IDs are dealt to buckets by their hash first - streams, in pieces of a bucket's IDs - and a
// workgroup then puts a bucket together in LDS, where such an access costs next to nothing:
//
//   k_overlap_hist    IDs per bucket of each of kPartBlocks stretches of the input
//   k_overlap_columns IDs of a bucket in the stretches before, and in all
//   k_overlap_split   deals the IDs, 4 096 a step: sorted by bucket in LDS, written out in runs
//   k_overlap_bucket  a bucket's distinct IDs with a bit per mini-batch that holds them; the pairs they add up to
//   k_overlap_sum     adds up the buckets
//
// The hash (near_hash) is one to one on 64 bits.  Its upper bits are the bucket; the others, shifted up,
// leave as many low bits free: an item is the rest of the hash and the mini-batch in 8 bytes, a slot of the table the rest of
// the hash and the mask of the mini-batches.  An empty slot is 0 (a mask never is).
//
// Four mini-batches of 1.15 M nodes, us, kernels of a traced window: 233 in one table (fill 13, insert 197, count 24), 89 here (IDs
// per bucket 10, columns 5, split 44, buckets 25, sum 6).  What is left is the split: 37 MB in and out at 1.7 TB/s, chains of LDS
// steps between barriers (1 024 threads of four IDs instead of 512 of eight: 47).  Buckets: tables of 8 192 slots with 4 500 IDs 39,
// of 4 096 with 2 250 25 (four workgroups to a compute unit instead of two; 256 threads 28).
#include "hash_table.h"
#include "internal.h"

namespace fastgl {
namespace {

constexpr int kMostBatches = 8;              // a mask's bits
constexpr int kLeastBits = 8, kMostBits = 11;        // of a bucket's number: the mask takes their place
constexpr int kMostBuckets = 1 << kMostBits;
constexpr int kPartBlocks = 512;             // stretches of the input: two workgroups per compute unit
constexpr int kHistThreads = 1024;
constexpr int kSplitThreads = 512;
constexpr int kSplitItems = 8;
constexpr int kSplitStep = kSplitThreads * kSplitItems;
constexpr int kBucketThreads = 512;
// Distinct IDs that a table of 1 << bits slots takes: beyond, every thread may still add one.
constexpr int most_held(int bits) { return bits > 12 ? 7168 : 3072; }
constexpr int kSmallTable = 12, kLargeTable = 13;            // 32 and 64 KB: four and two workgroups per compute unit
static_assert(most_held(kSmallTable) + kBucketThreads < 1 << kSmallTable && most_held(kLargeTable) + kBucketThreads < 1 << kLargeTable,
              "a search ends at an empty slot");
// IDs of a bucket: buckets are doubled beyond, up to kMostBuckets; with more than kSmallIds then, the tables are the large ones.
constexpr int64_t kBucketMean = 2400, kSmallIds = (int64_t)2560 << kMostBits;
constexpr int kPer = kMostBuckets / kSplitThreads;           // consecutive buckets of a thread
static_assert(kMostBatches <= kLeastBits && kPer * kSplitThreads == kMostBuckets, "layout");

struct BucketArgs {
    const int64_t *gid;
    int64_t offsets[kMostBatches + 1];
    int n;
    int64_t total, per;          // IDs; of a stretch
    int bits;                    // 1 << bits buckets
    int32_t *cnt;                // [kPartBlocks][buckets] IDs per bucket; then of the stretches before
    int32_t *tot, *first;        // [buckets] IDs; where they start
    unsigned long long *items;   // [total]
    int32_t *sums;               // [pairs][buckets]
    unsigned long long *counts;
    int32_t *violations;
};

// Negative IDs are in no bucket.
__global__ __launch_bounds__(kHistThreads) void k_overlap_hist(BucketArgs a)
{
    __shared__ int h[kMostBuckets];
    const int t = threadIdx.x, buckets = 1 << a.bits;
    for (int d = t; d < kMostBuckets; d += kHistThreads) h[d] = 0;
    __syncthreads();
    const int64_t beg = blockIdx.x * a.per, end = beg + a.per < a.total ? beg + a.per : a.total;
    constexpr int kBatch = 8;    // loads in flight (past the end they re-read the last ID)
    for (int64_t i0 = beg + t; i0 < end; i0 += (int64_t)kBatch * kHistThreads) {
        int64_t gid[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int64_t i = i0 + (int64_t)u * kHistThreads;
            gid[u] = a.gid[i < end ? i : end - 1];
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            if (i0 + (int64_t)u * kHistThreads < end && gid[u] >= 0) atomicAdd(&h[near_hash(gid[u]) >> (64 - a.bits)], 1);
    }
    __syncthreads();
    for (int d = t; d < buckets; d += kHistThreads) a.cnt[(int64_t)blockIdx.x * buckets + d] = h[d];
}

// 64 buckets per workgroup, one per lane; a wavefront sums a strip of the stretches, then walks it again with its prefix.
__global__ __launch_bounds__(kHistThreads) void k_overlap_columns(BucketArgs a)
{
    constexpr int kWaves = kHistThreads / kWave, kRows = kPartBlocks / kWaves;
    __shared__ int part[kWaves][kWave];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave, buckets = 1 << a.bits;
    int32_t *col = a.cnt + (int64_t)w * kRows * buckets + blockIdx.x * kWave + lane;     // buckets: a multiple of 64
    int v[kRows], sum = 0;
#pragma unroll
    for (int r = 0; r < kRows; ++r) v[r] = col[(int64_t)r * buckets];
#pragma unroll
    for (int r = 0; r < kRows; ++r) sum += v[r];
    part[w][lane] = sum;
    __syncthreads();
    int base = 0, total = 0;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
        const int c = part[k][lane];
        base += k < w ? c : 0;
        total += c;
    }
    if (w == 0) a.tot[blockIdx.x * kWave + lane] = total;
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        col[(int64_t)r * buckets] = base;
        base += v[r];
    }
}

__global__ __launch_bounds__(kSplitThreads) void k_overlap_split(BucketArgs a)
{
    __shared__ unsigned long long stage[kSplitStep];
    __shared__ uint16_t bucket[kSplitStep];
    __shared__ int cnt[kMostBuckets], next[kMostBuckets], delta[kMostBuckets];
    const int t = threadIdx.x, buckets = 1 << a.bits;
    const int64_t beg = blockIdx.x * a.per, end = beg + a.per < a.total ? beg + a.per : a.total;
    int64_t gid[kSplitItems];
    auto load_step = [&](int64_t step) {     // no branch around the loads: they go out together
#pragma unroll
        for (int i = 0; i < kSplitItems; ++i) {
            const int64_t p = step + i * kSplitThreads + t;
            gid[i] = a.gid[p < end ? p : end - 1];
        }
    };
    if (beg < end) load_step(beg);
    {   // where this stretch's IDs of a bucket go
        int tv[kPer], before[kPer], sum = 0, at;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int d = kPer * t + k;
            tv[k] = d < buckets ? a.tot[d] : 0;
            before[k] = d < buckets ? a.cnt[(int64_t)blockIdx.x * buckets + d] : 0;
            sum += tv[k];
        }
        block_exclusive_scan(sum, 0, at);
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int d = kPer * t + k;
            next[d] = at + before[k];
            if (blockIdx.x == 0 && d < buckets) a.first[d] = at;
            at += tv[k];
        }
    }
    for (int64_t step = beg; step < end; step += kSplitStep) {
#pragma unroll
        for (int k = 0; k < kPer; ++k) cnt[kPer * t + k] = 0;
        __syncthreads();
        unsigned long long item[kSplitItems];
        int d[kSplitItems], rank[kSplitItems];
#pragma unroll
        for (int i = 0; i < kSplitItems; ++i) {
            const int64_t p = step + i * kSplitThreads + t;
            int b = 0;
#pragma unroll
            for (int x = 1; x < kMostBatches; ++x) b += x < a.n && p >= a.offsets[x];
            const uint64_t h = near_hash(gid[i]);
            d[i] = p < end && gid[i] >= 0 ? (int)(h >> (64 - a.bits)) : -1;
            item[i] = h << a.bits | (unsigned)b;
            rank[i] = d[i] >= 0 ? atomicAdd(&cnt[d[i]], 1) : 0;
        }
        if (step + kSplitStep < end) load_step(step + kSplitStep);
        __syncthreads();
        int own[kPer], sum = 0, at;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            own[k] = cnt[kPer * t + k];
            sum += own[k];
        }
        const int valid = block_exclusive_scan(sum, 0, at);
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            cnt[kPer * t + k] = at;
            delta[kPer * t + k] = next[kPer * t + k] - at;
            next[kPer * t + k] += own[k];
            at += own[k];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kSplitItems; ++i) {
            if (d[i] < 0) continue;
            const int to = cnt[d[i]] + rank[i];
            stage[to] = item[i];
            bucket[to] = (uint16_t)d[i];
        }
        __syncthreads();
        for (int j = t; j < valid; j += kSplitThreads) a.items[delta[bucket[j]] + j] = stage[j];
        __syncthreads();                     // the arrays are the next step's
    }
}

// A bucket of more distinct IDs than a table may hold (IDs that were chosen for their hashes) is put together in passes: what finds no
// room and is not in the table either moves to the front of the bucket's items, which are the next pass's.  A pass takes more than
// kMostHeld distinct IDs off, whatever their hashes: n of them in one bucket cost this workgroup n / kMostHeld passes over half of
// them on average.
template <int NB, int BITS>
__global__ __launch_bounds__(kBucketThreads) void k_overlap_bucket(BucketArgs a)
{
    constexpr int PAIRS = NB * (NB + 1) / 2, kSlots = 1 << BITS, kMostHeld = most_held(BITS), kBatch = 8;
    __shared__ __align__(16) unsigned long long table[kSlots];
    __shared__ int held, left, sum[PAIRS];
    const int t = threadIdx.x;
    unsigned long long *in = a.items + a.first[blockIdx.x];
    int items = a.tot[blockIdx.x];
    int c[PAIRS];
#pragma unroll
    for (int k = 0; k < PAIRS; ++k) c[k] = 0;
    while (items > 0) {
        for (int s = t; s < kSlots / 2; s += kBucketThreads) reinterpret_cast<uint4 *>(table)[s] = make_uint4(0, 0, 0, 0);
        if (t == 0) held = left = 0;
        __syncthreads();
        const bool may_fill = items > kMostHeld;
        bool full = false;
        for (int i0 = t; i0 < items && !full; i0 += kBatch * kBucketThreads) {
            unsigned long long w[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int i = i0 + u * kBucketThreads;
                w[u] = in[i < items ? i : items - 1];
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const unsigned long long key = w[u] & ~(unsigned long long)0xFF, bit = 1ull << (w[u] & 7);
                const bool todo = i0 + u * kBucketThreads < items && !full;
                uint32_t slot = (uint32_t)(w[u] >> (64 - BITS));
                while (todo) {
                    unsigned long long v = *(volatile unsigned long long *)&table[slot];
                    if (v == 0) {
                        v = atomicCAS(&table[slot], 0ull, key | bit);
                        if (v == 0) {
                            if (may_fill) full = atomicAdd(&held, 1) >= kMostHeld;
                            break;
                        }
                    }
                    if ((v ^ key) <= 0xFF) {
                        if (!(v & bit)) atomicOr(&table[slot], bit);
                        break;
                    }
                    slot = (slot + 1) & (kSlots - 1);
                }
            }
        }
        __syncthreads();
        const bool over = may_fill && held > kMostHeld;       // the same for the workgroup; no thread adds to the table any more
        for (int base = 0; over && base < items; base += kBatch * kBucketThreads) {
            unsigned long long w[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int i = base + u * kBucketThreads + t;
                w[u] = in[i < items ? i : items - 1];
            }
            __syncthreads();                 // up to here the items have been read: there is room for as many
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                if (base + u * kBucketThreads + t >= items) continue;
                const unsigned long long key = w[u] & ~(unsigned long long)0xFF, bit = 1ull << (w[u] & 7);
                uint32_t slot = (uint32_t)(w[u] >> (64 - BITS));
                unsigned long long v;
                while ((v = *(volatile unsigned long long *)&table[slot]) != 0 && (v ^ key) > 0xFF) slot = (slot + 1) & (kSlots - 1);
                if (v == 0) in[atomicAdd(&left, 1)] = w[u];
                else if (!(v & bit)) atomicOr(&table[slot], bit);
            }
        }
        __syncthreads();
        for (int s = t; s < kSlots; s += kBucketThreads) {
            const unsigned m = (unsigned)table[s];
            int k = 0;
#pragma unroll
            for (int x = 0; x < NB; ++x)
#pragma unroll
                for (int y = x; y < NB; ++y, ++k) c[k] += (m >> x) & (m >> y) & 1;
        }
        items = left;                        // 0 but after an overflow
        __syncthreads();                     // the table, `held` and `left` are the next pass's
    }
    if (t < PAIRS) sum[t] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PAIRS; ++k) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) c[k] += __shfl_xor(c[k], o);
        if ((t & (kWave - 1)) == 0) atomicAdd(&sum[k], c[k]);
    }
    __syncthreads();
    if (t < PAIRS) a.sums[((int64_t)t << a.bits) + blockIdx.x] = sum[t];
}

// One workgroup, a wavefront per pair.  What is in no mini-batch's distinct IDs is negative or repeated: a violation.
template <int NB>
__global__ __launch_bounds__(kHistThreads) void k_overlap_sum(BucketArgs a)
{
    constexpr int PAIRS = NB * (NB + 1) / 2, kWaves = kHistThreads / kWave;
    __shared__ int sum[PAIRS];
    const int lane = threadIdx.x & (kWave - 1), buckets = 1 << a.bits;
    for (int k = threadIdx.x / kWave; k < PAIRS; k += kWaves) {
        int s = 0;
#pragma unroll 4
        for (int b = lane; b < buckets; b += kWave) s += a.sums[((int64_t)k << a.bits) + b];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        if (lane == 0) sum[k] = s;
    }
    __syncthreads();
    auto pair = [](int x, int y) { return x * NB - x * (x - 1) / 2 + y - x; };       // x <= y
    if ((int)threadIdx.x < a.n * a.n) {
        const int i = threadIdx.x / a.n, j = threadIdx.x % a.n;
        a.counts[threadIdx.x] = (unsigned long long)sum[i < j ? pair(i, j) : pair(j, i)];
    }
    if (threadIdx.x == 0) {
        int found = 0;
        for (int i = 0; i < a.n; ++i) found += sum[pair(i, i)];
        *a.violations = (int32_t)a.total - found;
    }
}

struct Layout {
    size_t items, cnt, tot, first, sums, total;
};

Layout layout(int64_t total, int bits)
{
    const size_t buckets = (size_t)1 << bits;
    Layout L;
    size_t off = 0;
    L.items = off; off += align_up((size_t)total * 8, 256);
    L.cnt = off; off += kPartBlocks * buckets * 4;
    L.tot = off; off += buckets * 4;
    L.first = off; off += buckets * 4;
    L.sums = off; off += buckets * 4 * (kMostBatches * (kMostBatches + 1) / 2);
    L.total = off;
    return L;
}

}  // namespace

fastgl_status launch_overlap_buckets(const int64_t *gid, const int64_t *offsets, int n, int64_t *counts, int32_t *violations,
                                     char *ws, size_t ws_bytes, hipStream_t s)
{
    BucketArgs a = {};
    a.gid = gid; a.n = n; a.total = offsets[n];
    for (int b = 0; b <= n; ++b) a.offsets[b] = offsets[b];
    a.bits = kLeastBits;
    while (a.bits < kMostBits && a.total > kBucketMean << a.bits) ++a.bits;
    const Layout L = layout(a.total, a.bits);
    if (n < 1 || n > kMostBatches || L.total > ws_bytes) {
        set_error("overlap counts: %d mini-batches in buckets", n);          // not reached
        return FASTGL_ERR_UNSUPPORTED;
    }
    a.per = ceil_div(a.total, kPartBlocks);
    a.items = (unsigned long long *)(ws + L.items);
    a.cnt = (int32_t *)(ws + L.cnt);
    a.tot = (int32_t *)(ws + L.tot);
    a.first = (int32_t *)(ws + L.first);
    a.sums = (int32_t *)(ws + L.sums);
    a.counts = (unsigned long long *)counts;
    a.violations = violations;
    const unsigned buckets = 1u << a.bits;
    hipLaunchKernelGGL(k_overlap_hist, dim3(kPartBlocks), dim3(kHistThreads), 0, s, a);
    FASTGL_LAUNCH_CHECK("fastgl_overlap_counts (IDs per bucket)");
    hipLaunchKernelGGL(k_overlap_columns, dim3(buckets / kWave), dim3(kHistThreads), 0, s, a);
    FASTGL_LAUNCH_CHECK("fastgl_overlap_counts (columns)");
    hipLaunchKernelGGL(k_overlap_split, dim3(kPartBlocks), dim3(kSplitThreads), 0, s, a);
    FASTGL_LAUNCH_CHECK("fastgl_overlap_counts (split)");
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(buckets), dim3(kBucketThreads), 0, s, a); };
    if (a.total <= kSmallIds) n <= 4 ? go(k_overlap_bucket<4, kSmallTable>) : go(k_overlap_bucket<8, kSmallTable>);
    else n <= 4 ? go(k_overlap_bucket<4, kLargeTable>) : go(k_overlap_bucket<8, kLargeTable>);
    FASTGL_LAUNCH_CHECK("fastgl_overlap_counts (buckets)");
    if (n <= 4) hipLaunchKernelGGL(k_overlap_sum<4>, dim3(1), dim3(kHistThreads), 0, s, a);
    else hipLaunchKernelGGL(k_overlap_sum<8>, dim3(1), dim3(kHistThreads), 0, s, a);
    FASTGL_LAUNCH_CHECK("fastgl_overlap_counts (sum)");
    return FASTGL_OK;
}

}  // namespace fastgl
