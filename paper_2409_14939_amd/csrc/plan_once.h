// The plan of a small block in ONE launch.  Included by bookkeeping.hip.
//
// A plan built in stages is a chain of 2 (forward only) to 9 launches, each of which waits for the one
// before: for a block of a few thousand edges that is 20 us of launch latency around 2 us of work.  Here
// nobody waits for anybody: every workgroup recomputes from the block's own arrays what it needs from the
// others.  That costs reads (every bucket's workgroup scans all source ids, at most 256 KB out of L2) and chains of
// steps in the workgroups that there is one of (the lists of long rows, a chunk): the limits below are where
// those chains, growing with the block, take as long as the launches they save.
//
//   bucket      512 consecutive source ids: counts the edges per source of its bucket and the edges of the
//               buckets before it, writes the bucket's rows of indptr_T, out-degrees, scale factors and row
//               sets, collects the first chunk of the bucket's edges (4 096) in order and places them stably
//               (counts per wavefront and source, column scan, lane match - as k_plan_buckets does); the
//               destination row of an edge comes from a binary search in row pointers held in LDS.  Every workgroup
//               looks at all source ids, so small buckets cost reads, but the chain from there on is as long as the
//               edges of a bucket (15 369 edges over 6 597 sources, two layers: 25 us with 2 048 ids, 13 now)
//   further chunks  one workgroup for each that there can be, (edges - 1) / 4 096 whatever the buckets are: finds from
//               the buckets' counts which chunk of which bucket is its own.  With all chunks of a bucket in one workgroup a
//               block whose hubs share a bucket was a chain: 49 152 edges over 12 288 sources, evenly spread / half / nearly
//               all of them in one bucket: 27 / 92 / 145 us, now 27 / 34 / 35 (chunks of 8 192: 27 / 41 / 42; of 2 048: 30 /
//               31 / 31, but they are more workgroups than the device holds where a call has many blocks)
//   source degrees  the first half of that for 2 048 ids, for a forward-only plan of a GCN-normalised pass
//   long sources    one workgroup: degrees of all sources, ordered list of the long ones
//   destination rows  1 024 rows per workgroup: degrees, scale factors, row sets
//   long destinations one workgroup: ordered list of the long destination rows
//
// 256 seeds, fan-out 5 (1 276 edges, 1 276 sources), us a plan: 24 in stages (9 launches), 9 here.
#pragma once
#include "plan_device.h"

namespace fastgl {

constexpr int kBucketBits = 11;
constexpr int kBucketIds = 1 << kBucketBits;

constexpr int kOnceThreads = 1024;
constexpr int kOnceWaves = kOnceThreads / kWave;
// Limits, us a plan in one launch / in stages (calls one after the other; a call that is waited for adds 3 to both).
// Edges of a forward-only plan with source degrees: 16-bit row pointers and edge ids; 65 535 edges: 14 / 19.
constexpr int kOnceEdges = 65535;
// Edges of a full plan: 20 000 over 2 000 sources 19 / 36 evenly spread, 22 / 41 with 95 % in one bucket.  With at most
// four edges per source more of them: 48 000 over 28 800 24 / 36 and 34 / 50; 49 152 over 12 288 27 / 40 and 35 / 49, 8 000
// of 40 000 of one source 35 / 50.  One source of many edges: 20 000 of 49 152 40 / 50, 46 000 49 / 53, 20 000 of 30 000
// 34 / 52, 19 000 of 20 000 30 / 50.
constexpr int kOnceFullEdges = 20480;
constexpr int kOnceSparseEdges = 49152;
// Destination rows: one workgroup scans all of them for long ones, 1 024 a step.  Forward-only: 8 192 rows 6.7 / 8.4,
// 16 384 rows 11 / 8.7, 65 536 rows 38 / 8.8, for any number of edges.  With source degrees (more launches to save)
// and full plans (row pointers in LDS): 24 576 rows 16 / 18 and 22 / 29.
constexpr int kOnceRowsFwd = 8192;
constexpr int kOnceRows = 24576;
// Sources of a full plan: one workgroup counts their degrees in LDS and scans them for long ones: 5 000 edges over
// 32 768 sources 18 / 25, over 65 536 (two windows of counters) 33 / 25, over 262 144 127 / 25.  Source degrees alone
// need no list: 128 buckets, 262 144 sources, 14 / 19.
constexpr int kOnceSourcesFull = 32768;
constexpr int kOnceSources = 1 << 18;
constexpr int kOnceChunk = 4096;           // edges of a bucket that one workgroup places
constexpr int kOnceMaxJobs = 8;
// Workgroups that the device holds at once (one per compute unit).  A launch of more, several blocks of many sources,
// has buckets of 2 048 ids: 8 blocks of 16 000 edges over 30 000 sources 30 us with 512 ids, 19 so; 4 blocks 18 and 18.
constexpr int kOnceGroups = 256;
constexpr int kOnceBits = 9;               // source ids of a bucket of a full plan, in launches of up to kOnceGroups workgroups
constexpr int kOnceIds = 1 << kOnceBits;
static_assert(kOnceIds <= kOnceThreads && kBucketIds == 2 * kOnceThreads, "one or two sources per thread");

struct OnceJob {
    const int32_t *indptr, *indices;
    RowsArgs dst, src;            // src.rowptr is not read; src.len_out / rsq / split NULL where not wanted
    int32_t *indptr_T, *indices_T, *perm;
    int32_t num_dst, num_src, num_edges;
    int32_t buckets, further, row_groups;    // workgroups of those roles
    int32_t full;                 // with the transpose
};

struct OnceArgs {
    int njobs;
    int first[kOnceMaxJobs + 1];
    OnceJob job[kOnceMaxJobs];
};

struct OnceShared {
    union {
        struct {
            int start[kBucketIds];                      // edges per source, then where its next edges go (within the bucket)
            uint32_t list[kOnceChunk];                  // collected edges: id | source within the bucket << 16
            uint16_t rows[kOnceRows + 8];               // indptr
            unsigned tab[kOnceWaves * kBucketIds / 2];  // per wavefront and source: count, then offset (16 bits each)
        };
        unsigned degree[kOnceSourcesFull / 2];          // 16-bit counters, two to a word
    };
};
constexpr size_t kOnceLdsFull = sizeof(OnceShared);
constexpr size_t kOnceLdsFullSmall = sizeof(OnceShared) - sizeof(unsigned) * kOnceWaves * (kBucketIds - kOnceIds) / 2;
static_assert(kOnceLdsFullSmall >= sizeof(unsigned) * kOnceSourcesFull / 2, "room for the degrees");
constexpr size_t kOnceLdsDegrees = sizeof(int) * kBucketIds;   // a forward-only plan needs no more than this

// The block's source ids, 64 per round; a wavefront owns the rounds r0 .. r1 - 1.
struct KeyRun {
    const int32_t *keys;
    int n, r0, r1;
    __device__ __forceinline__ KeyRun(const int32_t *k, int n_) : keys(k), n(n_)
    {
        const int rounds = (n + kWave - 1) / kWave, w = threadIdx.x / kWave, per = (rounds + kOnceWaves - 1) / kOnceWaves;
        r0 = w * per < rounds ? w * per : rounds;
        r1 = r0 + per < rounds ? r0 + per : rounds;
    }
    // f(edge id, source id, the edge exists), round by round; the loads of 8 rounds are in flight together
    template <class F>
    __device__ __forceinline__ void each(F f) const
    {
        const int lane = threadIdx.x & (kWave - 1);
        constexpr int kBatch = 8;
        for (int r = r0; r < r1; r += kBatch) {
            int32_t key[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int e = (r + u) * kWave + lane;
                key[u] = keys[e < n ? e : n - 1];       // past the end the last key again
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int e = (r + u) * kWave + lane;
                if (r + u < r1) f(e, key[u], e < n);    // the same for the whole wavefront
            }
        }
    }
};

// Ordered list of the rows longer than the threshold, their chunks, and how many there are of both.  len(i): length
// of row i; n = 0: none can be long.
template <class LEN>
__device__ __forceinline__ void once_long_rows(const RowsArgs &A, int n, int *lds, LEN len)
{
    int nl = 0, nc = 0;
    for (int base = 0; base < n; base += kOnceThreads) {
        const int i = base + threadIdx.x;
        const int l = i < n ? len(i) : 0;
        const int isl = l > kLongThreshold ? 1 : 0;
        if (!__syncthreads_or(isl)) continue;
        const int nch = isl ? (l + kLongChunk - 1) / kLongChunk : 0;
        int tl, tc;
        const int el = block_excl_scan(isl, &tl, lds), ec = block_excl_scan(nch, &tc, lds);
        if (isl) {
            A.long_rows[nl + el] = (int32_t)i;
            A.chunk_ptr[nl + el] = nc + ec;
        }
        nl += tl;
        nc += tc;
    }
    if (threadIdx.x != 0) return;
    A.chunk_ptr[nl] = nc;
    A.totals[0] = nl;
    A.totals[1] = nc;
}

// BITS: 1 << BITS source ids; FULL: with the transpose.
// Bucket d; FULL: places the share-th chunk of its edges.
template <int BITS, bool FULL>
__device__ __forceinline__ void once_bucket(const OnceJob &J, int d, int share, OnceShared &M, int *lds)
{
    constexpr int kIds = 1 << BITS, kPer = kIds > kOnceThreads ? kIds / kOnceThreads : 1;   // sources per thread
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
    // kCopies counters of a source, by lane: many edges of one source are a chain of additions to one word
    // (49 152 edges, 20 000 of one source, us a plan: 56 with one counter, 40 with four, 50 in stages; evenly spread 28.8
    // and 29.3, 1 276 edges 8.2 and 8.4)
    constexpr int kCopies = kBucketIds / kIds;
    static_assert(kCopies == 1 || (kCopies == 4 && kPer == 1), "copies are added up by the thread that has the source");
    int4 *const copies = reinterpret_cast<int4 *>(M.start);
    const int copy = lane & (kCopies - 1);
    const KeyRun run(J.indices, J.num_edges);
    for (int i = t; i < kIds * kCopies / 4; i += kOnceThreads) copies[i] = make_int4(0, 0, 0, 0);
    if (FULL)
        for (int i = t; i <= J.num_dst; i += kOnceThreads) M.rows[i] = (uint16_t)J.indptr[i];
    __syncthreads();
    // edges of the bucket (per source too) and of the buckets before it
    int mine = 0, before = 0;
    run.each([&](int, int32_t key, bool ok) {
        const int b = key >> BITS;
        const bool in = ok && b == d;
        mine += __popcll(__ballot(in));
        before += __popcll(__ballot(ok && b < d));
        if (in) atomicAdd(&M.start[(key & (kIds - 1)) * kCopies + copy], 1);
    });
    if (lane == 0) {
        lds[32 + w] = mine;
        lds[48 + w] = before;
    }
    __syncthreads();
    int listed = 0, total = 0, B0 = 0;       // of the wavefronts before this one; of all; edges before the bucket
#pragma unroll
    for (int k = 0; k < kOnceWaves; ++k) {
        if (k < w) listed += lds[32 + k];
        total += lds[32 + k];
        B0 += lds[48 + k];
    }
    const bool holds = kPer * t < kIds;      // this thread has sources: the same for a wavefront
    int c[kPer], sum_c = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        if constexpr (kCopies == 4) {
            const int4 v = copies[holds ? t : 0];
            c[k] = holds ? v.x + v.y + v.z + v.w : 0;
        } else {
            c[k] = holds ? M.start[kPer * t + k] : 0;
        }
        sum_c += c[k];
    }
    int all;
    int at = block_excl_scan(sum_c, &all, lds);
    int nl = 0, nc = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {         // the bucket's rows
        const int64_t r = (int64_t)d * kIds + kPer * t + k;
        const bool valid = holds && r < J.num_src;
        if (holds) {
            if constexpr (kCopies == 4) copies[t] = make_int4(at, 0, 0, 0);
            else M.start[kPer * t + k] = at;
        }
        if (share == 0) {
            if (FULL && valid) J.indptr_T[r] = B0 + at;
            row_emit(J.src, r, valid, B0 + at, c[k], nl, nc);
        }
        at += c[k];
    }
    if constexpr (FULL) {
        if (share == 0 && d == J.buckets - 1 && t == 0) J.indptr_T[J.num_src] = J.num_edges;
        const int f0 = share * kOnceChunk;
        if (f0 < total) {                    // the same for the workgroup
            int span = 1;
            while (span < J.num_dst) span <<= 1;
            const int n = total - f0 < kOnceChunk ? total - f0 : kOnceChunk;
            uint4 *z = reinterpret_cast<uint4 *>(M.tab);
            unsigned *tab = M.tab + w * (kIds / 2);
            for (int k = t; k < kOnceWaves * kIds / 2 / 4; k += kOnceThreads) z[k] = make_uint4(0u, 0u, 0u, 0u);
            int to = listed - f0;            // place in this chunk's list of the next edge of this wavefront
            auto collect = [&](auto first) {
                run.each([&](int e, int32_t key, bool ok) {
                    const bool in = ok && (key >> BITS) == d;
                    const unsigned long long m = __ballot(in);
                    const int p = to + lanes_below((unsigned)m, (unsigned)(m >> 32));
                    if (!decltype(first)::value && in && p < 0)   // of an earlier chunk
                        atomicAdd(&M.start[(key & (kIds - 1)) * kCopies + copy], 1);
                    if (in && p >= 0 && p < n) M.list[p] = (uint32_t)e | ((uint32_t)(key & (kIds - 1)) << 16);
                    to += __popcll(m);
                });
            };
            if (share == 0) {
                collect(std::true_type());
            } else {
                __syncthreads();             // M.start is written
                collect(std::false_type());
            }
            __syncthreads();
            // this wavefront's run of the list: seg entries, a multiple of 64
            const int seg = ((n + kOnceThreads - 1) / kOnceThreads) * kWave;
            const int s0 = w * seg < n ? w * seg : n, s1 = s0 + seg < n ? s0 + seg : n;
            for (int i = s0 + lane; i < s1; i += kWave) {
                const int k = (int)(M.list[i] >> 16);
                atomicAdd(&tab[k >> 1], 1u << ((k & 1) * 16));
            }
            __syncthreads();
            if (kCopies > 1 && share > 0 && t < kIds) {
                const int4 v = copies[t];
                M.start[t * kCopies] = v.x + v.y + v.z + v.w;
            }
            if (t < kIds / 2) {              // column scan over the wavefronts, two sources to a word
                unsigned sum = 0;
#pragma unroll
                for (int k = 0; k < kOnceWaves; ++k) {
                    const unsigned v = M.tab[k * (kIds / 2) + t];
                    M.tab[k * (kIds / 2) + t] = sum;
                    sum += v;
                }
            }
            __syncthreads();
            constexpr int kSide = 2;         // rounds of 64 edges side by side
            for (int i0 = s0; i0 < s1; i0 += kSide * kWave) {
                int kk[kSide], ee[kSide], row[kSide];
#pragma unroll
                for (int u = 0; u < kSide; ++u) {
                    const int i = i0 + u * kWave + lane;
                    const uint32_t v = i < s1 ? M.list[i] : 0u;
                    kk[u] = i < s1 ? (int)(v >> 16) : -1;
                    ee[u] = (int)(v & 0xFFFFu);
                    row[u] = 0;
                }
                // destination rows: the last row that starts at or before the edge
                for (int step = span >> 1; step > 0; step >>= 1) {
#pragma unroll
                    for (int u = 0; u < kSide; ++u) {
                        const int q = row[u] + step;
                        row[u] = q < J.num_dst && (int)M.rows[q < J.num_dst ? q : 0] <= ee[u] ? q : row[u];
                    }
                }
#pragma unroll
                for (int u = 0; u < kSide; ++u) {
                    const bool ok = kk[u] >= 0;
                    const int k = ok ? kk[u] : 0, sh = (k & 1) * 16;
                    unsigned mlo, mhi;
                    match_lanes<BITS>(k, ok, mlo, mhi);
                    const int lower = lanes_below(mlo, mhi);
                    const int prior = (int)((tab[k >> 1] >> sh) & 0xFFFFu);
                    // the LDS read above is issued before this update by the same wavefront
                    if (ok && lower == 0) atomicAdd(&tab[k >> 1], (unsigned)(__popc(mlo) + __popc(mhi)) << sh);
                    const int pos = B0 + M.start[k * kCopies] + prior + lower;
                    if (ok && pos < J.num_edges) {
                        J.indices_T[pos] = row[u];
                        if (J.perm) J.perm[pos] = ee[u];
                    }
                }
            }
        }
    }
}

// Which chunk behind the first of which bucket is the x-th?  There are at most (edges - 1) / kOnceChunk.
template <int BITS>
__device__ __forceinline__ bool once_further(const OnceJob &J, int x, OnceShared &M, int &bucket, int &share)
{
    constexpr int kSpread = 32;              // counters of a bucket: the edges of a wavefront mostly have the same one
    static_assert(kOnceSourcesFull >> BITS <= kWave && kWave * kSpread <= kBucketIds, "a bucket per lane");
    const int lane = threadIdx.x & (kWave - 1);
    for (int i = threadIdx.x; i < kWave * kSpread; i += kOnceThreads) M.start[i] = 0;
    __syncthreads();
    KeyRun(J.indices, J.num_edges).each([&](int, int32_t key, bool ok) {
        if (ok && (uint32_t)key < (uint32_t)kOnceSourcesFull) atomicAdd(&M.start[(key >> BITS) * kSpread + (lane & (kSpread - 1))], 1);
    });
    __syncthreads();
    int total = 0;
    for (int i = 0; i < kSpread; ++i) total += M.start[lane * kSpread + ((lane + i) & (kSpread - 1))];
    const int mine = total > kOnceChunk ? (total - 1) / kOnceChunk : 0;
    int upto = mine;
    for (int k = 1; k < kWave; k <<= 1) {
        const int v = __shfl_up(upto, k);
        upto += lane >= k ? v : 0;
    }
    __syncthreads();                         // the counters have been read
    const unsigned long long has = __ballot(upto > x);
    if (!has) return false;                  // the same for the workgroup
    bucket = __ffsll((long long)has) - 1;
    share = x - __shfl(upto - mine, bucket) + 1;
    return true;
}

__device__ __forceinline__ void once_long_sources(const OnceJob &J, OnceShared &M, int *lds)
{
    const int n = J.num_edges > kLongThreshold ? J.num_src : 0;
    if (n > 0) {
        for (int i = threadIdx.x; i < kOnceSourcesFull / 2; i += kOnceThreads) M.degree[i] = 0;
        __syncthreads();
        KeyRun(J.indices, J.num_edges).each([&](int, int32_t k, bool ok) {
            if (ok && (uint32_t)k < (uint32_t)kOnceSourcesFull) atomicAdd(&M.degree[k >> 1], 1u << ((k & 1) * 16));
        });
        __syncthreads();
    }
    once_long_rows(J.src, n, lds, [&](int i) { return (int)((M.degree[i >> 1] >> ((i & 1) * 16)) & 0xFFFFu); });
}

// Workgroups of a job, in this order: buckets, their further chunks, long sources (with the transpose), long destinations,
// row groups.  BITS: 1 << BITS sources to a bucket of a full plan; 0: there is none.
template <int BITS>
__global__ __launch_bounds__(kOnceThreads) void k_plan_once(OnceArgs A)
{
    extern __shared__ __align__(16) unsigned char dyn[];
    OnceShared &M = *reinterpret_cast<OnceShared *>(dyn);
    __shared__ int lds[64];
    int j = 0;
    while (j + 1 < A.njobs && (int)blockIdx.x >= A.first[j + 1]) ++j;
    const OnceJob &J = A.job[j];
    int b = blockIdx.x - A.first[j];
    if (b < J.buckets + J.further) {
        if constexpr (BITS > 0) {
            int share = 0;
            if (b >= J.buckets && !once_further<BITS>(J, b - J.buckets, M, b, share)) return;
            if (J.full) {
                once_bucket<BITS, true>(J, b, share, M, lds);
                return;
            }
        }
        once_bucket<kBucketBits, false>(J, b, 0, M, lds);
        return;
    }
    b -= J.buckets + J.further;
    if constexpr (BITS > 0) {
        if (J.full && b == 0) {
            once_long_sources(J, M, lds);
            return;
        }
    }
    b -= J.full ? 1 : 0;
    if (b == 0) {
        const int32_t *p = J.indptr;
        once_long_rows(J.dst, J.num_edges > kLongThreshold ? J.num_dst : 0, lds, [&](int i) { return p[i + 1] - p[i]; });
        return;
    }
    const int64_t r = (int64_t)(b - 1) * kOnceThreads + threadIdx.x;
    const bool valid = r < J.num_dst;
    const int e0 = valid ? J.indptr[r] : 0, len = valid ? J.indptr[r + 1] - e0 : 0;
    int nl = 0, nc = 0;
    row_emit(J.dst, r, valid, e0, len, nl, nc);
}

}  // namespace fastgl
