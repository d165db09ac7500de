// The plan of a small block in ONE launch.  Included by bookkeeping.hip.
//
// A plan built in stages is a chain of 2 (forward only) to 9 launches, each of which waits for the one
// before: for a block of a few thousand edges that is 20 us of launch latency around 2 us of work.  Here
// nobody waits for anybody: every workgroup recomputes from the block's own arrays what it needs from the
// others.  That costs reads (every bucket's workgroup scans all source ids, at most 256 KB out of L2) and chains of
// steps in the workgroups that there is one of (the lists of long rows, a bucket's chunks): the limits below are where
// those chains, growing with the block, take as long as the launches they save.
//
//   bucket      2 048 consecutive source ids: counts the edges per source of its bucket and the edges of the
//               buckets before it, writes the bucket's rows of indptr_T, out-degrees, scale factors and row
//               sets, collects the bucket's edges in order (8 192 at a time) and places them stably
//               (counts per wavefront and source, column scan, lane match - as k_plan_buckets does); the
//               destination row of an edge comes from a binary search in row pointers held in LDS
//   source degrees  the first half of that, for a forward-only plan of a GCN-normalised pass
//   long sources    one workgroup: degrees of all sources, ordered list of the long ones
//   destination rows  1 024 rows per workgroup: degrees, scale factors, row sets
//   long destinations one workgroup: ordered list of the long destination rows
//
// 256 seeds, fan-out 5 (1 276 edges, 1 276 sources), us a plan: 24 in stages (9 launches), 11 here.
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
// Edges of a full plan: two chunks of a bucket at most. One bucket's workgroup places its edges chunk by chunk, so a
// block whose sources fall into few buckets is a chain: 44 080 edges over 10 359 sources 76 / 43; 16 384: 20 / 35.
constexpr int kOnceFullEdges = 16384;
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
constexpr int kOnceChunk = 8192;           // edges of a bucket placed at a time
constexpr int kOnceRounds = kOnceChunk / kOnceThreads;   // 64-edge rounds per wavefront
constexpr int kOnceMaxJobs = 8;
static_assert(kBucketIds == 2 * kOnceThreads, "two sources per thread");

struct OnceJob {
    const int32_t *indptr, *indices;
    RowsArgs dst, src;            // src.rowptr is not read; src.len_out / rsq / split NULL where not wanted
    int32_t *indptr_T, *indices_T, *perm;
    int32_t num_dst, num_src, num_edges;
    int32_t buckets, row_groups;  // workgroups of those roles
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
            unsigned tab[kOnceWaves][kBucketIds / 2];   // per wavefront and source: count, then offset (16 bits each)
            uint32_t list[kOnceChunk];                  // collected edges: id | source within the bucket << 16
            uint16_t rows[kOnceRows + 2];               // indptr
        };
        unsigned degree[kOnceSourcesFull / 2];          // 16-bit counters, two to a word
    };
};
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

__device__ __forceinline__ void once_bucket(const OnceJob &J, int d, OnceShared &M, int *lds)
{
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
    const KeyRun run(J.indices, J.num_edges);
    M.start[t] = 0;
    M.start[t + kOnceThreads] = 0;
    if (J.full)
        for (int i = t; i <= J.num_dst; i += kOnceThreads) M.rows[i] = (uint16_t)J.indptr[i];
    __syncthreads();
    // edges of the bucket (per source too) and of the buckets before it
    int mine = 0, before = 0;
    run.each([&](int, int32_t key, bool ok) {
        const int b = key >> kBucketBits;
        const bool in = ok && b == d;
        mine += __popcll(__ballot(in));
        before += __popcll(__ballot(ok && b < d));
        if (in) atomicAdd(&M.start[key & (kBucketIds - 1)], 1);
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
    const int c0 = M.start[2 * t], c1 = M.start[2 * t + 1];
    int all;
    const int e0 = block_excl_scan(c0 + c1, &all, lds);
    M.start[2 * t] = e0;
    M.start[2 * t + 1] = e0 + c0;
    int nl = 0, nc = 0;
#pragma unroll
    for (int k = 0; k < 2; ++k) {            // the bucket's rows
        const int64_t r = (int64_t)d * kBucketIds + 2 * t + k;
        const bool valid = r < J.num_src;
        const int at = B0 + e0 + (k ? c0 : 0), len = k ? c1 : c0;
        if (valid && J.full) J.indptr_T[r] = at;
        row_emit(J.src, r, valid, at, len, nl, nc);
    }
    if (!J.full) return;
    if (d == J.buckets - 1 && t == 0) J.indptr_T[J.num_src] = J.num_edges;

    for (int f0 = 0; f0 < total; f0 += kOnceChunk) {
        const int n = total - f0 < kOnceChunk ? total - f0 : kOnceChunk;
        uint4 *z = reinterpret_cast<uint4 *>(&M.tab[0][0]);
#pragma unroll
        for (int k = 0; k < (int)(sizeof(M.tab) / sizeof(uint4)) / kOnceThreads; ++k) z[k * kOnceThreads + t] = make_uint4(0u, 0u, 0u, 0u);
        int at = listed - f0;                // place in this chunk's list of the next edge of this wavefront
        run.each([&](int e, int32_t key, bool ok) {
            const bool in = ok && (key >> kBucketBits) == d;
            const unsigned long long m = __ballot(in);
            const int p = at + lanes_below((unsigned)m, (unsigned)(m >> 32));
            if (in && p >= 0 && p < n) M.list[p] = (uint32_t)e | ((uint32_t)(key & (kBucketIds - 1)) << 16);
            at += __popcll(m);
        });
        __syncthreads();
        // this wavefront's run of the list: seg entries, a multiple of 64
        const int seg = ((n + kOnceThreads - 1) / kOnceThreads) * kWave;
        const int s0 = w * seg < n ? w * seg : n, s1 = s0 + seg < n ? s0 + seg : n;
        int kk[kOnceRounds], ee[kOnceRounds], row[kOnceRounds];
#pragma unroll
        for (int u = 0; u < kOnceRounds; ++u) {
            const int i = s0 + u * kWave + lane;
            const uint32_t v = i < s1 ? M.list[i] : 0u;
            kk[u] = i < s1 ? (int)(v >> 16) : -1;
            ee[u] = (int)(v & 0xFFFFu);
            row[u] = 0;
            if (kk[u] >= 0) atomicAdd(&M.tab[w][kk[u] >> 1], 1u << ((kk[u] & 1) * 16));
        }
        // destination rows: the last row that starts at or before the edge; the rounds' searches side by side
        int span = 1;
        while (span < J.num_dst) span <<= 1;
        for (int step = span >> 1; step > 0; step >>= 1) {
#pragma unroll
            for (int u = 0; u < kOnceRounds; ++u) {
                const int q = row[u] + step;
                if (s0 + u * kWave < s1 && q < J.num_dst && (int)M.rows[q] <= ee[u]) row[u] = q;
            }
        }
        __syncthreads();
        unsigned sum = 0;                    // column scan over the wavefronts, two sources to a word
#pragma unroll
        for (int k = 0; k < kOnceWaves; ++k) {
            const unsigned v = M.tab[k][t];
            M.tab[k][t] = sum;
            sum += v;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kOnceRounds; ++u) {
            if (s0 + u * kWave >= s1) break;                 // the same for the whole wavefront
            const bool ok = kk[u] >= 0;
            const int k = ok ? kk[u] : 0, sh = (k & 1) * 16;
            unsigned mlo, mhi;
            match_lanes<kBucketBits>(k, ok, mlo, mhi);
            const int lower = lanes_below(mlo, mhi);
            const int prior = (int)((M.tab[w][k >> 1] >> sh) & 0xFFFFu);
            // the LDS read above is issued before this update by the same wavefront
            if (ok && lower == 0) atomicAdd(&M.tab[w][k >> 1], (unsigned)(__popc(mlo) + __popc(mhi)) << sh);
            const int pos = B0 + M.start[k] + prior + lower;
            if (ok && pos < J.num_edges) {
                J.indices_T[pos] = row[u];
                if (J.perm) J.perm[pos] = ee[u];
            }
        }
        __syncthreads();
        M.start[2 * t] += (int)(sum & 0xFFFFu);
        M.start[2 * t + 1] += (int)(sum >> 16);
    }
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

// Workgroups of a job, in this order: buckets, long sources (with the transpose), long destinations, row groups.
__global__ __launch_bounds__(kOnceThreads) void k_plan_once(OnceArgs A)
{
    extern __shared__ __align__(16) unsigned char dyn[];
    OnceShared &M = *reinterpret_cast<OnceShared *>(dyn);
    __shared__ int lds[64];
    int j = 0;
    while (j + 1 < A.njobs && (int)blockIdx.x >= A.first[j + 1]) ++j;
    const OnceJob &J = A.job[j];
    int b = blockIdx.x - A.first[j];
    if (b < J.buckets) {
        once_bucket(J, b, M, lds);
        return;
    }
    b -= J.buckets;
    if (J.full && b == 0) {
        once_long_sources(J, M, lds);
        return;
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
