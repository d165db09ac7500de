// Device pieces shared by the kernels that build a plan: workgroup-wide scans and sums, what one row
// contributes to a plan, and the lane match of the stable sorts.
#pragma once
#include "internal.h"

namespace fastgl {

// -------------------------------------------------- block-wide primitives ----
__device__ __forceinline__ int wave_incl_scan(int v)
{
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        int t = __shfl_up(v, o, kWave);
        if (lane >= o) v += t;
    }
    return v;
}

// Exclusive scan over all threads of the block (any multiple of 64 up to 1024);
// *total = block sum.  `lds` needs 16 ints and is free again on return.
__device__ __forceinline__ int block_excl_scan(int v, int *total, int *lds)
{
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave, nw = blockDim.x / kWave;
    int inc = wave_incl_scan(v);
    if (lane == kWave - 1) lds[w] = inc;
    __syncthreads();
    int off = 0, tot = 0;
    for (int i = 0; i < nw; ++i) {
        int s = lds[i];
        if (i < w) off += s;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}

// Block sums of two values at once.  `lds` needs 32 ints and is free again on return.
__device__ __forceinline__ void block_sum2(int &a, int &b, int *lds)
{
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave, nw = blockDim.x / kWave;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        a += __shfl_xor(a, o, kWave);
        b += __shfl_xor(b, o, kWave);
    }
    if (lane == 0) {
        lds[w] = a;
        lds[16 + w] = b;
    }
    __syncthreads();
    int sa = 0, sb = 0;
    for (int i = 0; i < nw; ++i) {
        sa += lds[i];
        sb += lds[16 + i];
    }
    __syncthreads();
    a = sa;
    b = sb;
}

// ---------------------------------------- degrees + long-row buckets (roles) ----
struct RowsArgs {
    const int32_t *rowptr;   // [n+1]
    int64_t n, per;          // block b owns rows [b*per, min(n,(b+1)*per))
    int nb;
    int32_t *len_out;        // [n] or NULL
    float *inv, *rsq;        // [n] or NULL: 1/max(len,1), 1/sqrt(max(len,1))
    int32_t *counts;         // [2*nb] per-block (long rows, chunks)
    int32_t *long_rows, *chunk_ptr, *totals;
    int32_t *edge_row;       // [nnz] or NULL: edge_row[e] = row that owns edge e
    int32_t *split;          // [nsets+1] or NULL: first row of every equal-work row set
    int64_t nsets;
};

// What one row contributes: its length and scale factors, the long-row counts, and the
// equal-work row sets that start right after it.  Called by every thread of a wavefront
// together (rows that start many sets are written by the whole wavefront); valid = the
// thread has a row.  e0 = first edge of row r, len = its length.
__device__ __forceinline__ void row_emit(const RowsArgs &A, int64_t r, bool valid, int e0, int len, int &nl,
                                         int &nc)
{
    const int lane = threadIdx.x & (kWave - 1);
    if (valid) {
        if (A.len_out) A.len_out[r] = len;
        double d = (double)(len < 1 ? 1 : len);
        if (A.inv) A.inv[r] = (float)(1.0 / d);
        if (A.rsq) A.rsq[r] = (float)(1.0 / sqrt(d));
        if (len > kLongThreshold) {
            nl += 1;
            nc += (len + kLongChunk - 1) / kLongChunk;
        }
    }
    if (A.split) {
        // Equal-work row sets: set g starts at the first row whose work prefix
        // W[r] = rowptr[r] + r reaches g * kWorkPerGroup.  Row r+1 is that row for
        // every g in (W[r]/work, W[r+1]/work]; the thread of row r writes them.
        int64_t g0 = 1, g1 = 0;   // empty
        if (valid) {
            g0 = ((int64_t)e0 + r) / kWorkPerGroup + 1;
            g1 = ((int64_t)e0 + len + r + 1) / kWorkPerGroup;
            if (r == 0) A.split[0] = 0;
            if (r == A.n - 1 && g1 < A.nsets) A.split[A.nsets] = (int32_t)A.n;   // partial last set
        }
        const bool big = g1 - g0 >= kWave;
        if (!big)
            for (int64_t g = g0; g <= g1; ++g) A.split[g] = (int32_t)(r + 1);
        unsigned long long m = __ballot(big);
        while (m) {
            const int leader = __ffsll((long long)m) - 1;
            const int64_t lg0 = __shfl(g0, leader, kWave), lg1 = __shfl(g1, leader, kWave);
            const int64_t lr = __shfl(r, leader, kWave);
            for (int64_t g = lg0 + lane; g <= lg1; g += kWave) A.split[g] = (int32_t)(lr + 1);
            m &= m - 1;
        }
    }
}

// Lanes of the wavefront whose `bits`-bit value equals this lane's (lanes with ok == false match
// nobody and nobody matches them).  One ballot per bit; lo / hi = the mask's halves.
template <int BITS>
__device__ __forceinline__ void match_lanes(int v, bool ok, unsigned &lo, unsigned &hi)
{
    const unsigned long long act = __ballot(ok);
    unsigned dlo = 0, dhi = 0;   // lanes that differ from this one in some bit
#pragma unroll
    for (int bit = 0; bit < BITS; ++bit) {
        const int neg = (int)((unsigned)v << (31 - bit)) >> 31;   // all ones where the bit is set
        const unsigned long long bl = __ballot(neg < 0);
        dlo |= (unsigned)bl ^ (unsigned)neg;
        dhi |= (unsigned)(bl >> 32) ^ (unsigned)neg;
    }
    lo = ok ? (unsigned)act & ~dlo : 0u;
    hi = ok ? (unsigned)(act >> 32) & ~dhi : 0u;
}

__device__ __forceinline__ int lanes_below(unsigned lo, unsigned hi)   // set bits of the mask below this lane
{
    return (int)__builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
}

}  // namespace fastgl
