// Learned edge weights: gradient of Eq. 1 with respect to the weights (a sampled dense-dense
// product read at the block's edges) and the softmax over a destination's incoming edges.  See
// include/fastgl_edge.h for the contract.
//
// k_edge_dot: bound by HBM / fabric bandwidth like the aggregation itself - per edge one gathered row
// of X and one (cached, rows are consecutive) row of grad_out.  Work is dealt out per EDGE, not
// per row, so the degree distribution does not matter: a group of 2^k lanes covers the row pieces of
// one edge, several edges are in flight per group, and the lanes' partial dot products are added
// with cross-lane reads.  The destination of every edge comes from a small expansion pass.
// Pieces are of 16 bytes, of narrower rows the largest power of two that fits, of rows of any length and alignment; the groups
// of a workgroup take neighbouring batches of edges, so that what they load of edge numbers and store lies together.
// 2.56 M edges, us with the expansion pass; pieces of 16 bytes or one element and all edges of a group in a row -> pieces of
// any size -> neighbouring batches (before that: element by element where a row is no whole number of pieces):
//   f32   2 columns (98) 61 -> 50 -> 43;  3 (78) 78 -> 70 -> 50;  5 (76) 82 -> 82 -> 59;  9 (93) 110 -> 110 -> 67;
//         13 (96) 122 -> 122 -> 75;  33 (299) 127 -> 127 -> 121;  64 (140) 140 -> 140 -> 130;  256 (582) 582 -> 582 -> 528
//   bf16  4 (98) 72 -> 50 -> 43;  7 (66) 66 -> 73 -> 54;  9 (69) 78 -> 78 -> 58;  25 (105) 115 -> 115 -> 76;  100 (156) 152 -> 152 -> 140
//
// Softmax: many rows of fewer than 10 edges on average are walked 32 to a wavefront (walk_short_rows); of others a group of 8, 32 or 64
// lanes walks one destination row three times (maximum, sum of exponentials, write).  Rows longer than kLongRow are taken by whole workgroups of the
// same launch that look for them (softmax_long_rows).  exp and the sums are fp64, so the result is the correctly
// rounded quotient up to one unit in the last place.  Forward, us: 2.56 M edges in rows of 5, none long: 34 (a queue
// of long rows with launches of its own: 40; no workgroups that look: 32); 32 neighbouring rows of 20 000 among short
// ones: 51 (queue: 62; taken by the workgroup that met them, one after the other: 1 630); 512 of 2 000: 14 (29; 161).
#include <type_traits>

#include "fastgl_edge.h"
#include "internal.h"

namespace fastgl {
namespace {

constexpr int kLongRow = 1024;       // softmax rows longer than this are taken by a whole workgroup
constexpr int kMostSeekers = 512;    // workgroups of a softmax launch that look for them, two per compute unit
constexpr int kEdgeUnroll = 4;       // edges in flight per lane group in k_edge_dot (reduce4 assumes 4)
constexpr int kEdgeSteps = 8;        // batches of that many edges per lane group

// ---------------------------------------------------------------- edge -> destination row
// A group of 8 lanes writes the row number over the edges of one row (rows of sampled blocks are
// short; a row of 10^4 edges costs one group ~10^3 steps).
__global__ __launch_bounds__(256) void k_edge_rows(const int32_t *__restrict__ indptr, int64_t num_dst, int64_t E,
                                                   int32_t *__restrict__ edge_row)
{
    (void)E;
    const int64_t u = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 3;
    if (u >= num_dst) return;
    const int b = indptr[u], e = indptr[u + 1];
    for (int k = b + (threadIdx.x & 7); k < e; k += 8) edge_row[k] = (int32_t)u;
}

// ---------------------------------------------------------------- dL/dw_e
template <typename ACC>
__device__ __forceinline__ ACC group_sum(ACC v, int lanes);

template <>
__device__ __forceinline__ double group_sum<double>(double v, int lanes)
{
    for (int d = lanes >> 1; d > 0; d >>= 1) v += __shfl_xor(v, d);
    return v;
}

template <>
__device__ __forceinline__ float group_sum<float>(float v, int lanes)
{
    for (int d = lanes >> 1; d > 0; d >>= 1) v += __shfl_xor(v, d);
    return v;
}

// Sums of four values over a group of `lanes` >= 4 lanes with 2 + 1 + (log2(lanes) - 2) exchanges
// instead of 4 log2(lanes): the first exchange leaves each half of the group with two of the four
// sums, the second each quarter with one, the rest finish that one.  Returns the sum of value
// number `which` (0..3, set here) - the same in every lane of a quarter.
template <typename ACC>
__device__ __forceinline__ ACC reduce4(const ACC (&v)[4], int l, int lanes, int &which)
{
    int d = lanes >> 1;
    const bool up = (l & d) != 0;
    const ACC r0 = (up ? v[2] : v[0]) + __shfl_xor(up ? v[0] : v[2], d);
    const ACC r1 = (up ? v[3] : v[1]) + __shfl_xor(up ? v[1] : v[3], d);
    d >>= 1;
    const bool up2 = (l & d) != 0;
    ACC r = (up2 ? r1 : r0) + __shfl_xor(up2 ? r0 : r1, d);
    for (d >>= 1; d > 0; d >>= 1) r += __shfl_xor(r, d);
    which = (up ? 2 : 0) + (up2 ? 1 : 0);
    return r;
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// Dot product of one piece (PIECE bytes at byte offset `off` of both rows; a power of two, at least an element), which needs
// no more alignment than an element.  RAGGED: without its first `skip` elements.
template <bool BF16, int PIECE, bool RAGGED, typename ACC>
__device__ __forceinline__ ACC piece_dot(const char *__restrict__ x, const char *__restrict__ g, int64_t off, int skip)
{
    ACC s = 0;
    if constexpr (PIECE >= 4) {
        using W = Words<BF16 ? 2 : 4>;
        using Piece = typename std::conditional<PIECE == 16, typename W::x4,
                                                typename std::conditional<PIECE == 8, typename W::x2, typename W::x1>::type>::type;
        const Piece a = *reinterpret_cast<const Piece *>(x + off), b = *reinterpret_cast<const Piece *>(g + off);
        auto add = [&](int e, float u, float v) {
            const ACC t = (ACC)u * (ACC)v;
            s += !RAGGED || e >= skip ? t : (ACC)0;
        };
#pragma unroll
        for (int i = 0; i < PIECE / 4; ++i) {
            uint32_t p, q;
            if constexpr (PIECE > 4) {
                p = a[i];
                q = b[i];
            } else {
                p = a;
                q = b;
            }
            if constexpr (BF16) {
                add(2 * i, bf16_lo(p), bf16_lo(q));
                add(2 * i + 1, bf16_hi(p), bf16_hi(q));
            } else {
                add(i, __uint_as_float(p), __uint_as_float(q));
            }
        }
    } else {
        const uint32_t a = *reinterpret_cast<const uint16_t *>(x + off), b = *reinterpret_cast<const uint16_t *>(g + off);
        s = (ACC)bf16_lo(a) * (ACC)bf16_lo(b);
    }
    return s;
}

struct DotArgs {
    const int32_t *indptr, *indices, *edge_row;
    const char *X, *G;
    const float *src_scale;      // [num_src] or NULL
    float *grad_w;
    int64_t E, row_bytes;
    int pieces;                  // ceil(row_bytes / PIECE); the last one ends with the row
    int skip;                    // elements of the last piece that the one before it has
    int lanes;                   // lanes per edge group: power of two <= 64
    int steps;                   // batches of kEdgeUnroll edges per group, at most kEdgeSteps
    int mode;                    // 0 none, 1: 1/len, 2: 1/sqrt(len) of the destination row
};

// c_u * s_v of the aggregation mode.
__device__ __forceinline__ double edge_scale(const DotArgs &a, int32_t u, int32_t v)
{
    double scale = 1.0;
    if (a.mode) {
        const int len = a.indptr[u + 1] - a.indptr[u];
        const double d = len < 1 ? 1.0 : (double)len;
        scale = a.mode == 1 ? 1.0 / d : 1.0 / sqrt(d);
    }
    if (a.src_scale) scale *= (double)a.src_scale[v];
    return scale;
}

// Rows of at least kStagedLanes pieces: the workgroup's edges are consecutive, and their row and column numbers go
// through LDS in one coalesced load per thread and array instead of one load per edge, the same for all lanes of a
// group - half of all loads (2.56 M edges of 64 floats: 143 -> 129 us).  Narrower rows leave a workgroup more edges
// than LDS should hold.
constexpr int kStagedLanes = 8;
constexpr int kGroupEdges = kEdgeUnroll * kEdgeSteps;    // at most

template <bool BF16, int PIECE, bool RAGGED, bool STAGED>
__global__ __launch_bounds__(256) void k_edge_dot(const DotArgs a)
{
    using ACC = typename std::conditional<BF16, float, double>::type;
    constexpr int kStaged = STAGED ? 256 / kStagedLanes * kGroupEdges : 1;
    __shared__ int32_t row_s[kStaged], col_s[kStaged];
    const int lanes = a.lanes;
    const int groups_per_block = 256 / lanes;
    const int grp = threadIdx.x / lanes, l = threadIdx.x % lanes;
    const int step_edges = groups_per_block * kEdgeUnroll, block_edges = step_edges * a.steps;
    const int64_t block_first = (int64_t)blockIdx.x * block_edges;
    if constexpr (STAGED) {
        for (int i = threadIdx.x; i < block_edges; i += 256) {
            const int64_t e = block_first + i < a.E ? block_first + i : a.E - 1;   // a clamped edge is computed and dropped
            row_s[i] = a.edge_row[e];
            col_s[i] = a.indices[e];
        }
        __syncthreads();
    }
    // a group takes a.steps batches of kEdgeUnroll consecutive edges, next to those of its neighbours; without staging the
    // row and column of the next batch's edges are fetched while the current batch's rows are in flight
    const int64_t first = block_first + grp * kEdgeUnroll;
    int32_t u[kEdgeUnroll], v[kEdgeUnroll], un[kEdgeUnroll], vn[kEdgeUnroll];
    auto numbers = [&](int step) {
#pragma unroll
        for (int k = 0; k < kEdgeUnroll; ++k) {
            if constexpr (STAGED) {
                un[k] = row_s[step * step_edges + grp * kEdgeUnroll + k];
                vn[k] = col_s[step * step_edges + grp * kEdgeUnroll + k];
            } else {
                const int64_t at = first + step * step_edges + k, e = at < a.E ? at : a.E - 1;
                un[k] = a.edge_row[e];
                vn[k] = a.indices[e];
            }
        }
    };
    numbers(0);
    for (int step = 0; step < a.steps; ++step) {
        const int64_t e0 = first + step * step_edges;
        if (e0 >= a.E) break;                                        // uniform over the group
#pragma unroll
        for (int k = 0; k < kEdgeUnroll; ++k) {
            u[k] = un[k];
            v[k] = vn[k];
        }
        if (step + 1 < a.steps) numbers(step + 1);
        ACC acc[kEdgeUnroll];
#pragma unroll
        for (int k = 0; k < kEdgeUnroll; ++k) acc[k] = 0;
        for (int p = l; p < a.pieces; p += lanes) {
            const bool last = RAGGED && p == a.pieces - 1;
            const int64_t off = last ? a.row_bytes - PIECE : (int64_t)p * PIECE;
#pragma unroll
            for (int k = 0; k < kEdgeUnroll; ++k)
                acc[k] += piece_dot<BF16, PIECE, RAGGED, ACC>(a.X + (int64_t)v[k] * a.row_bytes,
                                                              a.G + (int64_t)u[k] * a.row_bytes, off, last ? a.skip : 0);
        }
        if (lanes >= 4) {
            int k;
            const ACC dot = reduce4<ACC>(acc, l, lanes, k);
            if ((l & (lanes / 4 - 1)) == 0 && e0 + k < a.E)          // first lane of each quarter
                a.grad_w[e0 + k] = (float)((double)dot * edge_scale(a, u[k], v[k]));
        } else {
#pragma unroll
            for (int k = 0; k < kEdgeUnroll; ++k) {
                const ACC dot = group_sum<ACC>(acc[k], lanes);
                if (l == 0 && e0 + k < a.E) a.grad_w[e0 + k] = (float)((double)dot * edge_scale(a, u[k], v[k]));
            }
        }
    }
}

// ---------------------------------------------------------------- short rows, many to a wavefront
// What the kernels on rows of a few edges are bound by is latency and instructions: with 8 lanes per row most lanes are idle.  Here a
// wavefront takes 16 or 32 neighbouring rows.  Their edges lie one after the other: all lanes load them, in order, into LDS; then 4 or 2
// lanes put their row together there, and per-edge results go out in order again.  Rows of more than kLaneRow edges per such lane are
// put together by the wavefront, one after the other; rows that do not fit LDS together are left to dense_sets.
constexpr int kStage = 512;          // edges in LDS: 17 KB a workgroup, eight of them on a compute unit
constexpr int kLaneRow = 16;
constexpr int kWalkLoads = 4;        // edges in flight per lane
constexpr int kWalkWaves = 4;        // of a workgroup
constexpr int kRowsOfDst = 32, kRowsOfSrc = 16;      // of a wavefront: sources come in order of their first appearance, the much used ones together
constexpr int kFewLanes = 32, kGroupRow = 64;        // groups of fewer lanes leave rows beyond kGroupRow edges to the wavefront

// Blocks of fewer rows, and of more edges to a row, are left to groups of 8 lanes, whose kernels are shorter.  us, groups / walked, in
// blocks of sampled neighbours, by number of destinations (their edges on average):
//                           59 K (7)    98 K (7)    155 K (5)   229 K (5)    261 K (5)    513 K (5)     192 K (9)     133 K (15)
//   softmax                 5.0 / 5.0   6.6 / 5.8   8.5 / 7.1   12.2 / 8.8   13.8 / 9.7   23.8 / 15.8   13.8 / 11.0   11.8 / 13.6
//   its gradient            3.7 / 4.0   4.4 / 4.5   6.1 / 5.4   8.2 / 6.9    9.2 / 7.2    16.4 / 11.8   8.7 / 7.8     7.7 / 10.0
//   scores                  3.1 / 4.0   4.4 / 5.0   5.4 / 5.6   7.6 / 8.3    9.1 / 8.3    17.8 / 15.4   11.5 / 11.8   12.0 / 14.0
//   their gradient's sums   4.0 / 3.7   5.7 / 5.3   7.2 / 6.6   10.2 / 9.2   10.9 / 8.7   20.2 / 16.0   12.0 / 12.5   13.0 / 14.6
// All neighbours of 1 M nodes, 6 edges on average and up to 1 900, in any order: 94 / 63, 55 / 38, 60 / 53, 62 / 45;  by degree:
// 102 / 109, 77 / 71, 131 / 133, 95 / 97.  Sums of sources, by their number: 195 K (3) 14.7 / 15.3, 307 K (3) 17.0 / 17.6, 321 K (2)
// 15.3 / 16.4, 345 K (1.5) 14.4 / 10.5, 375 K (3) 22.1 / 21.7, 442 K (2) 18.6 / 15.6, 732 K (2) 30.8 / 23.9, 1.15 M (2) 59.6 / 49.9;
// all neighbours, 1 M (6) 154 / 149, by degree 209 / 183, 754 K (7) 110 / 117, 524 K (8) 113 / 145.
constexpr int64_t kShortMean = 10, kSoftmaxRows = (int64_t)3 << 15, kScoreRows = (int64_t)1 << 18;
constexpr int64_t kShortSrcMean = 6, kScoreSources = (int64_t)1 << 18;

// Rows whose lengths are a power of two start at different banks.
__device__ __forceinline__ int stage_slot(int k) { return k + (k >> 4); }
constexpr int stage_slots(int edges) { return edges + edges / 16; }

__device__ __forceinline__ void stage_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");       // a wavefront's own LDS accesses are in order
    __builtin_amdgcn_wave_barrier();
}

inline unsigned walk_blocks(int64_t num_rows, int rows) { return (unsigned)ceil_div(num_rows, (int64_t)rows * kWalkWaves); }

// Sets of rows that do not fit LDS together: workgroups of the same launch look for them, each at sets that are far
// apart (where rows are in order of their length thousands of long ones lie together), and take them by groups of 8 lanes.  The walk
// alone took a block by degree, 8 edges on average, four times as long as the groups (258 / 62 us); with 512 such workgroups 74, with
// 1 024 66, with 2 048 65.
constexpr int kMostDense = 1024;
inline int dense_seekers(int64_t nnz) { return (int)(nnz / kStage < kMostDense ? nnz / kStage : kMostDense); }

// group(r, limit): row r < limit by 8 lanes.
template <int ROWS, class Group>
__device__ __forceinline__ void dense_sets(const int32_t *__restrict__ rowptr, int64_t num_rows, int seekers, const Group &group)
{
    __shared__ int32_t set[256];
    __shared__ int n_dense;
    const int64_t sets = (num_rows + ROWS - 1) / ROWS;
    auto end_of = [&](int64_t at) { return (at + 1) * ROWS < num_rows ? (at + 1) * ROWS : num_rows; };
    for (int64_t base = blockIdx.x; base < sets; base += 256 * (int64_t)seekers) {
        if (threadIdx.x == 0) n_dense = 0;
        __syncthreads();
        const int64_t at = base + (int64_t)threadIdx.x * seekers;
        if (at < sets && rowptr[end_of(at)] - rowptr[at * ROWS] > kStage) set[atomicAdd(&n_dense, 1)] = (int32_t)at;
        __syncthreads();
        const int n = n_dense;
        for (int q = 0; q < n; ++q) group((int64_t)set[q] * ROWS + threadIdx.x / 8, end_of(set[q]));
        __syncthreads();
    }
}

// Op: Word, what LDS holds of an edge;  load(k0, end, w): edges k0 + 64 i's;  own(r): what a row
// brings along;  row(st, lo, hi, r, own, l, lanes): row r, edges lo .. hi - 1 of LDS, by a group of lanes, this one lane l
// of it;  EDGES: result(word) goes to op.out[k] afterwards.
template <int ROWS, class Op>
__device__ __forceinline__ void walk_short_rows(const int32_t *__restrict__ rowptr, int64_t num_rows, int64_t first,
                                                typename Op::Word *st, const Op &op)
{
    static_assert(ROWS <= 32, "a set's rows have 8 lanes each in dense_sets");
    typedef typename Op::Word Word;
    constexpr int lanes = kWave / ROWS;
    const int lane = threadIdx.x & (kWave - 1), q = lane / lanes;
    const int64_t limit = first + ROWS < num_rows ? first + ROWS : num_rows;
    const int base = rowptr[first], end = rowptr[limit];
    if (end - base > kStage) return;         // dense_sets has them
    const int64_t r = first + q;
    const int qb = rowptr[r < limit ? r : limit], qe = rowptr[r + 1 < limit ? r + 1 : limit];     // rows that there are not are empty
    const float own = op.own(r < limit ? r : limit - 1);
    for (int k0 = base + lane; k0 - lane < end; k0 += kWave * kWalkLoads) {
        Word w[kWalkLoads];
        op.load(k0, end, w);                 // no branch around the loads: they go out together
#pragma unroll
        for (int i = 0; i < kWalkLoads; ++i)
            if (k0 + i * kWave < end) st[stage_slot(k0 + i * kWave - base)] = w[i];
    }
    stage_fence();
    const bool mine = r < limit, wide = qe - qb > kLaneRow * lanes;
    if (mine && !wide) op.row(st, qb - base, qe - base, r, own, lane % lanes, lanes);
    for (unsigned long long todo = __ballot(mine && wide && lane % lanes == 0); todo; todo &= todo - 1) {
        const int w = (int)__ffsll((long long)todo) - 1;
        op.row(st, __builtin_amdgcn_readlane(qb, w) - base, __builtin_amdgcn_readlane(qe, w) - base, first + w / lanes,
               __shfl(own, w), lane, kWave);
    }
    stage_fence();
    if (Op::EDGES)
        for (int k = base + lane; k < end; k += kWave) op.out[k] = op.result(st[stage_slot(k - base)]);
}

// ---------------------------------------------------------------- softmax
struct SoftmaxArgs {
    const int32_t *indptr;
    int64_t num_dst;
    const float *in0;            // fwd: score;  bwd: alpha
    const float *in1;            // fwd: unused; bwd: grad_alpha
    float *out;
    int backward;
    int seekers;                 // workgroups for the rows longer than kLongRow
};

__device__ __forceinline__ double lanes_max(double v, int lanes)
{
    for (int d = lanes >> 1; d > 0; d >>= 1) v = fmax(v, __shfl_xor(v, d));
    return v;
}

// One row by `lanes` lanes starting at lane `l` of its group; every lane of the group returns.
__device__ __forceinline__ void softmax_row_fwd(const float *__restrict__ score, float *__restrict__ alpha, int b,
                                                int e, int l, int lanes)
{
    double m = -INFINITY;
    for (int k = b + l; k < e; k += lanes) m = fmax(m, (double)score[k]);
    m = lanes_max(m, lanes);
    double z = 0.0;
    for (int k = b + l; k < e; k += lanes) z += exp((double)score[k] - m);
    z = group_sum<double>(z, lanes);
    for (int k = b + l; k < e; k += lanes) alpha[k] = (float)(exp((double)score[k] - m) / z);
}

__device__ __forceinline__ void softmax_row_bwd(const float *__restrict__ alpha, const float *__restrict__ da,
                                                float *__restrict__ ds, int b, int e, int l, int lanes)
{
    double s = 0.0;
    for (int k = b + l; k < e; k += lanes) s += (double)alpha[k] * (double)da[k];
    s = group_sum<double>(s, lanes);
    for (int k = b + l; k < e; k += lanes) ds[k] = (float)((double)alpha[k] * ((double)da[k] - s));
}

// Sum / max over a 256-thread workgroup, result to every thread.
__device__ __forceinline__ double block_reduce(double v, bool take_max)
{
    __shared__ double part[4];
    v = take_max ? lanes_max(v, 64) : group_sum<double>(v, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    return take_max ? fmax(fmax(part[0], part[1]), fmax(part[2], part[3])) : (part[0] + part[1]) + (part[2] + part[3]);
}

// A long row by the workgroup.
__device__ __forceinline__ void softmax_row_block(const SoftmaxArgs &a, int b, int e)
{
    const int l = threadIdx.x;
    if (!a.backward) {
        double m = -INFINITY;
        for (int k = b + l; k < e; k += 256) m = fmax(m, (double)a.in0[k]);
        m = block_reduce(m, true);
        double z = 0.0;
        for (int k = b + l; k < e; k += 256) z += exp((double)a.in0[k] - m);
        z = block_reduce(z, false);
        for (int k = b + l; k < e; k += 256) a.out[k] = (float)(exp((double)a.in0[k] - m) / z);
    } else {
        double s = 0.0;
        for (int k = b + l; k < e; k += 256) s += (double)a.in0[k] * (double)a.in1[k];
        s = block_reduce(s, false);
        for (int k = b + l; k < e; k += 256) a.out[k] = (float)((double)a.in0[k] * ((double)a.in1[k] - s));
    }
}

// The rows longer than kLongRow: workgroup b of n looks at rows b, b + n, ... and takes the long ones among them, so
// that neighbouring long rows (blocks whose destinations are ordered by degree) go to different workgroups.
__device__ __forceinline__ void softmax_long_rows(const SoftmaxArgs &a)
{
    __shared__ int32_t row[256];
    __shared__ int n_long;
    for (int64_t first = blockIdx.x; first < a.num_dst; first += 256 * (int64_t)a.seekers) {
        if (threadIdx.x == 0) n_long = 0;
        __syncthreads();
        const int64_t u = first + (int64_t)threadIdx.x * a.seekers;
        if (u < a.num_dst && a.indptr[u + 1] - a.indptr[u] > kLongRow) row[atomicAdd(&n_long, 1)] = (int32_t)u;
        __syncthreads();
        const int n = n_long;
        for (int q = 0; q < n; ++q) softmax_row_block(a, a.indptr[row[q]], a.indptr[row[q] + 1]);
        __syncthreads();
    }
}

// Row u < limit by a group of lanes, rows up to kLongRow; consecutive rows by a wavefront's groups.
template <int lanes>
__device__ __forceinline__ void softmax_group_rows(const SoftmaxArgs &a, int64_t u, int64_t limit)
{
    const int l = threadIdx.x % lanes;
    int b = 0, e = 0;
    if (u < limit) {
        b = a.indptr[u];
        e = a.indptr[u + 1];
        if (e - b > kLongRow) e = b;
    }
    // all lanes of a group hold the same (b, e): the cross-lane sums below see whole groups
    auto walk = [&](int beg, int end, int lane, int n) {
        if (a.backward)
            softmax_row_bwd(a.in0, a.in1, a.out, beg, end, lane, n);
        else
            softmax_row_fwd(a.in0, a.out, beg, end, lane, n);
    };
    bool wide = lanes < kFewLanes && e - b > kGroupRow;
    unsigned long long rows = lanes < kFewLanes ? __ballot(wide && l == 0) : 0;
    if (rows) {              // one after the other, unless the groups are done sooner (400 K rows by degree, gradient: 67 -> 55 us)
        int longest = 0, all = 0;
        for (unsigned long long todo = rows; todo; todo &= todo - 1) {
            const int w = (int)__ffsll((long long)todo) - 1, len = __builtin_amdgcn_readlane(e, w) - __builtin_amdgcn_readlane(b, w);
            longest = len > longest ? len : longest;
            all += len + 2 * kWave;
        }
        if (longest * (kWave / lanes) <= all) {
            wide = false;
            rows = 0;
        }
    }
    if (!wide) walk(b, e, l, lanes);
    if (lanes < kFewLanes)
        for (unsigned long long todo = rows; todo; todo &= todo - 1) {
            const int w = (int)__ffsll((long long)todo) - 1;
            walk(__builtin_amdgcn_readlane(b, w), __builtin_amdgcn_readlane(e, w), threadIdx.x & (kWave - 1), kWave);
        }
}

template <int lanes>
__global__ __launch_bounds__(256) void k_edge_softmax_rows(const SoftmaxArgs a)
{
    if ((int)blockIdx.x < a.seekers) {
        softmax_long_rows(a);
        return;
    }
    softmax_group_rows<lanes>(a, ((int64_t)(blockIdx.x - a.seekers) * blockDim.x + threadIdx.x) / lanes, a.num_dst);
}

// Rows of a wavefront's walk.  The exponentials stay in LDS from the sum to the quotient.
struct SoftmaxFwd {
    typedef double Word;
    static constexpr bool EDGES = true;
    const float *score;
    float *out;
    __device__ __forceinline__ void load(int k0, int end, Word (&w)[kWalkLoads]) const
    {
#pragma unroll
        for (int i = 0; i < kWalkLoads; ++i) {
            const int k = k0 + i * kWave;
            w[i] = (double)score[k < end ? k : end - 1];
        }
    }
    __device__ __forceinline__ float own(int64_t) const { return 0.f; }
    __device__ __forceinline__ float result(Word w) const { return (float)w; }
    __device__ __forceinline__ void row(Word *st, int lo, int hi, int64_t, float, int l, int lanes) const
    {
        double m = -INFINITY, z = 0.0;
        for (int k = lo + l; k < hi; k += lanes) m = fmax(m, st[stage_slot(k)]);
        m = lanes_max(m, lanes);
        for (int k = lo + l; k < hi; k += lanes) {
            const double x = exp(st[stage_slot(k)] - m);
            st[stage_slot(k)] = x;
            z += x;
        }
        z = group_sum<double>(z, lanes);
        for (int k = lo + l; k < hi; k += lanes) st[stage_slot(k)] /= z;
    }
};

struct SoftmaxBwd {
    typedef float2 Word;                     // alpha and its gradient; then the score's gradient
    static constexpr bool EDGES = true;
    const float *alpha, *da;
    float *out;
    __device__ __forceinline__ void load(int k0, int end, Word (&w)[kWalkLoads]) const
    {
#pragma unroll
        for (int i = 0; i < kWalkLoads; ++i) {
            const int k = k0 + i * kWave, at = k < end ? k : end - 1;
            w[i] = make_float2(alpha[at], da[at]);
        }
    }
    __device__ __forceinline__ float own(int64_t) const { return 0.f; }
    __device__ __forceinline__ float result(Word w) const { return w.x; }
    static __device__ __forceinline__ double term(Word w) { return (double)w.x * (double)w.y; }
    static __device__ __forceinline__ void put(Word *st, int k, double s)
    {
        const Word w = st[stage_slot(k)];
        st[stage_slot(k)].x = (float)((double)w.x * ((double)w.y - s));
    }
    __device__ __forceinline__ void row(Word *st, int lo, int hi, int64_t, float, int l, int lanes) const
    {
        double s = 0.0;
        for (int k = lo + l; k < hi; k += lanes) s += term(st[stage_slot(k)]);
        s = group_sum<double>(s, lanes);
        for (int k = lo + l; k < hi; k += lanes) put(st, k, s);
    }
};

__global__ __launch_bounds__(256) void k_edge_softmax_short(const SoftmaxArgs a)
{
    __shared__ __align__(16) char stage[kWalkWaves][stage_slots(kStage) * 8];
    if ((int)blockIdx.x < a.seekers) {
        softmax_long_rows(a);
        dense_sets<kRowsOfDst>(a.indptr, a.num_dst, a.seekers, [&](int64_t u, int64_t limit) { softmax_group_rows<8>(a, u, limit); });
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t first = ((int64_t)(blockIdx.x - a.seekers) * kWalkWaves + wave) * kRowsOfDst;
    if (first >= a.num_dst) return;
    if (a.backward)
        walk_short_rows<kRowsOfDst>(a.indptr, a.num_dst, first, reinterpret_cast<float2 *>(stage[wave]), SoftmaxBwd{a.in0, a.in1, a.out});
    else
        walk_short_rows<kRowsOfDst>(a.indptr, a.num_dst, first, reinterpret_cast<double *>(stage[wave]), SoftmaxFwd{a.in0, a.out});
}

template <int lanes>
void launch_softmax(const SoftmaxArgs &a, hipStream_t s)
{
    const dim3 grid((unsigned)(a.seekers + ceil_div(a.num_dst * lanes, 256)));
    hipLaunchKernelGGL(k_edge_softmax_rows<lanes>, grid, dim3(256), 0, s, a);
}

struct EdgeLayout {
    size_t edge_row, total;
};

EdgeLayout edge_layout(int64_t num_dst, int64_t E)
{
    (void)num_dst;
    EdgeLayout L;
    size_t off = 0;
    L.edge_row = off; off += align_up((size_t)(E > 0 ? E : 1) * 4, 256);
    // room that the softmax calls no longer use stays part of the size the interface asks for
    L.total = off + align_up((size_t)(E / kLongRow + 1) * 4, 256) + 256;
    return L;
}

fastgl_status check_csr(const int32_t *indptr, int64_t num_dst, int64_t E)
{
    if (num_dst < 0 || E < 0) {
        set_error("negative size (num_dst=%lld num_edges=%lld)", (long long)num_dst, (long long)E);
        return FASTGL_ERR_INVALID_ARG;
    }
    if (num_dst > kMaxIndex || E > kMaxIndex) {
        set_error("sizes must not exceed 2^31-1-1024 (int32 indices with look-ahead)");
        return FASTGL_ERR_UNSUPPORTED;
    }
    if (!indptr || ((uintptr_t)indptr & 3)) {
        set_error("indptr is NULL or misaligned");
        return FASTGL_ERR_INVALID_ARG;
    }
    if (E > 0 && num_dst == 0) {
        set_error("edges need at least one destination node");
        return FASTGL_ERR_INVALID_ARG;
    }
    return FASTGL_OK;
}

fastgl_status check_workspace(void *workspace, size_t have, size_t need)
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

template <bool BF16, int PIECE, bool RAGGED>
void launch_dot(const DotArgs &a, hipStream_t s)
{
    const int groups_per_block = 256 / a.lanes;
    const dim3 grid((unsigned)ceil_div(a.E, (int64_t)groups_per_block * kEdgeUnroll * a.steps));
    if (a.lanes >= kStagedLanes) hipLaunchKernelGGL((k_edge_dot<BF16, PIECE, RAGGED, true>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_edge_dot<BF16, PIECE, RAGGED, false>), grid, dim3(256), 0, s, a);
}

fastgl_status softmax(bool backward, const int32_t *indptr, int64_t num_dst, int64_t E, const float *in0,
                      const float *in1, float *out, void *workspace, size_t workspace_bytes, void *stream)
{
    fastgl_status st = check_csr(indptr, num_dst, E);
    if (st != FASTGL_OK) return st;
    if (E == 0) return FASTGL_OK;
    if (!in0 || !out || (backward && !in1) || (((uintptr_t)in0 | (uintptr_t)in1 | (uintptr_t)out) & 3)) {
        set_error("per-edge array is NULL or misaligned");
        return FASTGL_ERR_INVALID_ARG;
    }
    const EdgeLayout L = edge_layout(num_dst, E);
    st = check_workspace(workspace, workspace_bytes, L.total);
    if (st != FASTGL_OK) return st;
    SoftmaxArgs a = {};
    a.indptr = indptr; a.num_dst = num_dst; a.in0 = in0; a.in1 = in1; a.out = out;
    a.backward = backward;
    a.seekers = (int)(E / kLongRow < kMostSeekers ? E / kLongRow : kMostSeekers);   // no more than there can be long rows
    hipStream_t s = (hipStream_t)stream;
    // by the block's mean row length (rows of sampled blocks are short)
    const int64_t mean = E / (num_dst > 0 ? num_dst : 1);
    if (mean < kShortMean && num_dst >= kSoftmaxRows) {
        a.seekers = dense_seekers(E);                       // as many as there can be long rows, or more
        hipLaunchKernelGGL(k_edge_softmax_short, dim3(a.seekers + walk_blocks(num_dst, kRowsOfDst)), dim3(256), 0, s, a);
    } else if (mean < 24) launch_softmax<8>(a, s);
    else if (mean < 96) launch_softmax<32>(a, s);
    else launch_softmax<64>(a, s);
    FASTGL_LAUNCH_CHECK("edge softmax");
    return FASTGL_OK;
}


// ---------------------------------------------------------------- attention logits of a GAT head
// score_e = LeakyReLU(el[u] + er[v]) and the sums of its gradient over rows.  The same kernels run on
// the block's CSR (rows = destinations, col = neighbours) and on its transpose (rows = neighbours,
// col = destinations, eid = original edge ids): `row_val` belongs to the row index, `col_val` to col.
struct ScoreArgs {
    const int32_t *rowptr, *col, *eid;     // eid NULL: the edge id is the position
    int64_t num_rows;
    const float *row_val, *col_val;
    const float *grad_score;               // backward only
    float *out;                            // forward: [E] scores; backward: [num_rows] sums
    double slope;
};

// Rows of a wavefront's walk: what the edge's other end has, and the edge's gradient or its score.
template <bool BACKWARD>
struct ScoreRows {
    typedef float2 Word;
    static constexpr bool EDGES = !BACKWARD;
    const ScoreArgs &a;
    float *out;
    __device__ __forceinline__ void load(int k0, int end, Word (&w)[kWalkLoads]) const
    {
        int at[kWalkLoads], col[kWalkLoads], id[kWalkLoads];
#pragma unroll
        for (int i = 0; i < kWalkLoads; ++i) {
            const int k = k0 + i * kWave;
            at[i] = k < end ? k : end - 1;
            col[i] = a.col[at[i]];
            id[i] = BACKWARD && a.eid ? a.eid[at[i]] : at[i];
        }
#pragma unroll
        for (int i = 0; i < kWalkLoads; ++i) w[i] = make_float2(a.col_val[col[i]], BACKWARD ? a.grad_score[id[i]] : 0.f);
    }
    __device__ __forceinline__ float own(int64_t r) const { return a.row_val[r]; }
    __device__ __forceinline__ float result(Word w) const { return w.y; }
    __device__ __forceinline__ double term(double mine, Word w) const
    {
        return (double)w.y * (mine + (double)w.x > 0.0 ? 1.0 : a.slope);          // the sum's sign is exact
    }
    __device__ __forceinline__ float score(double mine, Word w) const
    {
        const double x = mine + (double)w.x;
        return (float)(x > 0.0 ? x : a.slope * x);
    }
    __device__ __forceinline__ void row(Word *st, int lo, int hi, int64_t r, float own, int l, int lanes) const
    {
        const double mine = (double)own;
        double acc = 0.0;
        for (int k = lo + l; k < hi; k += lanes) {
            const Word w = st[stage_slot(k)];
            if (BACKWARD) acc += term(mine, w);
            else st[stage_slot(k)].y = score(mine, w);
        }
        if (BACKWARD) {
            acc = group_sum<double>(acc, lanes);
            if (l == 0) out[r] = (float)acc;
        }
    }
    __device__ __forceinline__ void whole(int b, int e, int64_t r, float own) const
    {
        const int l = threadIdx.x & (kWave - 1);
        const double mine = (double)own;
        double acc = 0.0;
        for (int k0 = b + l; k0 - l < e; k0 += kWave * kWalkLoads) {
            Word w[kWalkLoads];
            load(k0, e, w);
#pragma unroll
            for (int i = 0; i < kWalkLoads; ++i) {
                const int k = k0 + i * kWave;
                if (k >= e) continue;
                if (BACKWARD) acc += term(mine, w[i]);
                else out[k] = score(mine, w[i]);
            }
        }
        if (BACKWARD) {
            acc = group_sum<double>(acc, kWave);
            if (l == 0) out[r] = (float)acc;
        }
    }
};

// Row r < limit by a group of lanes; consecutive rows by a wavefront's groups.
template <int lanes, bool BACKWARD>
__device__ __forceinline__ void score_group_rows(const ScoreArgs &a, int64_t r, int64_t limit)
{
    const int l = threadIdx.x % lanes;
    int b = 0, e = 0;
    double mine = 0.0;
    if (r < limit) {
        b = a.rowptr[r];
        e = a.rowptr[r + 1];
        mine = (double)a.row_val[r];
    }
    const bool wide = lanes < kFewLanes && e - b > kGroupRow;
    double acc = 0.0;
    for (int k = b + l; k < e && !wide; k += lanes) {
        const double x = mine + (double)a.col_val[a.col[k]];      // rounded in fp64, its sign is exact
        if (!BACKWARD)
            a.out[k] = (float)(x > 0.0 ? x : a.slope * x);
        else
            acc += (double)a.grad_score[a.eid ? a.eid[k] : k] * (x > 0.0 ? 1.0 : a.slope);
    }
    if (BACKWARD) {
        acc = group_sum<double>(acc, lanes);       // every lane of the group takes part
        if (l == 0 && r < limit && !wide) a.out[r] = (float)acc;
    }
    if (lanes < kFewLanes)
        for (unsigned long long todo = __ballot(wide && l == 0); todo; todo &= todo - 1) {
            const int w = (int)__ffsll((long long)todo) - 1;
            ScoreRows<BACKWARD>{a, a.out}.whole(__builtin_amdgcn_readlane(b, w), __builtin_amdgcn_readlane(e, w), r - (threadIdx.x & (kWave - 1)) / lanes + w / lanes,
                                                __shfl((float)mine, w));
        }
}

template <int lanes, bool BACKWARD>
__global__ __launch_bounds__(256) void k_edge_score(const ScoreArgs a)
{
    score_group_rows<lanes, BACKWARD>(a, ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / lanes, a.num_rows);
}

template <int ROWS, bool BACKWARD>
__global__ __launch_bounds__(256) void k_edge_score_short(const ScoreArgs a, int seekers)
{
    __shared__ float2 stage[kWalkWaves][stage_slots(kStage)];
    if ((int)blockIdx.x < seekers) {
        dense_sets<ROWS>(a.rowptr, a.num_rows, seekers, [&](int64_t r, int64_t limit) { score_group_rows<8, BACKWARD>(a, r, limit); });
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t first = ((int64_t)(blockIdx.x - seekers) * kWalkWaves + wave) * ROWS;
    if (first < a.num_rows) walk_short_rows<ROWS>(a.rowptr, a.num_rows, first, stage[wave], ScoreRows<BACKWARD>{a, a.out});
}

template <bool BACKWARD>
void launch_score(const ScoreArgs &a, int64_t nnz, hipStream_t s)
{
    const int64_t mean = nnz / (a.num_rows > 0 ? a.num_rows : 1);
    const int seekers = dense_seekers(nnz);
    if constexpr (BACKWARD)
        if (a.eid && mean < kShortSrcMean && a.num_rows >= kScoreSources) {
            hipLaunchKernelGGL((k_edge_score_short<kRowsOfSrc, true>), dim3(seekers + walk_blocks(a.num_rows, kRowsOfSrc)),
                               dim3(256), 0, s, a, seekers);
            return;
        }
    if (!a.eid && mean < kShortMean && a.num_rows >= kScoreRows)
        hipLaunchKernelGGL((k_edge_score_short<kRowsOfDst, BACKWARD>), dim3(seekers + walk_blocks(a.num_rows, kRowsOfDst)),
                           dim3(256), 0, s, a, seekers);
    else if (mean < 24)
        hipLaunchKernelGGL((k_edge_score<8, BACKWARD>), dim3((unsigned)ceil_div(a.num_rows * 8, 256)), dim3(256), 0, s, a);
    else if (mean < 96)
        hipLaunchKernelGGL((k_edge_score<32, BACKWARD>), dim3((unsigned)ceil_div(a.num_rows * 32, 256)), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL((k_edge_score<64, BACKWARD>), dim3((unsigned)ceil_div(a.num_rows * 64, 256)), dim3(256), 0, s, a);
}

fastgl_status check_score_args(const int32_t *indptr, const int32_t *indices, int64_t num_dst, int64_t num_src,
                               int64_t E, const float *el, const float *er, float slope)
{
    fastgl_status st = check_csr(indptr, num_dst, E);
    if (st != FASTGL_OK) return st;
    if (num_src < 0 || num_src >= INT32_MAX) {
        set_error("num_src out of range");
        return FASTGL_ERR_INVALID_ARG;
    }
    if (!(slope == slope) || slope - slope != 0.f) {
        set_error("slope must be finite");
        return FASTGL_ERR_INVALID_ARG;
    }
    if (E > 0 && (!indices || !el || !er || num_src == 0 || (((uintptr_t)indices | (uintptr_t)el | (uintptr_t)er) & 3))) {
        set_error("NULL or misaligned array (indices, el or er), or no source nodes");
        return FASTGL_ERR_INVALID_ARG;
    }
    return FASTGL_OK;
}

}  // namespace
}  // namespace fastgl

using namespace fastgl;

extern "C" {

size_t fastgl_edge_workspace_bytes(int64_t num_dst, int64_t num_edges)
{
    if (num_dst < 0 || num_edges < 0 || num_edges >= INT32_MAX) return 0;
    return edge_layout(num_dst, num_edges).total;
}

int32_t fastgl_edge_softmax_long_row(void) { return kLongRow; }

fastgl_status fastgl_edge_weight_grad(const int32_t *indptr, const int32_t *indices, int64_t num_dst,
                                      int64_t num_src, int64_t num_edges, int64_t feat, fastgl_agg_mode mode,
                                      fastgl_dtype dtype, const void *X, const void *grad_out,
                                      const fastgl_plan *plan, float *grad_w, void *workspace,
                                      size_t workspace_bytes, void *stream)
{
    fastgl_status st = check_csr(indptr, num_dst, num_edges);
    if (st != FASTGL_OK) return st;
    if (num_src < 0 || num_src >= INT32_MAX) {
        set_error("num_src out of range");
        return FASTGL_ERR_INVALID_ARG;
    }
    if (feat <= 0 || feat > ((int64_t)1 << 24)) {
        set_error("feat must be in [1, 2^24] (got %lld)", (long long)feat);
        return FASTGL_ERR_INVALID_ARG;
    }
    if ((int)mode < 0 || (int)mode > 2 || (int)dtype < 0 || (int)dtype > 1) {
        set_error("unknown aggregation mode %d or dtype %d", (int)mode, (int)dtype);
        return FASTGL_ERR_INVALID_ARG;
    }
    if (num_edges == 0) return FASTGL_OK;
    if (!indices || !X || !grad_out || !grad_w || num_src == 0) {
        set_error("NULL array (indices, X, grad_out or grad_w) or no source nodes");
        return FASTGL_ERR_INVALID_ARG;
    }
    const int64_t elem = dtype == FASTGL_F32 ? 4 : 2;
    if ((((uintptr_t)X | (uintptr_t)grad_out) & (uintptr_t)(elem - 1)) || (((uintptr_t)indices | (uintptr_t)grad_w) & 3)) {
        set_error("misaligned buffer");
        return FASTGL_ERR_INVALID_ARG;
    }
    const float *src_scale = nullptr;
    if (mode == FASTGL_AGG_GCN) {
        if (!plan || plan->indptr != indptr || plan->indices != indices || plan->num_dst != num_dst ||
            plan->num_src != num_src || plan->num_edges != num_edges ||
            !(plan->parts & (FASTGL_PLAN_BWD | FASTGL_PLAN_SRC_DEG))) {
            set_error("GCN mode needs a plan of this block that holds the source degrees");
            return FASTGL_ERR_INVALID_ARG;
        }
        src_scale = plan->src_rsqrt;
    }
    const EdgeLayout L = edge_layout(num_dst, num_edges);
    st = check_workspace(workspace, workspace_bytes, L.total);
    if (st != FASTGL_OK) return st;

    DotArgs a = {};
    a.indptr = indptr; a.indices = indices;
    a.edge_row = (int32_t *)((char *)workspace + L.edge_row);
    a.X = (const char *)X; a.G = (const char *)grad_out;
    a.src_scale = src_scale; a.grad_w = grad_w;
    a.E = num_edges; a.row_bytes = feat * elem;
    a.mode = mode == FASTGL_AGG_MEAN ? 1 : (mode == FASTGL_AGG_GCN ? 2 : 0);
    // of rows of any length and alignment (piece_dot): as much as a row has, up to 16 bytes
    int piece = 16;
    while (piece > a.row_bytes) piece /= 2;
    a.pieces = (int)ceil_div(a.row_bytes, (int64_t)piece);
    a.skip = (int)((a.pieces * (int64_t)piece - a.row_bytes) / elem);
    a.lanes = 1;
    while (a.lanes < 64 && a.lanes < a.pieces) a.lanes *= 2;
    // fewer edges per group where there are few: four workgroups per compute unit (10 302 edges of 56 floats, 21
    // workgroups of 8 batches each 18.4 us; 161 of one batch 4.5)
    a.steps = kEdgeSteps;
    while (a.steps > 1 && ceil_div(num_edges, (int64_t)(256 / a.lanes) * kEdgeUnroll * a.steps) < 1024) a.steps /= 2;
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(k_edge_rows, dim3((unsigned)ceil_div(num_dst * 8, 256)), dim3(256), 0, s, indptr, num_dst,
                       num_edges, (int32_t *)a.edge_row);
    FASTGL_LAUNCH_CHECK("fastgl_edge_weight_grad (edge rows)");
    const bool bf = dtype == FASTGL_BF16;
    auto go = [&](auto size) {
        constexpr int P = decltype(size)::value;
        if (bf) a.skip ? launch_dot<true, P, true>(a, s) : launch_dot<true, P, false>(a, s);
        else if constexpr (P > 4) a.skip ? launch_dot<false, P, true>(a, s) : launch_dot<false, P, false>(a, s);
        else if constexpr (P == 4) launch_dot<false, 4, false>(a, s);
    };
    switch (piece) {
    case 16: go(std::integral_constant<int, 16>()); break;
    case 8: go(std::integral_constant<int, 8>()); break;
    case 4: go(std::integral_constant<int, 4>()); break;
    default: launch_dot<true, 2, false>(a, s); break;
    }
    FASTGL_LAUNCH_CHECK("fastgl_edge_weight_grad");
    return FASTGL_OK;
}

fastgl_status fastgl_edge_softmax_fwd(const int32_t *indptr, int64_t num_dst, int64_t num_edges,
                                      const float *score, float *alpha, void *workspace, size_t workspace_bytes,
                                      void *stream)
{
    return softmax(false, indptr, num_dst, num_edges, score, nullptr, alpha, workspace, workspace_bytes, stream);
}

fastgl_status fastgl_edge_softmax_bwd(const int32_t *indptr, int64_t num_dst, int64_t num_edges,
                                      const float *alpha, const float *grad_alpha, float *grad_score,
                                      void *workspace, size_t workspace_bytes, void *stream)
{
    return softmax(true, indptr, num_dst, num_edges, alpha, grad_alpha, grad_score, workspace, workspace_bytes,
                   stream);
}

fastgl_status fastgl_edge_score_fwd(const int32_t *indptr, const int32_t *indices, int64_t num_dst, int64_t num_src,
                                    int64_t num_edges, const float *el, const float *er, float slope, float *score,
                                    void *stream)
{
    fastgl_status st = check_score_args(indptr, indices, num_dst, num_src, num_edges, el, er, slope);
    if (st != FASTGL_OK) return st;
    if (num_edges == 0) return FASTGL_OK;
    if (!score || ((uintptr_t)score & 3)) {
        set_error("score is NULL or misaligned");
        return FASTGL_ERR_INVALID_ARG;
    }
    ScoreArgs a = {};
    a.rowptr = indptr; a.col = indices; a.num_rows = num_dst;
    a.row_val = el; a.col_val = er; a.out = score; a.slope = (double)slope;
    launch_score<false>(a, num_edges, (hipStream_t)stream);
    FASTGL_LAUNCH_CHECK("fastgl_edge_score_fwd");
    return FASTGL_OK;
}

fastgl_status fastgl_edge_score_bwd(const int32_t *indptr, const int32_t *indices, int64_t num_dst, int64_t num_src,
                                    int64_t num_edges, const float *el, const float *er, float slope,
                                    const float *grad_score, const fastgl_plan *plan, float *grad_el, float *grad_er,
                                    void *stream)
{
    fastgl_status st = check_score_args(indptr, indices, num_dst, num_src, num_edges, el, er, slope);
    if (st != FASTGL_OK) return st;
    if ((((uintptr_t)grad_score | (uintptr_t)grad_el | (uintptr_t)grad_er) & 3) || (num_edges > 0 && !grad_score)) {
        set_error("grad_score is NULL, or a gradient array is misaligned");
        return FASTGL_ERR_INVALID_ARG;
    }
    hipStream_t s = (hipStream_t)stream;
    if (grad_er && num_src > 0) {   // checked before the first launch: a refused call leaves nothing on the stream
        const int need = FASTGL_PLAN_BWD | FASTGL_PLAN_PERM;
        if (!plan || plan->indptr != indptr || plan->indices != indices || plan->num_dst != num_dst ||
            plan->num_src != num_src || plan->num_edges != num_edges || (plan->parts & need) != need) {
            set_error("grad_er needs a plan of this block built with FASTGL_PLAN_BWD | FASTGL_PLAN_PERM");
            return FASTGL_ERR_INVALID_ARG;
        }
    }
    if (grad_el && num_dst > 0) {
        if (!el && num_edges == 0) el = grad_el;       // rows without edges read nothing but their own value
        ScoreArgs a = {};
        a.rowptr = indptr; a.col = indices; a.num_rows = num_dst;
        a.row_val = el; a.col_val = er; a.grad_score = grad_score; a.out = grad_el; a.slope = (double)slope;
        launch_score<true>(a, num_edges, s);
        FASTGL_LAUNCH_CHECK("fastgl_edge_score_bwd (grad_el)");
    }
    if (grad_er && num_src > 0) {
        if (!er && num_edges == 0) er = grad_er;
        ScoreArgs a = {};
        a.rowptr = plan->indptr_T; a.col = plan->indices_T; a.eid = plan->perm; a.num_rows = num_src;
        a.row_val = er; a.col_val = el; a.grad_score = grad_score; a.out = grad_er; a.slope = (double)slope;
        launch_score<true>(a, num_edges, s);
        FASTGL_LAUNCH_CHECK("fastgl_edge_score_bwd (grad_er)");
    }
    return FASTGL_OK;
}

}  // extern "C"
