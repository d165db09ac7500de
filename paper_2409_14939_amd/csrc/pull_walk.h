// Device code shared by the aggregation kernels: how a lane holds a slice of a
// feature row (load, multiply-add, round, store) and how a group of lanes walks
// the edges of consecutive rows as one flat list.  Included by aggregate.hip (the
// pull kernel of paper Section 2.1 Eq. 1 / Section 4.2 Eq. 5) and layer.hip (the
// aggregation fused with the update of Eq. 2).
#pragma once
#include <type_traits>

#include "internal.h"

namespace fastgl {

// Row gathers in flight per lane: groups of 16 lanes (and most of 32), of at most kBatchLanes, and of a whole wavefront (and of
// 32 lanes in large f32 launches and with column tiles).  A group loads as many column ids at a time (a chunk) as it has
// lanes, one of at most kBatchLanes lanes only those of the next batch: all neighbours of 65 536 nodes, width 32, forward / backward 96 / 91 us so, 110 / 98 with chunks of two batches.
// 16 lanes, 2.56 M weighted edges of 64 floats: 108 us, 4 in flight 110, batches of 4 111.
constexpr int kUnroll = 6;
constexpr int kUnrollNarrow = 4;
constexpr int kUnrollWave = 8;
constexpr int kBatchLanes = 8;

template <int DT> struct AccT { using type = double; };
template <> struct AccT<FASTGL_BF16> { using type = float; };

template <int DT, int VB> struct Slice {
    static constexpr int ES = DT == FASTGL_F32 ? 4 : 2;                       // bytes of an element
    static constexpr int NW = VB >= 4 ? VB / 4 : 1;                           // 32-bit words held per lane
    static constexpr int NE = DT == FASTGL_F32 ? VB / 4 : VB / 2;             // elements per lane
    using acc_t = typename AccT<DT>::type;
    using u32x4 = typename Words<ES>::x4;
    using u32x2 = typename Words<ES>::x2;
    using u32x1 = typename Words<ES>::x1;

    __device__ static __forceinline__ void load(const char *p, uint32_t (&r)[NW])
    {
        if constexpr (VB == 16) {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(p);
            r[0] = v[0]; r[1] = v[1]; r[2] = v[2]; r[3] = v[3];
        } else if constexpr (VB == 8) {
            const u32x2 v = *reinterpret_cast<const u32x2 *>(p);
            r[0] = v[0]; r[1] = v[1];
        } else if constexpr (VB == 4) {
            r[0] = *reinterpret_cast<const u32x1 *>(p);
        } else {
            r[0] = *reinterpret_cast<const uint16_t *>(p);
        }
    }

    // Waits for a slice here, whatever branch its use stands in: a load that a branch may leave unused is waited for
    // before the next one into its registers, and with it everything that was loaded ahead.
    __device__ static __forceinline__ void arrived(uint32_t (&r)[NW])
    {
#pragma unroll
        for (int i = 0; i < NW; ++i) asm volatile("" : "+v"(r[i]));
    }

    template <bool HASW>
    __device__ static __forceinline__ void fma(acc_t (&acc)[NE], const uint32_t (&r)[NW], acc_t w)
    {
        if constexpr (DT == FASTGL_F32) {
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                double x = (double)__uint_as_float(r[i]);
                acc[i] = HASW ? __builtin_fma(x, w, acc[i]) : acc[i] + x;
            }
        } else if constexpr (VB >= 4) {
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                float lo = __uint_as_float(r[i] << 16), hi = __uint_as_float(r[i] & 0xFFFF0000u);
                acc[2 * i] = HASW ? __builtin_fmaf(lo, w, acc[2 * i]) : acc[2 * i] + lo;
                acc[2 * i + 1] = HASW ? __builtin_fmaf(hi, w, acc[2 * i + 1]) : acc[2 * i + 1] + hi;
            }
        } else {
            float lo = __uint_as_float(r[0] << 16);
            acc[0] = HASW ? __builtin_fmaf(lo, w, acc[0]) : acc[0] + lo;
        }
    }

    // Two values to bf16, nearest even, NaN stays NaN: one instruction (in integer arithmetic it was eight for each,
    // and a kernel of 34 KB that small launches waited for).
    __device__ static __forceinline__ uint32_t to_bf16(float lo, float hi)
    {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        const bf16x2 v = {(__bf16)lo, (__bf16)hi};
        return __builtin_bit_cast(uint32_t, v);
    }

    __device__ static __forceinline__ void store(char *p, const acc_t (&acc)[NE], acc_t scale)
    {
        uint32_t r[NW];
        if constexpr (DT == FASTGL_F32) {
#pragma unroll
            for (int i = 0; i < NW; ++i) r[i] = __float_as_uint((float)(acc[i] * scale));
        } else if constexpr (VB >= 4) {
#pragma unroll
            for (int i = 0; i < NW; ++i) r[i] = to_bf16(acc[2 * i] * scale, acc[2 * i + 1] * scale);
        } else {
            r[0] = to_bf16(acc[0] * scale, 0.f);
        }
        // output rows are written once and never read back by this kernel: streaming
        // stores keep them from displacing gathered rows in L2 / Infinity Cache
        if constexpr (VB == 16) {
            u32x4 v = {r[0], r[1], r[2], r[3]};
            __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(p));
        } else if constexpr (VB == 8) {
            u32x2 v = {r[0], r[1]};
            __builtin_nontemporal_store(v, reinterpret_cast<u32x2 *>(p));
        } else if constexpr (VB == 4) {
            __builtin_nontemporal_store(r[0], reinterpret_cast<u32x1 *>(p));
        } else {
            __builtin_nontemporal_store((uint16_t)r[0], reinterpret_cast<uint16_t *>(p));
        }
    }
};

struct PullParams {
    const int32_t *rowptr, *col, *eid;
    const float *edge_w, *col_scale;
    const char *in;
    char *out;
    const int32_t *split;     // [nsets+1] first row of every fine row set (equal work each)
    int64_t nsets;            // fine row sets
    int64_t nwaves;           // wavefronts per column tile = ceil(nsets / sets_per_wave)
    int32_t ntiles;           // column tiles per row
    int32_t by_tile;          // column tiles: all rows of one tile after the other; 0: the tiles of a row together
    const int32_t *hot;       // not NULL: by tile if *hot >= hot_min
    int64_t hot_min;
    int32_t G, lg_G;          // lanes per group (power of two), its logarithm
    int32_t unit_shift;       // rows start at multiples of 1 << unit_shift bytes (no more than a slice)
    int32_t sets_per_wave;    // consecutive fine row sets one wavefront takes
    int64_t num_rows;
    int32_t row_mode;
    int32_t long_thr;         // rows longer than this are left to the chunk kernels
    int64_t row_bytes;        // bytes of one feature row
    int64_t feat;
    uint64_t tile_inv;        // ceil(2^64 / ntiles): division by multiplication (unused for one tile)
    uint64_t wave_inv;        // ceil(2^64 / nwaves)
    int64_t chunk_waves;      // wavefronts per column tile that take chunks of long rows
    int64_t num_blocks;       // launched blocks (multiple of kXcds)
    const int32_t *long_rows, *chunk_ptr, *n_long, *n_chunks;
    char *partials;
};

template <typename acc_t>
__device__ __forceinline__ acc_t row_scale(int mode, int len)
{
    acc_t d = (acc_t)(len < 1 ? 1 : len);
    if (mode == 1) return (acc_t)1 / d;
    if (mode == 2) return (acc_t)1 / (acc_t)sqrt((double)d);
    return (acc_t)1;
}

template <typename T> __device__ __forceinline__ T shfl_t(T v, int src);
template <> __device__ __forceinline__ float shfl_t<float>(float v, int src) { return __shfl(v, src, kWave); }
template <> __device__ __forceinline__ double shfl_t<double>(double v, int src) { return __shfl(v, src, kWave); }

// The value of one lane (the same for all: a scalar).
__device__ __forceinline__ int lane_value(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }
__device__ __forceinline__ float lane_value(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ double lane_value(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane), __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Weights of the edges.  kColWeight: col_scale, kEdgeWeight: edge_w in edge order, kPermWeight: edge_w by edge id,
// floats; kTwoWeights: edge_w * col_scale, in the type of the sums (fp64 holds it exactly, so one float fewer is handed
// round for a single weight).
enum { kNoWeight = 0, kColWeight = 1, kEdgeWeight = 2, kPermWeight = 3, kTwoWeights = 4 };
template <int W, typename acc_t> struct WeightT { using type = float; };
template <typename acc_t> struct WeightT<kTwoWeights, acc_t> { using type = acc_t; };

// Column ids, edge ids and weights of consecutive edges, one per lane of a group; past the end kend > 0 those of the
// block's first edge.  No control flow around the loads: one behind a branch is waited for where the branch ends, and
// these are to arrive while the rows of the edges before them are gathered.  Past the end it is the first edge because
// everybody's loads keep its cache line in L2; that of the last edge before the end has been displaced by then and came
// once more from memory (2.56 M weighted edges of 64 floats: 628 -> 606 MB read, 110.9 -> 108.5 us; transposed, with edge
// ids, 875 -> 840 MB, 165.2 -> 161.8).
__device__ __forceinline__ int load_col(const PullParams &P, int k, int kend) { return P.col[k < kend ? k : 0]; }

template <int W>
__device__ __forceinline__ int load_eid(const PullParams &P, int k, int kend)
{
    const int at = k < kend ? k : 0;
    if constexpr (W == kPermWeight) return P.eid[at];
    if constexpr (W == kTwoWeights) {
        const int id = (P.eid ? P.eid : P.col)[at];       // which one is a scalar
        return P.eid ? id : at;
    }
    return W == kEdgeWeight ? at : 0;
}

template <int W, typename acc_t>
__device__ __forceinline__ typename WeightT<W, acc_t>::type load_weight(const PullParams &P, int c, int eid)
{
    if constexpr (W == kColWeight) return P.col_scale[c];
    else if constexpr (W == kTwoWeights) return (acc_t)P.edge_w[eid] * (acc_t)P.col_scale[c];
    else if constexpr (W == kNoWeight) return 1;
    else return P.edge_w[eid];
}

// What happens to a finished row of a walk is its SINK's business:
// sink(row index, sums of this lane's slice, the row's scale factor).  RowStore
// writes the scaled, rounded row to the output matrix.
template <int DT, int VB>
struct RowStore {
    char *out;
    int64_t row_bytes, lane_off;
    bool active;
    __device__ __forceinline__ void operator()(int64_t row, const typename Slice<DT, VB>::acc_t (&acc)[Slice<DT, VB>::NE],
                                               typename Slice<DT, VB>::acc_t scale) const
    {
        if (active) Slice<DT, VB>::store(out + row * row_bytes + lane_off, acc, scale);
    }
};

// The unscaled sum of a chunk of a long row.
template <int DT, int VB>
__device__ __forceinline__ void put_partial(const PullParams &P, int64_t chunk, int64_t lane_off, bool active,
                                            const typename Slice<DT, VB>::acc_t (&acc)[Slice<DT, VB>::NE])
{
    using S = Slice<DT, VB>;
    if (!active) return;
    typename S::acc_t *dst = reinterpret_cast<typename S::acc_t *>(P.partials) + chunk * P.feat + lane_off / S::ES;
#pragma unroll
    for (int i = 0; i < S::NE; ++i) dst[i] = acc[i];
}

// Byte offset of the slice of lane `sub` of column tile `tile`. Of a row that is no multiple of a slice the last slice
// starts early enough to end with the row: its first elements are the ones before, too, and both lanes that have them
// store the same sums.
template <int VB>
__device__ __forceinline__ int64_t slice_offset(const PullParams &P, int64_t slice)
{
    const int64_t off = slice * VB, last = P.row_bytes - VB;
    return off < last ? off : last;
}

// What the groups of a wavefront share about its window of up to 64 rows; lane i writes row i.
template <typename acc_t, int NE>
struct RowWindow {
    int end[kWave];           // first edge behind the row
    acc_t scale[kWave];
    acc_t head[NE][kWave];    // a lane's sums of the first row that its group closes, the start of which others may have
};
template <int DT, int VB> using Window = RowWindow<typename Slice<DT, VB>::acc_t, Slice<DT, VB>::NE>;

// The 64 / G groups of a wavefront walk the edges of rows [ia, ib) of its window as ONE flat list, cut into as many
// equal runs as there are groups, so that no group has more to do than the others whatever the row lengths are, and
// every group has U row gathers in flight (sampled blocks have rows of 1-15 edges, transposed ones of 0-3, and now and
// then one of 200).  A group closes a row (hands its sum and scale factor to the sink, clears the sum) whenever its
// edge index passes the row's end.  Of a row that several groups share, the first ones' sums are carried to the group
// that closes it (a segmented scan over the groups, once per window).  ebeg: first edge of row ia; rows of the window
// are in `win`, their ends also in `pe` of lane i.  The scale factors (a division and a square root in fp64, some fifty
// instructions) are made by all lanes at once: made where a row is closed, they were issued once per row of every
// group.  Column ids are fetched two chunks ahead and weights one chunk ahead of use.
// PARTIAL: the only "row" is a chunk of a long row; its unscaled sum goes to slot r0 of the partial-sum buffer and the
// sink is not called.
//
// Instructions per edge count next to the gathers.  Column ids are turned into positions in units of the rows' common
// alignment by the lane that loads them (32 bits: the host sees to that), and lanes beyond the row's end gather its
// first slice instead of being masked out.
template <int DT, int VB, int W, bool PARTIAL, int U, bool BATCH, class Sink>
__device__ __forceinline__ void walk_flat(const PullParams &P, Window<DT, VB> &win, int64_t r0,
                                          int ia, int ib, int ebeg, int pe, int lane, int64_t lane_off, bool active,
                                          const Sink &sink)
{
    using S = Slice<DT, VB>;
    using acc_t = typename S::acc_t;
    using w_t = typename WeightT<W, acc_t>::type;
    const int G = P.G, groups = kWave >> P.lg_G, sub = lane & (G - 1), gbase = lane & ~(G - 1), q = lane >> P.lg_G;
    const int eend = lane_value(pe, ib - 1), total = eend - ebeg, per = (total + groups - 1) >> (6 - P.lg_G);
    auto run_begin = [&](int i) { return ebeg + (i * per < total ? i * per : total); };
    const int beg = run_begin(q), end = run_begin(q + 1);
    const uint32_t row_units = (uint32_t)(P.row_bytes >> P.unit_shift), my_unit = active ? (uint32_t)(lane_off >> P.unit_shift) : 0u;
    // group q > 0 starts in the first row that ends behind `beg`
    int row = ia;
    if constexpr (!PARTIAL) {
        for (int i = 1; i < groups; ++i) {
            const int before = __popcll(__ballot(lane >= ia && lane < ib && pe <= run_begin(i)));
            row = q == i ? ia + before : row;
        }
    }
    int rend = PARTIAL ? eend : win.end[row < ib ? row : ib - 1];
    acc_t acc[S::NE];
    int head_row = q > 0 ? -1 : 0;      // -1: none closed yet
#pragma unroll
    for (int i = 0; i < S::NE; ++i) acc[i] = (acc_t)0;

    auto close_row = [&]() {
        if (head_row < 0) {
            head_row = row;
#pragma unroll
            for (int i = 0; i < S::NE; ++i) win.head[i][lane] = acc[i];
        } else {
            sink(r0 + row, acc, win.scale[row]);
        }
#pragma unroll
        for (int i = 0; i < S::NE; ++i) acc[i] = (acc_t)0;
        ++row;
        rend = win.end[row < ib ? row : ib - 1];
    };

    // column ids and weights a chunk of the run at a time: as many edges as the group has lanes, or (BATCH) one batch
    const int chunk = BATCH ? U : G, mine = BATCH && sub >= U ? U - 1 : sub;
    int c0 = 0, nxt_c = 0, nxt_e = 0;
    w_t cur_w = 1;
    if (total > 0) {                    // a scalar; a group without edges loads what it has no use for
        c0 = load_col(P, beg + mine, end);
        const int e0 = load_eid<W>(P, beg + mine, end);
        nxt_c = load_col(P, beg + chunk + mine, end);
        nxt_e = load_eid<W>(P, beg + chunk + mine, end);
        cur_w = load_weight<W, acc_t>(P, c0, e0);
    }
    uint32_t cur_at = (uint32_t)c0 * row_units;
    // Edges j0 .. of the chunk at k0, which has n of them.  FULL: no masks.  Otherwise loads of edges that are not there
    // are masked out (a redundant load costs the address unit as much as any other: 222 -> 219 and 259 -> 256 us of the
    // headline mini-batch's input layer), except for groups that go batch by batch: past the end their lanes have the
    // block's first edge.
    auto batch = [&](auto full, int k0, int j0, int n) {
        constexpr bool FULL = decltype(full)::value;
        uint32_t raw[U][S::NW];
#pragma unroll
        for (int t = 0; t < U; ++t) {
            const int j = BATCH || FULL || j0 + t < G ? j0 + t : G - 1;
            const uint32_t at = (uint32_t)__shfl((int)cur_at, gbase + j, kWave) + my_unit;
            if (BATCH || FULL || j < n) S::load(P.in + ((uint64_t)at << P.unit_shift), raw[t]);
        }
#pragma unroll
        for (int t = 0; t < U; ++t) {
            const int j = j0 + t;
            acc_t w = (acc_t)1;
            if (W != kNoWeight) w = (acc_t)shfl_t<w_t>(cur_w, gbase + (BATCH || FULL || j < G ? j : G - 1));
            if (!BATCH && !FULL) S::arrived(raw[t]);
            if (FULL || j < n) {
                if constexpr (!PARTIAL)
                    while (k0 + j >= rend) close_row();
                S::template fma<W != kNoWeight>(acc, raw[t], w);
            }
        }
    };
    for (int k0 = beg; k0 < end; k0 += chunk) {
        const int n = end - k0 < chunk ? end - k0 : chunk;
        const int nn_c = load_col(P, k0 + 2 * chunk + mine, end), nn_e = load_eid<W>(P, k0 + 2 * chunk + mine, end);
        const w_t nxt_w = load_weight<W, acc_t>(P, nxt_c, nxt_e);
        if constexpr (BATCH) batch(std::false_type(), k0, 0, n);
        else
            for (int j0 = 0; j0 < n; j0 += U) {
                if (__all(j0 + U <= n)) batch(std::true_type(), k0, j0, n);
                else batch(std::false_type(), k0, j0, n);
            }
        cur_at = (uint32_t)nxt_c * row_units;
        cur_w = nxt_w;
        nxt_c = nn_c;
        nxt_e = nn_e;
    }
    if constexpr (PARTIAL) {
        for (int d = G; d < kWave; d <<= 1)
#pragma unroll
            for (int i = 0; i < S::NE; ++i) acc[i] += shfl_t<acc_t>(acc[i], lane ^ d);
        if (q == 0) put_partial<DT, VB>(P, r0, lane_off, active, acc);
    } else {
        while (row < ib && rend <= end) close_row();
        if (per >= total) return;                       // one group had all edges
        // acc: the start of a row that a later group closes.  Where a group closed none, inclusive scan over the groups
        // since the last one that did; group 0 carries nothing in.
        int closed = head_row >= 0;
        const bool scan = __ballot(!closed) != 0;
        for (int d = G; scan && d < kWave; d <<= 1) {
            const int from = lane >= d ? lane - d : lane;
            const int c = __shfl(closed, from, kWave);
            const bool take = lane >= d && !closed;
#pragma unroll
            for (int i = 0; i < S::NE; ++i) {
                const acc_t v = shfl_t<acc_t>(acc[i], from);
                acc[i] = take ? v + acc[i] : acc[i];
            }
            closed = take ? c : closed;
        }
#pragma unroll
        for (int i = 0; i < S::NE; ++i) acc[i] = shfl_t<acc_t>(acc[i], lane >= G ? lane - G : lane);
        if (q > 0 && head_row >= 0) {
#pragma unroll
            for (int i = 0; i < S::NE; ++i) acc[i] += win.head[i][lane];
            sink(r0 + head_row, acc, win.scale[head_row]);
        }
    }
}

// The same for a group that is a whole wavefront (rows of more than 32 slices): what the lanes of a group
// share - the edge, its column, its weight, the row's end - is a scalar, so that an edge costs a few scalar
// instructions, the load, and the conversions and multiply-adds of the slice.  r0, ia, ib and ebeg must be
// scalars already (readfirstlane).
template <int DT, int VB, int W, bool PARTIAL, int U, class Sink>
__device__ __forceinline__ void walk_wave(const PullParams &P, int64_t r0, int ia, int ib, int ebeg, int pe,
                                          typename Slice<DT, VB>::acc_t scale, int lane, int64_t lane_off, bool active,
                                          const Sink &sink)
{
    using S = Slice<DT, VB>;
    using acc_t = typename S::acc_t;
    using w_t = typename WeightT<W, acc_t>::type;
    const int eend = lane_value(pe, ib - 1);
    const uint32_t my_off = active ? (uint32_t)lane_off : 0u;
    int row = ia;
    int rend = lane_value(pe, row);
    acc_t acc[S::NE];
#pragma unroll
    for (int i = 0; i < S::NE; ++i) acc[i] = (acc_t)0;

    auto close_row = [&]() {
        if constexpr (PARTIAL) put_partial<DT, VB>(P, r0, lane_off, active, acc);
        else sink(r0 + row, acc, lane_value(scale, row));
#pragma unroll
        for (int i = 0; i < S::NE; ++i) acc[i] = (acc_t)0;
        ++row;
        rend = lane_value(pe, row < ib ? row : ib - 1);
    };

    int cur_c = 0, nxt_c = 0, nxt_e = 0;
    w_t cur_w = 1;
    if (ebeg < eend) {
        cur_c = load_col(P, ebeg + lane, eend);
        const int e0 = load_eid<W>(P, ebeg + lane, eend);
        nxt_c = load_col(P, ebeg + kWave + lane, eend);
        nxt_e = load_eid<W>(P, ebeg + kWave + lane, eend);
        cur_w = load_weight<W, acc_t>(P, cur_c, e0);
    }
    for (int k0 = ebeg; k0 < eend; k0 += kWave) {
        const int n = eend - k0 < kWave ? eend - k0 : kWave;
        const int nn_c = load_col(P, k0 + 2 * kWave + lane, eend), nn_e = load_eid<W>(P, k0 + 2 * kWave + lane, eend);
        const w_t nxt_w = load_weight<W, acc_t>(P, nxt_c, nxt_e);
        auto batch = [&](int j0, int m) {               // m edges
            uint32_t raw[U][S::NW];
#pragma unroll
            for (int t = 0; t < U; ++t)
                if (t < m) S::load(P.in + (int64_t)lane_value(cur_c, j0 + t) * P.row_bytes + my_off, raw[t]);
#pragma unroll
            for (int t = 0; t < U; ++t) {
                if (m < U) S::arrived(raw[t]);
                if (t < m) {
                    acc_t w = (acc_t)1;
                    if (W != kNoWeight) w = (acc_t)lane_value(cur_w, j0 + t);
                    if constexpr (!PARTIAL)
                        while (k0 + j0 + t >= rend) close_row();
                    S::template fma<W != kNoWeight>(acc, raw[t], w);
                }
            }
        };
        int j0 = 0;
        for (; j0 + U <= n; j0 += U) batch(j0, U);      // U divides kWave
        if (j0 < n) batch(j0, n - j0);
        cur_c = nxt_c;
        cur_w = nxt_w;
        nxt_c = nn_c;
        nxt_e = nn_e;
    }
    while (row < ib) close_row();
}

}  // namespace fastgl
