// Pull-mode block aggregation for gfx950 (paper Section 2.1 Eq. 1 forward;
// Section 4.2 Eq. 5 backward, run as the same pull over the transposed CSR).
//
//   out[r,:] = rowscale(len_r) * sum_{k in row r} a_k * colscale[col_k] * in[col_k,:]
//
// Mapping to the machine.  A feature row is cut into slices of 16 bytes (rows of
// any length: the last slice ends with the row) and a "group" of G lanes (a power
// of two, 4 to 64) covers G consecutive slices.  A wavefront owns a set of
// consecutive rows (x one column tile) from start to end, so each output element
// has a single writer and the summation order is fixed: results do not depend on
// scheduling.  The order follows from the block (which rows a wavefront shares out)
// and the sizes, not from where buffers lie.
// The row sets come from the plan and carry equal work (edges + rows), and the groups of a wavefront share its edges equally (walk_flat), so
// skewed degree distributions overload neither a wavefront nor a group.
// The partial sum lives in registers (the paper keeps it in shared memory on its
// GPU; with one lane per slice registers serve the same purpose at no traffic).
// The lanes of a group fetch column ids and weights with one coalesced load and
// hand them round with cross-lane reads, then issue up to 8 independent row
// gathers before the first use.  Output rows leave with streaming stores.
//
// Bound by the fabric (random rows: 7.1 TB/s from the Infinity Cache, 5.5-6 from HBM) where a block is large, by the
// chain of dependent loads (row sets, row pointers, column ids, weights, rows) and the fetch of the code where it is
// small.  Measured, us, rows walked by one group each / shared by the groups of a wavefront:
//   all neighbours of 65 536 nodes (rows of up to 256 edges and chunks of longer ones), 32 columns: forward 149 / 96,
//   backward 123 / 84;  of 5 313 nodes, 8 columns bf16, both directions: 391 / 20 (a group was a single lane)
//   reddit-shaped layer, 602 columns (8-byte slices, five column tiles / 16-byte slices, three): 83 / 81, 100 / 92
//   256 rows, 64 columns: 4.6 / 4.0, backward 8.2 / 5.4
//   rows of 400 and 256 bytes, 2.56 M edges: 217 / 218, 104 / 109 - nothing to share out there
//
// f32 rows accumulate in fp64, bf16 rows in fp32; one rounding at the store.
//
// Rows longer than kLongThreshold edges are cut into chunks of kLongChunk edges that any
// wavefront can take (in the same launch); the partial sums go to the workspace and are
// added in chunk order by a second, small kernel, so the result is still deterministic.
#include "pull_walk.h"

namespace fastgl {

constexpr int kXcdRun = 16;
constexpr int kReduceBlocks = 2048;   // workgroups for the long rows, whose number the host does not know

// Which (row sets, column tile) a wavefront works on.
//
// Workgroup ids are dealt round-robin to the 8 XCDs, each with its own L2.
// Consecutive logical workgroups are handed to an XCD in runs of kXcdRun, so
// that neighbouring rows (which share output cache lines and first-touch source
// rows) share an L2, while every XCD still samples the whole row range: blocks
// whose hubs all sit at low ids stay balanced.  The column tiles of a row set
// sit in neighbouring wavefronts, or (TILES: column_tiles) as far apart as can be.
struct WaveId {
    int64_t w;        // index of the wavefront's first fine row set / P.sets_per_wave
    int tile;         // column tile
};

template <bool TILES>
__device__ __forceinline__ WaveId map_wave(const PullParams &P)
{
    const uint32_t x = blockIdx.x % kXcds, q = blockIdx.x / kXcds;
    const uint64_t lb = ((uint64_t)(q / kXcdRun) * kXcds + x) * kXcdRun + q % kXcdRun;
    const uint64_t v = lb * (kBlock / kWave) + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    WaveId r;
    bool by_tile = TILES && P.by_tile;
    if (TILES && P.hot) by_tile = *P.hot >= P.hot_min;
    if (by_tile) {
        const uint64_t div = P.nwaves > 1 ? __umul64hi(v, P.wave_inv) : v;    // v < 2^34, ntiles < 2^20, nwaves < 2^28: exact
        const bool none = div >= (uint32_t)P.ntiles;                            // wavefronts that fill the last workgroups
        r.tile = none ? 0 : (int)div;
        r.w = none ? P.nwaves : (int64_t)(v - div * (uint64_t)P.nwaves);
    } else {
        const uint64_t div = P.ntiles > 1 ? __umul64hi(v, P.tile_inv) : v;
        r.w = (int64_t)div;
        r.tile = (int)(v - div * (uint32_t)P.ntiles);
    }
    return r;
}

// Chunks of long rows.  The number of chunks lives in device memory, so the host
// never needs to know the degrees; the wavefronts of a column tile stride over the
// chunks and write fp64 / fp32 partial sums of their tile to the workspace.
template <int DT, int VB, int W, int U, bool WAVE, bool BATCH>
__device__ __forceinline__ void pull_chunks(const PullParams &P, Window<DT, VB> &win, int n_long,
                                            int64_t total, const WaveId &id, int lane, int64_t lane_off, bool active)
{
    if (id.w >= P.chunk_waves) return;
    for (int64_t chunk = id.w; chunk < total; chunk += P.chunk_waves) {
        int lo = 0, hi = n_long;   // chunk_ptr[lo] <= chunk < chunk_ptr[hi]
        while (hi - lo > 1) {
            int mid = lo + ((hi - lo) >> 1);
            if (P.chunk_ptr[mid] <= chunk) lo = mid; else hi = mid;
        }
        const int row = P.long_rows[lo];
        const int rbeg = P.rowptr[row], rend = P.rowptr[row + 1];
        const int beg = rbeg + ((int)chunk - P.chunk_ptr[lo]) * kLongChunk;
        const int end = beg + kLongChunk < rend ? beg + kLongChunk : rend;
        const RowStore<DT, VB> unused = {nullptr, 0, 0, false};     // a chunk's sum goes to the partial-sum buffer
        if constexpr (WAVE) walk_wave<DT, VB, W, true, U>(P, chunk, 0, 1, beg, end, 0, lane, lane_off, active, unused);
        else walk_flat<DT, VB, W, true, U, BATCH>(P, win, chunk, 0, 1, beg, end, lane, lane_off, active, unused);
    }
}

// One launch covers every row.  Each wavefront first takes its share of the long-row
// chunks (usually none), then its own rows: the consecutive rows
// of a few fine row sets, which the plan cut so that every set carries the same
// work (edges + rows), whatever the degree distribution is.  Rows that are long
// are skipped here; k_reduce_chunks finishes them.
template <int DT, int VB, int W, int U, bool WAVE, bool BATCH>
__global__ __launch_bounds__(kBlock) void k_pull_rows(PullParams P)
{
    using acc_t = typename Slice<DT, VB>::acc_t;
    __shared__ Window<DT, VB> windows[WAVE ? 1 : kBlock / kWave];
    const int lane = threadIdx.x & (kWave - 1);
    Window<DT, VB> &win = windows[WAVE ? 0 : threadIdx.x / kWave];
    const WaveId id = map_wave<!WAVE && !BATCH && U == kUnrollWave>(P);
    const int64_t slice = WAVE ? (int64_t)id.tile * kWave + lane : (int64_t)id.tile * P.G + (lane & (P.G - 1));
    const int64_t lane_off = slice_offset<VB>(P, slice);
    const bool active = slice * VB < P.row_bytes;
    // all that the wavefront needs to know first, loaded together
    const int64_t s0 = id.w * P.sets_per_wave, s1 = s0 + P.sets_per_wave;
    const int n_long = P.long_rows ? *P.n_long : 0, n_chunks = P.long_rows ? *P.n_chunks : 0;
    const int64_t rbeg = P.split[s0 < P.nsets ? s0 : P.nsets], rend = P.split[s1 < P.nsets ? s1 : P.nsets];
    if (n_chunks > 0) pull_chunks<DT, VB, W, U, WAVE, BATCH>(P, win, n_long, n_chunks, id, lane, lane_off, active);
    const RowStore<DT, VB> sink = {P.out, P.row_bytes, lane_off, active};
    for (int64_t r0 = rbeg; r0 < rend; r0 += kWave) {
        const int nrows = rend - r0 < kWave ? (int)(rend - r0) : kWave;
        int pb = 0, pe = 0;
        if (lane < nrows) {
            pb = P.rowptr[r0 + lane];
            pe = P.rowptr[r0 + lane + 1];
        }
        const acc_t scale = row_scale<acc_t>(P.row_mode, pe - pb);
        if constexpr (!WAVE) {
            // the window is this wavefront's alone: its LDS accesses are carried out in order
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            win.end[lane] = pe;
            win.scale[lane] = scale;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        const unsigned long long lm = __ballot(lane < nrows && pe - pb > P.long_thr);
        int i = 0;
        while (i < nrows) {
            if ((lm >> i) & 1ull) {   // a long row: its chunks were handled above
                ++i;
                continue;
            }
            const unsigned long long rest = lm >> i;
            const int j = rest ? i + (__ffsll((long long)rest) - 1) : nrows;
            if constexpr (WAVE) walk_wave<DT, VB, W, false, U>(P, r0, i, j, lane_value(pb, i), pe, scale, lane, lane_off, active, sink);
            else walk_flat<DT, VB, W, false, U, BATCH>(P, win, r0, i, j, lane_value(pb, i), pe, lane, lane_off, active, sink);
            i = j;
        }
    }
}

// Long rows: the partial sums of a row's chunks, scaled and stored.  A unit is a (row, column tile).  Where there are more units than
// workgroups, one of no more chunks than a workgroup has groups (256 / G) is added up by one group; others by a workgroup: its
// groups sum consecutive ranges of the chunks, each in chunk order with 8 loads in flight, and the ranges are added in order.  Bound by
// latency: most rows have few chunks, a row of 25 000 edges has 200, a chain of 25 loads for one group.  All-neighbours block (65 536
// rows, 2 570 of them long, up to 26 000 edges, and 640 K, 3 642 long, up to 1 800), forward + backward in a program, us, 1 024 workgroups
// and one to every unit in turn -> now: 32 columns 10.8 + 10.5 -> 11.1 + 5.6;  256 columns 28.7 + 12.5 -> 26.4 + 12.4.  One loop for both
// ways takes 96 registers instead of 107 (five workgroups to a compute unit instead of four): 12.1 + 6.0, 27.2 + 11.6;  blocks of a few
// hundred rows with some long ones the same in all three.
template <int DT, int VB>
__global__ __launch_bounds__(kBlock) void k_reduce_chunks(PullParams P)
{
    using S = Slice<DT, VB>;
    using acc_t = typename S::acc_t;
    __shared__ acc_t range_sum[S::NE][kBlock];
    __shared__ int many[kBlock], n_many;
    const int64_t total = (int64_t)(*P.n_long) * P.ntiles;
    if (blockIdx.x >= total) return;
    const int tid = threadIdx.x, sub = tid & (P.G - 1), part = tid >> P.lg_G, parts = kBlock >> P.lg_G;
    auto add_chunks = [&](int lo, int hi, int64_t lane_off, acc_t (&acc)[S::NE]) {
        const acc_t *src = reinterpret_cast<const acc_t *>(P.partials) + lane_off / S::ES;
        for (int c0 = lo; c0 < hi; c0 += 8) {
            acc_t load[8][S::NE];
#pragma unroll
            for (int k = 0; k < 8; ++k)
#pragma unroll
                for (int i = 0; i < S::NE; ++i)
                    load[k][i] = c0 + k < hi ? src[(int64_t)(c0 + k) * P.feat + i] : (acc_t)0;
#pragma unroll
            for (int k = 0; k < 8; ++k)
#pragma unroll
                for (int i = 0; i < S::NE; ++i) acc[i] += load[k][i];
        }
    };
    const bool spread = total > gridDim.x;         // else every unit has a workgroup, and nobody looks for them
    for (int64_t unit = (int64_t)blockIdx.x * parts + part; spread && unit < total; unit += (int64_t)gridDim.x * parts) {
        const int li = (int)(unit / P.ntiles), tile = (int)(unit - (int64_t)li * P.ntiles);
        const int64_t slice = (int64_t)tile * P.G + sub, lane_off = slice_offset<VB>(P, slice);
        const int row = P.long_rows[li], first = P.chunk_ptr[li], last = P.chunk_ptr[li + 1];
        if (last - first > parts || slice * VB >= P.row_bytes) continue;
        const int len = P.rowptr[row + 1] - P.rowptr[row];
        acc_t acc[S::NE];
#pragma unroll
        for (int i = 0; i < S::NE; ++i) acc[i] = (acc_t)0;
        add_chunks(first, last, lane_off, acc);
        S::store(P.out + (int64_t)row * P.row_bytes + lane_off, acc, row_scale<acc_t>(P.row_mode, len));
    }
    for (int64_t base = blockIdx.x; base < total; base += (int64_t)gridDim.x * kBlock) {
        int n = 1;
        if (spread) {
            if (tid == 0) n_many = 0;
            __syncthreads();
            const int64_t at = base + (int64_t)tid * gridDim.x;
            if (at < total) {
                const int li = (int)(at / P.ntiles);
                if (P.chunk_ptr[li + 1] - P.chunk_ptr[li] > parts) many[atomicAdd(&n_many, 1)] = tid;      // in any order: units are independent
            }
            __syncthreads();
            n = n_many;
        }
        for (int m = 0; m < n; ++m) {
            const int64_t unit = spread ? base + (int64_t)many[m] * gridDim.x : base;
            const int li = (int)(unit / P.ntiles), tile = (int)(unit - (int64_t)li * P.ntiles);
            const int64_t slice = (int64_t)tile * P.G + sub, lane_off = slice_offset<VB>(P, slice);
            const bool active = slice * VB < P.row_bytes;
            const int row = P.long_rows[li], first = P.chunk_ptr[li], last = P.chunk_ptr[li + 1];
            const int per = (last - first + parts - 1) / parts;
            const int lo = first + part * per, hi = lo + per < last ? lo + per : last;
            acc_t acc[S::NE];
#pragma unroll
            for (int i = 0; i < S::NE; ++i) acc[i] = (acc_t)0;
            if (active) add_chunks(lo, hi, lane_off, acc);
            __syncthreads();                       // the previous unit's sums have been read
#pragma unroll
            for (int i = 0; i < S::NE; ++i) range_sum[i][tid] = acc[i];
            __syncthreads();
            if (part != 0 || !active) continue;    // the barriers of the next unit are reached by all
            for (int q = 1; q < parts && q * per < last - first; ++q)
#pragma unroll
                for (int i = 0; i < S::NE; ++i) acc[i] += range_sum[i][q * P.G + sub];
            const int len = P.rowptr[row + 1] - P.rowptr[row];
            S::store(P.out + (int64_t)row * P.row_bytes + lane_off, acc, row_scale<acc_t>(P.row_mode, len));
        }
        __syncthreads();                           // the list is the next units'
    }
}

// A row's last slice ends with the row (slice_offset): rows of any length move 16 bytes per lane.
template <int DT, int VB>
__global__ __launch_bounds__(kBlock) void k_gather_rows(const char *__restrict__ table,
                                                        const int64_t *__restrict__ ids, int64_t num_units,
                                                        int32_t ntiles, uint64_t tile_inv, int32_t lg_G, int64_t row_bytes,
                                                        char *__restrict__ out)
{
    using S = Slice<DT, VB>;
    const int tid = threadIdx.x;
    const int sub = tid & ((1 << lg_G) - 1);
    const int64_t unit = ((int64_t)blockIdx.x * kBlock + tid) >> lg_G;
    if (unit >= num_units) return;
    const int64_t row = ntiles > 1 ? (int64_t)__umul64hi((uint64_t)unit, tile_inv) : unit;   // unit * ntiles < 2^64
    const int tile = (int)(unit - row * ntiles);
    const int64_t at = (((int64_t)tile << lg_G) + sub) * VB, lane_off = at < row_bytes - VB ? at : row_bytes - VB;
    if (at >= row_bytes) return;
    uint32_t r[S::NW];
    S::load(table + ids[row] * row_bytes + lane_off, r);
    char *p = out + row * row_bytes + lane_off;
    if constexpr (VB == 16) *reinterpret_cast<typename S::u32x4 *>(p) = typename S::u32x4{r[0], r[1], r[2], r[3]};
    else if constexpr (VB == 8) *reinterpret_cast<typename S::u32x2 *>(p) = typename S::u32x2{r[0], r[1]};
    else if constexpr (VB == 4) *reinterpret_cast<typename S::u32x1 *>(p) = r[0];
    else *reinterpret_cast<uint16_t *>(p) = (uint16_t)r[0];
}

// ------------------------------------------------------------- host side ----
// Width of a slice: 16 bytes, or as much of that as fits a row.  Rows need not be whole slices (slice_offset).
static int slice_bytes(int64_t row_bytes)
{
    int vb = 16;
    while (vb > row_bytes) vb >>= 1;
    return vb;
}

// ceil(2^64 / n): the upper half of its product with x is x / n while x * n < 2^64.  0 for n = 1.
static uint64_t tile_inverse(int64_t n) { return n > 1 ? UINT64_MAX / (uint64_t)n + 1 : 0; }

static void group_shape(int64_t row_bytes, int vb, int smallest, int *G, int *ntiles)
{
    const int64_t slices = ceil_div(row_bytes, (int64_t)vb);
    int g = smallest;
    while (g < kWave && g < slices) g <<= 1;
    *G = g;
    *ntiles = (int)ceil_div(slices, g);
}

// Are rows wider than 32 slices gathered in column tiles of 32?  The choice decides in which order the edges of a row are
// added, so it looks at sizes alone.  Not where the columns of long rows ascend, nor where tiles would share cache lines
// (602 columns: 83 us whole, 93 in tiles).  1 024 row sets keep the wavefronts of a tile many.
constexpr int kTileLanes = 32;

static bool column_tiles(int64_t num_rows, int64_t num_cols, int64_t nnz, int64_t row_bytes)
{
    return row_bytes > kTileLanes * 16 && row_bytes % (kTileLanes * 16) == 0 &&
           num_cols * row_bytes >= (int64_t)128 << 20 && num_cols * (row_bytes / 16) <= (int64_t)UINT32_MAX &&
           nnz >= 5 * num_cols && num_row_sets(num_rows, nnz) >= 1024;
}

// All rows of one tile after the other: the gathers of a pass come from a table that is so much smaller, and more of its
// often used rows stay in the caches.  But every pass reads the column ids and their scale factors again, and factors of
// more than 2^18 columns fall out of L2 in between: then only where columns that are read more than kLongThreshold
// times have a quarter of the edges, which a plan with the transpose knows (on the device; sums are the same either way).
// us, whole rows / tiles of a row together / one tile after the other, columns drawn evenly, and in proportion to rank^-0.8
// and ^-1.1 (12 % to 22 % and 44 % to 60 % of the edges are such columns'):
//   256 f32 mean  200 MB read 12 times: 336 / 340 / 330, 292 / 290 / 272, 165 / 170 / 154;  600 MB: 979 / 978 / 990, 922 / 911 / 838,
//                 528 / 529 / 470;  900 MB: 1 526 / 1 525 / 1 497, 1 322 / 1 327 / 1 298, 810 / 812 / 723
//   256 f32 gcn   200 MB: 359 / 354 / 352, 310 / 301 / 292, 182 / 188 / 175;  600 MB: 1 075 / 1 072 / 1 145, 1 020 / 1 005 / 1 002,
//                 597 / 598 / 572;  900 MB: 1 638 / 1 636 / 1 771, 1 470 / 1 471 / 1 535, 919 / 923 / 887
//   512 bf16 gcn  600 MB: 1 073 / 1 097 / 1 146, 1 020 / 1 030 / 1 006, 595 / 608 / 574
//   1 024 f32 gcn 600 MB: 1 002 / 989 / 1 000, 962 / 930 / 775, 658 / 657 / 523
// all neighbours in a power-law graph (656 MB read 9 times, 36 %): 256 f32 gcn 820 / 790 / 753, mean 777 / 765 / 690; 512 bf16
// gcn 880 / 840 / 795; another (557 MB, 6 times, 25 %) 469 / 446 / 436; (608 MB, 9 times, 4 %) 837 / 821 / 873
constexpr int64_t kScaleInL2 = (int64_t)1 << 18;

static void tile_order(const PullDesc &d, PullParams &P)
{
    if ((uintptr_t)d.in & 127) return;                         // tiles would share cache lines: together
    P.by_tile = !d.col_scale || d.num_cols <= kScaleInL2;
    P.hot = P.by_tile ? nullptr : d.hot_chunks;
    P.hot_min = ceil_div(d.nnz, (int64_t)4 * kLongChunk);
}

// 32 lanes have 8 gathers in flight where there are wavefronts enough to hide the longer way through the code, f32.  us, rows
// of 2 to 8 edges (twice as many columns as rows), 6 in flight / 8, 100 columns sum, 100 gcn, 128 weighted:
//   16 000 rows (6 000 wavefronts) 9.4 / 10.7, 11.1 / 11.6, 11.1 / 11.7;  64 000 (12 000) 29.4 / 29.9, 31.5 / 32.3, 31.7 / 32.0;
//   128 000 (24 000, as the larger ones) 55.7 / 55.2, 59.9 / 59.9, 56.6 / 56.6;  256 000 110.4 / 109.8, 122.3 / 121.2, 113.9 / 112.6;
//   512 000 216.2 / 215.7, 247.2 / 247.7, 221.7 / 221.0;  2.56 M edges of a products-shaped block 200.0 / 197.6, 218.0 / 216.4
// bf16 gains nothing on average and loses up to 1.2 % with scale factors (256 columns, 512 000 rows: 252.8 / 255.7).
constexpr int64_t kManyWaves = 16384;

template <int DT, int VB, int W>
static void launch_rows(const PullParams &P, hipStream_t s)
{
    const dim3 grid((unsigned)P.num_blocks);
    if (P.G == kWave) hipLaunchKernelGGL((k_pull_rows<DT, VB, W, kUnrollWave, true, false>), grid, dim3(kBlock), 0, s, P);
    else if (P.G <= kBatchLanes) hipLaunchKernelGGL((k_pull_rows<DT, VB, W, kUnrollNarrow, false, true>), grid, dim3(kBlock), 0, s, P);
    else if (P.G == kTileLanes && (P.ntiles > 1 || (DT == FASTGL_F32 && P.nwaves >= kManyWaves))) hipLaunchKernelGGL((k_pull_rows<DT, 16, W, kUnrollWave, false, false>), grid, dim3(kBlock), 0, s, P);
    else hipLaunchKernelGGL((k_pull_rows<DT, 16, W, kUnroll, false, false>), grid, dim3(kBlock), 0, s, P);
}

template <int DT, int VB>
static fastgl_status launch_typed(const PullParams &P, unsigned reduce_blocks, hipStream_t s)
{
    if (P.num_blocks > 0) {
        if (P.edge_w && P.col_scale) launch_rows<DT, VB, kTwoWeights>(P, s);
        else if (P.edge_w && P.eid) launch_rows<DT, VB, kPermWeight>(P, s);
        else if (P.edge_w) launch_rows<DT, VB, kEdgeWeight>(P, s);
        else if (P.col_scale) launch_rows<DT, VB, kColWeight>(P, s);
        else launch_rows<DT, VB, kNoWeight>(P, s);
        FASTGL_LAUNCH_CHECK("k_pull_rows");
    }
    if (reduce_blocks) {
        hipLaunchKernelGGL((k_reduce_chunks<DT, VB>), dim3(reduce_blocks), dim3(kBlock), 0, s, P);
        FASTGL_LAUNCH_CHECK("k_reduce_chunks");
    }
    return FASTGL_OK;
}

fastgl_status launch_pull(const PullDesc &d, hipStream_t s)
{
    if (d.num_rows == 0) return FASTGL_OK;
    const int elem = d.dtype == FASTGL_F32 ? 4 : 2;
    PullParams P;
    P.rowptr = d.rowptr; P.col = d.col; P.eid = d.eid;
    P.edge_w = d.edge_w; P.col_scale = d.col_scale;
    P.in = (const char *)d.in; P.out = (char *)d.out;
    P.row_bytes = d.feat * elem;
    P.feat = d.feat;
    P.row_mode = d.row_mode;
    P.by_tile = 0;
    P.hot = nullptr; P.hot_min = 0;
    const int vb = slice_bytes(P.row_bytes);
    int G, ntiles;
    group_shape(P.row_bytes, vb, kUnrollNarrow, &G, &ntiles);   // a group loads as many column ids at a time as it has lanes
    P.unit_shift = 1;
    while ((1 << P.unit_shift) < vb && P.row_bytes % (2 << P.unit_shift) == 0) ++P.unit_shift;
    // walk_flat counts units in 32 bits; beyond that (more than 2^27 rows of 32 slices) a whole wavefront takes a row
    if (d.num_cols * (P.row_bytes >> P.unit_shift) > (int64_t)UINT32_MAX) {
        G = kWave;
        ntiles = (int)ceil_div(ceil_div(P.row_bytes, (int64_t)vb), (int64_t)G);
    }
    const bool tiles = d.any_order && column_tiles(d.num_rows, d.num_cols, d.nnz, P.row_bytes);
    if (tiles) {
        G = kTileLanes;
        ntiles = (int)(P.row_bytes / (kTileLanes * vb));
        tile_order(d, P);
    }
    P.G = G; P.ntiles = ntiles;
    P.lg_G = __builtin_ctz((unsigned)G);
    P.num_rows = d.num_rows;
    P.split = d.split;
    P.nsets = d.nsets;
    // Fine sets per wavefront: as few as leave every compute unit four wavefronts, until a group has kUnrollNarrow edges
    // to gather (512 rows of 16 floats with 430 edges: 4 sets 11.6 us, 1 set 5.2); up to a set (16 edges and rows) per group
    // while that gives at least the 4 096 wavefronts that the device holds at once; more when there are plenty: that amortises
    // the row-pointer / column-id latency over more gathers while keeping >= 16 K wavefronts (at least 8 K: all neighbours,
    // width 32, forward 98 -> 106 us, 2.56 M edges of 64 floats 113 -> 118; at least 32 K: 104 and 117).
    const int groups = kWave / G;
    int spw = 1;
    while (spw < groups / kUnrollNarrow && d.nsets / (spw * 2) * ntiles >= 1024) spw *= 2;
    while (spw < groups && d.nsets / (spw * 2) * ntiles >= 4096) spw *= 2;
    while (spw >= groups && spw < 8 * groups && d.nsets / (spw * 2) * ntiles >= 16384) spw *= 2;
    P.sets_per_wave = spw;
    P.nwaves = ceil_div(d.nsets, (int64_t)spw);
    P.tile_inv = tile_inverse(ntiles);
    P.wave_inv = tile_inverse(P.nwaves);
    const bool with_long = d.long_rows != nullptr && d.nnz > kLongThreshold;
    P.long_thr = with_long ? kLongThreshold : INT32_MAX;
    P.long_rows = with_long ? d.long_rows : nullptr;
    P.chunk_ptr = d.chunk_ptr; P.n_long = d.n_long; P.n_chunks = d.n_chunks;
    P.partials = (char *)d.partials;
    P.num_blocks = ceil_div(ceil_div(P.nwaves * ntiles, (int64_t)(kBlock / kWave)), (int64_t)kXcds * kXcdRun) * kXcdRun * kXcds;
    P.chunk_waves = tiles ? P.nwaves : P.num_blocks * (kBlock / kWave) / ntiles;
    if (P.num_blocks > 0x7FFFFFFFLL) {
        set_error("block too large for one launch (%lld workgroups)", (long long)P.num_blocks);
        return FASTGL_ERR_UNSUPPORTED;
    }
    // workgroups for the long rows: no more than there can be
    const int64_t most_long = cap_long_rows(d.nnz) * ntiles;
    const unsigned reduce_blocks = !with_long ? 0u : (unsigned)(most_long < kReduceBlocks ? most_long : kReduceBlocks);
#define FASTGL_CASE(DT, VB) return launch_typed<DT, VB>(P, reduce_blocks, s)
    if (d.dtype == FASTGL_F32) {
        switch (vb) {
            case 16: FASTGL_CASE(FASTGL_F32, 16);
            case 8: FASTGL_CASE(FASTGL_F32, 8);
            default: FASTGL_CASE(FASTGL_F32, 4);
        }
    } else {
        switch (vb) {
            case 16: FASTGL_CASE(FASTGL_BF16, 16);
            case 8: FASTGL_CASE(FASTGL_BF16, 8);
            case 4: FASTGL_CASE(FASTGL_BF16, 4);
            default: FASTGL_CASE(FASTGL_BF16, 2);
        }
    }
#undef FASTGL_CASE
}

fastgl_status launch_gather_rows(const void *table, const int64_t *ids, int64_t n, int64_t feat,
                                 fastgl_dtype dtype, void *out, hipStream_t s)
{
    if (n == 0) return FASTGL_OK;
    const int elem = dtype == FASTGL_F32 ? 4 : 2;
    const int64_t row_bytes = feat * elem;
    const int vb = slice_bytes(row_bytes);
    int G, ntiles;
    group_shape(row_bytes, vb, 1, &G, &ntiles);
    const int64_t units = n * ntiles;
    const int64_t nblocks = ceil_div(units * G, kBlock);
    if (nblocks > 0x7FFFFFFFLL) {
        set_error("gather too large for one launch");
        return FASTGL_ERR_UNSUPPORTED;
    }
    dim3 grid((unsigned)nblocks);
    const int lg_G = __builtin_ctz((unsigned)G);
    const char *t = (const char *)table;
    char *o = (char *)out;
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(kBlock), 0, s, t, ids, units, ntiles, tile_inverse(ntiles), lg_G, row_bytes, o); };
    if (dtype == FASTGL_F32) {
        switch (vb) {
            case 16: go(k_gather_rows<FASTGL_F32, 16>); break;
            case 8: go(k_gather_rows<FASTGL_F32, 8>); break;
            default: go(k_gather_rows<FASTGL_F32, 4>); break;
        }
    } else {
        switch (vb) {
            case 16: go(k_gather_rows<FASTGL_BF16, 16>); break;
            case 8: go(k_gather_rows<FASTGL_BF16, 8>); break;
            case 4: go(k_gather_rows<FASTGL_BF16, 4>); break;
            default: go(k_gather_rows<FASTGL_BF16, 2>); break;
        }
    }
    FASTGL_LAUNCH_CHECK("k_gather_rows");
    return FASTGL_OK;
}

}  // namespace fastgl

extern "C" int32_t fastgl_aggregate_column_tiles(int64_t num_dst, int64_t num_src, int64_t num_edges, int64_t feat, fastgl_dtype dtype)
{
    using namespace fastgl;
    const int64_t row_bytes = feat * (dtype == FASTGL_F32 ? 4 : 2);
    if (num_dst < 0 || num_src < 0 || num_edges < 0 || feat <= 0 || feat > (int64_t)1 << 24) return 0;
    return column_tiles(num_dst, num_src, num_edges, row_bytes) ? (int32_t)(row_bytes / (kTileLanes * 16)) : 1;
}
