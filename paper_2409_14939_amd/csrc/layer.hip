// One sampled GNN layer in one call: aggregation (paper Section 2.1, Eq. 1) followed by the update
// Y = act(H W + b) (Eq. 2).  See include/fastgl_update.h for the contract of fastgl_layer_fwd.
//
// For a narrow layer on few target nodes - the class-score layer of a sampled GCN: a few thousand
// seeds, 256 features in, a few dozen classes out - both steps run in ONE kernel: the aggregated
// rows never travel to memory and back (they are written once, for the backward pass, only if the
// caller asks for them).  The product of such a layer is a fraction of a GFLOP, a microsecond of
// the vector ALUs, and the kernel is bound by its row gathers like the aggregation kernel is, so
// the product is done with plain fp32 multiply-adds rather than on the matrix cores.
//
//   workgroup = 4 wavefronts; a wavefront owns RPW consecutive target rows and a quarter of the K terms
//   1. lane n loads its column of the wavefront's quarter of W (K x N) into registers, all loads in flight
//      together, behind the row pointers'
//   2. each wavefront walks the edges of its rows as one flat list (the aggregation kernel's
//      walk: 64 lanes x 16 bytes cover a row of up to 256 floats, 8 row gathers in flight, fp64
//      sums), scales and rounds each finished row to fp32 exactly as the aggregation kernel does,
//      and keeps it in LDS
//   3. lane n forms the sum of its quarter's terms for ALL rows of the workgroup, k ascending, one fp32
//      multiply-add per term (H[r][k..k+3] is one broadcast 16-byte read); the four sums go through LDS and
//      y[r][n] = ((s0 + s1) + (s2 + s3)) + b[n]
// Bound by latency where there are few rows: the rows' gathers and W come in together, and the chain of
// multiply-adds is a quarter of K long.  K = 256, N = 47, us,
// W through LDS and K terms per wavefront -> now: 16 rows of 15 edges 21.6 -> 8.5, 8 000 rows 42 -> 37.
//
// Every other shape takes the two kernels of the separate calls, back to back on the stream.
#include "fastgl_update.h"
#include "pull_walk.h"

namespace fastgl {
namespace {

constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kMaxFusedK = 256;     // 64 lanes x 4 floats
constexpr int kFusedCols = 64;      // one lane per output column
constexpr int kQuarter = kMaxFusedK / kWavesPerBlock;   // most terms of a wavefront
// Rows of a wavefront: one, two or four while that gives at most three workgroups per compute unit (every workgroup reads W
// once); beyond that two again, which leave the unit more wavefronts, for half as many rows more, and up to 65 536 rows where a row gathers
// much (kMuch: columns times edges).  us right after X was written, GCN, 1 / 2 / 4 rows, by K -> N and edges of a row:
//   rows      256 -> 47, 15       256 -> 47, 5        100 -> 47, 15       100 -> 47, 5        64 -> 16, 10
//   2 048     13.8 / 15.4 / 24.0  11.2 / 12.8 / 19.0  10.7 / 12.1 / 17.2                      8.9 / 9.9 / 13.1
//   3 000     16.3 / 17.8 / 23.4  12.9 / 14.0 / 19.6  12.0 / 13.2 / 17.7                      9.9 / 10.8 / 13.5
//   4 000     21.5 / 20.0 / 25.4  17.3 / 14.9 / 20.3  16.4 / 13.8 / 18.0                      13.6 / 10.9 / 13.6
//   6 000     26.5 / 25.5 / 30.4  20.2 / 18.0 / 22.3  19.2 / 16.4 / 20.2                      15.4 / 12.3 / 14.7
//   8 000     29.7 / 31.9 / 32.2  19.4 / 19.9 / 19.8  20.3 / 20.1 / 18.6  14.6 / 12.9 / 12.4  15.8 / 14.6 / 12.7
//   12 000    40.0 / 40.8 / 43.4  26.6 / 23.6 / 24.6  27.8 / 24.0 / 23.2  20.4 / 15.7 / 14.3  21.8 / 16.9 / 14.8
//   13 000    42.6 / 44.6 / 56.4  28.9 / 27.6 / 35.6  30.4 / 28.2 / 32.2  22.3 / 18.8 / 20.7  23.8 / 20.1 / 21.2
//   16 000    49.5 / 50.0 / 62.4  34.2 / 30.8 / 37.8  36.0 / 31.7 / 35.3  27.2 / 20.9 / 22.6  28.6 / 22.4 / 22.5
//   20 000    59.1 / 59.8 / 71.6  41.6 / 36.5 / 42.7  43.1 / 38.4 / 39.2  32.2 / 25.2 / 24.5  34.7 / 27.0 / 25.0
//   32 000    109 / 99 / 109      62.8 / 53.0 / 60.6  66.6 / 55.8 / 57.5  49.2 / 36.6 / 34.6  53.0 / 39.7 / 35.1
//   64 000    225 / 201 / 210     123 / 99 / 109      133 / 106 / 106     95.9 / 67.5 / 61.1  102 / 74 / 63
//   100 000   351 / 318 / 324     217 / 176 / 169     245 / 198 / 181     146 / 103 / 90      157 / 113 / 96
constexpr int64_t kOneRow = 3 * 256 * kWavesPerBlock, kManyRows = (int64_t)1 << 16, kMuch = 1024;

struct LayerParams {
    PullParams pull;                // rowptr, col, eid, edge_w, col_scale, in, G = 64, row_mode, row_bytes, feat
    const float *W, *bias;          // [K][N], [N] or NULL
    float *H, *Y;                   // [rows][K] or NULL, [rows][N]
    int64_t rows;
    int32_t K, N, relu;
};

// A finished row: scaled and rounded to fp32 once (the value the aggregation kernel would store),
// kept in LDS for the product and, if asked for, streamed to H.
struct RowToLds {
    float *lds_rows;                // this wavefront's rows, [rows][K]
    float *H;
    int64_t row0;                   // first row of the wavefront
    int32_t K, sub;
    bool active;
    __device__ __forceinline__ void operator()(int64_t row, const double (&acc)[4], double scale) const
    {
        if (!active) return;
        const float4 v = make_float4((float)(acc[0] * scale), (float)(acc[1] * scale), (float)(acc[2] * scale),
                                     (float)(acc[3] * scale));
        *reinterpret_cast<float4 *>(lds_rows + (row - row0) * K + 4 * sub) = v;
        if (H) {
            typedef float f32x4 __attribute__((ext_vector_type(4)));
            const f32x4 w = {v.x, v.y, v.z, v.w};
            __builtin_nontemporal_store(w, reinterpret_cast<f32x4 *>(H + row * K + 4 * sub));
        }
    }
};

template <int WEIGHTS, int RPW>
__global__ __launch_bounds__(kBlock) void k_layer_rows(const LayerParams L)
{
    constexpr int ROWS = RPW * kWavesPerBlock;
    __shared__ __attribute__((aligned(16))) float h_lds[ROWS * kMaxFusedK];     // [ROWS][K]
    __shared__ float part[kWavesPerBlock][ROWS][kFusedCols];
    const PullParams &P = L.pull;
    const int K = L.K, N = L.N;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int64_t row0 = (int64_t)blockIdx.x * ROWS + wave * RPW;
    const int nrows = L.rows - row0 < RPW ? (int)(L.rows - row0) : RPW;         // may be <= 0
    int pb = 0, pe = 0;
    if (lane < nrows) {
        pb = P.rowptr[row0 + lane];
        pe = P.rowptr[row0 + lane + 1];
    }

    // 1. this wavefront's terms of W: k_first .. + terms, K and both of them multiples of 4
    const int per = 4 * ((K + 4 * kWavesPerBlock - 1) / (4 * kWavesPerBlock)), k_first = wave * per;
    const int terms = K - k_first < per ? K - k_first : per;                    // may be <= 0
    float w[kQuarter];
    const float *w_col = L.W + (lane < N ? lane : N - 1);
#pragma unroll
    for (int i = 0; i < kQuarter; ++i) {
        const int k = k_first + i;
        w[i] = w_col[(int64_t)(k < K ? k : K - 1) * N];
    }
    __builtin_amdgcn_sched_barrier(0);

    // 2. aggregate this wavefront's rows into LDS
    if (nrows > 0) {
        const bool active = 4 * lane < K;
        const RowToLds sink = {h_lds + wave * RPW * K, L.H, row0, K, lane, active};
        walk_wave<FASTGL_F32, 16, WEIGHTS, false, kUnrollWave>(P, row0, 0, nrows, lane_value(pb, 0), pe,
                                                               row_scale<double>(P.row_mode, pe - pb), lane,
                                                               (int64_t)lane * 16, active, sink);
    }
    __syncthreads();

    // 3. lane = output column; rows that do not exist hold whatever LDS held: computed, never stored
    float acc[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) acc[r] = 0.f;
#pragma unroll
    for (int i = 0; i < kQuarter; i += 4) {
        if (i < terms) {                                                        // the same for the wavefront
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const float4 h = *reinterpret_cast<const float4 *>(h_lds + r * K + k_first + i);
                acc[r] = __builtin_fmaf(h.x, w[i], acc[r]);
                acc[r] = __builtin_fmaf(h.y, w[i + 1], acc[r]);
                acc[r] = __builtin_fmaf(h.z, w[i + 2], acc[r]);
                acc[r] = __builtin_fmaf(h.w, w[i + 3], acc[r]);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) part[wave][r][lane] = acc[r];
    __syncthreads();
    if (lane >= N) return;
    const float b = L.bias ? L.bias[lane] : 0.f;
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        if (i >= nrows) break;
        const int r = wave * RPW + i;
        float v = ((part[0][r][lane] + part[1][r][lane]) + (part[2][r][lane] + part[3][r][lane])) + b;
        if (L.relu) v = v > 0.f ? v : 0.f;
        L.Y[(row0 + i) * N + lane] = v;
    }
}

bool fuses(int64_t K, int64_t N, fastgl_dtype dtype, const void *X, const void *H)
{
    return dtype == FASTGL_F32 && K > 0 && K % 4 == 0 && K <= kMaxFusedK && N > 0 && N <= kFusedCols &&
           (((uintptr_t)X | (uintptr_t)H) & 15) == 0;
}

template <int WEIGHTS>
void launch_layer(const LayerParams &L, int64_t edges, hipStream_t s)
{
    const bool much = L.rows <= kManyRows && L.K * edges >= kMuch * L.rows;
    if (L.rows <= kOneRow)
        hipLaunchKernelGGL((k_layer_rows<WEIGHTS, 1>), dim3((unsigned)ceil_div(L.rows, kWavesPerBlock)), dim3(kBlock), 0, s, L);
    else if (L.rows <= 2 * kOneRow || (L.rows > 4 * kOneRow && (L.rows <= 6 * kOneRow || much)))
        hipLaunchKernelGGL((k_layer_rows<WEIGHTS, 2>), dim3((unsigned)ceil_div(L.rows, 2 * kWavesPerBlock)), dim3(kBlock), 0, s, L);
    else
        hipLaunchKernelGGL((k_layer_rows<WEIGHTS, 4>), dim3((unsigned)ceil_div(L.rows, 4 * kWavesPerBlock)), dim3(kBlock), 0, s, L);
}

}  // namespace
}  // namespace fastgl

using namespace fastgl;

extern "C" {

int fastgl_layer_fwd_fuses(int64_t K, int64_t N, fastgl_dtype dtype)
{
    return fuses(K, N, dtype, nullptr, nullptr) ? 1 : 0;
}

fastgl_status fastgl_layer_fwd(const int32_t *indptr, const int32_t *indices, const float *edge_w, int64_t num_dst,
                               int64_t num_src, int64_t num_edges, int64_t K, fastgl_agg_mode mode,
                               fastgl_dtype dtype, const void *X, const void *W, const float *bias, int64_t N,
                               int relu, void *H, void *Y, const fastgl_plan *plan, void *workspace,
                               size_t workspace_bytes, void *stream)
{
    if (N < 0 || N >= ((int64_t)1 << 24)) {
        set_error("N must be in [0, 2^24) (got %lld)", (long long)N);
        return FASTGL_ERR_INVALID_ARG;
    }
    const bool fused = fuses(K, N, dtype, X, H);
    if (!H && !fused && num_dst > 0 && N > 0) {
        set_error("H is NULL but this shape (K=%lld N=%lld) runs as two kernels, which hand H over in memory",
                  (long long)K, (long long)N);
        return FASTGL_ERR_INVALID_ARG;
    }
    // the aggregation's own checks; with H == NULL they are given Y's address only to pass the
    // "output pointer is not NULL" test - nothing is stored there by the aggregation
    size_t need = 0;
    fastgl_status st = aggregate_check(false, indptr, indices, edge_w, num_dst, num_src, num_edges, K, mode, dtype, X,
                                       H ? H : Y, plan, &need);
    if (st != FASTGL_OK) return st;
    const uintptr_t el = dtype == FASTGL_F32 ? 4 : 2;
    if (num_dst > 0 && N > 0 && (!W || !Y)) {
        set_error("W or Y is NULL");
        return FASTGL_ERR_INVALID_ARG;
    }
    if ((((uintptr_t)W | (uintptr_t)Y | (uintptr_t)H) & (el - 1)) || ((uintptr_t)bias & 3)) {
        set_error("matrices must be aligned to their element size");
        return FASTGL_ERR_INVALID_ARG;
    }
    if (!workspace || ((uintptr_t)workspace & 255)) {
        set_error("workspace must be a 256-byte aligned device buffer");
        return FASTGL_ERR_INVALID_ARG;
    }
    if (workspace_bytes < need) {
        set_error("workspace too small: %zu < %zu bytes", workspace_bytes, need);
        return FASTGL_ERR_WORKSPACE;
    }
    if (num_dst == 0 || (N == 0 && !H)) return FASTGL_OK;

    if (!fused) {
        // two kernels back to back: aggregation into H, then the update phase's kernel
        st = aggregate_run(false, indptr, indices, edge_w, num_dst, num_src, num_edges, K, mode, dtype, X, H, plan,
                           workspace, stream);
        if (st != FASTGL_OK || N == 0) return st;
        return dtype == FASTGL_F32
                   ? fastgl_update_fwd((const float *)H, (const float *)W, bias, num_dst, K, N, relu, (float *)Y, stream)
                   : fastgl_update_fwd_bf16((const uint16_t *)H, (const uint16_t *)W, bias, num_dst, K, N, relu,
                                            (uint16_t *)Y, stream);
    }

    fastgl_plan local;
    PullDesc d;
    st = aggregate_prepare(false, indptr, indices, edge_w, num_dst, num_src, num_edges, K, mode, dtype, X, H, plan,
                           workspace, stream, &local, &d);
    if (st != FASTGL_OK) return st;
    LayerParams L = {};
    PullParams &P = L.pull;
    P.rowptr = d.rowptr; P.col = d.col; P.eid = d.eid;
    P.edge_w = d.edge_w; P.col_scale = d.col_scale;
    P.in = (const char *)d.in; P.out = nullptr;
    P.G = kWave; P.ntiles = 1;
    P.row_mode = d.row_mode;
    P.row_bytes = K * 4;
    P.feat = K;
    P.num_rows = num_dst;
    L.W = (const float *)W; L.bias = bias;
    L.H = (float *)H; L.Y = (float *)Y;
    L.rows = num_dst; L.K = (int32_t)K; L.N = (int32_t)N; L.relu = relu != 0;
    hipStream_t s = (hipStream_t)stream;
    if (d.edge_w && d.col_scale) launch_layer<kTwoWeights>(L, num_edges, s);
    else if (d.edge_w) launch_layer<kEdgeWeight>(L, num_edges, s);
    else if (d.col_scale) launch_layer<kColWeight>(L, num_edges, s);
    else launch_layer<kNoWeight>(L, num_edges, s);
    FASTGL_LAUNCH_CHECK("fastgl_layer_fwd");
    return FASTGL_OK;
}

}  // extern "C"
