// Update phase (paper Section 2.1, Eq. 2) with at most kNarrowCols result columns: attention
// projections (N = 1), class scores of few classes.  See include/fastgl_update.h for the contract.
//
// With N <= 8 the products are a matrix-vector product (Y), an outer product (dH) and a weighted column
// sum (dW): 2 N flops per element of H, bound by reading H once (Y, dW) or writing dH once.  The tiled
// matrix-core kernel spends 128 result columns of work on them and waits for a narrow column of loads
// per step.  Here a group of G lanes (a power of two, quads of four elements per lane) covers a row, as
// in the aggregation kernel, and several rows are in flight per lane; products are plain fp32
// multiply-adds (one rounding per term, sums of four lanes' chains added pairwise).
// M = 1 150 398, K = 64, N = 1, fp32, us in the step of an attention head (part of H still in the Infinity Cache):
// dH 148 -> 55, dW 239 -> 47 (6.3 TB/s); a call with cold caches, the reduction included: 152 -> 59, 358 -> 114.
// Y comes from here for up to kNarrowRows rows (update.hip): 20 000 rows 18.7 -> 7.6.
#include "update_internal.h"

namespace fastgl {
namespace {

constexpr int kRows = 4;            // rows in flight per lane group

template <bool BF16>
__device__ __forceinline__ float elem_f32(const void *p, int64_t i)
{
    if (BF16) return __uint_as_float((uint32_t)static_cast<const uint16_t *>(p)[i] << 16);
    return static_cast<const float *>(p)[i];
}

// Four elements k .. k+3 of a row that starts at element `row`; elements at or beyond K read as 0.
// VEC: K is a multiple of 4 and rows are aligned to quads.
template <bool VEC, bool BF16>
__device__ __forceinline__ float4 load4(const void *p, int64_t row, int64_t k, int64_t K)
{
    typedef typename QuadBits<BF16>::elem E;
    const E *q = static_cast<const E *>(p) + row + k;
    if (VEC) return quad_to_f32(*reinterpret_cast<const typename QuadBits<BF16>::type *>(q));
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = k + i < K ? elem_f32<BF16>(q, i) : 0.f;
    return make_float4(v[0], v[1], v[2], v[3]);
}

__device__ __forceinline__ float part_of(const float4 &v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }

// W[k .. k+3][0 .. N) as fp32; rows at or beyond K and columns at or beyond N are 0.
template <int NMAX, bool BF16>
__device__ __forceinline__ void load_w(const NarrowArgs &a, int64_t k, float (&w)[4][NMAX])
{
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int n = 0; n < NMAX; ++n) w[i][n] = k + i < a.K && n < a.N ? elem_f32<BF16>(a.W, (k + i) * a.N + n) : 0.f;
}

// dZ[m][0 .. N), gated; columns at or beyond N are 0.
template <int NMAX, bool BF16>
__device__ __forceinline__ void load_dz(const NarrowArgs &a, int64_t m, float (&z)[NMAX])
{
#pragma unroll
    for (int n = 0; n < NMAX; ++n) {
        z[n] = n < a.N ? elem_f32<BF16>(a.dY, m * a.N + n) : 0.f;
        if (a.gate && n < a.N) z[n] = elem_f32<BF16>(a.gate, m * a.N + n) > 0.f ? z[n] : 0.f;
    }
}

// Y = act(H W + b): a group of G lanes takes kRows rows at a time.
template <int NMAX, bool VEC, bool BF16>
__global__ __launch_bounds__(256) void k_narrow_fwd(const NarrowArgs a, int G)
{
    typedef typename QuadBits<BF16>::elem E;
    const int sub = threadIdx.x & (G - 1);
    const int64_t m0 = ((int64_t)blockIdx.x * (256 / G) + threadIdx.x / G) * kRows;
    if (m0 >= a.M) return;
    float acc[kRows][NMAX];
#pragma unroll
    for (int r = 0; r < kRows; ++r)
#pragma unroll
        for (int n = 0; n < NMAX; ++n) acc[r][n] = 0.f;
    for (int64_t k = 4 * sub; k < a.K; k += 4 * G) {
        float4 h[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r)     // rows past the end re-read the last one; they are not stored
            h[r] = load4<VEC, BF16>(a.H, (m0 + r < a.M ? m0 + r : a.M - 1) * a.K, k, a.K);
        float w[4][NMAX];
        load_w<NMAX, BF16>(a, k, w);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int r = 0; r < kRows; ++r)
#pragma unroll
                for (int n = 0; n < NMAX; ++n) acc[r][n] = __builtin_fmaf(part_of(h[r], i), w[i][n], acc[r][n]);
    }
    for (int d = G >> 1; d > 0; d >>= 1)
#pragma unroll
        for (int r = 0; r < kRows; ++r)
#pragma unroll
            for (int n = 0; n < NMAX; ++n) acc[r][n] += __shfl_xor(acc[r][n], d);
    if (sub != 0) return;
    E *y = static_cast<E *>(a.out);
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        if (m0 + r >= a.M) break;
#pragma unroll
        for (int n = 0; n < NMAX; ++n) {
            if (n >= a.N) break;
            float v = acc[r][n] + (a.bias ? a.bias[n] : 0.f);
            if (a.relu) v = v > 0.f ? v : 0.f;
            if constexpr (BF16) y[(m0 + r) * a.N + n] = f32_to_bf16(v);
            else y[(m0 + r) * a.N + n] = v;
        }
    }
}

// dH = dZ W^T: a lane writes one quad of kRows rows (blockIdx.y: which 4 G columns of dH).
template <int NMAX, bool VEC, bool BF16>
__global__ __launch_bounds__(256) void k_narrow_dh(const NarrowArgs a, int G)
{
    typedef typename QuadBits<BF16>::elem E;
    const int sub = threadIdx.x & (G - 1);
    const int64_t m0 = ((int64_t)blockIdx.x * (256 / G) + threadIdx.x / G) * kRows;
    const int64_t k = 4 * ((int64_t)blockIdx.y * G + sub);
    if (m0 >= a.M || k >= a.K) return;
    float w[4][NMAX], z[kRows][NMAX];
#pragma unroll
    for (int r = 0; r < kRows; ++r) load_dz<NMAX, BF16>(a, m0 + r < a.M ? m0 + r : a.M - 1, z[r]);
    load_w<NMAX, BF16>(a, k, w);
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        if (m0 + r >= a.M) break;
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i] = 0.f;                     // a sum that starts at +0: a gated-off row is +0 everywhere
#pragma unroll
            for (int n = 0; n < NMAX; ++n) v[i] = __builtin_fmaf(z[r][n], w[i][n], v[i]);
        }
        E *dst = static_cast<E *>(a.out) + (m0 + r) * a.K + k;
        if (VEC) {
            if constexpr (BF16) {
                typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                const u32x2 q = {(uint32_t)f32_to_bf16(v[0]) | ((uint32_t)f32_to_bf16(v[1]) << 16),
                                 (uint32_t)f32_to_bf16(v[2]) | ((uint32_t)f32_to_bf16(v[3]) << 16)};
                __builtin_nontemporal_store(q, reinterpret_cast<u32x2 *>(dst));
            } else {
                typedef float f32x4 __attribute__((ext_vector_type(4)));
                const f32x4 q = {v[0], v[1], v[2], v[3]};
                __builtin_nontemporal_store(q, reinterpret_cast<f32x4 *>(dst));
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (k + i >= a.K) break;
                if constexpr (BF16) dst[i] = f32_to_bf16(v[i]);
                else dst[i] = v[i];
            }
        }
    }
}

// Partials of dW and db over one slab of rows (blockIdx.x) for 4 G columns of H (blockIdx.y): every
// lane keeps the sums of its quad over the rows of its row lane, the 256 / G row lanes are added in LDS
// in a fixed order.  H may be NULL: db alone.
template <int NMAX, bool VEC, bool BF16>
__global__ __launch_bounds__(256) void k_narrow_dw(const NarrowArgs a, int G)
{
    __shared__ float red[256][4 * NMAX + 1];
    __shared__ float redz[256][NMAX];
    const int t = threadIdx.x, sub = t & (G - 1), lanes = 256 / G;
    const int64_t beg = (int64_t)blockIdx.x * a.slab, end = beg + a.slab < a.M ? beg + a.slab : a.M;
    const int64_t k = 4 * ((int64_t)blockIdx.y * G + sub);
    float acc[4][NMAX], zs[NMAX];
#pragma unroll
    for (int n = 0; n < NMAX; ++n) {
        zs[n] = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i][n] = 0.f;
    }
    const bool mine = a.H && k < a.K;
    for (int64_t m = beg + t / G; m < end; m += (int64_t)kRows * lanes) {
        float4 h[kRows];
        float z[kRows][NMAX];
#pragma unroll
        for (int r = 0; r < kRows; ++r) {   // rows past the end re-read the last one and count as 0
            const int64_t row = m + (int64_t)r * lanes < end ? m + (int64_t)r * lanes : end - 1;
            h[r] = mine ? load4<VEC, BF16>(a.H, row * a.K, k, a.K) : make_float4(0.f, 0.f, 0.f, 0.f);
            load_dz<NMAX, BF16>(a, row, z[r]);
        }
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const bool in = m + (int64_t)r * lanes < end;
#pragma unroll
            for (int n = 0; n < NMAX; ++n) {
                const float zr = in ? z[r][n] : 0.f;
                zs[n] += zr;
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[i][n] = __builtin_fmaf(in ? part_of(h[r], i) : 0.f, zr, acc[i][n]);
            }
        }
    }
#pragma unroll
    for (int n = 0; n < NMAX; ++n) {
        redz[t][n] = zs[n];
#pragma unroll
        for (int i = 0; i < 4; ++i) red[t][i * NMAX + n] = acc[i][n];
    }
    __syncthreads();
    float *part = a.part + (int64_t)blockIdx.x * (a.K * a.N + a.N);
    const int per = 4 * G * a.N;            // results of this workgroup: [4 G columns of H][N]
    for (int o = t; o < per; o += 256) {
        const int kk = o / a.N, n = o - kk * a.N;
        const int64_t col = 4 * (int64_t)blockIdx.y * G + kk;
        if (col >= a.K) continue;
        float s = red[kk >> 2][(kk & 3) * NMAX + n];
        for (int l = 1; l < lanes; ++l) s += red[l * G + (kk >> 2)][(kk & 3) * NMAX + n];
        part[col * a.N + n] = s;
    }
    if (blockIdx.y == 0 && t < a.N) {
        float s = redz[0][t];
        for (int l = 1; l < lanes; ++l) s += redz[l * G][t];
        part[a.K * a.N + t] = s;
    }
}

// Lanes per row: enough quads for the row, at most a wavefront.
int group_lanes(int64_t K)
{
    int g = 1;
    while (g < kWave && 4 * (int64_t)g < K) g <<= 1;
    return g;
}

bool quads(const void *p, int64_t K, bool bf16) { return K % 4 == 0 && ((uintptr_t)p & (bf16 ? 7 : 15)) == 0; }

enum { FWD, DH, DW };

template <int WHAT, int NMAX, bool VEC, bool BF16>
void launch(const NarrowArgs &a, int G, dim3 grid, hipStream_t s)
{
    if constexpr (WHAT == FWD) hipLaunchKernelGGL((k_narrow_fwd<NMAX, VEC, BF16>), grid, dim3(256), 0, s, a, G);
    else if constexpr (WHAT == DH) hipLaunchKernelGGL((k_narrow_dh<NMAX, VEC, BF16>), grid, dim3(256), 0, s, a, G);
    else hipLaunchKernelGGL((k_narrow_dw<NMAX, VEC, BF16>), grid, dim3(256), 0, s, a, G);
}

template <int WHAT, int NMAX>
void launch_typed(const NarrowArgs &a, bool vec, bool bf16, int G, dim3 grid, hipStream_t s)
{
    if (bf16) vec ? launch<WHAT, NMAX, true, true>(a, G, grid, s) : launch<WHAT, NMAX, false, true>(a, G, grid, s);
    else vec ? launch<WHAT, NMAX, true, false>(a, G, grid, s) : launch<WHAT, NMAX, false, false>(a, G, grid, s);
}

template <int WHAT>
fastgl_status launch_any(const NarrowArgs &a, bool bf16, const void *rows_of, hipStream_t s, const char *what)
{
    const int G = group_lanes(a.K);
    const int64_t x = WHAT == DW ? ceil_div(a.M, a.slab) : ceil_div(a.M, (int64_t)kRows * (256 / G));
    const int64_t y = WHAT == FWD ? 1 : (a.K > 0 ? ceil_div(a.K, 4 * (int64_t)G) : 1);
    if (x >= INT32_MAX || y > 65535) {
        set_error("%s: too many tiles", what);
        return FASTGL_ERR_UNSUPPORTED;
    }
    const dim3 grid((unsigned)x, (unsigned)y);
    const bool vec = quads(rows_of, a.K, bf16);
    if (a.N == 1) launch_typed<WHAT, 1>(a, vec, bf16, G, grid, s);
    else if (a.N == 2) launch_typed<WHAT, 2>(a, vec, bf16, G, grid, s);
    else if (a.N <= 4) launch_typed<WHAT, 4>(a, vec, bf16, G, grid, s);
    else launch_typed<WHAT, 8>(a, vec, bf16, G, grid, s);
    FASTGL_LAUNCH_CHECK(what);
    return FASTGL_OK;
}

}  // namespace

fastgl_status launch_narrow_fwd(const NarrowArgs &a, bool bf16, hipStream_t s)
{
    return launch_any<FWD>(a, bf16, a.H, s, "fastgl_update_fwd (narrow)");
}

fastgl_status launch_narrow_dh(const NarrowArgs &a, bool bf16, hipStream_t s)
{
    return launch_any<DH>(a, bf16, a.out, s, "fastgl_update_bwd (narrow dH)");
}

fastgl_status launch_narrow_dw(const NarrowArgs &a, bool bf16, hipStream_t s)
{
    return launch_any<DW>(a, bf16, a.H, s, "fastgl_update_bwd (narrow dW)");
}

// Rows per partial: about 1 024 workgroups (four per compute unit), at least 64 rows each so that the
// partials stay a small part of what is read; a multiple of 32, at most 2 048 as for every shape.
int64_t narrow_slab_rows(int64_t M)
{
    const int64_t rows = ceil_div(ceil_div(M > 0 ? M : 1, 1024), 32) * 32;
    return rows < 64 ? 64 : (rows > 2048 ? 2048 : rows);
}

}  // namespace fastgl
