// Shared by the translation units of the update phase: the problem of one call, and the kernels for
// result shapes that the tiled matrix-core kernel of update.hip does not suit.
#pragma once
#include "internal.h"

namespace fastgl {

// fp32 -> bf16, round to nearest even (NaN stays NaN): one instruction.
__device__ __forceinline__ uint16_t f32_to_bf16(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

// A quad (four consecutive elements) of an fp32 or bf16 row.
template <bool BF16>
struct QuadBits;
template <>
struct QuadBits<false> {
    typedef float4 type;
    typedef float elem;
};
template <>
struct QuadBits<true> {
    typedef uint2 type;           // four bf16
    typedef uint16_t elem;
};

__device__ __forceinline__ float4 quad_to_f32(float4 q) { return q; }
__device__ __forceinline__ float4 quad_to_f32(uint2 q)
{
    return make_float4(__uint_as_float(q.x << 16), __uint_as_float(q.x & 0xFFFF0000u), __uint_as_float(q.y << 16),
                       __uint_as_float(q.y & 0xFFFF0000u));
}

// ---- update_rows.hip: C[M][N] = A[M][Kc] B, A and C row-major; Kc >= 1, M >= 1, N >= 1
struct RowsGemm {
    const void *a, *gate;            // A; where gate (same layout) is <= 0 an element of A counts as 0; NULL: no gate
    const void *b;
    int64_t lda, ldb;
    const float *bias;               // [N] or NULL
    void *c;
    int64_t M, N, Kc;
    int64_t tiles_r;
    int32_t tiles_c, relu;
};
// b_col: B[k][n] = b[k * ldb + n] (no gate then), else b[n * ldb + k]
fastgl_status launch_rows_gemm(RowsGemm g, bool b_col, bool bf16, hipStream_t s, const char *what);

// c[i][j] = act(bias[j]) (0 without bias): what is left of either product with nothing to contract
fastgl_status launch_no_terms(bool bf16, void *c, const float *bias, int64_t rows, int64_t cols, bool relu, hipStream_t s,
                              const char *what);

// ---- update_narrow.hip: N <= kNarrowCols
constexpr int kNarrowCols = 8;

struct NarrowArgs {
    const void *H, *W, *dY, *gate;   // gate: where it is <= 0, dY counts as 0; NULL: everywhere dY
    const float *bias;
    void *out;                       // Y or dH
    float *part;                     // dW / db partials: [slab][K * N + N]
    int64_t M, K;
    int64_t slab;                    // rows per dW partial
    int32_t N, relu;
};

fastgl_status launch_narrow_fwd(const NarrowArgs &a, bool bf16, hipStream_t s);
fastgl_status launch_narrow_dh(const NarrowArgs &a, bool bf16, hipStream_t s);
fastgl_status launch_narrow_dw(const NarrowArgs &a, bool bf16, hipStream_t s);
int64_t narrow_slab_rows(int64_t M);

}  // namespace fastgl
