// Update phase of a sampled GCN layer (paper Section 2.1, Eq. 2) on the matrix cores of gfx950:
// Y = act(H W + b) and its three gradients.  See include/fastgl_update.h for the contract of every
// entry point.
//
// The tiled kernel here forms dW and db (Y and dH: update_rows.hip; up to 8 columns: update_narrow.hip).
// A workgroup of 4 wavefronts owns a 128 x 128 tile of the result (each wavefront a 64 x 64 quarter =
// 2 x 2 accumulators of v_mfma_f32_32x32x16_bf16), or a 128 x 64 tile (a wavefront 32 x 64), and walks the
// contracted dimension in steps of 16, staged through two LDS buffers; three workgroups share a compute unit.
//
// The bf16 instruction runs at 16 times the rate of the fp32 one, so fp32 operands are not
// multiplied as fp32: an element x is cut into three bf16 planes, x = x1 + x2 + x3 exactly
// (x1 = bf16(x), x2 = bf16(x - x1), x3 = x - x1 - x2: 8 + 8 + 8 significant bits, each rounding to
// nearest, so |x2| <= 2^-8 |x| and |x3| <= 2^-16 |x|), when a tile is written to LDS.  Of the nine
// plane products six are kept: a1 b3, a3 b1, a2 b2, a1 b2, a2 b1, a1 b1 (smallest first, all into
// the same fp32 accumulator); the three dropped ones are below 2^-23 |a||b| together, and below
// 2^-28 |a||b| on average.  bf16 storage needs one plane and one product.  An element that is not
// finite, or beyond the largest bf16 (3.39e38), turns the results it enters into NaN.
//
// Both operands have the contracted index outside (mem[contract][out]: H and dZ) and are copied to LDS as they lie in
// memory, four neighbouring columns per lane and load.  One plane of an operand tile (16 contracted x 128 out) in LDS:
// [pair p = contracted 2p, 2p+1][out] dwords, 128 + 8 per pair.  Lane half h (lanes 32h..32h+31) multiplies contracted
// indices 8h .. 8h+7 of both operands.
//
// Rows of any length and alignment: the four columns of a lane start early enough to end with the row, and move to
// their places in registers.  Columns that do not exist are not masked: what they hold stays in columns of the result
// that are not stored.  Only contracted indices past the end have to be zeros.
// Bound by the matrix cores and the memory for fp32 (1.25 GB of operands at 4.3 TB/s for 512 K rows), by the
// partial results' traffic for bf16 (as much as the operands for 87 000 rows; loads two steps ahead, and two steps to a
// barrier, change nothing).
// us with cold caches, gated, with the reduction; single-element loads for rows that are no whole quads, masks in tiles
// at the matrix' edge, and 4 loads in flight in the reduction -> now:
//   fp32  40 000 rows, 131 x 99: 87 -> 37;  300 000, 57 x 33: 95 -> 67;  100 000, 40 x 10: 35 -> 27;  512 K, 100 x 256: 307 -> 289
//   bf16  200 000, 99 x 128: 110 -> 68;  300 000, 128 x 64: 72 -> 69;  87 000, 128 x 256: 62 -> 61;  50 000, 256 x 256: 51 -> 51
#include <type_traits>

#include "fastgl_update.h"
#include "update_internal.h"

namespace fastgl {
namespace {

constexpr int kTile = 128;              // rows and columns of a workgroup's result tile
constexpr int kStep = 16;               // contracted indices per LDS stage
constexpr int kMaxSlabRows = 2048;      // most rows of H per dW / db partial
constexpr int kMinSlabRows = 32;
constexpr int kSlabRowStep = 32;        // slab heights considered: 32, 64, ..., 2048
constexpr int kRoundSlots = 768;        // workgroups the device this is tuned for holds at once (256 CUs x 3)

typedef float f32x16 __attribute__((ext_vector_type(16)));

struct Operand {
    const void *p;        // element (contracted k, out o) at p[k*ld + o]
    const void *gate;     // same layout, or NULL; where gate <= 0 the element reads as 0 (ReLU derivative)
    int64_t ld;           // out indices: fp32 or bf16 elements (the kernel's BF16 argument says which)
};

struct GemmArgs {
    Operand a, b;
    float *c;                   // [slab][c_slab]: [R][C] partial of every slab
    int64_t ldc, c_slab;
    int64_t R, C, Kc;           // result rows, result columns, contracted length
    int64_t slab, n_slabs;      // contracted indices per slab
    int tiles_r, tiles_c;
    float *colsum;              // [slab][colsum_slab]: sums of operand b over the slab
    int64_t colsum_slab;
};

// A quad = four consecutive elements.  Loading and everything after are split so that the loads of the next steps stay
// in flight during the MFMAs of the current one: loads have no control flow around them (a load behind a branch is
// waited for at the join) and no arithmetic on their result.
template <bool GATE, bool BF16>
struct Quad {
    typename QuadBits<BF16>::type v;
    typename QuadBits<BF16>::type g[GATE ? 1 : 0];
};

// Four elements from p on, which need no more alignment than an element has.
template <bool ONCE>
__device__ __forceinline__ float4 load_four(const float *p)
{
    const Words<4>::x4 *q = reinterpret_cast<const Words<4>::x4 *>(p);
    const Words<4>::x4 w = ONCE ? __builtin_nontemporal_load(q) : *q;
    return make_float4(__uint_as_float(w[0]), __uint_as_float(w[1]), __uint_as_float(w[2]), __uint_as_float(w[3]));
}
template <bool ONCE>
__device__ __forceinline__ uint2 load_four(const uint16_t *p)
{
    const Words<2>::x2 *q = reinterpret_cast<const Words<2>::x2 *>(p);
    const Words<2>::x2 w = ONCE ? __builtin_nontemporal_load(q) : *q;
    return make_uint2(w[0], w[1]);
}
// The same one by one, where a row has fewer: element i < n, the others the first one again.
template <class E>
__device__ __forceinline__ typename QuadBits<sizeof(E) == 2>::type load_few(const E *p, uint32_t off, int n)
{
    E e[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) e[i] = p[i < n ? off + i : 0u];
    if constexpr (sizeof(E) == 2) return make_uint2((uint32_t)e[0] | ((uint32_t)e[1] << 16), (uint32_t)e[2] | ((uint32_t)e[3] << 16));
    else return make_float4(e[0], e[1], e[2], e[3]);
}

__device__ __forceinline__ int clamp4(int64_t n) { return n >= 4 ? 4 : (n <= 0 ? 0 : (int)n); }

// Writes a wavefront's 32 FA x 64 part of the result tile at (r0, c0).
// Accumulator element e of lane (h, l32) is row 8*(e/4) + 4*h + e%4, column l32 of its 32 x 32 tile.
template <int FA>
__device__ __forceinline__ void write_tile(const GemmArgs &g, const f32x16 (&acc)[FA][2], int64_t r0, int64_t c0,
                                           int64_t slab_id, int wr, int wc, int h, int l32)
{
    const int64_t row0 = r0 + wr * 32 * FA + 4 * h, col0 = c0 + wc * 64 + l32;
    float *cb = g.c + slab_id * g.c_slab + row0 * g.ldc + col0;
    const bool whole = r0 + kTile <= g.R && c0 + 64 * FA <= g.C;       // uniform
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        if (!whole && col0 + 32 * j >= g.C) continue;
#pragma unroll
        for (int i = 0; i < FA; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int dr = 32 * i + 8 * (e >> 2) + (e & 3);
                if (whole || row0 + dr < g.R) cb[(int64_t)dr * g.ldc + 32 * j] = acc[i][j][e];
            }
    }
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kPairStride = kTile + 8;                        // dwords between pairs of a plane
constexpr int kPlaneBytes = (kStep / 2) * kPairStride * 4;

// Planes of the pair (x0, x1), packed as two bf16 per dword (x0 in the low half).
template <int PLANES>
__device__ __forceinline__ void split_pair(float x0, float x1, uint32_t (&w)[PLANES])
{
#pragma unroll
    for (int p = 0; p < PLANES; ++p) {
        const bf16x2 b = {(__bf16)x0, (__bf16)x1};
        w[p] = __builtin_bit_cast(uint32_t, b);
        if (p + 1 < PLANES) {
            x0 -= __uint_as_float(w[p] << 16);
            x1 -= __uint_as_float(w[p] & 0xFFFF0000u);
        }
    }
}

// One operand tile of 16 contracted x 128 out indices: global -> registers (fetch), registers -> bf16 planes in LDS
// (stage).  Lane t has out indices 4(t%32)..+3 of contracted 2(t/32) and 2(t/32) + 1.  SUM keeps a running sum per held
// out index of everything staged.  MASK = false is for steps that lie inside the contracted range.
// QUADS: rows of at least four elements; else element by element.
template <bool QUADS, bool GATE, bool BF16, int PLANES, bool SUM, bool ONCE>
struct PlaneMover {
    typedef typename QuadBits<BF16>::elem E;
    Quad<GATE, BF16> r[2];      // [slot]
    uint32_t off[2];            // of the slot's quad from the step's first row on
    uint32_t first;             // the same in the first row: an element that exists
    int moved;                  // columns that the quad starts early
    int n_out;                  // !QUADS: columns that exist
    bool any_moved;             // the same for the workgroup
    int64_t ld;
    const E *p, *gate;
    float sum[SUM ? 4 : 1];

    __device__ __forceinline__ void init(const Operand &op, int64_t o0, int64_t omax)
    {
        const int t = threadIdx.x;
        ld = op.ld; p = static_cast<const E *>(op.p); gate = static_cast<const E *>(op.gate);
        const int64_t o = o0 + 4 * (t & 31), last = omax - 4, at = QUADS && o > last ? last : o;
        first = QUADS ? (uint32_t)at : 0u;
        moved = (int)(o - at < 3 ? o - at : 3);          // more: none of the quad's columns exists
        any_moved = QUADS && (omax & 3) && o0 + kTile > omax;
        n_out = clamp4(omax - o);
#pragma unroll
        for (int s = 0; s < 2; ++s) off[s] = (uint32_t)(2 * (t >> 5) + s) * (uint32_t)ld + (uint32_t)at;
#pragma unroll
        for (int j = 0; j < (SUM ? 4 : 1); ++j) sum[j] = 0.f;
    }

    __device__ __forceinline__ static bool in_range(int s, int64_t k0, int64_t kend)
    {
        return k0 + 2 * (int)(threadIdx.x >> 5) + s < kend;
    }

    // A row beyond kend (of a step that is, of row 0) is loaded from the step's first row, all masked.
    template <bool MASK>
    __device__ __forceinline__ void fetch(int64_t k0, int64_t kend)
    {
        const int64_t origin = (k0 < kend ? k0 : 0) * ld;              // uniform
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const bool ok = !MASK || in_range(s, k0, kend);
            if constexpr (QUADS) {
                const uint32_t o = ok ? off[s] : first;
                r[s].v = load_four<ONCE>(p + origin + o);
                if constexpr (GATE) r[s].g[0] = load_four<ONCE>(gate + origin + o);
            } else {
                r[s].v = load_few(p + origin, off[s], ok ? n_out : 0);
                if constexpr (GATE) r[s].g[0] = load_few(gate + origin, off[s], ok ? n_out : 0);
            }
        }
    }

    // (k0, kend) must be those of the fetch that filled the registers.
    template <bool MASK>
    __device__ __forceinline__ void stage(char *lds, int64_t k0, int64_t kend)
    {
        const int t = threadIdx.x;
        float4 v[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            v[s] = quad_to_f32(r[s].v);
            if constexpr (GATE) {
                const float4 g = quad_to_f32(r[s].g[0]);
                v[s].x = g.x > 0.f ? v[s].x : 0.f;
                v[s].y = g.y > 0.f ? v[s].y : 0.f;
                v[s].z = g.z > 0.f ? v[s].z : 0.f;
                v[s].w = g.w > 0.f ? v[s].w : 0.f;
            }
            if (any_moved) {             // what moves up from behind the quad is a column that does not exist
                if (moved & 1) v[s] = make_float4(v[s].y, v[s].z, v[s].w, v[s].w);
                if (moved & 2) v[s] = make_float4(v[s].z, v[s].w, v[s].w, v[s].w);
            }
            if (MASK && !in_range(s, k0, kend)) v[s] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        uint32_t w[4][PLANES];
        split_pair<PLANES>(v[0].x, v[1].x, w[0]);
        split_pair<PLANES>(v[0].y, v[1].y, w[1]);
        split_pair<PLANES>(v[0].z, v[1].z, w[2]);
        split_pair<PLANES>(v[0].w, v[1].w, w[3]);
        char *dst = lds + ((t >> 5) * kPairStride + 4 * (t & 31)) * 4;
#pragma unroll
        for (int pl = 0; pl < PLANES; ++pl)
            *reinterpret_cast<uint4 *>(dst + pl * kPlaneBytes) = make_uint4(w[0][pl], w[1][pl], w[2][pl], w[3][pl]);
        if (SUM) {
            sum[0] += v[0].x + v[1].x;
            sum[1] += v[0].y + v[1].y;
            sum[2] += v[0].z + v[1].z;
            sum[3] += v[0].w + v[1].w;
        }
    }
};

// A tile of 64 out indices: lane t has out indices 2(t%32), +1 of contracted 2(t/32) and 2(t/32) + 1, so that all lanes
// have the same share; LDS as above, the first 64 dwords of every pair.
template <bool QUADS, bool GATE, bool BF16, int PLANES, bool SUM, bool ONCE>
struct HalfMover {
    typedef typename QuadBits<BF16>::elem E;
    typedef typename std::conditional<BF16, uint32_t, float2>::type Duo;
    Duo v[2], g[GATE ? 2 : 1];           // [slot]
    uint32_t off[2], first;
    int n_out;                           // !QUADS: columns that exist, 0 .. 2
    bool moved, any_moved;
    int64_t ld;
    const E *p, *gate;
    float sum[2];

    __device__ __forceinline__ void init(const Operand &op, int64_t o0, int64_t omax)
    {
        const int t = threadIdx.x;
        ld = op.ld; p = static_cast<const E *>(op.p); gate = static_cast<const E *>(op.gate);
        const int64_t o = o0 + 2 * (t & 31), last = omax - 2, at = QUADS && o > last ? last : o;
        first = QUADS ? (uint32_t)at : 0u;
        moved = o > at;
        any_moved = QUADS && (omax & 1) && o0 + kTile / 2 > omax;
        const int n = clamp4(omax - o);
        n_out = n < 2 ? n : 2;
#pragma unroll
        for (int s = 0; s < 2; ++s) off[s] = (uint32_t)(2 * (t >> 5) + s) * (uint32_t)ld + (uint32_t)at;
        sum[0] = sum[1] = 0.f;
    }

    __device__ __forceinline__ static bool in_range(int s, int64_t k0, int64_t kend)
    {
        return k0 + 2 * (int)(threadIdx.x >> 5) + s < kend;
    }

    __device__ __forceinline__ Duo load(const E *base, int s, bool ok) const
    {
        if constexpr (QUADS) {
            const E *q = base + (ok ? off[s] : first);
            if constexpr (BF16) {
                const Words<2>::x1 *at = reinterpret_cast<const Words<2>::x1 *>(q);
                return ONCE ? __builtin_nontemporal_load(at) : *at;
            } else {
                const Words<4>::x2 *at = reinterpret_cast<const Words<4>::x2 *>(q);
                const Words<4>::x2 w = ONCE ? __builtin_nontemporal_load(at) : *at;
                return make_float2(__uint_as_float(w[0]), __uint_as_float(w[1]));
            }
        } else {
            const int n = ok ? n_out : 0;
            const E x = base[n > 0 ? off[s] : 0u], y = base[n > 1 ? off[s] + 1 : 0u];
            if constexpr (BF16) return (uint32_t)x | ((uint32_t)y << 16);
            else return make_float2(x, y);
        }
    }
    __device__ __forceinline__ static float2 to_f32(float2 d) { return d; }
    __device__ __forceinline__ static float2 to_f32(uint32_t d)
    {
        return make_float2(__uint_as_float(d << 16), __uint_as_float(d & 0xFFFF0000u));
    }

    template <bool MASK>
    __device__ __forceinline__ void fetch(int64_t k0, int64_t kend)
    {
        const int64_t origin = (k0 < kend ? k0 : 0) * ld;              // uniform
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const bool ok = !MASK || in_range(s, k0, kend);
            v[s] = load(p + origin, s, ok);
            if constexpr (GATE) g[s] = load(gate + origin, s, ok);
        }
    }

    template <bool MASK>
    __device__ __forceinline__ void stage(char *lds, int64_t k0, int64_t kend)
    {
        const int t = threadIdx.x;
        float2 x[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            x[s] = to_f32(v[s]);
            if constexpr (GATE) {
                const float2 open = to_f32(g[s]);
                x[s].x = open.x > 0.f ? x[s].x : 0.f;
                x[s].y = open.y > 0.f ? x[s].y : 0.f;
            }
            if (any_moved && moved) x[s].x = x[s].y;
            if (MASK && !in_range(s, k0, kend)) x[s] = make_float2(0.f, 0.f);
        }
        uint32_t w[2][PLANES];
        split_pair<PLANES>(x[0].x, x[1].x, w[0]);
        split_pair<PLANES>(x[0].y, x[1].y, w[1]);
        char *dst = lds + ((t >> 5) * kPairStride + 2 * (t & 31)) * 4;
#pragma unroll
        for (int pl = 0; pl < PLANES; ++pl) *reinterpret_cast<uint2 *>(dst + pl * kPlaneBytes) = make_uint2(w[0][pl], w[1][pl]);
        if (SUM) {
            sum[0] += x[0].x + x[1].x;
            sum[1] += x[0].y + x[1].y;
        }
    }
};

// The eight values (contracted indices 8h .. 8h+7) of out index o in one plane.
__device__ __forceinline__ uint4 read_plane(const char *plane, int o, int h)
{
    const uint32_t *q = reinterpret_cast<const uint32_t *>(plane) + 4 * h * kPairStride + o;
    return make_uint4(q[0], q[kPairStride], q[2 * kPairStride], q[3 * kPairStride]);
}

// A wavefront's fragments of one step: [operand a / b][32-wide fragment][plane].
template <int PLANES, int FA>
struct Frags {
    uint4 a[FA][PLANES], b[2][PLANES];
};

template <int PLANES, int FA>
__device__ __forceinline__ void read_frags(const char *la, const char *lb, int wr, int wc, int l32, int h,
                                           Frags<PLANES, FA> &f)
{
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int pl = 0; pl < PLANES; ++pl) {
            if (i < FA) f.a[i][pl] = read_plane(la + pl * kPlaneBytes, wr * 32 * FA + i * 32 + l32, h);
            f.b[i][pl] = read_plane(lb + pl * kPlaneBytes, wc * 64 + i * 32 + l32, h);
        }
}

// All MFMAs of one step; consecutive MFMAs go to different accumulators.
template <int PLANES, int FA>
__device__ __forceinline__ void mma_frags(const Frags<PLANES, FA> &f, f32x16 (&acc)[FA][2])
{
    constexpr int kTerms = PLANES == 3 ? 6 : 1;
    constexpr int pa[6] = {0, 2, 1, 0, 1, 0}, pb[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
    for (int t = 0; t < kTerms; ++t)
#pragma unroll
        for (int i = 0; i < FA; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int x = PLANES == 3 ? pa[t] : 0, y = PLANES == 3 ? pb[t] : 0;
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f.a[i][x]),
                                                                   __builtin_bit_cast(bf16x8, f.b[j][y]), acc[i][j], 0, 0, 0);
            }
}

// One step of the contracted range: the loads of the next step are issued, this step is multiplied
// out of LDS buffer `cur`, and the next one is split into the other buffer.  No branch inside.
template <bool MASK, int PLANES, int FA, class MoverA, class MoverB>
__device__ __forceinline__ void one_step(MoverA &ma, MoverB &mb, char *la, char *lb, int cur, int64_t k0, int64_t kend,
                                         int wr, int wc, int l32, int h, f32x16 (&acc)[FA][2])
{
    constexpr int kBytes = PLANES * kPlaneBytes;
    ma.template fetch<MASK>(k0 + kStep, kend);
    mb.template fetch<MASK>(k0 + kStep, kend);
    __builtin_amdgcn_sched_barrier(0);       // the loads stay ahead of the step's other work
    Frags<PLANES, FA> f;
    read_frags<PLANES, FA>(la + cur * kBytes, lb + cur * kBytes, wr, wc, l32, h, f);
    mma_frags<PLANES, FA>(f, acc);
    ma.template stage<MASK>(la + (cur ^ 1) * kBytes, k0 + kStep, kend);
    mb.template stage<MASK>(lb + (cur ^ 1) * kBytes, k0 + kStep, kend);
    __syncthreads();
}

// The contracted range [kbeg, kend) of one result tile.  The first steps touch nothing but whole steps (a step also loads
// and converts the one after it) and run without masks; the others, at least one, mask what does not exist - a
// step beyond kend is a step of zeros.  The MFMAs are not behind any condition other than the two loop counts:
// accumulators that can reach the end by a path without MFMAs are given a second set of registers by the compiler.
template <int PLANES, int FA, class MoverA, class MoverB>
__device__ __forceinline__ void run_steps(MoverA &ma, MoverB &mb, char *la, char *lb, int64_t kbeg, int64_t kend, bool quads,
                                          int wr, int wc, int l32, int h, f32x16 (&acc)[FA][2])
{
    const int64_t len = kend > kbeg ? kend - kbeg : 0;
    const int64_t nstep = len > 0 ? (len + kStep - 1) / kStep : 1;
    int64_t plain = quads ? len / kStep - 1 : 0;
    plain = plain < 0 ? 0 : plain;                         // < nstep
    ma.template fetch<true>(kbeg, kend);
    mb.template fetch<true>(kbeg, kend);
    ma.template stage<true>(la, kbeg, kend);
    mb.template stage<true>(lb, kbeg, kend);
    __syncthreads();
    int64_t k0 = kbeg;
    int cur = 0;
    for (int64_t i = 0; i < plain; ++i, k0 += kStep, cur ^= 1)
        one_step<false, PLANES, FA>(ma, mb, la, lb, cur, k0, kend, wr, wc, l32, h, acc);
    int64_t i = plain;
    do {
        one_step<true, PLANES, FA>(ma, mb, la, lb, cur, k0, kend, wr, wc, l32, h, acc);
        k0 += kStep;
        cur ^= 1;
    } while (++i < nstep);
}

// FA: a wavefront's 32-row fragments.  2: the tile is 128 x 128.  1: it is 128 x 64, a wavefront has 32 rows of it.
template <bool QUADS, bool GATE, bool BF16, int FA, bool ONCE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_update_gemm(const GemmArgs g)
{
    constexpr int PLANES = BF16 ? 1 : 3;
    constexpr int kOperandBytes = PLANES * kPlaneBytes;
    __shared__ __attribute__((aligned(16))) char lds_a[2][kOperandBytes];
    __shared__ __attribute__((aligned(16))) char lds_b[2][kOperandBytes];

    const int64_t bid = blockIdx.x;
    const int xcd = (int)(bid % kXcds);
    const int64_t q = bid / kXcds;
    const int n_inner = g.tiles_r * g.tiles_c;
    const int inner = (int)(q % n_inner);
    const int64_t slab_id = (q / n_inner) * kXcds + xcd;
    if (slab_id >= g.n_slabs) return;
    const int64_t tile_r = inner / g.tiles_c;
    const int tile_c = inner % g.tiles_c;
    const int64_t kbeg = slab_id * g.slab, kend = kbeg + g.slab < g.Kc ? kbeg + g.slab : g.Kc;
    constexpr int kCols = 64 * FA;
    const int64_t r0 = tile_r * kTile, c0 = (int64_t)tile_c * kCols;

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wr = FA == 2 ? wave >> 1 : wave, wc = FA == 2 ? wave & 1 : 0;      // 2 x 2 or 4 x 1 wavefronts
    const int h = lane >> 5, l32 = lane & 31;

    f32x16 acc[FA][2];
#pragma unroll
    for (int i = 0; i < FA; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    PlaneMover<QUADS, false, BF16, PLANES, false, ONCE> ma;
    typename std::conditional<FA == 2, PlaneMover<QUADS, GATE, BF16, PLANES, true, ONCE>,
                              HalfMover<QUADS, GATE, BF16, PLANES, true, ONCE>>::type mb;
    ma.init(g.a, r0, g.R);
    mb.init(g.b, c0, g.C);
    run_steps<PLANES, FA>(ma, mb, lds_a[0], lds_b[0], kbeg, kend, QUADS, wr, wc, l32, h, acc);
    write_tile<FA>(g, acc, r0, c0, slab_id, wr, wc, h, l32);
    if (tile_r == 0) {
        // Every barrier above has been passed by all lanes, so the LDS is free: add up the eight
        // running sums of each column in a fixed order.
        float *red = reinterpret_cast<float *>(lds_b[0]);
        const int t = threadIdx.x;
#pragma unroll
        for (int j = 0; j < 2 * FA; ++j) red[(t >> 5) * kCols + 2 * FA * (t & 31) + j] = mb.sum[j];
        __syncthreads();
        if (t < kCols) {
            float s = red[t];
#pragma unroll
            for (int i = 1; i < 8; ++i) s += red[i * kCols + t];
            if (c0 + t < g.C) g.colsum[slab_id * g.colsum_slab + c0 + t] = s;
        }
    }
}

// out[e] = sum over slabs of part[s*stride + e], in fp64 and in a fixed order: the slabs are cut into
// PARTS consecutive ranges, each summed in slab order by one thread, and the range sums are
// added in range order.  The first n_w elements go to dW, the remaining n_b to db (either may be NULL).
// Few elements get 64 ranges: the launch is bound by the chain of loads of a thread, and a result of a
// narrow layer (65 elements, 562 slabs: 10.0 us with 8 ranges, 4.7 with 64) gives few threads to hide it.
// With thousands of elements the 16-byte pieces that 64 ranges read cost more (6 464: 10 -> 24 us).
constexpr int kReduceElemsWide = 1024;   // from this many elements on: 8 ranges

template <int PARTS>
__global__ __launch_bounds__(256) void k_update_reduce(const float *__restrict__ part, int64_t nslab, int64_t stride,
                                                       int64_t n_w, int64_t n_b, float *dW, float *db)
{
    constexpr int kElems = 256 / PARTS;
    __shared__ double partial[PARTS][kElems];
    const int el = threadIdx.x % kElems, pt = threadIdx.x / kElems;
    const int64_t e = (int64_t)blockIdx.x * kElems + el;
    const int64_t per = (nslab + PARTS - 1) / PARTS;
    const int64_t lo = pt * per, hi = lo + per < nslab ? lo + per : nslab;
    double s = 0.0;
    if (e < n_w + n_b) {
        const float *q = part + e;
        int64_t k = lo;
        constexpr int kAhead = 16;           // loads in flight: a range's chain is what the launch waits for
        for (; k + kAhead <= hi; k += kAhead) {
            float v[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) v[u] = q[(k + u) * stride];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) s += (double)v[u];
        }
        // what is left, with as many loads as that takes and not 16 (few rows have a slab or two to a range)
        auto rest = [&](auto count) {
            constexpr int n = decltype(count)::value;
            float v[n];
#pragma unroll
            for (int u = 0; u < n; ++u) v[u] = q[(k + u < hi ? k + u : hi - 1) * stride];
#pragma unroll
            for (int u = 0; u < n; ++u) s += k + u < hi ? (double)v[u] : 0.0;
        };
        if (hi - k > 4) rest(std::integral_constant<int, kAhead>());
        else if (hi - k > 1) rest(std::integral_constant<int, 4>());
        else if (hi > k) rest(std::integral_constant<int, 1>());
    }
    partial[pt][el] = s;
    __syncthreads();
    if (pt != 0 || e >= n_w + n_b) return;
    double t = partial[0][el];
#pragma unroll
    for (int i = 1; i < PARTS; ++i) t += partial[i][el];
    float *dst = e < n_w ? (dW ? dW + e : nullptr) : (db ? db + (e - n_w) : nullptr);
    if (dst) *dst = (float)t;
}

// Operands of so many bytes are loaded past the caches, where one tile reads them (launch_gemm has both sides).
constexpr int64_t kOnceBytes = (int64_t)128 << 20;

fastgl_status launch_gemm(GemmArgs &g, bool bf16, hipStream_t s, const char *what)
{
    // Up to 64 result columns: no matrix instructions and no conversions for columns that do not exist.
    // us, tiles of 128 columns -> 64:  fp32 M = 1.15 M, 100 x 64: 262 -> 212;  8 000, 256 x 47: 29 -> 16 (bf16,
    // 1 000 rows: 15 -> 10).
    const bool half = g.C <= kTile / 2;
    g.tiles_r = (int)ceil_div(g.R, kTile);
    g.tiles_c = (int)ceil_div(g.C, kTile);
    if (g.tiles_r == 0) g.tiles_r = 1;                     // column sums are still owed when R == 0
    const int64_t blocks = ceil_div(g.n_slabs, kXcds) * kXcds * g.tiles_r * g.tiles_c;
    if (blocks == 0) return FASTGL_OK;
    if (blocks >= INT32_MAX) {
        set_error("%s: too many tiles (%lld)", what, (long long)blocks);
        return FASTGL_ERR_UNSUPPORTED;
    }
    bool quads = g.a.ld >= 4 && g.b.ld >= 4;
    if (g.R == 0) {            // operand a has no elements: give its (all masked) loads a readable address
        g.a.p = g.b.p;
        g.a.gate = nullptr;
        quads = false;
    }
    const dim3 grid((unsigned)blocks);
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, g); };
    auto gated = [&](auto q, auto type, auto fa) {
        constexpr bool Q = decltype(q)::value, T = decltype(type)::value;
        constexpr int FA = decltype(fa)::value;
        auto pick = [&](auto once) {
            constexpr bool ONCE = decltype(once)::value;
            if (g.b.gate) go(k_update_gemm<Q, true, T, FA, ONCE>);
            else go(k_update_gemm<Q, false, T, FA, ONCE>);
        };
        // One tile: fp32 operands that one workgroup reads are loaded past the caches, from a size on that the caches no longer hold
        // together with what else a step has written.  us, cached / past the caches, operands just written, 512 MB written after them, and
        // gated with two more results written between them and the call:
        //   100 x 64    39 MB 16 / 17, 21 / 16, 17 / 19;  112 MB 26 / 31, 47 / 28, 29 / 30;  164 MB 36 / 40, 69 / 39, 48 / 41;  754 MB 199 / 158, 206 / 148, 206 / 160
        //   96 x 18     46 MB 19 / 22, 24 / 20, 20 / 23;  114 MB 33 / 38, 47 / 35, 35 / 44;  182 MB 49 / 54, 73 / 52, 54 / 54;  524 MB 146 / 136, 170 / 134, 165 / 145
        //   64 x 128    77 MB 29 / 30, 38 / 31, 31 / 31;  131 MB 40 / 40, 60 / 41, 56 / 50;  192 MB 55 / 56, 83 / 57, 83 / 62;  883 MB 246 / 222, 260 / 224, 281 / 247
        // An operand of several tiles is not, nor one beside it: 512 K rows, gated, 100 x 256, whose 256 columns
        // one tile reads, alone 241 / 233, in a training step 251 / 256;  91 K rows, gated, 256 x 256, each read by two tiles: 91 / 95.
        // bf16 gains nothing: 85 K rows, 128 x 256: 29.3 / 30.4.
        if constexpr (Q && !T)
            if (g.tiles_r == 1 && g.tiles_c == 1 && g.Kc * (g.R + g.C) * 4 >= kOnceBytes) return pick(std::true_type());
        pick(std::false_type());
    };
    auto typed = [&](auto q, auto fa) {
        if (bf16) gated(q, std::true_type(), fa);
        else gated(q, std::false_type(), fa);
    };
    auto wide = [&](auto fa) {
        if (quads) typed(std::true_type(), fa);
        else typed(std::false_type(), fa);
    };
    if (half) wide(std::integral_constant<int, 1>());
    else wide(std::integral_constant<int, 2>());
    FASTGL_LAUNCH_CHECK(what);
    return FASTGL_OK;
}

fastgl_status check_dims(int64_t M, int64_t K, int64_t N)
{
    if (M < 0 || K < 0 || N < 0) {
        set_error("negative size (M=%lld K=%lld N=%lld)", (long long)M, (long long)K, (long long)N);
        return FASTGL_ERR_INVALID_ARG;
    }
    if (M >= INT32_MAX || K >= ((int64_t)1 << 24) || N >= ((int64_t)1 << 24)) {
        set_error("M must stay below 2^31-1, K and N below 2^24");
        return FASTGL_ERR_UNSUPPORTED;
    }
    return FASTGL_OK;
}

// Few result columns: plain multiply-adds instead of matrix-core tiles (update_narrow.hip).  dW with the reduction, us
// with cold caches, K = 64, tiles of 128 columns -> multiply-adds: N = 1: 20 000 rows 38 -> 11, 1.15 M 358 -> 114;
// N = 8: 27 -> 14, 235 -> 143.  Y and dH: see kNarrowRows.  K beyond the grid's second dimension stays here.
bool narrow(int64_t K, int64_t N) { return N >= 1 && N <= kNarrowCols && K > 0 && K <= (int64_t)1 << 20; }

// With more rows than this, Y with few columns comes from the tall tiles of update_rows.hip (32 columns wide) too,
// and so does dH with 5 to 8.  us a call with cold caches, multiply-adds / tall tiles, K = 64:
//   Y   N = 1: 20 000 rows 7.6 / 9.2, 512 K 49 / 53, 1.15 M 98 / 103;   N = 2: 9.7 / 9.4, 56 / 54, 106 / 104;
//       N = 4: 13 / 9, 89 / 55, 189 / 104;   N = 8: 20 / 9, 183 / 56, 398 / 108
//   dH  N = 1: 6.4 / 9.7, 29 / 51, 59 / 104;   N = 3: 6.9 / 10.5, 42 / 71, 91 / 145;   N = 4: 9.1 / 8.9, 68 / 47,
//       143 / 101;   N = 8: 13 / 9, 127 / 47, 274 / 98
// So beyond the line Y is faster on tall tiles from two columns on, dH from four (the rule sends it there from five).
// Y with one column is NOT faster on them: the multiply-adds took 53 us in the step of an attention head, 1.15 M rows with part
// of H still in the Infinity Cache, the tall tiles 82 then and 66 now.  It goes to the tall tiles all the same, not for speed but to keep the
// order of its terms: another one would turn a few of millions of LeakyReLU signs from what earlier versions of the library
// gave.  Below the line the order is the multiply-adds'.
constexpr int64_t kNarrowRows = 16384;

// Rows per slab: a function of the shape alone, so results do not depend on the device or the run.
// The height that minimises a model of the launch: the (slab, tile) workgroups run in rounds of
// kRoundSlots, a workgroup costs its steps plus a fixed part, and every slab adds a partial result
// that is written once and read once by the reduction.  Integer arithmetic (picoseconds).
int64_t slab_rows(int64_t M, int64_t K, int64_t N)
{
    if (narrow(K, N)) return narrow_slab_rows(M);
    const int64_t tiles = (K > 0 ? ceil_div(K, kTile) : 1) * ceil_div(N, kTile);
    const int64_t partial = K * N + N;                 // floats per slab
    int64_t best = kMinSlabRows, best_cost = INT64_MAX;
    for (int64_t rows = kMinSlabRows; rows <= kMaxSlabRows; rows += kSlabRowStep) {
        const int64_t nslab = ceil_div(M > 0 ? M : 1, rows);
        const int64_t rounds = ceil_div(nslab * tiles, kRoundSlots);
        // 2.5 us per step of 16 rows with three workgroups on a CU, 8 steps' worth of prologue and
        // epilogue; 8 bytes of traffic per float of a partial at 4 TB/s
        const int64_t cost = rounds * (rows * 156250 + 20000000) + nslab * partial * 2;
        if (cost < best_cost) {
            best_cost = cost;
            best = rows;
        }
    }
    return best;
}

size_t bwd_workspace(int64_t M, int64_t K, int64_t N)
{
    const int64_t nslab = ceil_div(M, slab_rows(M, K, N));
    return align_up((size_t)nslab * (size_t)(K * N + N) * sizeof(float), 256);
}

}  // namespace
}  // namespace fastgl

using namespace fastgl;

namespace {

bool misaligned_to(const void *p, uintptr_t bytes) { return ((uintptr_t)p & (bytes - 1)) != 0; }

fastgl_status update_fwd(bool bf16, const void *H, const void *W, const float *bias, int64_t M, int64_t K, int64_t N,
                         int relu, void *Y, void *stream)
{
    fastgl_status st = check_dims(M, K, N);
    if (st != FASTGL_OK) return st;
    if (M == 0 || N == 0) return FASTGL_OK;
    if (!Y || (K > 0 && (!H || !W))) {
        set_error("H, W or Y is NULL");
        return FASTGL_ERR_INVALID_ARG;
    }
    const uintptr_t el = bf16 ? 2 : 4;
    if (misaligned_to(H, el) || misaligned_to(W, el) || misaligned_to(bias, 4) || misaligned_to(Y, el)) {
        set_error("matrices must be aligned to their element size");
        return FASTGL_ERR_INVALID_ARG;
    }
    if (narrow(K, N) && M <= kNarrowRows) {
        NarrowArgs a = {};
        a.H = H; a.W = W; a.bias = bias; a.out = Y;
        a.M = M; a.K = K; a.N = (int32_t)N; a.relu = relu != 0;
        return launch_narrow_fwd(a, bf16, (hipStream_t)stream);
    }
    if (K == 0) return launch_no_terms(bf16, Y, bias, M, N, relu != 0, (hipStream_t)stream, "fastgl_update_fwd (K = 0)");
    RowsGemm g = {};
    g.a = H; g.lda = K;
    g.b = W; g.ldb = N;
    g.bias = bias; g.c = Y;
    g.M = M; g.N = N; g.Kc = K; g.relu = relu != 0;
    return launch_rows_gemm(g, true, bf16, (hipStream_t)stream, "fastgl_update_fwd");
}

fastgl_status update_bwd(bool bf16, const void *H, const void *W, const void *Y, const void *dY, int64_t M, int64_t K,
                         int64_t N, int relu, void *dH, float *dW, float *db, void *workspace, size_t workspace_bytes,
                         void *stream)
{
    fastgl_status st = check_dims(M, K, N);
    if (st != FASTGL_OK) return st;
    const bool want_w = (dW && K > 0 && N > 0) || (db && N > 0);
    if ((M > 0 && N > 0 && !dY) || (relu && M > 0 && N > 0 && !Y)) {
        set_error("dY is NULL, or relu is set and Y is NULL");
        return FASTGL_ERR_INVALID_ARG;
    }
    if (dH && M > 0 && K > 0 && N > 0 && !W) {
        set_error("dH needs W");
        return FASTGL_ERR_INVALID_ARG;
    }
    if (dW && M > 0 && K > 0 && N > 0 && !H) {
        set_error("dW needs H");
        return FASTGL_ERR_INVALID_ARG;
    }
    const uintptr_t el = bf16 ? 2 : 4;
    if (misaligned_to(H, el) || misaligned_to(W, el) || misaligned_to(Y, el) || misaligned_to(dY, el) ||
        misaligned_to(dH, el) || misaligned_to(dW, 4) || misaligned_to(db, 4)) {
        set_error("matrices must be aligned to their element size");
        return FASTGL_ERR_INVALID_ARG;
    }
    const size_t need = want_w ? bwd_workspace(M, K, N) : 0;
    if (want_w && need > 0) {
        if (!workspace || ((uintptr_t)workspace & 255)) {
            set_error("workspace must be a 256-byte aligned device buffer");
            return FASTGL_ERR_INVALID_ARG;
        }
        if (workspace_bytes < need) {
            set_error("workspace too small: %zu < %zu bytes", workspace_bytes, need);
            return FASTGL_ERR_WORKSPACE;
        }
    }
    hipStream_t s = (hipStream_t)stream;
    const void *gate = relu ? Y : nullptr;

    NarrowArgs na = {};
    na.H = H; na.W = W; na.dY = dY; na.gate = gate; na.out = dH;
    na.M = M; na.K = K; na.N = (int32_t)N;
    if (dH && M > 0 && narrow(K, N) && (N <= 4 || M <= kNarrowRows)) {
        st = launch_narrow_dh(na, bf16, s);
        if (st != FASTGL_OK) return st;
    } else if (dH && M > 0 && K > 0 && N > 0) {
        RowsGemm g = {};
        g.a = dY; g.gate = gate; g.lda = N;
        g.b = W; g.ldb = N;
        g.c = dH;
        g.M = M; g.N = K; g.Kc = N;
        st = launch_rows_gemm(g, false, bf16, s, "fastgl_update_bwd (dH)");
        if (st != FASTGL_OK) return st;
    } else if (dH && M > 0 && K > 0) {
        st = launch_no_terms(bf16, dH, nullptr, M, K, false, s, "fastgl_update_bwd (dH, N = 0)");
        if (st != FASTGL_OK) return st;
    }
    if (want_w) {
        // dW[k][n] = sum_m H[m][k] dZ[m][n], db[n] = sum_m dZ[m][n]: slabs of rows m, partials per slab.
        const int64_t rows = slab_rows(M, K, N), nslab = ceil_div(M, rows);
        const int64_t stride = K * N + N;
        float *part = (float *)workspace;
        if (nslab > 0 && narrow(K, N)) {         // also for db alone: its bits do not depend on what else is asked for
            na.part = part; na.slab = rows;
            if (!dW) na.H = nullptr;
            st = launch_narrow_dw(na, bf16, s);
            if (st != FASTGL_OK) return st;
        } else if (nslab > 0) {
            GemmArgs g = {};
            g.a = Operand{H, nullptr, K};
            g.b = Operand{dY, gate, N};
            g.c = part; g.ldc = N; g.c_slab = stride;
            g.R = K; g.C = N; g.Kc = M; g.slab = rows;
            if (!H) {                            // db alone: column sums without a product
                g.a = Operand{dY, nullptr, 0};
                g.R = 0;
            }
            g.n_slabs = nslab;
            g.colsum = part + K * N; g.colsum_slab = stride;
            st = launch_gemm(g, bf16, s, "fastgl_update_bwd (dW)");
            if (st != FASTGL_OK) return st;
        }
        const int64_t n_w = K * N, total = n_w + N;
        if (total >= kReduceElemsWide)
            hipLaunchKernelGGL(k_update_reduce<8>, dim3((unsigned)ceil_div(total, 32)), dim3(256), 0, s, part, nslab, stride,
                               n_w, N, dW, db);
        else
            hipLaunchKernelGGL(k_update_reduce<64>, dim3((unsigned)ceil_div(total, 4)), dim3(256), 0, s, part, nslab, stride,
                               n_w, N, dW, db);
        FASTGL_LAUNCH_CHECK("fastgl_update_bwd (reduce)");
    }
    return FASTGL_OK;
}

}  // namespace

extern "C" {

fastgl_status fastgl_update_fwd(const float *H, const float *W, const float *bias, int64_t M, int64_t K,
                                int64_t N, int relu, float *Y, void *stream)
{
    return update_fwd(false, H, W, bias, M, K, N, relu, Y, stream);
}

fastgl_status fastgl_update_fwd_bf16(const uint16_t *H, const uint16_t *W, const float *bias, int64_t M, int64_t K,
                                     int64_t N, int relu, uint16_t *Y, void *stream)
{
    return update_fwd(true, H, W, bias, M, K, N, relu, Y, stream);
}

size_t fastgl_update_bwd_workspace_bytes(int64_t M, int64_t K, int64_t N)
{
    if (M < 0 || K < 0 || N < 0) return 0;
    return bwd_workspace(M, K, N);
}

fastgl_status fastgl_update_bwd(const float *H, const float *W, const float *Y, const float *dY, int64_t M,
                                int64_t K, int64_t N, int relu, float *dH, float *dW, float *db,
                                void *workspace, size_t workspace_bytes, void *stream)
{
    return update_bwd(false, H, W, Y, dY, M, K, N, relu, dH, dW, db, workspace, workspace_bytes, stream);
}

fastgl_status fastgl_update_bwd_bf16(const uint16_t *H, const uint16_t *W, const uint16_t *Y, const uint16_t *dY,
                                     int64_t M, int64_t K, int64_t N, int relu, uint16_t *dH, float *dW, float *db,
                                     void *workspace, size_t workspace_bytes, void *stream)
{
    return update_bwd(true, H, W, Y, dY, M, K, N, relu, dH, dW, db, workspace, workspace_bytes, stream);
}

int32_t fastgl_update_slab_rows(int64_t M, int64_t K, int64_t N)
{
    if (M < 0 || K < 0 || N < 0) return 0;
    return (int32_t)slab_rows(M, K, N);
}

}  // extern "C"
