// The two products of the update phase (paper Section 2.1, Eq. 2) whose first operand is a matrix of
// rows with the contracted index contiguous: Y = act(H W + b) and dH = dZ W^T.  See update.hip for how
// fp32 elements become three bf16 planes and which plane products are kept.
//
// C[M][N] = A[M][Kc] B.  A is tall (M is the number of nodes), B is a weight matrix of at most a few
// hundred KB that every workgroup reads from L2.
//
//   k_update_tall   bound by HBM for narrow layers, by the matrix cores for wide ones.  A wavefront owns
//     32 rows and NTILES x 32 columns.  Nobody else needs its rows, so A never passes through LDS: a lane
//     loads 64 contiguous bytes of its row per 32 contracted indices, two such chunks ahead where registers allow,
//     and cuts them into planes in registers.  B goes through LDS (all wavefronts of the workgroup read it), cut into
//     planes when it is written there, double buffered.  With NTILES = 8 a row is read and cut once for
//     256 columns.
//   k_update_held   k_update_tall's tiles for many rows of whole fp32 tiles: B stays in LDS, wavefronts go on alone.
//   k_update_small  bound by latency: too few rows to fill the chip with such tiles.  A workgroup owns
//     32 x 64 results and its 8 wavefronts share the contracted range; every wavefront loads the operands of two
//     steps up front (no staging, no barrier before the end) and the partial tiles are added in LDS.
//
// us a call with cold caches, first version (128 x 128 tiles, both operands through LDS) -> whole turns of 32 or 64
// indices, one chunk ahead -> now, fp32:
//   Y   M = 1.15 M, 100 -> 64: 381 -> 225 -> 218;  512 K, 100 -> 256: 257 -> 250 -> 220, 730 MB at 3.3 TB/s;
//       91 K, 256 -> 256: 97 -> 87 -> 84, 855 TFLOP/s of plane products where a large bf16 product reaches 1 135
//   dH, gated  M = 1.15 M, 64 -> 100: 347 -> 284 -> 272;  512 K, 256 -> 100: 316 -> 310;  91 K, 256 -> 256: 109 -> 121 -> 110
// (where buffers lie is worth 10 to 15 %: allocated otherwise, Y of 1.15 M rows took 202 -> 193 in the last step and Y of 512 K
// rows 279 -> 236, so that 250 -> 220 is a gain only as both sides had the same buffers);
// bf16: Y 300 K, 128 -> 256: 79 -> 78, gated dH 256 -> 128: 141 -> 128;  87 K, 128 -> 256: 26.8 -> 27.0 (1 % lost).
// What is left of the 512 K product: 178 us without the matrix instructions, 190 without the stores, 143 to move its bytes
// at 5.1 TB/s; priorities that let one of a unit's two workgroups run ahead of the other changed nothing.
// k_update_small, first version -> 4 wavefronts of 4 steps -> 8 of 2 (a launch that does nothing takes 6.4 so timed):
//   1 000, 256 -> 256: 34 -> 10.1 -> 8.8 (bf16 29 -> 8.0 -> 6.9);  16, 256 -> 47: 30 -> 9.4 -> 8.1;  2 600, 100 -> 256: 10.8 -> 9.6;
//   4 000, 256 -> 256: 14.3 -> 12.8 (16 wavefronts of 1 step: 13.6, 8.2 at 1 000 rows: their LDS leaves room for one workgroup)
//
// A step of 16 contracted indices goes into one matrix instruction per plane product (lane half h: indices 8 h .. + 7).
// Tall tiles add the steps in ascending order, so results do not depend on a tile's width; small tiles add eight
// partial sums of consecutive steps.  The tall loop ends with the last step that holds a term (K = 100: seven, which is
// where most of 250 -> 220 came from: with whole turns eight were multiplied).
#include <type_traits>

#include "update_internal.h"

namespace fastgl {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int kWaveRows = 32;
constexpr int kTallRows = 128;                 // 4 wavefronts
constexpr int kStageElems = 4096;              // elements of B per LDS stage
constexpr int kSmallCols = 64;
constexpr int kSmallWaves = 8;                 // share the contracted range of a small tile

// Eight consecutive elements, as loaded.
template <bool BF16>
struct Oct;
template <>
struct Oct<false> {
    float v[8];
};
template <>
struct Oct<true> {
    uint32_t v[4];
};

// Where the loads of a row of K elements go.  V: elements per load (4 floats, 8 bf16; 1: rows shorter than
// that).  A row needs no more alignment than a dword: a load that would run past the row's end starts at K - V
// instead (or, for V = 1, at the row's start), so that every load lies inside its row whatever K is, and
// settle() moves the elements to their places afterwards.  V = kOdd: bf16 rows of odd length, every other of
// which starts in the middle of a dword: eight elements come out of the five dwords they touch.
constexpr int kOdd = 9;

template <int V>
__device__ __forceinline__ int load_at(int k, int K)
{
    constexpr int N = V == kOdd ? 8 : V;
    if (V == 1) return k < K ? k : 0;
    return k < K - N ? k : K - N;
}

// Elements p .. p+7 out of the dwords w[0..4] that hold elements p & ~1 and up.
__device__ __forceinline__ void funnel(const uint32_t (&w)[5], uint32_t p, uint32_t (&v)[4])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = __builtin_amdgcn_alignbit(w[e + 1], w[e], 16u * (p & 1u));
}

// Elements k .. k+7 of a row.  No control flow around the loads: they stay in flight until they are used.
template <int V>
__device__ __forceinline__ void load_oct(const void *row_, int k, int K, Oct<false> &o)
{
    typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));
    const float *row = static_cast<const float *>(row_);
    if constexpr (V == 4) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const f32x4 q = *reinterpret_cast<const f32x4 *>(row + load_at<4>(k + 4 * i, K));
#pragma unroll
            for (int e = 0; e < 4; ++e) o.v[4 * i + e] = q[e];
        }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) o.v[i] = row[load_at<1>(k + i, K)];
    }
}
template <int V>
__device__ __forceinline__ void load_oct(const void *row_, int k, int K, Oct<true> &o)
{
    typedef uint32_t u32x4a __attribute__((ext_vector_type(4), aligned(4)));
    const uint16_t *row = static_cast<const uint16_t *>(row_);
    if constexpr (V == 8) {
        const u32x4a q = *reinterpret_cast<const u32x4a *>(row + load_at<8>(k, K));
#pragma unroll
        for (int e = 0; e < 4; ++e) o.v[e] = q[e];
    } else if constexpr (V == kOdd) {
        const uintptr_t at = (uintptr_t)(row + load_at<kOdd>(k, K)), base = at & ~(uintptr_t)3;
        const u32x4a q = *reinterpret_cast<const u32x4a *>(base);
        const uint32_t w[5] = {q[0], q[1], q[2], q[3], *reinterpret_cast<const uint32_t *>(base + (at & 2 ? 16 : 12))};
        funnel(w, (uint32_t)(at >> 1), o.v);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            o.v[i] = (uint32_t)row[load_at<1>(k + 2 * i, K)] | ((uint32_t)row[load_at<1>(k + 2 * i + 1, K)] << 16);
    }
}

__device__ __forceinline__ uint32_t keep(uint32_t w, bool lo, bool hi)
{
    return w & ((lo ? 0xFFFFu : 0u) | (hi ? 0xFFFF0000u : 0u));
}

// Elements k .. k+7 in their places, 0 beyond the row's end.  Needed (and called) only where a load may have
// run past the end.
template <int V>
__device__ __forceinline__ void settle(Oct<false> &o, int k, int K)
{
    if constexpr (V == 4) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int d = k + 4 * i - (K - 4);             // elements the load was moved back by, if positive
            const float q[4] = {o.v[4 * i], o.v[4 * i + 1], o.v[4 * i + 2], o.v[4 * i + 3]};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float v = 0.f;
#pragma unroll
                for (int j = e; j < 4; ++j) v = (d > 0 ? e + d : e) == j ? q[j] : v;
                o.v[4 * i + e] = v;
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) o.v[i] = k + i < K ? o.v[i] : 0.f;
    }
}
template <int V>
__device__ __forceinline__ void settle(Oct<true> &o, int k, int K)
{
    if constexpr (V == 8) {
        const int d = (k - (K - 8)) >> 1;                  // dwords; K is even
        const uint32_t q[4] = {o.v[0], o.v[1], o.v[2], o.v[3]};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t v = 0;
#pragma unroll
            for (int j = e; j < 4; ++j) v = (d > 0 ? e + d : e) == j ? q[j] : v;
            o.v[e] = v;
        }
    } else if constexpr (V == kOdd) {
        const int d = k - (K - 8) > 0 ? k - (K - 8) : 0;   // elements
        const uint32_t q[5] = {o.v[0], o.v[1], o.v[2], o.v[3], 0u};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t lo = 0, hi = 0;
#pragma unroll
            for (int j = e; j < 4; ++j) {
                lo = e + (d >> 1) == j ? q[j] : lo;
                hi = e + (d >> 1) == j ? q[j + 1] : hi;
            }
            o.v[e] = __builtin_amdgcn_alignbit(hi, lo, 16u * ((uint32_t)d & 1u));
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) o.v[i] = keep(o.v[i], k + 2 * i < K, k + 2 * i + 1 < K);
    }
}

// Zeroes what the gate closes.
__device__ __forceinline__ void gate_oct(Oct<false> &o, const Oct<false> &gate)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) o.v[i] = gate.v[i] > 0.f ? o.v[i] : 0.f;
}
__device__ __forceinline__ void gate_oct(Oct<true> &o, const Oct<true> &gate)
{
#pragma unroll
    for (int i = 0; i < 4; ++i)
        o.v[i] = keep(o.v[i], __uint_as_float(gate.v[i] << 16) > 0.f, __uint_as_float(gate.v[i] & 0xFFFF0000u) > 0.f);
}

// Planes of the pair (x0, x1), packed as two bf16 per dword (x0 in the low half): x = plane 0 + 1 + 2 exactly.
__device__ __forceinline__ void split_pair3(float x0, float x1, uint32_t (&w)[3])
{
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        const bf16x2 b = {(__bf16)x0, (__bf16)x1};
        w[p] = __builtin_bit_cast(uint32_t, b);
        if (p < 2) {
            x0 -= __uint_as_float(w[p] << 16);
            x1 -= __uint_as_float(w[p] & 0xFFFF0000u);
        }
    }
}

// The operand of a matrix instruction: eight contracted elements per lane, one uint4 per plane.
template <bool BF16>
struct Planes {
    static constexpr int N = BF16 ? 1 : 3;
    uint4 p[N];
};

__device__ __forceinline__ void to_planes(const Oct<false> &o, Planes<false> &f)
{
    uint32_t w[4][3];
#pragma unroll
    for (int i = 0; i < 4; ++i) split_pair3(o.v[2 * i], o.v[2 * i + 1], w[i]);
#pragma unroll
    for (int p = 0; p < 3; ++p) f.p[p] = make_uint4(w[0][p], w[1][p], w[2][p], w[3][p]);
}
__device__ __forceinline__ void to_planes(const Oct<true> &o, Planes<true> &f)
{
    f.p[0] = make_uint4(o.v[0], o.v[1], o.v[2], o.v[3]);
}

template <bool BF16>
__device__ __forceinline__ void mma(const Planes<BF16> &a, const Planes<BF16> &b, f32x16 &acc)
{
    constexpr int kTerms = BF16 ? 1 : 6;       // smallest products first
    constexpr int pa[6] = {0, 2, 1, 0, 1, 0}, pb[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
    for (int t = 0; t < kTerms; ++t) {
        const int x = BF16 ? 0 : pa[t], y = BF16 ? 0 : pb[t];
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a.p[x]), __builtin_bit_cast(bf16x8, b.p[y]),
                                                      acc, 0, 0, 0);
    }
}

// ------------------------------------------------------------------------------------ tall tiles
// The tall kernel's operands are read and its results written through buffer instructions: a load past the
// end of the matrix gives 0 and a store past it is dropped, so that ragged edges need no address clamps and
// no branches (a load or store behind a branch is waited for), and an address is one 32-bit addition.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __amdgpu_buffer_rsrc_t Rsrc;

constexpr int kRsrcFormat = 0x00020000;        // raw buffer of 32-bit elements
constexpr uint32_t kNowhere = 0x80000000u;     // beyond every buffer made here
constexpr int kStream = 2;                     // non-temporal
constexpr int64_t kMaxTallLd = (int64_t)1 << 21;   // row length up to which every offset inside a tile stays below 2^31 bytes

// Exactly `bytes` bytes: the element behind a matrix belongs to somebody else.  Stores are dropped there by this size
// alone (the rows of a tile past the last one are not masked), and the rows of a column operand past the last one
// are 0 by it: whatever lies there would meet A's zeros in the matrix instructions, and 0 times NaN is NaN.
__device__ __forceinline__ Rsrc buffer_from(const void *p, int64_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)(bytes < 0x7FFFFFFF ? bytes : 0x7FFFFFFF), kRsrcFormat);
}

// Size of an operand loaded by rows.  Rows of odd length are loaded in aligned dwords: the one that holds the last
// element counts as inside, its other half (of a row that does not exist) goes no further than funnel and settle.
template <int V>
__device__ __forceinline__ int64_t loadable(int64_t bytes)
{
    return V == kOdd ? (bytes + 3) & ~(int64_t)3 : bytes;
}

// Elements k .. k+7 of the row of K elements that starts at byte offset `row`.
template <int V>
__device__ __forceinline__ void buffer_oct(Rsrc r, uint32_t row, int k, int K, Oct<false> &o)
{
    if constexpr (V == 4) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const u32x4 q = __builtin_amdgcn_raw_buffer_load_b128(r, row + 4u * (uint32_t)load_at<4>(k + 4 * i, K), 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) o.v[4 * i + e] = __uint_as_float(q[e]);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            o.v[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, row + 4u * (uint32_t)load_at<1>(k + i, K), 0, 0));
    }
}
template <int V>
__device__ __forceinline__ void buffer_oct(Rsrc r, uint32_t row, int k, int K, Oct<true> &o)
{
    if constexpr (V == 8) {
        const u32x4 q = __builtin_amdgcn_raw_buffer_load_b128(r, row + 2u * (uint32_t)load_at<8>(k, K), 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) o.v[e] = q[e];
    } else if constexpr (V == kOdd) {
        const uint32_t at = row + 2u * (uint32_t)load_at<kOdd>(k, K), base = at & ~3u;
        const u32x4 q = __builtin_amdgcn_raw_buffer_load_b128(r, base, 0, 0);
        const uint32_t w[5] = {q[0], q[1], q[2], q[3], __builtin_amdgcn_raw_buffer_load_b32(r, base + (at & 2u ? 16 : 12), 0, 0)};
        funnel(w, at >> 1, o.v);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            o.v[i] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, row + 2u * (uint32_t)load_at<1>(k + 2 * i, K), 0, 0) |
                     ((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, row + 2u * (uint32_t)load_at<1>(k + 2 * i + 1, K), 0, 0) << 16);
    }
}

// Two neighbouring columns of B, eight contracted elements each, as loaded: rows of B `ld` bytes apart.  V: elements
// per load (1: bf16 rows that are no whole dwords, a single column of floats).
template <bool BF16>
struct ColPair {
    uint32_t v[BF16 ? 8 : 16];
};
template <int V>
__device__ __forceinline__ void buffer_cols(Rsrc r, uint32_t off, uint32_t ld, ColPair<false> &c)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if constexpr (V > 1) {
            const u32x2 q = __builtin_amdgcn_raw_buffer_load_b64(r, off + i * ld, 0, 0);
            c.v[2 * i] = q[0]; c.v[2 * i + 1] = q[1];
        } else {                             // a single column: nothing follows the last element
            c.v[2 * i] = __builtin_amdgcn_raw_buffer_load_b32(r, off + i * ld, 0, 0);
            c.v[2 * i + 1] = 0;
        }
    }
}
template <int V>
__device__ __forceinline__ void buffer_cols(Rsrc r, uint32_t off, uint32_t ld, ColPair<true> &c)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if constexpr (V > 1) c.v[i] = __builtin_amdgcn_raw_buffer_load_b32(r, off + i * ld, 0, 0);
        else
            c.v[i] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, off + i * ld, 0, 0) |
                     ((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, off + i * ld + 2, 0, 0) << 16);
    }
}
__device__ __forceinline__ Oct<false> column(const ColPair<false> &c, int which)
{
    Oct<false> o;
#pragma unroll
    for (int i = 0; i < 8; ++i) o.v[i] = __uint_as_float(c.v[2 * i + which]);
    return o;
}
__device__ __forceinline__ Oct<true> column(const ColPair<true> &c, int which)
{
    Oct<true> o;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        o.v[i] = which ? (c.v[2 * i] >> 16) | (c.v[2 * i + 1] & 0xFFFF0000u) : (c.v[2 * i] & 0xFFFFu) | (c.v[2 * i + 1] << 16);
    return o;
}

// LDS stage of B: [plane][octet slot][column] x 16 bytes (a lane's eight elements of one plane).
template <int NTILES, bool BCOL, bool GATE, int VA, int VB, bool BF16>
__global__ __launch_bounds__(256, NTILES == 8 || (NTILES <= 4 && GATE && !BF16) ? 2 : 3) void k_update_tall(const RowsGemm g)
{
    constexpr int NT = NTILES * 32, KS = NT < 64 ? 64 : kStageElems / NT, SLOTS = KS / 8, PL = Planes<BF16>::N;
    // Chunks of 32 contracted indices of A under way: two where the registers of the second cost neither a wavefront nor
    // spills (Y M = 512 K, 100 -> 256: 226 us with one, 220 with two; gated dH M = 1.15 M, 64 -> 100: 270 and 257).  Fp32
    // with a gate and 64 columns takes two wavefronts a SIMD for it (M = 40 K, 99 -> 131: 39 us with three and spills, 36).
    constexpr int AHEAD = !BF16 && (NTILES == 4 || (GATE && NTILES == 8)) ? 1 : 2;
    constexpr uint32_t EB = BF16 ? 2 : 4;
    __shared__ uint4 lds[2][PL][SLOTS][NT];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, h = lane >> 5, l32 = lane & 31;
    // consecutive workgroups of one XCD: the column tiles of one row tile
    const int64_t bid = blockIdx.x, q = bid / kXcds;
    const int64_t tile_r = (q / g.tiles_c) * kXcds + bid % kXcds;
    const int tile_c = (int)(q % g.tiles_c);
    if (tile_r >= g.tiles_r) return;
    const int64_t r0 = tile_r * kTallRows, c0 = (int64_t)tile_c * NT;
    const int Kc = (int)g.Kc;

    // A from the tile's first row on; B from its first element (row operand: the tile's first row) on
    const int64_t abytes = loadable<VA>((g.M - r0) * g.lda * EB);
    const Rsrc ra = buffer_from((const char *)g.a + r0 * g.lda * EB, abytes);
    const Rsrc rg = buffer_from(GATE ? (const char *)g.gate + r0 * g.lda * EB : nullptr, GATE ? abytes : 0);
    const Rsrc rb = BCOL ? buffer_from(g.b, g.Kc * g.ldb * EB)
                         : buffer_from((const char *)g.b + c0 * g.ldb * EB, loadable<VB>((g.N - c0) * g.ldb * EB));
    const uint32_t arow = (uint32_t)(wave * kWaveRows + l32) * (uint32_t)g.lda * EB;
    const uint32_t ldb = (uint32_t)g.ldb * EB;

    f32x16 acc[NTILES];
#pragma unroll
    for (int j = 0; j < NTILES; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;

    // Contracted indices per turn of the loop: no more than chunks and stages need (gated dH M = 512 K, 256 -> 100: 310 us
    // with 32, 323 with 64).
    constexpr int TURN = AHEAD == 1 && KS <= 32 ? 32 : 64;
    // The turns before the last one are a loop of their own, without the questions where the range ends, and the last one stands
    // behind it.  us, the questions in every turn / so, fp32:  Y 30 000 rows, 602 -> 256: 59.3 / 53.5, 200 000, 33 -> 57: 22.4 / 20.0;
    // dH 45 000, 32 -> 300: 23.4 / 19.1, gated 26.7 / 24.6;  bf16:  Y 400 000, 99 -> 131: 125 / 101, 256 -> 47: 70 / 62, gated dH 87 000
    // rows of 256: 44.6 / 39.7 (worst: 400 000, 100 <- 256 71.6 / 75.4).  Not for the fp32 forms that hold most registers:
    // Y 400 000, 256 -> 256: 305 / 339, gated dH 131 -> 99: 176 / 199.
    constexpr bool PLAIN = BF16 || !((NTILES == 8 && BCOL && !GATE) || (NTILES == 4 && GATE));
    Oct<BF16> ar[AHEAD][2], gr[AHEAD][GATE ? 2 : 1];
    auto load_a = [&](int to, int k0) {                       // this lane's octets of the chunk: indices k0 + 16 s + 8 h .. + 7
        const uint32_t row = arow + (k0 < Kc ? 0u : kNowhere);        // chunks past the end touch no memory
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            buffer_oct<VA>(ra, row, k0 + 16 * s + 8 * h, Kc, ar[to][s]);
            if constexpr (GATE) buffer_oct<VA>(rg, row, k0 + 16 * s + 8 * h, Kc, gr[to][s]);
        }
    };
    // which two octets of a stage a thread brings: BCOL two columns of one slot, else one column's two slots
    const int bc = BCOL ? 2 * (t % (NT / 2)) : t % NT;
    const int bs = BCOL ? t / (NT / 2) : 2 * (t / NT);
    // of an odd number of columns the last two are brought as a pair that starts one column early
    const bool shifted = BCOL && (VB > 1) && (g.N & 1) && c0 + bc == g.N - 1 && g.N > 1;
    const uint32_t bcol = (uint32_t)(c0 + bc - (shifted ? 1 : 0)) * EB;
    ColPair<BF16> bcols;
    Oct<BF16> brow[BCOL ? 1 : 2];
    const bool brings = NT >= 64 || bs < SLOTS;               // 32 columns: half of the threads
    auto load_b = [&](int k0) {                               // the stage of KS contracted indices from k0 on
        if (!brings) return;                                  // the same for a whole wavefront
        if constexpr (BCOL) {
            buffer_cols<VB>(rb, (uint32_t)(k0 + 8 * bs) * ldb + bcol, ldb, bcols);
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i)
                buffer_oct<VB>(rb, (uint32_t)bc * ldb, k0 + 8 * (bs + i), Kc, brow[i]);
        }
    };
    auto stage_b = [&](int buf, int k0) {
        if (!brings) return;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int slot = BCOL ? bs : bs + i, col = BCOL ? bc + i : bc;
            Oct<BF16> o;
            if constexpr (BCOL) {                             // rows of B past the end read as 0
                o = column(bcols, i);
                if (!BF16 && (g.N & 1) && i == 0) {
                    const Oct<BF16> second = column(bcols, 1);
#pragma unroll
                    for (int e = 0; e < (int)(sizeof(o.v) / sizeof(o.v[0])); ++e) o.v[e] = shifted ? second.v[e] : o.v[e];
                }
            } else {
                o = brow[i];
                if (k0 + KS > Kc) settle<VB>(o, k0 + 8 * slot, Kc);
            }
            Planes<BF16> f;
            to_planes(o, f);
#pragma unroll
            for (int p = 0; p < PL; ++p) lds[buf][p][slot][col] = f.p[p];
        }
    };

    load_b(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) load_a(i, 32 * i);
    float bias[NTILES];
#pragma unroll
    for (int j = 0; j < NTILES; ++j) bias[j] = 0.f;
    if (g.bias) {
#pragma unroll
        for (int j = 0; j < NTILES; ++j) {
            const int64_t col = c0 + 32 * j + l32;
            bias[j] = g.bias[col < g.N ? col : 0];
        }
    }
    stage_b(0, 0);
    int lk = KS;                                              // the stage whose loads are under way
    load_b(lk);
    __syncthreads();
    int cur = 0;
    // Order of a stage: the next one, whose loads were issued a stage ago, goes to the other LDS buffer; the
    // loads of the one after it are issued; then this one is multiplied.  Loads of B and A are issued in the
    // order in which they are waited for.
    Planes<BF16> fa[2];
    if constexpr (PLAIN) {
        auto turn = [&](auto last, int k0) {
            constexpr bool LAST = decltype(last)::value;
#include "update_tall_turn.inc"
        };
        int k0 = 0;
        for (; k0 + TURN < Kc; k0 += TURN) turn(std::false_type(), k0);
        turn(std::true_type(), k0);
    } else {
        constexpr bool LAST = true;
        for (int k0 = 0; k0 < Kc; k0 += TURN) {
#include "update_tall_turn.inc"
        }
    }

    // element e of lane (h, l32): row 8 (e / 4) + 4 h + e % 4, column l32 of its 32 x 32 tile
    const Rsrc rc = buffer_from((const char *)g.c + (r0 * g.N + c0) * EB, ((g.M - r0) * g.N - c0) * EB);
    const uint32_t ldc = (uint32_t)g.N * EB, coff = (uint32_t)(wave * kWaveRows + 4 * h) * ldc + (uint32_t)l32 * EB;
    const bool relu = g.relu != 0;
    auto write = [&](auto stream) {
#pragma unroll
        for (int j = 0; j < NTILES; ++j) {
            const uint32_t off = c0 + 32 * j + l32 < g.N ? coff + 32 * j * EB : kNowhere;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                float v = acc[j][e] + bias[j];
                if (relu) v = v > 0.f ? v : 0.f;
                const uint32_t at = off + (uint32_t)(8 * (e >> 2) + (e & 3)) * ldc;
                if constexpr (BF16) __builtin_amdgcn_raw_buffer_store_b16(f32_to_bf16(v), rc, at, 0, decltype(stream)::value);
                else __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rc, at, 0, decltype(stream)::value);
            }
        }
    };
    // streaming stores only where they fill whole cache lines (N = 100: 345 us with them, 280 without)
    if (ldc % 128 == 0) write(std::integral_constant<int, kStream>());
    else write(std::integral_constant<int, 0>());
}

// ---------------------------------------------------------------------- tall tiles, B in LDS for good
// Y of fp32 rows of four and more elements, many of them, N = 32 NTILES: one workgroup per compute unit keeps all of B in LDS,
// cut into planes once, and its wavefronts take tiles of 32 rows one after the other, each for itself: no barrier and no conversion of B in the
// loop, so that one wavefront's loads and stores run under the other's matrix instructions.  The steps of a tile are those of
// k_update_tall in the same order: the same results.  Y of 512 K rows, 100 -> 256, in a training step: 231 us with k_update_tall, 192;
// 730 MB, 143 to move them, and 156 for the matrix instructions at the 1 135 TFLOP/s of a large product.  Loads of A in whole lines that
// reach their lanes through LDS, past the caches or not, gained nothing.
constexpr int kHeldBlocks = 256;               // one per compute unit
constexpr int64_t kHeldLds = 160 * 1024;       // of a workgroup
constexpr int kHeldThreads = 512;              // two wavefronts per SIMD

// B in LDS, [plane][octet slot][column] x 16 bytes, and 16 bytes of zeros: the octet behind the last one of an odd number.
inline int64_t held_lds(int ntiles, int64_t Kc) { return ceil_div(Kc, 8) * ntiles * 32 * 3 * 16 + 16; }

// LAST: steps of the last turn, 1 to 4 (a constant: accumulators that reach the end by several paths take a second set of
// registers).
template <int NTILES, int LAST>
__global__ __launch_bounds__(kHeldThreads, 2) void k_update_held(const RowsGemm g)
{
    constexpr int NT = NTILES * 32, THREADS = kHeldThreads, WAVES = THREADS / kWave, PL = 3;
    extern __shared__ uint4 planes[];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), h = lane >> 5, l32 = lane & 31;
    const int Kc = (int)g.Kc, slots = (Kc + 7) >> 3;
    const uint32_t ldb = (uint32_t)g.ldb * 4;
    {
        const Rsrc rb = buffer_from(g.b, g.Kc * g.ldb * 4);
        for (int u = t; u < slots * (NT / 2); u += THREADS) {
            const int bc = 2 * (u % (NT / 2)), slot = u / (NT / 2);
            ColPair<false> c;                                  // rows of B past the end read as 0
            buffer_cols<4>(rb, (uint32_t)(8 * slot) * ldb + (uint32_t)bc * 4, ldb, c);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                Planes<false> f;
                to_planes(column(c, i), f);
#pragma unroll
                for (int p = 0; p < PL; ++p) planes[(p * slots + slot) * NT + bc + i] = f.p[p];
            }
        }
        if (t == 0) planes[PL * slots * NT] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
    }
    float bias[NTILES];
#pragma unroll
    for (int j = 0; j < NTILES; ++j) bias[j] = g.bias ? g.bias[32 * j + l32] : 0.f;

    const int64_t tiles = (g.M + kWaveRows - 1) / kWaveRows, stride = (int64_t)gridDim.x * WAVES;
    // Two chunks of 32 contracted indices under way: octets s of row l32, indices k0 + 16 s + 8 h .. + 7.  Chunks past the end
    // touch no memory.
    Oct<false> ar[2][2];
    auto load_a = [&](int to, int64_t tile, int k0) {
        const int64_t r0 = tile * kWaveRows;
        const bool there = tile < tiles && k0 < Kc;
        const Rsrc ra = buffer_from((const char *)g.a + (there ? r0 * g.lda * 4 : 0), there ? (g.M - r0) * g.lda * 4 : 0);
#pragma unroll
        for (int s = 0; s < 2; ++s) buffer_oct<4>(ra, (uint32_t)l32 * (uint32_t)g.lda * 4, k0 + 16 * s + 8 * h, Kc, ar[to][s]);
    };
    Planes<false> fa[2];
    const bool relu = g.relu != 0;
    int64_t tile = (int64_t)blockIdx.x * WAVES + wave;
#pragma unroll
    for (int i = 0; i < 2; ++i) load_a(i, tile, 32 * i);
    for (; tile < tiles; tile += stride) {
        f32x16 acc[NTILES];
#pragma unroll
        for (int j = 0; j < NTILES; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;
        // STEPS steps from k0 on; then = tile and index of what the chunks' registers are loaded with
        auto turn = [&](auto steps, int k0, int64_t then, int then_k0) {
            constexpr int STEPS = decltype(steps)::value;
            if (STEPS <= 2) load_a(1, then, then_k0 + 32);      // there is no second chunk
#pragma unroll
            for (int step = 0; step < STEPS; ++step) {
                const int cc = step >> 1, s = step & 1;
                if (s == 0) {
                    const int kc = k0 + 32 * cc;
                    if (kc + 32 > Kc)
#pragma unroll
                        for (int i = 0; i < 2; ++i) settle<4>(ar[cc][i], kc + 16 * i + 8 * h, Kc);
#pragma unroll
                    for (int i = 0; i < 2; ++i) to_planes(ar[cc][i], fa[i]);
                    __builtin_amdgcn_sched_barrier(0);
                    load_a(cc, then, then_k0 + 32 * cc);
                    __builtin_amdgcn_sched_barrier(0);
                }
                const int slot = (k0 + 16 * step) / 8 + h;
                const bool there = slot < slots;
                const uint4 *at = planes + (there ? slot * NT + l32 : PL * slots * NT);
                const int plane = there ? slots * NT : 0, next = there ? 32 : 0;
                Planes<false> fb[2];
#pragma unroll
                for (int p = 0; p < PL; ++p) fb[0].p[p] = at[p * plane];
#pragma unroll
                for (int j = 0; j < NTILES; ++j) {             // the next tile is read while this one is multiplied
                    if (j + 1 < NTILES)
#pragma unroll
                        for (int p = 0; p < PL; ++p) fb[(j + 1) & 1].p[p] = at[p * plane + (j + 1) * next];
                    mma<false>(fa[s], fb[j & 1], acc[j]);
                }
                __builtin_amdgcn_sched_group_barrier(0x100, PL, 0);
#pragma unroll
                for (int j = 0; j < NTILES; ++j) {
                    if (j + 1 < NTILES) __builtin_amdgcn_sched_group_barrier(0x100, PL, 0);    // LDS reads
                    __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);                         // matrix instructions
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        int k0 = 0;
        for (; k0 + 64 < Kc; k0 += 64) turn(std::integral_constant<int, 4>(), k0, tile, k0 + 64);
        turn(std::integral_constant<int, LAST>(), k0, tile + stride, 0);

        const int64_t r0 = tile * kWaveRows;
        const Rsrc rc = buffer_from((const char *)g.c + r0 * g.N * 4, (g.M - r0) * g.N * 4);
        // made anew for every tile: kept over the loop, the offsets of a lane's results would take more registers than there are
        uint32_t ldc = (uint32_t)g.N * 4;
        asm volatile("" : "+s"(ldc));
        const uint32_t coff = (uint32_t)(4 * h) * ldc + (uint32_t)l32 * 4;
        // past the caches: 512 K rows, 100 -> 256: 183 us alone without, 189 so, but the aggregation that reads Y next takes 172 and 150 us
#pragma unroll
        for (int j = 0; j < NTILES; ++j) {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                float v = acc[j][e] + bias[j];
                if (relu) v = v > 0.f ? v : 0.f;
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rc, coff + 32 * j * 4 + (uint32_t)(8 * (e >> 2) + (e & 3)) * ldc, 0, kStream);
            }
        }
    }
}

template <int NTILES, int LAST>
fastgl_status launch_held(const RowsGemm &g, hipStream_t s)
{
    FASTGL_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&k_update_held<NTILES, LAST>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)kHeldLds));
    hipLaunchKernelGGL((k_update_held<NTILES, LAST>), dim3(kHeldBlocks), dim3(kHeldThreads),
                       held_lds(NTILES, g.Kc), s, g);
    return FASTGL_OK;
}

template <int NTILES>
fastgl_status launch_held_steps(const RowsGemm &g, hipStream_t s)
{
    switch (ceil_div((g.Kc - 1) % 64 + 1, 16)) {
        case 1: return launch_held<NTILES, 1>(g, s);
        case 2: return launch_held<NTILES, 2>(g, s);
        case 3: return launch_held<NTILES, 3>(g, s);
        default: return launch_held<NTILES, 4>(g, s);
    }
}

// ----------------------------------------------------------------------------------- small tiles
template <bool BCOL, bool GATE, int VA, int VB, bool BF16>
__global__ __launch_bounds__(64 * kSmallWaves) void k_update_small(const RowsGemm g)
{
    constexpr int U = 2;                                       // steps of 16 contracted indices loaded together
    constexpr int kLd = kSmallCols + 4;                        // floats per row of a partial tile
    __shared__ __attribute__((aligned(16))) float part[kSmallWaves][kWaveRows][kLd];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, h = lane >> 5, l32 = lane & 31;
    const int64_t r0 = (int64_t)(blockIdx.x / g.tiles_c) * kWaveRows, c0 = (int64_t)(blockIdx.x % g.tiles_c) * kSmallCols;
    typedef typename QuadBits<BF16>::elem E;
    const int64_t row = r0 + l32 < g.M ? r0 + l32 : g.M - 1;
    const E *arow = static_cast<const E *>(g.a) + row * g.lda;
    const E *grow = GATE ? static_cast<const E *>(g.gate) + row * g.lda : nullptr;
    // wavefront w: a contiguous part of the steps
    const int Kc = (int)g.Kc, steps = (Kc + 15) / 16, per = (steps + kSmallWaves - 1) / kSmallWaves;
    const int s0 = wave * per, s1 = s0 + per < steps ? s0 + per : steps;

    f32x16 acc[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;
    for (int sb = s0; sb < s1; sb += U) {
        Oct<BF16> a[U], ga[GATE ? U : 1], b[U][2];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = 16 * (sb + u < s1 ? sb + u : s1 - 1) + 8 * h;          // a step past the end repeats the last one
            load_oct<VA>(arow, k, Kc, a[u]);
            if constexpr (GATE) load_oct<VA>(grow, k, Kc, ga[u]);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int64_t n = c0 + 32 * j + l32 < g.N ? c0 + 32 * j + l32 : 0;
                if constexpr (BCOL) {
                    const E *p = static_cast<const E *>(g.b) + n;
                    if constexpr (BF16) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const uint32_t lo = p[load_at<1>(k + 2 * i, Kc) * g.ldb], hi = p[load_at<1>(k + 2 * i + 1, Kc) * g.ldb];
                            b[u][j].v[i] = lo | (hi << 16);
                        }
                    } else {
#pragma unroll
                        for (int i = 0; i < 8; ++i) b[u][j].v[i] = p[load_at<1>(k + i, Kc) * g.ldb];
                    }
                } else {
                    load_oct<VB>(static_cast<const E *>(g.b) + n * g.ldb, k, Kc, b[u][j]);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (sb + u >= s1) break;                            // same for the whole wavefront
            const int k = 16 * (sb + u) + 8 * h;
            const bool tail = 16 * (sb + u) + 16 > Kc;          // same for the whole wavefront
            Planes<BF16> fa, fb;
            if constexpr (GATE) gate_oct(a[u], ga[u]);
            if (tail) settle<VA>(a[u], k, Kc);
            to_planes(a[u], fa);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if (tail) settle<BCOL ? 1 : VB>(b[u][j], k, Kc);
                to_planes(b[u][j], fb);
                mma<BF16>(fa, fb, acc[j]);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) part[wave][8 * (e >> 2) + 4 * h + (e & 3)][32 * j + l32] = acc[j][e];
    __syncthreads();
    E *c = static_cast<E *>(g.c);
    const int64_t col = c0 + lane;
    const float bias = g.bias && col < g.N ? g.bias[col] : 0.f;
#pragma unroll
    for (int i = 0; i < kWaveRows / kSmallWaves; ++i) {
        const int r = kSmallWaves * i + wave;
        float p[kSmallWaves];
#pragma unroll
        for (int w = 0; w < kSmallWaves; ++w) p[w] = part[w][r][lane];
#pragma unroll
        for (int n = kSmallWaves; n > 1; n /= 2)
#pragma unroll
            for (int w = 0; w < n / 2; ++w) p[w] = p[2 * w] + p[2 * w + 1];
        float v = p[0] + bias;
        if (g.relu) v = v > 0.f ? v : 0.f;
        if (r0 + r < g.M && col < g.N) {
            if constexpr (BF16) c[(r0 + r) * g.N + col] = f32_to_bf16(v);
            else c[(r0 + r) * g.N + col] = v;
        }
    }
}

template <bool BF16>
__global__ __launch_bounds__(256) void k_update_no_terms(void *c, const float *bias, int64_t n, int64_t cols, bool relu)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        float v = bias ? bias[i % cols] : 0.f;
        if (relu) v = v > 0.f ? v : 0.f;
        if constexpr (BF16) static_cast<uint16_t *>(c)[i] = f32_to_bf16(v);
        else static_cast<float *>(c)[i] = v;
    }
}

// ------------------------------------------------------------------------------------- host side
// Elements per load of rows of K elements, no gap between them, at p (and p2).
int row_vector(const void *p, const void *p2, int64_t K, bool bf16)
{
    if (!bf16) return K >= 4 ? 4 : 1;
    if (K < 8 || (((uintptr_t)p | (uintptr_t)p2) & 3)) return 1;
    return K % 2 == 0 ? 8 : kOdd;
}

template <int NTILES, bool BCOL, bool GATE, int VA, int VB, bool BF16>
void launch_one(const RowsGemm &g, unsigned blocks, hipStream_t s)
{
    if constexpr (NTILES == 0) hipLaunchKernelGGL((k_update_small<BCOL, GATE, VA, VB, BF16>), dim3(blocks), dim3(64 * kSmallWaves), 0, s, g);
    else hipLaunchKernelGGL((k_update_tall<NTILES, BCOL, GATE, VA, VB, BF16>), dim3(blocks), dim3(256), 0, s, g);
}

template <int NTILES, bool BCOL, bool GATE>
void launch_vectors(const RowsGemm &g, bool bf16, int va, int vb, unsigned blocks, hipStream_t s)
{
    if (!bf16) {
        if (NTILES == 1 && vb == 1) {
            if constexpr (NTILES == 1)
                va == 4 ? launch_one<NTILES, BCOL, GATE, 4, 1, false>(g, blocks, s) : launch_one<NTILES, BCOL, GATE, 1, 1, false>(g, blocks, s);
        } else if (va == 4) launch_one<NTILES, BCOL, GATE, 4, 4, false>(g, blocks, s);
        else launch_one<NTILES, BCOL, GATE, 1, BCOL ? 4 : 1, false>(g, blocks, s);
    } else if constexpr (BCOL) {                 // vb: are column pairs whole dwords
        if (va == 8) vb > 1 ? launch_one<NTILES, BCOL, GATE, 8, 8, true>(g, blocks, s) : launch_one<NTILES, BCOL, GATE, 8, 1, true>(g, blocks, s);
        else if (va == kOdd) vb > 1 ? launch_one<NTILES, BCOL, GATE, kOdd, 8, true>(g, blocks, s) : launch_one<NTILES, BCOL, GATE, kOdd, 1, true>(g, blocks, s);
        else vb > 1 ? launch_one<NTILES, BCOL, GATE, 1, 8, true>(g, blocks, s) : launch_one<NTILES, BCOL, GATE, 1, 1, true>(g, blocks, s);
    } else {                                     // rows of the same length on both sides
        if (va == 8 && vb == 8) launch_one<NTILES, BCOL, GATE, 8, 8, true>(g, blocks, s);
        else if (va == kOdd && vb == kOdd) launch_one<NTILES, BCOL, GATE, kOdd, kOdd, true>(g, blocks, s);
        else launch_one<NTILES, BCOL, GATE, 1, 1, true>(g, blocks, s);
    }
}

template <int NTILES>
void launch_tiles(const RowsGemm &g, bool b_col, bool bf16, int va, int vb, unsigned blocks, hipStream_t s)
{
    if (b_col) launch_vectors<NTILES, true, false>(g, bf16, va, vb, blocks, s);
    else if constexpr (NTILES == 1) return;      // dH: narrow K is rare, 64 columns then
    else if (g.gate) launch_vectors<NTILES, false, true>(g, bf16, va, vb, blocks, s);
    else launch_vectors<NTILES, false, false>(g, bf16, va, vb, blocks, s);
}

// Small tiles up to this many of them: two per compute unit.  Up to there the latency of one workgroup
// decides and theirs is the shorter; M = 4 000, K = N = 256: 11 us against 12 with tall tiles, M = 8 000:
// 18 against 12, M = 1 000: 7 against 12.
constexpr int64_t kMostSmall = 512;
// Tall tiles: of the widths that give every compute unit a workgroup, the one with the least work.  A
// workgroup's step takes about 0.55, 1.0 and 1.7 us with 64, 128 and 256 columns, so that idle compute units cost more
// than reading rows again (M = 16 000, K = N = 256: 29 us with 125 tiles of 256 columns, 18 with 250 of 128), while
// with enough rows narrow tiles cut every row more often (about 6 % and 25 % more work per column) and wide
// ones work on columns that do not exist (N = 100, M = 1.15 M: 285 us with 256 columns, 210 with 128).
constexpr int64_t kFull = 240;

int tall_tiles(int64_t M, int64_t N, bool b_col)
{
    const int64_t rows = ceil_div(M, kTallRows);
    if (b_col && N <= 32) return 1;
    int best = 2;
    int64_t best_cost = ceil_div(N, 64) * 64 * 20;
    for (int nt = 4; nt <= 8; nt *= 2) {
        const int64_t tiles = ceil_div(N, 32 * nt), cost = tiles * 32 * nt * (nt == 4 ? 17 : 16);
        if (rows * tiles >= kFull && cost <= best_cost) {
            best = nt;
            best_cost = cost;
        }
    }
    return best;
}

// Does k_update_held take these tiles?  B fits LDS, a tile has no columns that do not exist, and what is saved, cutting B anew in every
// workgroup, is more than what the tiles' end costs: the rounds in which its wavefronts take their tiles are nearly full and a tile has
// many steps, or there are hardly more tiles than wavefronts (256 columns).  us with the aggregation that reads the result, right after
// the operand was written, k_update_tall / k_update_held, by K -> N:
//   rows (rounds)    32 -> 256   64 -> 256   72 -> 256   88 -> 256   96 -> 256   100 -> 256
//   72 K  (1.1)      46 / 43     53 / 49                                         63 / 59
//   131 K (2.0)      70 / 67     78 / 81     83 / 85     87 / 83     86 / 90     91 / 82
//   196 K (3.0)      99 / 102    111 / 114   118 / 118   125 / 118   125 / 125   130 / 122
//   300 K (4.6)      149 / 152   167 / 172   178 / 173   191 / 181   186 / 177   198 / 185
//   420 K (6.4)      204 / 214   225 / 232   235 / 234   250 / 243   251 / 239   273 / 258
//   512 K (7.8)      245 / 247   271 / 265   287 / 279   300 / 291   312 / 293   324 / 306
//   rows (rounds)    32 -> 128   112 -> 128  128 -> 128  144 -> 128  160 -> 128  176 -> 128  200 -> 128
//   540 K (8.2)      134 / 135   206 / 212   238 / 224   236 / 228   238 / 231   251 / 246   291 / 276
//   655 K (10.0)     161 / 167   247 / 238   254 / 244   271 / 262   281 / 275   302 / 287   342 / 321
//   800 K (12.2)     196 / 200   300 / 302   306 / 313   331 / 334   342 / 342   365 / 359   412 / 389
//   1 M   (15.3)     246 / 250   378 / 378   382 / 380   412 / 412   430 / 427   451 / 441   516 / 487
// At 140 K and 215 K rows, rounds that are not full, it loses (100 -> 256 alone, cold: 74 / 75, 100 / 102), at 8 rounds and fewer with
// 128 columns as well; with columns that do not exist, or rows that are no whole lines (512 K rows: 64 -> 200 141 / 160, 37 -> 100 78 / 87),
// and in narrower tiles (100 -> 64 104 / 113, 256 -> 47 172 / 189).
bool held_fits(int ntiles, int64_t M, int64_t Kc, int64_t N)
{
    if ((ntiles != 8 && ntiles != 4) || N != 32 * ntiles || held_lds(ntiles, Kc) > kHeldLds) return false;
    const int64_t waves = kHeldBlocks * kHeldThreads / kWave, tiles = ceil_div(M, kWaveRows), rounds = ceil_div(tiles, waves);
    if (ntiles == 4) return rounds >= 9 && Kc > 144;
    if (rounds == 2) return 2 * tiles <= 3 * waves || Kc > 96;
    return rounds > 2 && Kc > 64 && 20 * tiles >= 17 * rounds * waves;
}

}  // namespace

fastgl_status launch_rows_gemm(RowsGemm g, bool b_col, bool bf16, hipStream_t s, const char *what)
{
    const int va = row_vector(g.a, g.gate, g.Kc, bf16);
    const int vb = !b_col ? row_vector(g.b, nullptr, g.Kc, bf16) : (bf16 ? g.ldb % 2 == 0 && ((uintptr_t)g.b & 3) == 0 : g.N > 1) ? 8 : 1;
    const int64_t ld = g.lda > g.ldb ? g.lda : g.ldb, small = ceil_div(g.M, kWaveRows) * ceil_div(g.N, kSmallCols);
    const bool far = ld > kMaxTallLd || g.N > kMaxTallLd || (b_col && (g.Kc + 64) * g.ldb >= (int64_t)1 << 29);
    int ntiles = small <= kMostSmall || far ? 0 : tall_tiles(g.M, g.N, b_col);
    g.tiles_c = ntiles ? (int)ceil_div(g.N, ntiles * 32) : (int)ceil_div(g.N, kSmallCols);
    g.tiles_r = ntiles ? ceil_div(g.M, kTallRows) : ceil_div(g.M, kWaveRows);
    const int64_t blocks = ntiles ? ceil_div(g.tiles_r, kXcds) * kXcds * g.tiles_c : g.tiles_r * g.tiles_c;
    if (blocks >= INT32_MAX) {
        set_error("%s: too many tiles (%lld)", what, (long long)blocks);
        return FASTGL_ERR_UNSUPPORTED;
    }
    if (b_col && !bf16 && va == 4 && held_fits(ntiles, g.M, g.Kc, g.N)) {
        const fastgl_status st = ntiles == 8 ? launch_held_steps<8>(g, s) : launch_held_steps<4>(g, s);
        if (st != FASTGL_OK) return st;
        FASTGL_LAUNCH_CHECK(what);
        return FASTGL_OK;
    }
    switch (ntiles) {
        case 0: launch_tiles<0>(g, b_col, bf16, va, vb, (unsigned)blocks, s); break;
        case 1: launch_tiles<1>(g, b_col, bf16, va, vb, (unsigned)blocks, s); break;
        case 2: launch_tiles<2>(g, b_col, bf16, va, vb, (unsigned)blocks, s); break;
        case 4: launch_tiles<4>(g, b_col, bf16, va, vb, (unsigned)blocks, s); break;
        default: launch_tiles<8>(g, b_col, bf16, va, vb, (unsigned)blocks, s); break;
    }
    FASTGL_LAUNCH_CHECK(what);
    return FASTGL_OK;
}

fastgl_status launch_no_terms(bool bf16, void *c, const float *bias, int64_t rows, int64_t cols, bool relu, hipStream_t s,
                              const char *what)
{
    const int64_t n = rows * cols, blocks = ceil_div(n, 1024);
    const dim3 grid((unsigned)(blocks < 65536 ? blocks : 65536));
    if (bf16) hipLaunchKernelGGL(k_update_no_terms<true>, grid, dim3(256), 0, s, c, bias, n, cols, relu);
    else hipLaunchKernelGGL(k_update_no_terms<false>, grid, dim3(256), 0, s, c, bias, n, cols, relu);
    FASTGL_LAUNCH_CHECK(what);
    return FASTGL_OK;
}

}  // namespace fastgl
