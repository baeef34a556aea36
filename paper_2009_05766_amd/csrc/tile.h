// Building blocks of the tiled kernels for layers of any shape (k_tile_fwd.hip, k_tile_dgrad.hip, k_tile_wgrad.hip): one
// workgroup computes a BM x BN block of a worker's product, its waves 32 x 32 tiles of it, in steps of BK contraction
// indices through LDS.  While a step is multiplied the next one is on its way into registers.
//
// Both operands lie in LDS as rows along the contraction (As[m][k], Bs[n][k]) in pieces of four neighbouring k, so that a
// lane reads what an instruction or two want as one 128-bit word.  A piece comes from memory in one of two ways:
//   along     the operand is contiguous along k there: a piece is one load
//   across    it is contiguous along m (or n): a thread loads a 4 x 4 block as four rows and turns it by naming registers
// fp32 operands are multiplied by v_mfma_f32_32x32x2_f32 (exact products, fp32 accumulation; the two lane halves take four
// consecutive k each, the order inside the sum is the same for both operands), bfloat16 operands (BF) by
// v_mfma_f32_32x32x16_bf16; values that are fp32 in memory are rounded on their way into LDS.
#pragma once
#include "bf16.h"
#include "kernels.h"
#include "layout.h"
#include "vec.h"

namespace netmax {

typedef float tile_f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t tile_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t tile_u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 tile_bf16x8;

// Grid of a tiled kernel, and a workgroup's id in it.
inline dim3 tile_grid(unsigned workgroups)
{
    const GridRows r = grid_rows(workgroups);
    return dim3(r.x, r.y);
}
__device__ __forceinline__ unsigned tile_block() { return blockIdx.y * GRID_ROW + blockIdx.x; }

// tiled_offset() with one 32 x 32 -> 64 bit multiply-add: j + (((j >> 11) (M - 1) + i) << 11); needs j < 2^43
__device__ __forceinline__ size_t tiled_offset_quick(int M, int i, int64_t j)
{
    const uint64_t t = (uint64_t)(uint32_t)(j >> TILE_SHIFT) * (uint32_t)(M - 1) + (uint32_t)i;
    return (size_t)j + (size_t)(t << TILE_SHIFT);
}

// A stretch of a worker's parameters that starts at parameter j: offset of parameter j + u as base + at(u), in 32 bits but for the last
// step (u < 2^32 - TILE, a block of 128 rows of at most 2^24 columns).  j is the same for all lanes.
struct TileSpan {
    size_t base; uint32_t rem, skip;
    __device__ __forceinline__ TileSpan(int M, int g, int64_t j)
        : base(((size_t)(j >> TILE_SHIFT) * M + g) << TILE_SHIFT), rem((uint32_t)(j & (TILE - 1))), skip((uint32_t)(M - 1) << TILE_SHIFT) {}
    __device__ __forceinline__ size_t at(uint32_t u) const
    {
        const uint32_t q = rem + u;
        return (uint64_t)(q >> TILE_SHIFT) * skip + q;
    }
};

// The value, hidden from the optimiser: addresses computed from it inside a loop are computed there, not kept in registers across it.
__device__ __forceinline__ int tile_opaque(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// Four neighbouring elements of memory: fp32, or bfloat16 (S16) as two packed words.
template <bool S16> struct Piece { f32x4 v; };
template <> struct Piece<true> { tile_u32x2 v; };

// V: one load of four elements that exist, at any address of an element (gfx950 takes wide loads there).  Otherwise element by
// element, n of them exist (at least one; the others repeat the last).
typedef float tile_f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t tile_u32x2_any __attribute__((ext_vector_type(2), aligned(2)));
template <bool V> __device__ __forceinline__ Piece<false> load_piece(const float *p, int n)
{
    Piece<false> r;
    if constexpr (V) r.v = *reinterpret_cast<const tile_f32x4_any *>(p);
    else {
#pragma unroll
        for (int e = 0; e < 4; ++e) r.v[e] = p[e < n ? e : n - 1];
    }
    return r;
}
template <bool V> __device__ __forceinline__ Piece<true> load_piece(const uint16_t *p, int n)
{
    Piece<true> r;
    if constexpr (V) r.v = *reinterpret_cast<const tile_u32x2_any *>(p);
    else {
        uint32_t h[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = p[e < n ? e : n - 1];
        r.v = tile_u32x2{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
    }
    return r;
}

// A row whose length is no multiple of four: its last piece is loaded from four elements before the end.  The piece with the last
// `left` (1 .. 3) of those first and zeros behind them; of more than three nothing changes, of less than one all zeros.
__device__ __forceinline__ Piece<false> piece_tail(Piece<false> p, int left)
{
    if (left < 4) {
        const f32x4 v = p.v;
        p.v[0] = left == 3 ? v[1] : left == 2 ? v[2] : left == 1 ? v[3] : 0.0f;
        p.v[1] = left == 3 ? v[2] : left == 2 ? v[3] : 0.0f;
        p.v[2] = left == 3 ? v[3] : 0.0f;
        p.v[3] = 0.0f;
    }
    return p;
}
__device__ __forceinline__ Piece<true> piece_tail(Piece<true> p, int left)
{
    if (left < 4) {
        const uint64_t v = left > 0 ? (((uint64_t)p.v[1] << 32) | p.v[0]) >> (16 * (4 - left)) : 0ull;
        p.v = tile_u32x2{(uint32_t)v, (uint32_t)(v >> 32)};
    }
    return p;
}

// Element e of a loaded piece as 16 bits, as the value of either kind.
__device__ __forceinline__ uint32_t piece_bits(const Piece<true> &p, int e) { return (p.v[e >> 1] >> (16 * (e & 1))) & 0xFFFFu; }

__device__ __forceinline__ float piece_value(const Piece<false> &p, int e) { return p.v[e]; }
__device__ __forceinline__ float piece_value(const Piece<true> &p, int e) { return __uint_as_float(piece_bits(p, e) << 16); }

template <bool BF, int BK> struct TileLds {
    typedef float elem;
    static constexpr int PITCH = BK + 4;             // rows start at multiples of 16 bytes, 32 of them meet all banks evenly
};
template <int BK> struct TileLds<true, BK> {
    typedef uint16_t elem;
    static constexpr int PITCH = BK + 8;
};

// Writes the piece k .. k + 3 of an operand row; only the first `left` of the four indices exist, the others become 0.
__device__ __forceinline__ void put_piece(float *dst, f32x4 v, int left)
{
    if (left < 4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = e < left ? v[e] : 0.0f;
    }
    *reinterpret_cast<f32x4 *>(dst) = v;
}
__device__ __forceinline__ void put_piece(uint16_t *dst, f32x4 v, int left)
{
    if (left < 4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = e < left ? v[e] : 0.0f;
    }
    *reinterpret_cast<tile_u32x2 *>(dst) = tile_u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
}
__device__ __forceinline__ void put_piece(uint16_t *dst, tile_u32x2 v, int left)
{
    if (left < 4) {
        v[0] = left >= 2 ? v[0] : (left == 1 ? v[0] & 0xFFFFu : 0u);
        v[1] = left == 3 ? v[1] & 0xFFFFu : 0u;
    }
    *reinterpret_cast<tile_u32x2 *>(dst) = v;
}

// A block loaded across: piece of row e = element e of the four loaded rows.
__device__ __forceinline__ f32x4 turned(const Piece<false> (&r)[4], int e) { return f32x4{r[0].v[e], r[1].v[e], r[2].v[e], r[3].v[e]}; }
__device__ __forceinline__ tile_u32x2 turned(const Piece<true> (&r)[4], int e)
{
    return tile_u32x2{piece_bits(r[0], e) | (piece_bits(r[1], e) << 16), piece_bits(r[2], e) | (piece_bits(r[3], e) << 16)};
}

// One step: acc[i][j] += As[m0 + 32 i ..][ka + k] Bs[n0 + 32 j ..][ka + k] over BK indices in LDS, of which `left` exist (the others are
// zeros; whole groups of 32 of them are left out).
template <int BK, int RI, int CJ, int PA, int PB>
__device__ __forceinline__ void tile_multiply(const float (*As)[PA], const float (*Bs)[PB], int m0, int n0, int lane,
                                              tile_f32x16 (&acc)[RI][CJ], int left = BK, int ka = 0)
{
#pragma unroll
    for (int ks = 0; ks < BK; ks += 8) {
        if (ks % 32 == 0 && ks > 0 && ks >= left) break;
        f32x4 a[RI], b[CJ];
#pragma unroll
        for (int i = 0; i < RI; ++i) a[i] = *reinterpret_cast<const f32x4 *>(&As[m0 + 32 * i + (lane & 31)][ka + ks + 4 * (lane >> 5)]);
#pragma unroll
        for (int j = 0; j < CJ; ++j) b[j] = *reinterpret_cast<const f32x4 *>(&Bs[n0 + 32 * j + (lane & 31)][ka + ks + 4 * (lane >> 5)]);
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < RI; ++i)
#pragma unroll
                for (int j = 0; j < CJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][c], b[j][c], acc[i][j], 0, 0, 0);
    }
}
template <int BK, int RI, int CJ, int PA, int PB>
__device__ __forceinline__ void tile_multiply(const uint16_t (*As)[PA], const uint16_t (*Bs)[PB], int m0, int n0, int lane,
                                              tile_f32x16 (&acc)[RI][CJ], int left = BK, int ka = 0)
{
#pragma unroll
    for (int ks = 0; ks < BK; ks += 16) {
        if (ks % 32 == 0 && ks > 0 && ks >= left) break;
        tile_u32x4 a[RI], b[CJ];
#pragma unroll
        for (int i = 0; i < RI; ++i) a[i] = *reinterpret_cast<const tile_u32x4 *>(&As[m0 + 32 * i + (lane & 31)][ka + ks + 8 * (lane >> 5)]);
#pragma unroll
        for (int j = 0; j < CJ; ++j) b[j] = *reinterpret_cast<const tile_u32x4 *>(&Bs[n0 + 32 * j + (lane & 31)][ka + ks + 8 * (lane >> 5)]);
#pragma unroll
        for (int i = 0; i < RI; ++i)
#pragma unroll
            for (int j = 0; j < CJ; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(tile_bf16x8, a[i]),
                                                                    __builtin_bit_cast(tile_bf16x8, b[j]), acc[i][j], 0, 0, 0);
    }
}

// momentum_mix4() of a single parameter: the same operations in the same order, so the same bits.
__device__ __forceinline__ void momentum_mix1(float x, float v, float g, float x_peer, float w, float alpha, float mu, float wd,
                                              float &x_new, float &v_new)
{
    v_new = fmaf(wd, x, fmaf(mu, v, g));
    const float h = fmaf(-alpha, v_new, x);
    x_new = fmaf(-w, h - x_peer, h);
}

// ---- fp32 operands as three bfloat16 planes -----------------------------------------------------------------------------
// x = hi + mid + lo, each the rounding of what the ones before leave (8 + 8 + 8 bits).  Exact while x rounds to a finite bfloat16
// and the last part is no subnormal number (true from |x| = 2^-102 on; below, bfloat16 may not have the bits that float has).  Of the
// nine products of two such sums the six largest are taken (mid lo, lo mid and lo lo are left out: at most 2^-24 of the product
// in all), smallest first, each group of sixteen contraction indices with one rounding per product: 6 x 32 cycles where
// v_mfma_f32_32x32x2_f32 takes 8 x 64.  Where the split is not exact the caller does the product again in fp32: `lost` tells it
// of a last part that is subnormal; a value that is not finite does not survive the split (inf - inf) and makes every sum it
// enters a NaN.
constexpr unsigned FP_SUBNORMAL_CLASS = 0x90;                         // of either sign (v_cmp_class_f32)
__device__ __forceinline__ void split2(float x0, float x1, uint32_t (&plane)[3], bool &lost)
{
    plane[0] = pack_bf16x2(x0, x1);
    const float r0 = x0 - __uint_as_float(plane[0] << 16), r1 = x1 - __uint_as_float(plane[0] & 0xFFFF0000u);
    plane[1] = pack_bf16x2(r0, r1);
    const float l0 = r0 - __uint_as_float(plane[1] << 16), l1 = r1 - __uint_as_float(plane[1] & 0xFFFF0000u);
    plane[2] = pack_bf16x2(l0, l1);
    lost |= __builtin_isfpclass(l0, FP_SUBNORMAL_CLASS);
    lost |= __builtin_isfpclass(l1, FP_SUBNORMAL_CLASS);
}

// Four neighbouring k of an operand row into the three planes (plane p of the row starts at dst + p * stride).
__device__ __forceinline__ void put_split(uint16_t *dst, int stride, f32x4 v, bool &lost)
{
    uint32_t a[3], b[3];
    split2(v[0], v[1], a, lost);
    split2(v[2], v[3], b, lost);
#pragma unroll
    for (int p = 0; p < 3; ++p) *reinterpret_cast<tile_u32x2 *>(dst + p * stride) = tile_u32x2{a[p], b[p]};
}
// Two neighbouring k.
__device__ __forceinline__ void put_split(uint16_t *dst, int stride, float x0, float x1, bool &lost)
{
    uint32_t a[3];
    split2(x0, x1, a, lost);
#pragma unroll
    for (int p = 0; p < 3; ++p) *reinterpret_cast<uint32_t *>(dst + p * stride) = a[p];
}
// The piece with only its first `left` elements kept, the others 0.
__device__ __forceinline__ f32x4 first_of(f32x4 v, int left)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = e < left ? v[e] : 0.0f;
    return v;
}

// LDS rows of 32 contraction indices.  Pieces of four k, eight lanes along a row: rows of 64 bytes, their four 16-byte units
// permuted by the row's group of four, so that neither the writes nor the 128-bit reads of sixteen rows meet a bank twice.
__device__ __forceinline__ int split_at(int row, int k) { return row * 32 + ((((k >> 3) ^ (row >> 2)) & 3) << 3) + (k & 7); }
// Pairs of k, sixteen lanes along a row, of columns four apart: rows of 80 bytes do the same for those.
constexpr int SPLIT_PITCH = 40;

// One step of 32 indices; As (split_at) and Bs (SPLIT_PITCH) hold three planes, `sa` and `sb` elements apart.
template <int RI, int CJ>
__device__ __forceinline__ void split_multiply(const uint16_t *As, int sa, const uint16_t *Bs, int sb, int m0, int n0, int lane,
                                               tile_f32x16 (&acc)[RI][CJ])
{
#pragma unroll
    for (int ks = 0; ks < 32; ks += 16) {
        const int k = ks + 8 * (lane >> 5);
        tile_bf16x8 a[RI][3], b[CJ][3];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
#pragma unroll
            for (int i = 0; i < RI; ++i)
                a[i][p] = *reinterpret_cast<const tile_bf16x8 *>(As + split_at(m0 + 32 * i + (lane & 31), k) + p * sa);
#pragma unroll
            for (int j = 0; j < CJ; ++j)
                b[j][p] = *reinterpret_cast<const tile_bf16x8 *>(Bs + (n0 + 32 * j + (lane & 31)) * SPLIT_PITCH + k + p * sb);
        }
        constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int q = 0; q < 6; ++q)
#pragma unroll
            for (int i = 0; i < RI; ++i)
#pragma unroll
                for (int j = 0; j < CJ; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][PA[q]], b[j][PB[q]], acc[i][j], 0, 0, 0);
    }
}

// Row of result register v in a 32 x 32 tile (the column is lane % 32).
__device__ __forceinline__ int tile_row(int lane, int v) { return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); }

template <int RI, int CJ> __device__ __forceinline__ void tile_clear(tile_f32x16 (&acc)[RI][CJ])
{
#pragma unroll
    for (int i = 0; i < RI; ++i)
#pragma unroll
        for (int j = 0; j < CJ; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
}

// ---- operands that cross LDS in steps of 64 bytes of every row (sixteen indices, bfloat16 32), straight from wide loads to the layout of the matrix
// instruction; blocks of 32 columns
constexpr int WF_COLS = 32, WF_PITCH = WF_COLS + 1;
typedef uint32_t tile_u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
template <bool BF> struct WaveOperand { typedef f32x4 piece; typedef float elem; typedef tile_f32x4_any any; };      // piece: 16 bytes of a row
template <> struct WaveOperand<true> { typedef tile_u32x4 piece; typedef uint16_t elem; typedef tile_u32x4_any any; };
template <int RT>
__device__ __forceinline__ void wave_multiply(const f32x4 (&a)[RT], const float *w, tile_f32x16 (&acc)[RT])
{
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < RT; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], w[e], acc[i], 0, 0, 0);
}
template <int RT>
__device__ __forceinline__ void wave_multiply(const tile_u32x4 (&a)[RT], const float *w, tile_f32x16 (&acc)[RT])
{
    const tile_u32x4 b = {pack_bf16x2(w[0], w[1]), pack_bf16x2(w[2], w[3]), pack_bf16x2(w[4], w[5]), pack_bf16x2(w[6], w[7])};
#pragma unroll
    for (int i = 0; i < RT; ++i)
        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(tile_bf16x8, a[i]), __builtin_bit_cast(tile_bf16x8, b), acc[i], 0, 0, 0);
}
// 16-byte unit of piece `at` (0 .. 3) of a row: sixteen rows' pieces, written or read together, then lie in different banks
__device__ __forceinline__ int wave_unit(int row, int at) { return 4 * row + ((at ^ (row >> 2)) & 3); }

// Parameters j .. j + 3 of a worker.  ALIGNED: they do not cross a layout tile.  Otherwise one load where they lie in a tile together, the last four of the tile
// for a lane where they do not, and the wave again by floats.
template <bool ALIGNED> __device__ __forceinline__ f32x4 load4_params(const float *X, int M, int g, int64_t j)
{
    if constexpr (ALIGNED) return load4(X + tiled_offset_quick(M, g, j));
    const int over = max((int)(j & (TILE - 1)) - (TILE - 4), 0);
    f32x4 r = *reinterpret_cast<const tile_f32x4_any *>(X + tiled_offset_quick(M, g, j - over));
    if (__any(over > 0)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = X[tiled_offset_quick(M, g, j + e)];
    }
    return r;
}

}  // namespace netmax
