// Grouped GEMMs of the perceptron gradient on the CDNA4 matrix cores, bf16 operands / fp32 accumulate.
// One group per worker (its own batch times its own weights), so every weight is used by only `batch`
// rows: the kernels are bound by streaming the fp32 master weights from HBM and the gradient back, and
// are organised around that (128-bit loads along the weights' contiguous dimension, conversion to
// bfloat16 on the way into LDS), with v_mfma_f32_32x32x16_bf16 doing the arithmetic.
//
// Lane layout of v_mfma_f32_32x32x16_bf16 (64 lanes, l = lane):
//   A operand: 8 values A[row = l % 32][k = 8 (l / 32) + 0..7]
//   B operand: 8 values B[k = 8 (l / 32) + 0..7][col = l % 32]
//   D:        16 values D[row = 4 (l / 32) + v % 4 + 8 (v / 4)][col = l % 32], v = 0..15
#include <algorithm>
#include "bf16.h"
#include "kernels.h"
#include "layout.h"
#include "softmax_xent.h"
#include "vec.h"

namespace netmax {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int MF_THREADS = 256;      // 4 waves
constexpr int MF_BM = 128, MF_BN = 128;        // weight-gradient and forward tile
// Contraction step BK of the forward and backward-data kernels: operand rows in LDS are BK + 8 bf16 long
// (16-byte aligned, conflict-free 128-bit reads).

__device__ __forceinline__ f32x16 mfma_bf16(u32x4 a, u32x4 b, f32x16 acc)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}

// tiled_offset() with one 32 x 32 -> 64 bit multiply-add: j + (((j >> 11) (M - 1) + i) << 11); needs j < 2^43
__device__ __forceinline__ size_t tiled_offset_fast(int M, int i, int64_t j)
{
    const uint64_t t = (uint64_t)(uint32_t)(j >> TILE_SHIFT) * (uint32_t)(M - 1) + (uint32_t)i;
    return (size_t)j + (size_t)(t << TILE_SHIFT);
}

__device__ __forceinline__ int d_row(int lane, int v) { return 4 * (lane >> 5) + (v & 3) + 8 * (v >> 2); }

// Position (in bf16 elements) of the 16-byte unit u of row n in an operand tile whose units are permuted
// inside each row by the row's 16-block index.  The forward kernel writes its weight tile four rows apart per
// lane (rows 4 nq + e); without the permutation those 8-byte writes meet only four bank groups (8-way
// conflict), with it the conflict is 2-way; reads of whole units stay conflict-free.
__device__ __forceinline__ int swz_unit(int n, int u) { return (u ^ ((n >> 4) & 3)) << 3; }

// One contraction step of the 128 x 128 tile from LDS: As[m][k], Bs[n][k], both k-contiguous.
// SWZ: Bs rows are stored with swz_unit().
template <int BK, bool SWZ>
__device__ __forceinline__ void tile_mma_128(const uint16_t (*As)[BK + 8], const uint16_t (*Bs)[BK + 8], int wm, int wn,
                                             int lane, f32x16 (&acc)[2][2])
{
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
        const int u = 2 * ks + (lane >> 5);
        u32x4 a[2], b[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) a[i] = *reinterpret_cast<const u32x4 *>(&As[64 * wm + 32 * i + (lane & 31)][8 * u]);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int n = 64 * wn + 32 * j + (lane & 31);
            b[j] = *reinterpret_cast<const u32x4 *>(&Bs[n][SWZ ? swz_unit(n, u) : 8 * u]);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = mfma_bf16(a[i], b[j], acc[i][j]);
    }
}

// ---------------------------------------------------------------------------------------------------
// Leaving a 128 x 128 result tile (waves 2 x 2, 64 x 64 each, final fp32 values in acc) as bfloat16 in both
// orientations.  The matrix-instruction layout gives a lane single elements of 32 different rows; written
// straight to memory that is 2-byte and 8-byte stores.  The tile goes through LDS instead, once row-major and
// once transposed, and leaves as whole 256-byte rows in 16-byte pieces.
constexpr int ST_PITCH = 128 + 8;                      // bf16 elements per staged row (272 B)
constexpr int ST_BYTES = 128 * ST_PITCH * 2;

// T[row][col] = bf16(acc) for the whole tile (2-byte LDS writes; lanes 0..31 neighbouring columns)
__device__ __forceinline__ void stage_rows(uint16_t (*T)[ST_PITCH], int wm, int wn, int lane, const f32x16 (&acc)[2][2])
{
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                T[64 * wm + 32 * i + d_row(lane, v)][64 * wn + 32 * j + (lane & 31)] = (uint16_t)bf16_bits(acc[i][j][v]);
}
// T[col][row] = bf16(acc): four consecutive rows per 8-byte LDS write
__device__ __forceinline__ void stage_cols(uint16_t (*T)[ST_PITCH], int wm, int wn, int lane, const f32x16 (&acc)[2][2])
{
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                u32x2 packed;
                packed.x = pack_bf16x2(acc[i][j][4 * q], acc[i][j][4 * q + 1]);
                packed.y = pack_bf16x2(acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
                *reinterpret_cast<u32x2 *>(&T[64 * wn + 32 * j + (lane & 31)][64 * wm + 32 * i + d_row(lane, 4 * q)]) = packed;
            }
}
// 128 staged rows of `len` valid bf16 elements each -> dst + r * stride, 16 bytes per thread and piece;
// only the first n_rows rows are written.
__device__ __forceinline__ void flush_rows(const uint16_t (*T)[ST_PITCH], int t, int n_rows, int len, uint16_t *dst, size_t stride)
{
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int chunk = t + q * MF_THREADS, r = chunk >> 4, c = (chunk & 15) * 8;
        if (r < n_rows && c < len) *reinterpret_cast<u32x4 *>(dst + (size_t)r * stride + c) = *reinterpret_cast<const u32x4 *>(&T[r][c]);
    }
}
// out[(g B + row) ld + c0 + col] and out_t[(g ld + c0 + col) B + row] from acc; all threads of the workgroup.
__device__ __forceinline__ void store_tile_bf16(uint16_t (*T)[ST_PITCH], int wm, int wn, int lane, int t, const f32x16 (&acc)[2][2],
                                                int g, int B, int64_t ld, int64_t c0, uint16_t *out, uint16_t *out_t)
{
    stage_rows(T, wm, wn, lane, acc);
    __syncthreads();
    flush_rows(T, t, B, 128, out + ((size_t)g * B) * ld + c0, (size_t)ld);
    __syncthreads();
    stage_cols(T, wm, wn, lane, acc);
    __syncthreads();
    flush_rows(T, t, 128, B, out_t + ((size_t)g * ld + c0) * B, (size_t)B);
}

// ---------------------------------------------------------------------------------------------------
// Forward: H = relu(A W + b) for one worker and one block of 128 output columns; all batch rows.
// A: gathered bf16 data rows (first layer) or the previous layer's bf16 activations [B][din].
// W: fp32 master weights [din][dout] inside the worker's parameter row (tile layout), read with 128-bit
// loads along dout, transposed 4 x 4 in registers and stored to LDS as bf16 [n][k].
// Output: bf16 activations, row-major [B][dout] and transposed [dout][B].
struct FwdMfmaArgs {
    const uint16_t *feats; const int64_t *row0; const int32_t *idx;   // first layer
    const uint16_t *a_prev;                                           // later layers: [M][B][din]
    const float *X; int64_t woff; int M, B; int64_t din, dout; int relu;
    uint16_t *out, *out_t;
};

template <bool FIRST, int BK>
__device__ __forceinline__ void fwd_mfma_body(const FwdMfmaArgs &p)
{
    constexpr int PITCH = BK + 8;
    constexpr int A_CH = MF_BM * BK / 8 / MF_THREADS;      // 16-byte chunks of A per thread and step
    constexpr int CPR = BK / 8;                            // chunks per A row
    constexpr int W_BL = BK / 32;                          // 4 (k) x 4 (n) blocks of W per thread and step
    // operand tiles during the contraction, the staging tile of the result afterwards
    constexpr int OPERAND_BYTES = (MF_BM + MF_BN) * PITCH * 2;
    __shared__ __attribute__((aligned(16))) unsigned char smem[OPERAND_BYTES > ST_BYTES ? OPERAND_BYTES : ST_BYTES];
    uint16_t (*As)[PITCH] = reinterpret_cast<uint16_t (*)[PITCH]>(smem);
    uint16_t (*Bs)[PITCH] = reinterpret_cast<uint16_t (*)[PITCH]>(smem + MF_BM * PITCH * 2);
    uint16_t (*T)[ST_PITCH] = reinterpret_cast<uint16_t (*)[ST_PITCH]>(smem);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
    int g;
    unsigned nblk;
    if (!decode_group(blockIdx.x, (unsigned)(p.dout / MF_BN), p.M, g, nblk)) return;
    const int64_t n0 = (int64_t)nblk * MF_BN;

    const uint16_t *a_src[A_CH];
    int a_row[A_CH], a_k[A_CH];
#pragma unroll
    for (int c = 0; c < A_CH; ++c) {
        const int chunk = t + c * MF_THREADS;
        a_row[c] = chunk / CPR;
        a_k[c] = (chunk % CPR) * 8;
        if (a_row[c] < p.B) {
            const int64_t row = FIRST ? p.row0[g] + p.idx[(size_t)g * p.B + a_row[c]] : (int64_t)g * p.B + a_row[c];
            a_src[c] = (FIRST ? p.feats : p.a_prev) + row * p.din + a_k[c];
        } else {
            a_src[c] = nullptr;
        }
    }
    // W: 4 (k) x 4 (n) blocks per thread.  One contraction step moves every load by BK rows of W =
    // BK * dout columns of the parameter row, a whole number of layout tiles (dout is a multiple of 128),
    // so the pointers advance by a constant.
    const int kg = t >> 5, nq = t & 31;
    const float *w_src[W_BL][4];
#pragma unroll
    for (int q = 0; q < W_BL; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            w_src[q][r] = p.X + tiled_offset(p.M, g, p.woff + n0 + 4 * nq + (int64_t)(4 * (kg + 8 * q) + r) * p.dout);
    const size_t w_step = (size_t)BK * (size_t)p.dout * (size_t)p.M;

    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    u32x4 ra[A_CH];
    f32x4_t rw[W_BL][4];
    auto fetch = [&](int64_t k0) {
#pragma unroll
        for (int c = 0; c < A_CH; ++c)
            ra[c] = a_src[c] ? *reinterpret_cast<const u32x4 *>(a_src[c] + k0) : (u32x4){0u, 0u, 0u, 0u};
#pragma unroll
        for (int q = 0; q < W_BL; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                rw[q][r] = *reinterpret_cast<const f32x4_t *>(w_src[q][r]);
                w_src[q][r] += w_step;
            }
    };
    auto stash = [&]() {
#pragma unroll
        for (int c = 0; c < A_CH; ++c) *reinterpret_cast<u32x4 *>(&As[a_row[c]][a_k[c]]) = ra[c];
#pragma unroll
        for (int q = 0; q < W_BL; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) {   // column n = 4 nq + e gets its four consecutive k
                u32x2 packed;
                packed.x = pack_bf16x2(rw[q][0][e], rw[q][1][e]);
                packed.y = pack_bf16x2(rw[q][2][e], rw[q][3][e]);
                const int n = 4 * nq + e, k4 = kg + 8 * q;       // k4: index of the group of four k
                *reinterpret_cast<u32x2 *>(&Bs[n][swz_unit(n, k4 >> 1) + 4 * (k4 & 1)]) = packed;
            }
    };

    fetch(0);
    for (int64_t k0 = 0; k0 < p.din; k0 += BK) {
        __syncthreads();            // the previous step's reads of LDS are done
        stash();
        __syncthreads();
        if (k0 + BK < p.din) fetch(k0 + BK);   // overlaps with the matrix instructions below
        tile_mma_128<BK, true>(As, Bs, wm, wn, lane, acc);
    }

    // epilogue: bias, ReLU, then bf16 in both layouts through LDS
    const float *bias = p.X;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int64_t col = n0 + 64 * wn + 32 * j + (lane & 31);
        const float bcol = bias[tiled_offset(p.M, g, p.woff + p.din * p.dout + col)];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float z = acc[i][j][v] + bcol;
                acc[i][j][v] = (p.relu && !(z > 0.0f)) ? 0.0f : z;
            }
    }
    __syncthreads();                 // the last step's reads of the operand tiles are done
    store_tile_bf16(T, wm, wn, lane, t, acc, g, p.B, p.dout, n0, p.out, p.out_t);
}

template <bool FIRST>
__global__ void __launch_bounds__(MF_THREADS) __attribute__((amdgpu_waves_per_eu(4, 4))) fwd_mfma_kernel(FwdMfmaArgs p)
{
    fwd_mfma_body<FIRST, 32>(p);
}
// ---------------------------------------------------------------------------------------------------
// Shared tail of the backward-data kernels.  The workgroup holds dA for all batch rows (waves 2 x 2, each
// 64 rows x 64 columns in acc[i][j]) of `c0 .. c0 + 127`: applies the ReLU mask of the layer's input, writes
// the error as bf16 [B][din] and transposed [din][B] (fp32 [B][din] too if out_f32 is given) and, because all
// rows of a column are here, the column sums = the bias gradient of the layer below, in a fixed order.
struct DgradOut {
    const uint16_t *act;          // bf16 activations of this layer's input [M][B][din] (ReLU mask)
    float *out_f32; uint16_t *out, *out_t;
    float *G; int64_t boff;       // bias gradient of the layer below: G[tile layout, boff + column]
};

// BURST: how many of the eight pieces of the activation tile a thread requests at a time (0: see below).
template <int BURST>
__device__ __forceinline__ void dgrad_tail(const DgradOut &o, int M, int g, int B, int64_t din, int64_t c0, int wm, int wn,
                                           int lane, int t, f32x16 (&acc)[2][2], uint16_t (*T)[ST_PITCH], float (*red)[2][64])
{
    const int wave = 2 * wm + wn;
    // the activations under the tile (ReLU mask) come in as whole rows
    // (all eight requested before the first is stored, rows past the batch clamped: a load under a bounds test is
    // waited for where the branches join, one round trip per load)
    if constexpr (BURST == 0) {
        // one piece at a time, each under its bounds test: for the kernel whose registers are all taken by the tile
        // (requesting the pieces together made it spill more and run 4 % slower)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int chunk = t + q * MF_THREADS, r = chunk >> 4, c = (chunk & 15) * 8;
            if (r < B) *reinterpret_cast<u32x4 *>(&T[r][c]) = *reinterpret_cast<const u32x4 *>(o.act + ((size_t)g * B + r) * din + c0 + c);
        }
    } else {
#pragma unroll
    for (int q0 = 0; q0 < 8; q0 += (BURST > 0 ? BURST : 8)) {
        u32x4 mask_rows[BURST > 0 ? BURST : 1];
#pragma unroll
        for (int q = 0; q < BURST; ++q) {
            const int chunk = t + (q0 + q) * MF_THREADS, r = chunk >> 4, c = (chunk & 15) * 8;
            mask_rows[q] = *reinterpret_cast<const u32x4 *>(o.act + ((size_t)g * B + (r < B ? r : B - 1)) * din + c0 + c);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < BURST; ++q) {
            const int chunk = t + (q0 + q) * MF_THREADS, r = chunk >> 4, c = (chunk & 15) * 8;
            if (r < B) *reinterpret_cast<u32x4 *>(&T[r][c]) = mask_rows[q];
        }
    }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int cl = 64 * wn + 32 * j + (lane & 31);
        float csum = 0.0f;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = 64 * wm + 32 * i + d_row(lane, v);
                const float d = (row < B && bf16_positive(T[row][cl])) ? acc[i][j][v] : 0.0f;
                acc[i][j][v] = d;
                csum += d;
            }
        red[wave][j][lane] = csum;
    }
    if (o.out_f32) {                 // only when the layer below runs on the general fp32-input kernels
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = 64 * wm + 32 * i + d_row(lane, v);
                    if (row < B) o.out_f32[((size_t)g * B + row) * din + c0 + 64 * wn + 32 * j + (lane & 31)] = acc[i][j][v];
                }
    }
    __syncthreads();                 // every mask is read before the tile is overwritten
    store_tile_bf16(T, wm, wn, lane, t, acc, g, B, din, c0, o.out, o.out_t);
    if (t < 128) {                   // red[] was complete before the barriers above
        const int cwn = t >> 6, cj = (t >> 5) & 1, cl = t & 31;
        float sum = 0.0f;
#pragma unroll
        for (int cwm = 0; cwm < 2; ++cwm)
#pragma unroll
            for (int half = 0; half < 2; ++half) sum += red[2 * cwm + cwn][cj][cl + 32 * half];
        o.G[tiled_offset(M, g, o.boff + c0 + t)] = sum;
    }
}

// Backward through a layer: dA = (dZ W^T) * [A > 0] for one worker, all batch rows and 128 input features
// (the output columns).  dZ: bf16 [B][dout]; W rows are contiguous along the contraction index, so they go
// to LDS untransposed (128-byte row pieces per step).
struct DgradMfmaArgs {
    const uint16_t *dz; const float *X; int64_t woff; int M, B; int64_t din, dout;
    DgradOut o;
};

template <int BK>
__device__ __forceinline__ void dgrad_mfma_body(const DgradMfmaArgs &p)
{
    constexpr int PITCH = BK + 8;
    constexpr int A_CH = MF_BM * BK / 8 / MF_THREADS;      // 16-byte chunks of dZ per thread and step
    constexpr int CPR = BK / 8;
    constexpr int W_CH = MF_BN * BK / 4 / MF_THREADS;      // 16-byte chunks of W per thread and step
    constexpr int WPR = BK / 4;
    constexpr int OPERAND_BYTES = (MF_BM + MF_BN) * PITCH * 2;
    __shared__ __attribute__((aligned(16))) unsigned char smem[OPERAND_BYTES > ST_BYTES ? OPERAND_BYTES : ST_BYTES];
    uint16_t (*As)[PITCH] = reinterpret_cast<uint16_t (*)[PITCH]>(smem);
    uint16_t (*Bs)[PITCH] = reinterpret_cast<uint16_t (*)[PITCH]>(smem + MF_BM * PITCH * 2);
    uint16_t (*T)[ST_PITCH] = reinterpret_cast<uint16_t (*)[ST_PITCH]>(smem);
    __shared__ float red[4][2][64];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
    int g;
    unsigned cblk;
    if (!decode_group(blockIdx.x, (unsigned)(p.din / MF_BN), p.M, g, cblk)) return;
    const int64_t c0 = (int64_t)cblk * MF_BN;     // first input feature (output column) of this block

    const uint16_t *a_src[A_CH];
    int a_row[A_CH], a_k[A_CH];
#pragma unroll
    for (int c = 0; c < A_CH; ++c) {
        const int chunk = t + c * MF_THREADS;
        a_row[c] = chunk / CPR;
        a_k[c] = (chunk % CPR) * 8;
        a_src[c] = a_row[c] < p.B ? p.dz + ((size_t)g * p.B + a_row[c]) * p.dout + a_k[c] : nullptr;
    }
    // W: 16-byte chunks, feature row = chunk / WPR, k offset 4 * (chunk % WPR)
    int w_row[W_CH], w_k[W_CH];
    int64_t w_col[W_CH];
#pragma unroll
    for (int r = 0; r < W_CH; ++r) {
        const int chunk = t + r * MF_THREADS;
        w_row[r] = chunk / WPR;
        w_k[r] = 4 * (chunk % WPR);
        w_col[r] = p.woff + (c0 + w_row[r]) * p.dout + w_k[r];
    }
    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    u32x4 ra[A_CH];
    f32x4_t rw[W_CH];
    auto fetch = [&](int64_t k0) {
#pragma unroll
        for (int c = 0; c < A_CH; ++c)
            ra[c] = a_src[c] ? *reinterpret_cast<const u32x4 *>(a_src[c] + k0) : (u32x4){0u, 0u, 0u, 0u};
#pragma unroll
        for (int r = 0; r < W_CH; ++r) rw[r] = *reinterpret_cast<const f32x4_t *>(p.X + tiled_offset(p.M, g, w_col[r] + k0));
    };
    auto stash = [&]() {
#pragma unroll
        for (int c = 0; c < A_CH; ++c) *reinterpret_cast<u32x4 *>(&As[a_row[c]][a_k[c]]) = ra[c];
#pragma unroll
        for (int r = 0; r < W_CH; ++r) {
            u32x2 packed;
            packed.x = pack_bf16x2(rw[r][0], rw[r][1]);
            packed.y = pack_bf16x2(rw[r][2], rw[r][3]);
            *reinterpret_cast<u32x2 *>(&Bs[w_row[r]][w_k[r]]) = packed;
        }
    };

    // The contraction starts at a different offset in every workgroup and wraps around: at any moment the
    // workgroups then read different parts of their weight rows, which spreads the requests over the memory
    // channels (all rows of W start at multiples of 4 dout bytes, the same offset in every row would meet
    // the same few channels).
    const int n_steps = (int)(p.dout / BK);
    const int shift = (int)((cblk * 5u + (unsigned)g * 3u) % (unsigned)n_steps);
    auto k_of = [&](int s) { int q = s + shift; if (q >= n_steps) q -= n_steps; return (int64_t)q * BK; };
    fetch(k_of(0));
    for (int s = 0; s < n_steps; ++s) {
        __syncthreads();
        stash();
        __syncthreads();
        if (s + 1 < n_steps) fetch(k_of(s + 1));
        tile_mma_128<BK, false>(As, Bs, wm, wn, lane, acc);
    }
    __syncthreads();                 // the last step's reads of the operand tiles are done
    dgrad_tail<0>(p.o, p.M, g, p.B, p.din, c0, wm, wn, lane, t, acc, T, red);
}

__global__ void __launch_bounds__(MF_THREADS) __attribute__((amdgpu_waves_per_eu(4, 4))) dgrad_mfma_kernel(DgradMfmaArgs p)
{
    dgrad_mfma_body<32>(p);
}

// ---------------------------------------------------------------------------------------------------
// Weight gradient: dW = A^T dZ for one worker and a strip of rows of W.  The contraction runs over
// the batch (<= 128), so whole operand blocks fit in LDS: the strip's A^T block [rows][B] is loaded once,
// then the workgroup walks along the strip in blocks of 128 columns; the dZ^T block of the next step is
// fetched into registers while the matrix instructions of the current one run.  Both operands are the
// transposed bf16 copies (batch-contiguous), read with coalesced 128-bit loads.  The fp32 product leaves
// straight from the accumulators as 128-byte row pieces (non-temporal) into the gradient row.
struct WgradMfmaArgs {
    const uint16_t *a_t, *dz_t; int M, B; int64_t din, dout, woff; float *G;
    const uint16_t *feats; const int64_t *row0; const int32_t *idx;      // first layer: A^T is gathered from the data rows
};

constexpr int WG_PITCH = 128 + 8;            // bf16 elements per operand row in LDS (272 B)

// The strip's A^T block [ROWS][B] into LDS.  Layers above the first read it from the transposed bf16 activations
// (batch-contiguous rows, whole 16-byte chunks).  The first layer (feats != nullptr) takes it from the data rows of
// the worker's batch themselves: every batch row holds the strip's ROWS features as ROWS * 2 contiguous bytes; a
// thread loads eight of them and scatters them into eight rows of the block.  Neighbouring lanes take neighbouring
// batch rows (the same feature chunk): their 2-byte LDS writes fall into one row of the block, and the eight chunks
// of a data row's line are fetched from memory once and hit in the cache afterwards.
template <int ROWS>
__device__ __forceinline__ void load_at_block(uint16_t (*At)[WG_PITCH], int t, int g, int B, int64_t din, int64_t r0,
                                              const uint16_t *a_t, const uint16_t *feats, const int64_t *row0,
                                              const int32_t *idx)
{
    // No load sits under a branch (one under a bounds test is waited for where the branches join: a round trip per
    // load instead of one for all): indices past the end are clamped and what they load is not stored.
    if (feats) {
        constexpr int KC = ROWS / 8;                             // 16-byte chunks of a batch row inside the strip
        constexpr int N = KC * 128 / MF_THREADS;                 // chunks per thread at the largest batch
        const int n = KC * B;
        int kcs[N], bs[N];
        int32_t rows[N];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const int c = t + q * MF_THREADS, cc = c < n ? c : n - 1;
            kcs[q] = cc / B;
            bs[q] = cc - kcs[q] * B;
            rows[q] = idx[(size_t)g * B + bs[q]];                // all batch-row numbers first, then all rows
        }
        const uint16_t *base = feats + (size_t)row0[g] * din + r0;
        u32x4 v[N];
#pragma unroll
        for (int q = 0; q < N; ++q) v[q] = *reinterpret_cast<const u32x4 *>(base + (size_t)rows[q] * din + 8 * kcs[q]);
#pragma unroll
        for (int q = 0; q < N; ++q) {
            if (t + q * MF_THREADS < n) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    At[8 * kcs[q] + 2 * e][bs[q]] = (uint16_t)(v[q][e] & 0xFFFFu);
                    At[8 * kcs[q] + 2 * e + 1][bs[q]] = (uint16_t)(v[q][e] >> 16);
                }
            }
        }
        return;
    }
    const int chunks_per_row = B >> 3;
    const uint16_t *a_src = a_t + ((size_t)g * din + r0) * B;
    constexpr int N = ROWS * 16 / MF_THREADS;                    // chunks per thread at the largest batch
    const int n = ROWS * chunks_per_row;
    int rws[N], cols[N];
    u32x4 v[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const int c = t + q * MF_THREADS, cc = c < n ? c : n - 1;
        rws[q] = cc / chunks_per_row;
        cols[q] = (cc - rws[q] * chunks_per_row) * 8;
        v[q] = *reinterpret_cast<const u32x4 *>(a_src + (size_t)rws[q] * B + cols[q]);
    }
#pragma unroll
    for (int q = 0; q < N; ++q)
        if (t + q * MF_THREADS < n) *reinterpret_cast<u32x4 *>(&At[rws[q]][cols[q]]) = v[q];
}

// STRIP: rows of W per workgroup (128 or 64), BN: columns per block step (128 or 64); waves 2 x 2, each
// STRIP / 2 rows x BN / 2 columns.
constexpr int WG_STAGE_PITCH = 132;                  // floats per row of the staged output block
template <int STRIP, int BN>
__device__ __forceinline__ void wgrad_mfma_body(const WgradMfmaArgs &p)
{
    constexpr int RI = STRIP / 64;                               // 32-row tiles per wave
    constexpr int CJ = BN / 64;                                  // 32-column tiles per wave
    constexpr int Z_CHUNKS = BN * 128 / 8 / MF_THREADS;
    __shared__ __attribute__((aligned(16))) uint16_t At[STRIP][WG_PITCH];
    __shared__ __attribute__((aligned(16))) uint16_t Zt[BN][WG_PITCH];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
    const unsigned nx = (unsigned)(p.dout / BN), ny = (unsigned)(p.din / STRIP);
    int g;
    unsigned strip;
    if (!decode_group(blockIdx.x, ny, p.M, g, strip)) return;
    const int64_t r0 = (int64_t)strip * STRIP;
    const int chunks_per_row = p.B >> 3;                        // 16-byte chunks; at most 16
    const uint16_t *z_src = p.dz_t + (size_t)g * p.dout * p.B;
    load_at_block<STRIP>(At, t, g, p.B, p.din, r0, p.a_t, p.feats, p.row0, p.idx);
    int c_row[Z_CHUNKS], c_col[Z_CHUNKS];
#pragma unroll
    for (int q = 0; q < Z_CHUNKS; ++q) {
        const int c = t + q * MF_THREADS;
        c_row[q] = c / chunks_per_row;
        c_col[q] = (c - c_row[q] * chunks_per_row) * 8;
    }
    const int n_chunks = BN * chunks_per_row;
    const int64_t lane_col = p.woff + (r0 + 32 * RI * wm + 4 * (lane >> 5)) * p.dout + 32 * CJ * wn + (lane & 31);
    u32x4 rz[Z_CHUNKS];
    auto fetch_z = [&](unsigned nb) {
#pragma unroll
        for (int q = 0; q < Z_CHUNKS; ++q)
            if (t + q * MF_THREADS < n_chunks)
                rz[q] = *reinterpret_cast<const u32x4 *>(z_src + ((size_t)nb * BN + c_row[q]) * p.B + c_col[q]);
    };
    fetch_z(0);

    for (unsigned nb = 0; nb < nx; ++nb) {
        __syncthreads();                                        // the previous block's reads of Zt are done
#pragma unroll
        for (int q = 0; q < Z_CHUNKS; ++q)
            if (t + q * MF_THREADS < n_chunks) *reinterpret_cast<u32x4 *>(&Zt[c_row[q]][c_col[q]]) = rz[q];
        __syncthreads();
        if (nb + 1 < nx) fetch_z(nb + 1);

        f32x16 acc[RI][CJ];
#pragma unroll
        for (int i = 0; i < RI; ++i)
#pragma unroll
            for (int j = 0; j < CJ; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
        for (int b0 = 0; b0 < p.B; b0 += 16) {
            const int kofs = b0 + 8 * (lane >> 5);
            u32x4 a[RI], b[CJ];
#pragma unroll
            for (int i = 0; i < RI; ++i) a[i] = *reinterpret_cast<const u32x4 *>(&At[32 * RI * wm + 32 * i + (lane & 31)][kofs]);
#pragma unroll
            for (int j = 0; j < CJ; ++j) b[j] = *reinterpret_cast<const u32x4 *>(&Zt[32 * CJ * wn + 32 * j + (lane & 31)][kofs]);
#pragma unroll
            for (int i = 0; i < RI; ++i)
#pragma unroll
                for (int j = 0; j < CJ; ++j) acc[i][j] = mfma_bf16(a[i], b[j], acc[i][j]);
        }
        if constexpr (STRIP == 64 && BN == 128) {
            // The block goes through LDS (the space of the dZ^T block, which every wave has finished reading) and
            // leaves as whole 512-byte row pieces, 16 bytes per lane, in one burst of stores per workgroup (measured:
            // 15 us less per iteration of the 3072-1024-1024 perceptron than 4-byte stores straight from the accumulators).
            float (*T)[WG_STAGE_PITCH] = reinterpret_cast<float (*)[WG_STAGE_PITCH]>(&Zt[0][0]);
            static_assert(sizeof(float) * 64 * WG_STAGE_PITCH <= sizeof(uint16_t) * BN * WG_PITCH, "the staged block fits the operand block");
            __syncthreads();
#pragma unroll
            for (int j = 0; j < CJ; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) T[32 * wm + d_row(lane, v)][64 * wn + 32 * j + (lane & 31)] = acc[0][j][v];
            __syncthreads();
            const int cq = (t & 31) * 4, r_in = t >> 5;              // 32 lanes along the 128 columns, 8 rows per pass
#pragma unroll
            for (int pass = 0; pass < 8; ++pass) {
                const int row = pass * 8 + r_in;
                const int64_t jj = p.woff + (r0 + row) * p.dout + (int64_t)nb * BN + cq;
                __builtin_nontemporal_store(*reinterpret_cast<const f32x4_t *>(&T[row][cq]),
                                            reinterpret_cast<f32x4_t *>(p.G + tiled_offset_fast(p.M, g, jj)));
            }
        } else {
        // column index inside the parameter row = lane part (fixed) + a part that is the same for the whole wave
#pragma unroll
        for (int i = 0; i < RI; ++i)
#pragma unroll
            for (int j = 0; j < CJ; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int64_t uni = (int64_t)(32 * i + (v & 3) + 8 * (v >> 2)) * p.dout + (int64_t)nb * BN + 32 * j;
                    __builtin_nontemporal_store(acc[i][j][v], p.G + tiled_offset_fast(p.M, g, lane_col + uni));
                }
        }
    }
}

// 64-row strips: 51 KB of LDS, three workgroups per compute unit, whose arithmetic and store phases overlap
// better than those of two workgroups with 128-row strips (measured: 13 % less time for both layers of the
// 3072-1024-1024 perceptron).
constexpr int WG_STRIP = 64;
__global__ void __launch_bounds__(MF_THREADS) __attribute__((amdgpu_waves_per_eu(3, 3))) wgrad_mfma_kernel(WgradMfmaArgs p)
{
    wgrad_mfma_body<WG_STRIP, 128>(p);
}

// ---------------------------------------------------------------------------------------------------
// Weight gradient with the second-step update applied in place of the store, or beside it (KEEP_G): one workgroup = one worker and
// 128 columns of W, along which it walks in strips of 32 rows.  The product dW = A^T dZ of a strip is computed as above (the same
// steps in the same order), turned through LDS into rows, and every thread then updates four neighbouring parameters per row:
// v' = mu v + dW + wd x, h = x - alpha v', x' = h - w (h - x_peer) (Eq. (c0), (c1)) with 128-bit loads and stores.
// Workgroups are ordered block by block: all M workers of a block run side by side on one XCD (as the mix kernel
// orders its tiles), so the strip a worker pulls from its peer is in that XCD's L2.
// Bound by memory: x, v, x', v' and the operands that are read again for every block.  The dZ^T block stays in LDS for the whole walk, A^T's
// next strip and x, v and the peer's x travel while the present one is multiplied.  3072-1024 and 1024-1024, batch 128, 48
// workers: 464 and 144 us (5.2 and 5.6 TB/s of the 16 bytes a parameter; 4.0 GB with operands and peers across the fabric); with one block of 64 x 128 per workgroup, its operands
// loaded, multiplied and then x, v and the peer's x asked for, 725 us together.  Without products and operands it would take 460 and 133,
// whatever the number of workgroups per compute unit (one to three) and the height of a strip (32, 64, 128 rows: the same within 3 %).
struct WgradMixArgs {
    const uint16_t *a_t, *dz_t; int M, B; int64_t din, dout, woff; unsigned walk, apart; float *G;
    MixArgs mix;
    const uint16_t *feats; const int64_t *row0; const int32_t *idx;      // first layer: A^T is gathered from the data rows
};
constexpr int WM_ROWS = 32, WM_COLS = 128;
constexpr int WM_TILE_PITCH = WM_COLS + 4;           // floats per staged row

template <bool GATHERED, bool KEEP_G>
__global__ void __launch_bounds__(MF_THREADS) __attribute__((amdgpu_waves_per_eu(3, 3))) wgrad_mix_mfma_kernel(WgradMixArgs p)
{
    constexpr int STAGE = WM_ROWS * WM_TILE_PITCH * 4;
    static_assert(STAGE >= WM_ROWS * WG_PITCH * 2, "A's strip lies where the staged block will");
    __shared__ __attribute__((aligned(16))) uint16_t Zt[WM_COLS][WG_PITCH];
    __shared__ __attribute__((aligned(16))) unsigned char smem[STAGE];
    uint16_t (*At)[WG_PITCH] = reinterpret_cast<uint16_t (*)[WG_PITCH]>(smem);
    float (*T)[WM_TILE_PITCH] = reinterpret_cast<float (*)[WM_TILE_PITCH]>(smem);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    // workgroup id -> (columns and strips, worker): ids are dealt round-robin to the XCDs; a block's workers are consecutive slots
    const unsigned nbx = (unsigned)(p.dout / WM_COLS), strips = (unsigned)(p.din / WM_ROWS), walks = (strips + p.walk - 1) / p.walk;
    const unsigned xcd = blockIdx.x % MF_XCD, slot = blockIdx.x / MF_XCD;
    const unsigned blk = (slot / (unsigned)p.M) * MF_XCD + xcd;
    const int g = (int)(slot % (unsigned)p.M);
    if (blk >= nbx * walks) return;
    const unsigned first = blk / nbx * p.walk, n = min(p.walk, strips - first);
    const int64_t r0 = (int64_t)first * WM_ROWS, n0 = (int64_t)(blk % nbx) * WM_COLS;
    const int chunks_per_row = p.B >> 3;
    const uint16_t *z_src = p.dz_t + ((size_t)g * p.dout + n0) * p.B;

    // A's strip: two pieces of eight elements per thread, of a row of A^T, or of a data row (neighbouring lanes then take neighbouring
    // batch rows).  Pieces past the end are read from the last one's place and not stored.
    constexpr int AN = WM_ROWS * 16 / MF_THREADS;
    const int a_chunks = WM_ROWS * chunks_per_row;
    const uint16_t *a_src[AN];
    int a_row[AN], a_col[AN];
#pragma unroll
    for (int q = 0; q < AN; ++q) {
        const int c = min(t + q * MF_THREADS, a_chunks - 1);
        if constexpr (GATHERED) {
            a_row[q] = c / p.B * 8;
            a_col[q] = c % p.B;
            a_src[q] = p.feats + (size_t)(p.row0[g] + p.idx[(size_t)g * p.B + a_col[q]]) * p.din + r0 + a_row[q];
        } else {
            a_row[q] = c / chunks_per_row;
            a_col[q] = c % chunks_per_row * 8;
            a_src[q] = p.a_t + ((size_t)g * p.din + r0 + a_row[q]) * p.B + a_col[q];
        }
    }
    const size_t a_step = GATHERED ? WM_ROWS : (size_t)WM_ROWS * p.B;
    // A strip of data rows is half of their 128-byte lines: two strips are asked for together (walks of more than one strip have an
    // even number of them), the second one stays in registers.  us per iteration of 3072-1024-1024-10, batch 128, each strip for itself
    // and two together: calls of eight iterations, 48 workers 907 and 891, of four, 128 workers 2435 and 2392; calls of one, 48 workers 900 and 892, 64 workers 1226 and
    // 1231, 128 workers 2469 and 2410.
    u32x4 ra[AN], rs[GATHERED ? AN : 1];
    const bool pairs = GATHERED && p.walk > 1;
    auto fetch_a = [&](unsigned k) {
#pragma unroll
        for (int q = 0; q < AN; ++q) ra[q] = *reinterpret_cast<const u32x4 *>(a_src[q] + k * a_step);
        if constexpr (GATHERED)
            if (pairs) {
#pragma unroll
                for (int q = 0; q < AN; ++q) rs[q] = *reinterpret_cast<const u32x4 *>(a_src[q] + (k + 1) * a_step);
            }
    };
    unsigned at = p.apart ? (unsigned)g / p.apart % n & ~1u : 0;     // where this worker's walk begins; it goes on from the first strip
    auto stash_a = [&]() {
#pragma unroll
        for (int q = 0; q < AN; ++q) {
            if (t + q * MF_THREADS >= a_chunks) continue;
            if constexpr (GATHERED) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    At[a_row[q] + 2 * e][a_col[q]] = (uint16_t)(ra[q][e] & 0xFFFFu);
                    At[a_row[q] + 2 * e + 1][a_col[q]] = (uint16_t)(ra[q][e] >> 16);
                }
            } else {
                *reinterpret_cast<u32x4 *>(&At[a_row[q]][a_col[q]]) = ra[q];
            }
        }
    };
    fetch_a(at);
    {
        constexpr int ZN = WM_COLS * 16 / MF_THREADS;
        const int z_chunks = WM_COLS * chunks_per_row;
        u32x4 rz[ZN];
#pragma unroll
        for (int q = 0; q < ZN; ++q) {
            const int c = min(t + q * MF_THREADS, z_chunks - 1);
            rz[q] = *reinterpret_cast<const u32x4 *>(z_src + 8 * (size_t)c);
        }
#pragma unroll
        for (int q = 0; q < ZN; ++q) {
            const int c = t + q * MF_THREADS;
            if (c < z_chunks) *reinterpret_cast<u32x4 *>(&Zt[c / chunks_per_row][c % chunks_per_row * 8]) = rz[q];
        }
    }
    const MixArgs &mx = p.mix;
    int m = mx.peer[g];
    if ((unsigned)m >= (unsigned)p.M) m = g;             // an index outside [0, M) is treated as a self draw
    const float wi = mx.w[(size_t)g * p.M + m];
    const int64_t peer_shift = ((int64_t)m - g) * TILE;
    constexpr int PASSES = WM_ROWS / 8;
    const int cq = (t & 31) * 4, r_in = t >> 5;          // 32 lanes along the 128 columns, 8 rows per pass
    const int64_t jb = p.woff + (r0 + r_in) * p.dout + n0 + cq;

    for (unsigned s = 0; s < n; ++s) {
        size_t own[PASSES];
        f32x4_t x[PASSES], v[PASSES], xp[PASSES];
        const int64_t j0 = jb + (int64_t)at * WM_ROWS * p.dout;
        stash_a();
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PASSES; ++u) {
            own[u] = tiled_offset_fast(p.M, g, j0 + (int64_t)(8 * u) * p.dout);
            x[u] = *reinterpret_cast<const f32x4_t *>(mx.Xcur + own[u]);
            v[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t *>(mx.V + own[u]));
        }
#pragma unroll
        for (int u = 0; u < PASSES; ++u) xp[u] = *reinterpret_cast<const f32x4_t *>(mx.Xcur + own[u] + peer_shift);
        at = at + 1 < n ? at + 1 : 0;
        if (s + 1 < n) {
            if (!pairs || at % 2 == 0) fetch_a(at);
            else if constexpr (GATHERED) {
#pragma unroll
                for (int q = 0; q < AN; ++q) ra[q] = rs[q];
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        f32x16 acc;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
        for (int b0 = 0; b0 < p.B; b0 += 16) {
            const int kofs = b0 + 8 * (lane >> 5);
            const u32x4 a = *reinterpret_cast<const u32x4 *>(&At[lane & 31][kofs]);
            acc = mfma_bf16(a, *reinterpret_cast<const u32x4 *>(&Zt[32 * wave + (lane & 31)][kofs]), acc);
        }
        __syncthreads();                                  // the strip is read; its space becomes the staged block
#pragma unroll
        for (int e = 0; e < 16; ++e) T[d_row(lane, e)][32 * wave + (lane & 31)] = acc[e];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PASSES; ++u) {
            const f32x4_t gr = *reinterpret_cast<const f32x4_t *>(&T[8 * u + r_in][cq]);
            f32x4_t xn, vn;
            momentum_mix4(x[u], v[u], gr, xp[u], wi, mx.alpha, mx.mu, mx.wd, xn, vn);
            if constexpr (KEEP_G) __builtin_nontemporal_store(gr, reinterpret_cast<f32x4_t *>(p.G + own[u]));
            __builtin_nontemporal_store(xn, reinterpret_cast<f32x4_t *>(mx.Xnext + own[u]));
            __builtin_nontemporal_store(vn, reinterpret_cast<f32x4_t *>(mx.V + own[u]));
        }
        __syncthreads();                                  // the staged block is read; the next strip takes its place
    }
}

// ---------------------------------------------------------------------------------------------------
// Last layer with few classes (dout <= 32): the same three products with the class dimension padded to
// one 32-wide matrix-instruction tile.  The weight matrix is tiny (din x dout), the work is bound by
// reading / writing the [B][din] activations and errors.

// logits = A W + b.  One workgroup per worker; W^T goes to LDS as bf16 [32][din], each wave takes 32
// batch rows.  One compute unit pulls a worker's 256 KB of activations (1024 features, batch 128): bound by how much of them is on
// the way.  A wave asks for four pieces of 64 features ahead, the first ones before W is turned, as lines of 128 bytes by eight lanes
// (a lane per row asks for 64 lines an instruction), and turns them to the matrix instruction's layout in LDS of its own.  The logits
// stay in LDS for the softmax, whose chain of loads from memory was the other half.  us, before, with the pieces, and with both:
// 1024-10, batch 128, 48 workers 26.5, 22.9, 18.7; 2048-10, 4 workers 33.6, 25.7, 23.0; 128-30, batch 96, 8 workers 22.1, 21.7, 12.2; 640-10,
// batch 32, 61 workers 16.7, 16.2, 14.2.  From 256 workers on, what counts as well is how many workgroups a compute unit holds: W^T has rows of the real classes only,
// pieces of the real batch.  us, before, with 32 rows and 128, now: 1024-2, batch 128, 520 workers 49, 55, 39; 128-4, batch 32, 700 workers 11.6, 19.2, 10.9; 2048-10, batch
// 128, 4 workers 32, 23, 19.9, 48 workers 33.6, 24, 20.9.
struct FwdSmallArgs {
    const uint16_t *a_prev; const float *X; int64_t woff; int M, B; int64_t din, dout; float *out;
    SoftmaxArgs sm;                  // what follows the logits in the same workgroup
};
constexpr int SMALL_MAX_DIN = 2048;
constexpr int FS_KS = 64, FS_PITCH = FS_KS + 8;                         // features of a piece, elements of its rows in LDS
// LDS: W^T and the pieces of the batch's waves; then the logits
constexpr size_t fwd_small_lds(int64_t din, int64_t dout, int B) { return sizeof(uint16_t) * (size_t)(dout * (din + 8) + (int64_t)B * FS_PITCH); }
static_assert(sizeof(uint16_t) * FS_PITCH >= sizeof(float) * SOFTMAX_PITCH, "the logits fit the space of the pieces");

// FS_DEPTH pieces ahead; WAVES workgroups fit the registers of a compute unit.
template <int FS_DEPTH, int WAVES>
__global__ void __launch_bounds__(MF_THREADS, WAVES) fwd_small_mfma_kernel(FwdSmallArgs p)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t Wt[];      // [dout][din + 8]
    const int g = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int din = (int)p.din, dout = (int)p.dout, pitch = din + 8;
    static_assert(MF_THREADS / 64 * 32 >= 128, "a wave for every 32 rows of the largest batch");
    const int m0 = 32 * wave, pieces = din / FS_KS;                    // din is a multiple of 128: at least two pieces
    const bool mine = m0 < p.B;
    const int label = softmax_label(p.sm, g);
    const uint16_t *a_src = p.a_prev + ((size_t)g * p.B + (mine ? m0 : 0) + (lane >> 3)) * p.din + 8 * (lane & 7);
    u32x4 ra[FS_DEPTH][4];
    auto request = [&](int d, int k) {                                 // past the end: the last piece again, never used
        const uint16_t *src = a_src + (k < pieces ? k : pieces - 1) * FS_KS;
#pragma unroll
        for (int u = 0; u < 4; ++u) ra[d][u] = *reinterpret_cast<const u32x4 *>(src + (size_t)(8 * u) * p.din);
    };
    if (mine) {
#pragma unroll
        for (int d = 0; d < FS_DEPTH; ++d) request(d, d);
    }
    // W[k][n] -> Wt[n][k]: the din x dout block is contiguous in the parameter row and starts at a multiple of four
    // columns, so it is read as float4 (a float4 never straddles a layout tile)
    {
        // eight pieces per thread are requested together (past the end: the first piece again, not stored)
        const unsigned n_w = (unsigned)(din * dout), udout = (unsigned)dout;
        for (unsigned base = 4u * t; base < n_w; base += 8u * 4u * MF_THREADS) {
            f32x4_t w[8];
#pragma unroll
            for (unsigned u = 0; u < 8; ++u) {
                const unsigned e4 = base + u * 4u * MF_THREADS;
                w[u] = *reinterpret_cast<const f32x4_t *>(p.X + tiled_offset(p.M, g, p.woff + (e4 < n_w ? e4 : 0u)));
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (unsigned u = 0; u < 8; ++u) {
                const unsigned e4 = base + u * 4u * MF_THREADS;
                if (e4 < n_w) {
#pragma unroll
                    for (unsigned c = 0; c < 4; ++c) {
                        const unsigned e = e4 + c, k = e / udout, n = e - k * udout;
                        Wt[n * pitch + k] = (uint16_t)bf16_bits(w[u][c]);
                    }
                }
            }
        }
    }
    __syncthreads();
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    const int col = lane & 31;
    const float bcol = p.X[tiled_offset(p.M, g, p.woff + (int64_t)din * dout + (col < dout ? col : dout - 1))];
    if (mine) {
        uint16_t *own = Wt + dout * pitch + wave * 32 * FS_PITCH, *to = own + (lane >> 3) * FS_PITCH + 8 * (lane & 7);
        const uint16_t *a_ptr = own + (lane & 31) * FS_PITCH + 8 * (lane >> 5), *b_ptr = Wt + (col < dout ? col : dout - 1) * pitch + 8 * (lane >> 5);      // columns past the last class repeat it
        auto consume = [&](int d, int k) {
#pragma unroll
            for (int u = 0; u < 4; ++u) *reinterpret_cast<u32x4 *>(to + 8 * u * FS_PITCH) = ra[d][u];
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int s = 0; s < FS_KS / 16; ++s)
                acc = mfma_bf16(*reinterpret_cast<const u32x4 *>(a_ptr + 16 * s), *reinterpret_cast<const u32x4 *>(b_ptr + k * FS_KS + 16 * s), acc);
            __builtin_amdgcn_wave_barrier();
        };
        int k = 0;
        for (; k + FS_DEPTH <= pieces; k += FS_DEPTH) {
#pragma unroll
            for (int d = 0; d < FS_DEPTH; ++d) {
                consume(d, k + d);
                request(d, k + d + FS_DEPTH);
            }
        }
#pragma unroll
        for (int d = 0; d < FS_DEPTH - 1; ++d)
            if (k + d < pieces) consume(d, k + d);
    }
    // the workgroup holds all logits of its worker: loss, dZ and the last layer's bias gradient follow at once
    __syncthreads();                                                   // W has been read; the logits take its place
    float *rows = reinterpret_cast<float *>(Wt);
    if (mine) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = m0 + d_row(lane, v);
            const float z = acc[v] + bcol;
            rows[row * SOFTMAX_PITCH + col] = z;
            if (col < dout) p.out[((size_t)g * p.B + row) * p.dout + col] = z;
        }
    }
    __syncthreads();
    softmax_xent_block<32, MF_THREADS>(p.sm, g, label, rows);
}

// dW = A^T dZ with dout <= 32: one workgroup = one worker x 128 rows of W, one 32-row tile per wave;
// both operands come straight from the transposed bf16 copies.
struct WgradSmallArgs {
    const uint16_t *a_t, *dz_t; int M, B; int64_t din, dout, woff; float *G;
};

__global__ void __launch_bounds__(MF_THREADS) wgrad_small_mfma_kernel(WgradSmallArgs p)
{
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    int g;
    unsigned strip;
    if (!decode_group(blockIdx.x, (unsigned)(p.din / 128), p.M, g, strip)) return;
    const int64_t r0 = (int64_t)strip * 128 + 32 * wave;
    const uint16_t *a_ptr = p.a_t + ((size_t)g * p.din + r0 + (lane & 31)) * p.B + 8 * (lane >> 5);
    const int n = lane & 31;
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    // the batch is at most 128: all eight steps' operands are requested before the first product (steps past the batch
    // and classes past dout repeat a valid address and are masked)
    const uint16_t *b_ok = p.dz_t + ((size_t)g * p.dout + (n < p.dout ? n : 0)) * p.B + 8 * (lane >> 5);
    const uint32_t keep = n < p.dout ? 0xFFFFFFFFu : 0u;
    u32x4 av[8], bv[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const int b0 = 16 * s < p.B ? 16 * s : 0;
        av[s] = *reinterpret_cast<const u32x4 *>(a_ptr + b0);
        bv[s] = *reinterpret_cast<const u32x4 *>(b_ok + b0);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 8; ++s)
        if (16 * s < p.B) acc = mfma_bf16(av[s], (u32x4){bv[s][0] & keep, bv[s][1] & keep, bv[s][2] & keep, bv[s][3] & keep}, acc);
    if (n < p.dout) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
            p.G[tiled_offset(p.M, g, p.woff + (r0 + d_row(lane, v)) * p.dout + n)] = acc[v];
    }
}

// dA = (dZ W^T) * [A > 0] with dout <= 32: the contraction is one or two matrix-instruction steps.
// One workgroup = one worker x 128 input features x all batch rows; waves 2 x 2, 64 x 64 each.
struct DgradSmallArgs {
    const uint16_t *dz; const float *X; int64_t woff; int M, B; int64_t din, dout;
    DgradOut o;
};

__global__ void __launch_bounds__(MF_THREADS) dgrad_small_mfma_kernel(DgradSmallArgs p)
{
    __shared__ __attribute__((aligned(16))) uint16_t T[128][ST_PITCH];
    __shared__ float red[4][2][64];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
    int g;
    unsigned cblk;
    if (!decode_group(blockIdx.x, (unsigned)(p.din / 128), p.M, g, cblk)) return;
    const int64_t c0 = (int64_t)cblk * 128;
    const int steps = p.dout <= 16 ? 1 : 2;
    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    for (int s = 0; s < steps; ++s) {
        const int nbase = 16 * s + 8 * (lane >> 5);
        u32x4 a[2], b[2];
        // All 32 values are requested before any is used: unconditional loads (row / class clamped into the operand,
        // the value masked afterwards; a load under the bounds test, or selected by it, is waited for one by one).
        uint32_t zr[2][8];
        float xr[2][8];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int row = 64 * wm + 32 * i + (lane & 31);
            const uint16_t *zrow = p.dz + ((size_t)g * p.B + (row < p.B ? row : p.B - 1)) * p.dout;
#pragma unroll
            for (int e = 0; e < 8; ++e) zr[i][e] = zrow[nbase + e < p.dout ? nbase + e : 0];
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int64_t feat = c0 + 64 * wn + 32 * j + (lane & 31);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                xr[j][e] = p.X[tiled_offset(p.M, g, p.woff + feat * p.dout + (nbase + e < p.dout ? nbase + e : 0))];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int row = 64 * wm + 32 * i + (lane & 31);
            uint32_t h[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) h[e] = zr[i][e] & ((row < p.B && nbase + e < p.dout) ? 0xFFFFu : 0u);
            a[i] = (u32x4){h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            float w[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) w[e] = __uint_as_float(__float_as_uint(xr[j][e]) & (nbase + e < p.dout ? 0xFFFFFFFFu : 0u));
            b[j] = (u32x4){pack_bf16x2(w[0], w[1]), pack_bf16x2(w[2], w[3]), pack_bf16x2(w[4], w[5]), pack_bf16x2(w[6], w[7])};
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = mfma_bf16(a[i], b[j], acc[i][j]);
    }
    dgrad_tail<8>(p.o, p.M, g, p.B, p.din, c0, wm, wn, lane, t, acc, T, red);
}

// ---------------------------------------------------------------------------------------------------
bool mfma_layer_ok(const MlpPlan &p, int l)
{
    const int64_t din = p.dims[l], dout = p.dims[l + 1];
    return p.bf16 && p.B % 32 == 0 && p.B <= 128 && din % 128 == 0 && dout % 128 == 0 && p.woff[l] % 4 == 0;
}

// the last layer when it has at most 32 outputs (see the "few classes" kernels above)
bool mfma_small_last_ok(const MlpPlan &p)
{
    const int l = p.n_layers - 1;
    const int64_t din = p.dims[l], dout = p.dims[l + 1];
    return p.bf16 && l > 0 && dout <= 32 && p.B % 32 == 0 && p.B <= 128 && din % 128 == 0 && din <= SMALL_MAX_DIN &&
           p.woff[l] % 4 == 0;
}

void prepare_kernels()
{

    // fwd_small_mfma_kernel keeps W^T in more than the default 64 KB of dynamic LDS
    const int lds = (int)fwd_small_lds(SMALL_MAX_DIN, 32, 128);
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(fwd_small_mfma_kernel<4, 3>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(fwd_small_mfma_kernel<2, 4>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
}

// Outputs of the backward-data kernel of layer l: the error of layer l - 1 and that layer's bias gradient.
static DgradOut dgrad_out(const MlpPlan &p, int l, int cur, float *G, bool want_f32)
{
    DgradOut o;
    o.act = p.hb[l]; o.out_f32 = want_f32 ? p.dz[cur ^ 1] : nullptr; o.out = p.dzb[cur ^ 1]; o.out_t = p.dzt[cur ^ 1];
    o.G = G; o.boff = p.woff[l - 1] + p.dims[l - 1] * p.dims[l];
    return o;
}

void launch_fwd_small(hipStream_t s, const MlpPlan &p, const float *X, float *G)
{
    const int l = p.n_layers - 1;
    FwdSmallArgs a;
    a.a_prev = p.hb[l]; a.X = X; a.woff = p.woff[l]; a.M = p.M; a.B = p.B; a.din = p.dims[l]; a.dout = p.dims[l + 1];
    a.out = p.act[l + 1];
    a.sm = softmax_args(p, G);
    const dim3 grid(p.M), block(MF_THREADS);
    const size_t lds = fwd_small_lds(a.din, a.dout, a.B), fit = (160 << 10) / (lds + MF_THREADS * sizeof(float));
    // Four pieces ahead, where two and the fourth workgroup on a compute unit don't save a round of them.  us, four and two, batch 32: 700 workers 128-10 11.2 and 11.3, 1024-2
    // 18.8 and 19.8, 820 workers (a round of two) 18.4 and 12.3, 28.1 and 21.1, 1366 workers (two rounds) 21.3 and 20.8, 35.4 and 38.6, 2500
    // workers (three of four) 36.8 and 30.9, 62.7 and 60.1.
    auto rounds = [&](size_t most) {
        const size_t at_once = MF_XCD * XCD_CUS * std::min(fit, most);
        return (p.M + at_once - 1) / at_once;
    };
    if (rounds(4) < rounds(3)) hipLaunchKernelGGL((fwd_small_mfma_kernel<2, 4>), grid, block, lds, s, a);
    else hipLaunchKernelGGL((fwd_small_mfma_kernel<4, 3>), grid, block, lds, s, a);
}

void launch_wgrad_small(hipStream_t s, const MlpPlan &p, float *G, int cur)
{
    const int l = p.n_layers - 1;
    WgradSmallArgs a;
    a.a_t = p.ht[l]; a.dz_t = p.dzt[cur]; a.M = p.M; a.B = p.B; a.din = p.dims[l]; a.dout = p.dims[l + 1];
    a.woff = p.woff[l]; a.G = G;
    hipLaunchKernelGGL(wgrad_small_mfma_kernel, dim3(grouped_grid(p.M, (unsigned)(a.din / 128))), dim3(MF_THREADS), 0, s, a);
}

void launch_dgrad_small(hipStream_t s, const MlpPlan &p, const float *X, float *G, int cur, bool want_f32)
{
    const int l = p.n_layers - 1;
    DgradSmallArgs a;
    a.dz = p.dzb[cur]; a.X = X; a.woff = p.woff[l]; a.M = p.M; a.B = p.B; a.din = p.dims[l]; a.dout = p.dims[l + 1];
    a.o = dgrad_out(p, l, cur, G, want_f32);
    hipLaunchKernelGGL(dgrad_small_mfma_kernel, dim3(grouped_grid(p.M, (unsigned)(a.din / 128))), dim3(MF_THREADS), 0, s, a);
}

void launch_fwd_mfma(hipStream_t s, const MlpPlan &p, int l, const float *X)
{
    FwdMfmaArgs a;
    a.feats = (const uint16_t *)p.feats; a.row0 = p.row0; a.idx = p.idx; a.a_prev = l > 0 ? p.hb[l] : nullptr;
    a.X = X; a.woff = p.woff[l]; a.M = p.M; a.B = p.B; a.din = p.dims[l]; a.dout = p.dims[l + 1];
    a.relu = (l + 1 < p.n_layers); a.out = p.hb[l + 1]; a.out_t = p.ht[l + 1];
    const dim3 grid(grouped_grid(p.M, (unsigned)(a.dout / MF_BN)));
    if (l == 0) hipLaunchKernelGGL(fwd_mfma_kernel<true>, grid, dim3(MF_THREADS), 0, s, a);
    else hipLaunchKernelGGL(fwd_mfma_kernel<false>, grid, dim3(MF_THREADS), 0, s, a);
}

void launch_dgrad_mfma(hipStream_t s, const MlpPlan &p, int l, const float *X, float *G, int cur, bool want_f32)
{
    DgradMfmaArgs a;
    a.dz = p.dzb[cur]; a.X = X; a.woff = p.woff[l]; a.M = p.M; a.B = p.B; a.din = p.dims[l]; a.dout = p.dims[l + 1];
    a.o = dgrad_out(p, l, cur, G, want_f32);
    hipLaunchKernelGGL(dgrad_mfma_kernel, dim3(grouped_grid(p.M, (unsigned)(a.din / MF_BN))), dim3(MF_THREADS), 0, s, a);
}

// Strips a walk of wgrad_mix_mfma_kernel, and the bytes that a parameter then costs: 16 of x, v, x' and v', dZ^T of the 128 columns once a walk, the strip's rows of
// A^T, all that by how much longer the XCD with the most blocks is at work than they are on average.  Of the walks of one, two, four and eight strips the one that costs
// least, if the compute units have two walks each.  At batches of up to 64, where dZ^T is small beside the strip's 64 KB of x, v, x' and v', one strip: with one and
// with eight, batch 64, 64 workers 1024-512 372 and 370 us an iteration, batch 32, 61 workers 2304-640 740 and 783.
// us per iteration with one, two, four and eight strips (fused), bytes by this count: batch 128, 63 workers 1152-896-10 364, 323, 320, 336 (26.4, 22.3, 20.3,
// 24.1), 640-384-10 134, 123, 120, 131 (27.7, 23.5, 21.3, 40.5), 1024-512-10 203, 190, 185, 182 (26, 22, 20, 19), 128 workers 1664-384-10 462, 408, 400, 420 (26.7,
// 22.6, 20.5, 23.4); one and eight, 128 workers 3072-1024-1024-10 2977 and 2527; too few walks: 4 workers 2944-896-640-25 617 and 674.  Walks whose blocks
// are whole rounds over the XCDs, or eight rounds and more, were the only ones before: that left one strip to 127 workers 1152-384-10 (341 us, 302 now; a block of 64 x
// 128 per workgroup 333) and 48 workers 640-640-10 (150 and 138).  The others have to save 8 %: batch 96, 100 workers 1152-896-10 (126 and 63 blocks) 467 us with
// two strips and 475 with four (7 % by the count).  At multiples of 64 workers (see `apart`) a walk of four has two places to begin: not those there, batch 96, 64
// workers 1152-896-10 312 us with two strips and 321 with four; but 128 workers 1280-512-10, batch 128 (40 blocks) 412 and 402.
struct WgradWalk { unsigned strips; double operands, uneven; };
static WgradWalk wgrad_walk(int M, int B, int64_t din, int64_t dout)
{
    const unsigned strips = (unsigned)(din / WM_ROWS), cols = (unsigned)(dout / WM_COLS);
    WgradWalk best{};
    double least = 0.0;
    for (unsigned walk = 1; walk <= (B > 64 ? 8u : 1u); walk *= 2) {
        const unsigned blocks = (strips + walk - 1) / walk * cols, rounds = (blocks + MF_XCD - 1) / MF_XCD;
        const double operands = B / 64.0 + B / (16.0 * walk), uneven = rounds * MF_XCD * (double)walk / ((double)strips * cols), bytes = (16.0 + operands) * uneven;
        const bool even = blocks % MF_XCD == 0 || blocks >= 8 * MF_XCD;
        if (walk > 1 && ((uint64_t)M * blocks < 2 * MF_XCD * XCD_CUS || (walk > 2 && M % 64 == 0 && !even))) continue;
        if (walk == 1 || bytes < (even ? 1.0 : 0.92) * least) {
            best = WgradWalk{walk, operands, uneven};
            least = bytes;
        }
    }
    return best;
}

// The update inside the weight gradients of netmax_run, by the bytes a parameter that it saves: 24 with the separate mix (g written and read), against x, v, x' and v',
// the operands as long as all workers' do not stay in an XCD's 4 MB of L2, and most of the uneven share (XCDs that are done leave the others their part
// of the memory).  Operands count half, as repeated reads of them mostly end in the last cache, but in full beside g, which counts as 2.  Both and the uneven
// share count for less where x, v, x' and v' of all workers stay in the last cache themselves (18 M floats, 288 MB) and an XCD holds more workers than there
// are (96).  Every parameter that is none of these layers' costs 2.25 more, in the mix of what is left, than in the mix of everything
// (1.25 from 96 workers on).
// us, four iterations, separate and in the gradients, saved bytes a parameter of the model: batch 128, 64 workers 3000-1000-128-128-10 4820 and 5068 (-2.3), 200-1024-1024-10
// 2482 and 2326 (5.0); 18 workers 128-1408-17 344 and 301 (4.5), 10 workers 128-2048-4 347 and 276 (5.6), 27 workers 128-1280-6 340 and 305 (5.5).
// One iteration, which keeps g: batch 128, 127 workers 384-384-10 151 and 168 (-6.4), 48 workers 784-384-384-10 205 and 211 (-3.7), 127 workers 1024-1024-10
// 787 and 712 (3.0), 10 workers 128-2048-4 90 and 68 (1.8), 27 workers 128-1280-6 89 and 79 (1.8); batch 96, 122 workers 640-640-10 307 and 328 (-2.4); batch 64, 96
// workers 3072-512-512-10 935 and 839 (1.0); batch 32, 128 workers 1024-1024-10 692 and 633 (3.4).
double wgrad_mix_saves(const MlpPlan &p, bool keep_g)
{
    const double rest = p.M >= 96 ? 1.25 : 2.25, memory = std::min(1.0, std::max({0.4, (double)p.M * (double)p.ld / 18e6, p.M / 96.0}));
    double saved = -rest * (double)p.ld;
    for (int l = 0; l < p.n_layers; ++l) {
        if (!mfma_layer_ok(p, l)) continue;
        const int64_t din = p.dims[l], dout = p.dims[l + 1];
        const WgradWalk w = wgrad_walk(p.M, p.B, din, dout);
        const bool in_l2 = p.M * (din + dout) * p.B * 2 <= (int64_t)7 << 19;
        const double moved = 16.0 + (keep_g ? 2.0 : 0.0) + (in_l2 ? 0.0 : memory * (keep_g ? 1.0 : 0.5) * w.operands);
        saved += (double)(din * dout) * (24.0 + rest - moved * (1.0 + 0.85 * memory * (w.uneven - 1.0)));
    }
    return saved / (double)p.ld;
}

void launch_wgrad_mix_mfma(hipStream_t s, const MlpPlan &p, int l, float *G, int cur, const MixArgs &mix)
{
    WgradMixArgs a;
    a.a_t = p.ht[l]; a.dz_t = p.dzt[cur]; a.M = p.M; a.B = p.B; a.din = p.dims[l]; a.dout = p.dims[l + 1];
    a.woff = p.woff[l]; a.G = G; a.mix = mix;
    a.feats = l == 0 ? (const uint16_t *)p.feats : nullptr; a.row0 = p.row0; a.idx = p.idx;
    a.walk = wgrad_walk(p.M, p.B, a.din, a.dout).strips;
    // A tile of the layout is 8 KB of every worker.  At a multiple of 512 KB from tile to tile the workers, strip by strip in step, fall
    // on few of the memory's channels: eight workers at a time begin their walk a strip further on.  64 workers 3072-1024-1024 1341 and
    // 1237 us, 128 workers 2527 and 2495; 32 and 48 workers would lose 2 to 10 % (the peer's strip is no longer in the L2).
    a.apart = p.M % 64 == 0 ? 8 : 0;
    const unsigned blocks = ((unsigned)(a.din / WM_ROWS) + a.walk - 1) / a.walk * (unsigned)(a.dout / WM_COLS);
    const dim3 grid((blocks + MF_XCD - 1) / MF_XCD * MF_XCD * (unsigned)p.M), block(MF_THREADS);
    if (l == 0) {
        if (mix.keep_g) hipLaunchKernelGGL((wgrad_mix_mfma_kernel<true, true>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((wgrad_mix_mfma_kernel<true, false>), grid, block, 0, s, a);
    } else {
        if (mix.keep_g) hipLaunchKernelGGL((wgrad_mix_mfma_kernel<false, true>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((wgrad_mix_mfma_kernel<false, false>), grid, block, 0, s, a);
    }
}

void launch_wgrad_mfma(hipStream_t s, const MlpPlan &p, int l, float *G, int cur)
{
    WgradMfmaArgs a;
    a.a_t = p.ht[l]; a.dz_t = p.dzt[cur]; a.M = p.M; a.B = p.B; a.din = p.dims[l]; a.dout = p.dims[l + 1];
    a.woff = p.woff[l]; a.G = G;
    a.feats = l == 0 ? (const uint16_t *)p.feats : nullptr; a.row0 = p.row0; a.idx = p.idx;
    hipLaunchKernelGGL(wgrad_mfma_kernel, dim3(grouped_grid(p.M, (unsigned)(a.din / WG_STRIP))), dim3(MF_THREADS), 0, s, a);
}

}  // namespace netmax
