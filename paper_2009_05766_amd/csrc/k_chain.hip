// Forward pass and error of layers on bfloat16 operands in few blocks (the stochastic gradient of Algorithm 2's first-step update).  The tiled
// kernels (k_grad_mfma.hip, k_tile_fwd.hip, k_tile_dgrad.hip) ask for a step of 32 to 128 contraction indices while they multiply the one before and
// wait for it at two barriers; where a few workgroups have the chip to themselves that is a memory round trip a step, and most compute units have
// nothing to do.  Here a workgroup takes 32 columns and RT x 32 batch rows.  Its four waves ask for a chunk of four steps of 32 indices, one
// each, two chunks ahead; a chunk crosses LDS (two buffers in turn, one barrier), and wave i multiplies tile i.  Every result is one chain of
// v_mfma_f32_32x32x16_bf16 over the indices in the order of the kernels in whose place these stand: their results bit for bit.
// Column sums of an error (the bias gradient of the layer below) are added in those kernels' order as well.
// us, before and now: forward 8 x 1024-1024, batch 32, 27 and 11.6, 9 x 2432-256 56 and 16, 16 x 3072-1024, batch 128, 81 and 48 (4.1 TB/s of W); errors 8 x 1024-1024,
// batch 32, 30 and 8.4, batch 128 36 and 14.  (Eight waves that share the indices and add their parts are 1 to 3 us faster still, in another order of sums: after four
// iterations of a network with two hidden layers roundings of activations that fall the other way have travelled to 1e-2 of the momentum.)
#include "tile.h"
#include <type_traits>

namespace netmax {

constexpr int CH_WAVES = 4, CH_THREADS = 64 * CH_WAVES, CH_STEP = 32, CH_SETS = 2, CH_PITCH = WF_COLS + 1;

// 64 bytes of every row of the batch tiles and of the 32 columns: a step's operands in LDS.
template <int RT> constexpr int chain_step_units() { return (RT + 1) * 32 * 4; }
// LDS of a workgroup: two chunks, later the block's results in fp32.
template <int RT> constexpr int chain_lds()
{
    constexpr int operands = 2 * CH_WAVES * chain_step_units<RT>() * 16, results = 32 * RT * CH_PITCH * 4;
    return operands > results ? operands : results;
}

// What a lane loads of a 16-byte piece of an operand row, and the piece.
template <bool WIDE> struct ChainRaw { f32x4 v[2]; };                 // eight floats that become bfloat16
template <> struct ChainRaw<false> { tile_u32x4 v; };                 // eight bfloat16 as they are
__device__ __forceinline__ tile_u32x4 chain_piece(const ChainRaw<false> &r) { return r.v; }
__device__ __forceinline__ tile_u32x4 chain_pack(f32x4 a, f32x4 b)
{
    return tile_u32x4{pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(b[0], b[1]), pack_bf16x2(b[2], b[3])};
}
__device__ __forceinline__ tile_u32x4 chain_piece(const ChainRaw<true> &r) { return chain_pack(r.v[0], r.v[1]); }

// acc += one step's product for tile `wave`; `at`: the step's operands.
template <int RT> __device__ __forceinline__ void chain_multiply(const tile_u32x4 *at, int wave, int lane, tile_f32x16 &acc)
{
    const int row = lane & 31, half = lane >> 5;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int u = wave_unit(row, 2 * j + half);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(tile_bf16x8, at[32 * 4 * wave + u]), __builtin_bit_cast(tile_bf16x8, at[32 * 4 * RT + u]),
                                                      acc, 0, 0, 0);
    }
}

// The whole steps of a contraction.  request(set, s): this wave's loads of step s; put(set, to): what they brought, into the step's operands in LDS.
// Steps past the last one are asked for as the last one again and never multiplied.
template <int RT, class Request, class Put>
__device__ __forceinline__ void chain_steps(int total, int wave, int lane, tile_u32x4 *smem, tile_f32x16 &acc, Request request, Put put)
{
    constexpr int STEP = chain_step_units<RT>();
    if (total == 0) return;
    auto mine = [&](int chunk) { return min(CH_WAVES * chunk + wave, total - 1); };
#pragma unroll
    for (int d = 0; d < CH_SETS; ++d) request(d, mine(d));
    const int chunks = (total + CH_WAVES - 1) / CH_WAVES;
    auto chunk = [&](int c, int d) {
        tile_u32x4 *buf = smem + (c & 1) * (CH_WAVES * STEP);
        put(d, buf + wave * STEP);
        __syncthreads();                                              // the chunk is in LDS; the one before the last has been read
        request(d, mine(c + CH_SETS));
        if (wave < RT) {
            if (CH_WAVES * c + CH_WAVES <= total) {
#pragma unroll
                for (int s = 0; s < CH_WAVES; ++s) chain_multiply<RT>(buf + s * STEP, wave, lane, acc);
            } else {
                for (int s = 0; CH_WAVES * c + s < total; ++s) chain_multiply<RT>(buf + s * STEP, wave, lane, acc);
            }
        }
    };
    int c = 0;
    for (; c + CH_SETS <= chunks; c += CH_SETS) {
#pragma unroll
        for (int d = 0; d < CH_SETS; ++d) chunk(c + d, d);
    }
#pragma unroll
    for (int d = 0; d < CH_SETS - 1; ++d)
        if (c + d < chunks) chunk(c + d, d);
}

// The block's results, in LDS, as bfloat16 to `rows` ([..][ld], 32 columns of RT x 32 rows) and transposed to `cols` ([..][B]); each may be absent.
template <int RT>
__device__ __forceinline__ void chain_store(const float (*F)[CH_PITCH], int t, int n_rows, int n_cols, uint16_t *rows, int64_t ld, uint16_t *cols, int64_t B)
{
    if (rows && ld % 8 == 0) {
        for (int e = t; e < 32 * RT * 4; e += CH_THREADS) {
            const int r = e >> 2, c = (e & 3) * 8;
            if (r < n_rows && c < n_cols)
                *reinterpret_cast<tile_u32x4 *>(rows + (size_t)r * ld + c) =
                    chain_pack(f32x4{F[r][c], F[r][c + 1], F[r][c + 2], F[r][c + 3]}, f32x4{F[r][c + 4], F[r][c + 5], F[r][c + 6], F[r][c + 7]});
        }
    } else if (rows) {
        for (int e = t; e < 32 * RT * 32; e += CH_THREADS) {
            const int r = e >> 5, c = e & 31;
            if (r < n_rows && c < n_cols) rows[(size_t)r * ld + c] = (uint16_t)bf16_bits(F[r][c]);
        }
    }
    if (cols)                                                         // who asks for it has a batch of whole 32 rows
        for (int e = t; e < 32 * RT * 4; e += CH_THREADS) {
            const int c = e / (4 * RT), r = e % (4 * RT) * 8;
            if (r < n_rows && c < n_cols)
                *reinterpret_cast<tile_u32x4 *>(cols + (size_t)c * B + r) =
                    chain_pack(f32x4{F[r][c], F[r + 1][c], F[r + 2][c], F[r + 3][c]}, f32x4{F[r + 4][c], F[r + 5][c], F[r + 6][c], F[r + 7][c]});
        }
}

struct ChainFwd {
    const uint16_t *feats; const int64_t *row0; const int32_t *idx;   // first layer: gathered data rows
    const uint16_t *act;                                              // else the activation below, [M][B][din]
    const float *X; int64_t woff; int M, B, din, dout, relu;
    float *out; uint16_t *out_bf16, *out_bf16_t;                      // [M][B][dout], and [M][dout][B]; each may be absent
};

// Z = A W + b.  A lane's operands of W are neighbouring rows of its column, each a load of a float (32 lanes 128 bytes of a row).  TAIL: indices behind
// the last whole step.
template <int RT, bool TAIL>
__global__ void __launch_bounds__(CH_THREADS) chain_fwd_kernel(ChainFwd p)
{
    __shared__ __attribute__((aligned(16))) unsigned char smem[chain_lds<RT>()];
    tile_u32x4 *units = reinterpret_cast<tile_u32x4 *>(smem);
    const int t = threadIdx.x, lane = t & 63, row = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const unsigned nblk = (unsigned)((p.dout + WF_COLS - 1) / WF_COLS), mblk = (unsigned)((p.B + 32 * RT - 1) / (32 * RT));
    int g;
    unsigned local;
    if (!decode_group(tile_block(), nblk * mblk, p.M, g, local)) return;
    const int n0 = (int)(local % nblk) * WF_COLS, m0 = (int)(local / nblk) * 32 * RT, K = p.din, total = K / CH_STEP;
    const int col = min(n0 + row, p.dout - 1);                        // columns past the end repeat the last one
    const float bias = p.X[tiled_offset_quick(p.M, g, p.woff + (int64_t)K * p.dout + col)];
    const uint32_t skip = (uint32_t)(p.M - 1) << (TILE_SHIFT + 2), dout4 = (uint32_t)p.dout * 4u, w_first = (uint32_t)col * 4u + (uint32_t)(8 * half) * dout4;
    // pieces that this lane brings into LDS: `pa` of rows pr and pr + 16 of every tile (rows past the batch repeat the last one), and of column
    // `row` the indices 8 half + 0 .. 7 and 16 more
    const int pa = lane & 3, pr = lane >> 2;
    const uint16_t *a_row[RT][2];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int r = min(m0 + 32 * i + 16 * h + pr, p.B - 1);
            a_row[i][h] = (p.feats ? p.feats : p.act) + (p.feats ? p.row0[g] + p.idx[(size_t)g * p.B + r] : (int64_t)g * p.B + r) * K;
        }
    tile_u32x4 a[CH_SETS][RT][2];
    float w[CH_SETS][16];
    auto request = [&](int d, int s) {
        const int64_t j0 = p.woff + (int64_t)s * CH_STEP * p.dout;
        const float *base = p.X + (((size_t)(j0 >> TILE_SHIFT) * p.M + g) << TILE_SHIFT);
        const uint32_t from = w_first + (uint32_t)(j0 & (TILE - 1)) * 4u;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const uint32_t q = from + (uint32_t)(e < 8 ? e : 8 + e) * dout4;
            w[d][e] = *(const float *)((const char *)base + (__umul24(q >> (TILE_SHIFT + 2), skip) + q));
        }
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) a[d][i][h] = *reinterpret_cast<const tile_u32x4_any *>(a_row[i][h] + (s * CH_STEP + 8 * pa));
    };
    auto put_w = [&](const float (&x)[16], tile_u32x4 *to) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
            to[32 * 4 * RT + wave_unit(row, 2 * j + half)] = chain_pack(f32x4{x[8 * j], x[8 * j + 1], x[8 * j + 2], x[8 * j + 3]}, f32x4{x[8 * j + 4], x[8 * j + 5], x[8 * j + 6], x[8 * j + 7]});
    };
    auto put = [&](int d, tile_u32x4 *to) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) to[32 * 4 * i + wave_unit(16 * h + pr, pa)] = a[d][i][h];
        put_w(w[d], to);
    };
    // what is behind the last whole step: asked for first, a tile by each wave; what does not exist counts as zero
    uint16_t at[2][8];
    float wt[16];
    const int from = total * CH_STEP, left = K - from;
    if constexpr (TAIL) {
#pragma unroll
        for (int e = 0; e < 16; ++e) wt[e] = p.X[tiled_offset_quick(p.M, g, p.woff + (int64_t)min(from + (e < 8 ? 0 : 8) + 8 * half + e, K - 1) * p.dout + col)];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint16_t *r = a_row[0][h];
#pragma unroll
            for (int i = 1; i < RT; ++i) r = wave == i ? a_row[i][h] : r;
#pragma unroll
            for (int e = 0; e < 8; ++e) at[h][e] = r[min(from + 8 * pa + e, K - 1)];
        }
    }
    tile_f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    chain_steps<RT>(total, wave, lane, units, acc, request, put);
    if constexpr (TAIL) {
        tile_u32x4 *buf = units + ((total + CH_WAVES - 1) / CH_WAVES & 1) * (CH_WAVES * chain_step_units<RT>());      // the other buffer's turn
        if (wave < RT) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                tile_u32x4 x;
#pragma unroll
                for (int e = 0; e < 8; e += 2) x[e / 2] = (8 * pa + e < left ? (uint32_t)at[h][e] : 0u) | (8 * pa + e + 1 < left ? (uint32_t)at[h][e + 1] << 16 : 0u);
                buf[32 * 4 * wave + wave_unit(16 * h + pr, pa)] = x;
            }
        }
        if (wave == 0) {
#pragma unroll
            for (int e = 0; e < 16; ++e) wt[e] = (e < 8 ? 0 : 8) + 8 * half + e < left ? wt[e] : 0.0f;
            put_w(wt, buf);
        }
        __syncthreads();
        if (wave < RT) chain_multiply<RT>(buf, wave, lane, acc);
    }
    __syncthreads();                                                  // the operands' space becomes the results
    float (*F)[CH_PITCH] = reinterpret_cast<float (*)[CH_PITCH]>(smem);
    if (wave < RT) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float z = acc[v] + bias;
            F[32 * wave + tile_row(lane, v)][row] = p.relu && !(z > 0.0f) ? 0.0f : z;
        }
    }
    __syncthreads();
    const int rows = min(32 * RT, p.B - m0), cols = min(WF_COLS, p.dout - n0);
    if (p.out)
        for (int e = t; e < 32 * RT * 32; e += CH_THREADS)
            if ((e >> 5) < rows && (e & 31) < cols) p.out[((size_t)g * p.B + m0 + (e >> 5)) * p.dout + n0 + (e & 31)] = F[e >> 5][e & 31];
    chain_store<RT>(F, t, rows, cols, p.out_bf16 ? p.out_bf16 + ((size_t)g * p.B + m0) * p.dout + n0 : nullptr, p.dout,
                    p.out_bf16_t ? p.out_bf16_t + ((size_t)g * p.dout + n0) * p.B + m0 : nullptr, p.B);
}

struct ChainDgrad {
    const void *dz;                                                   // [M][B][dout], bfloat16 (ZB) or float
    const float *X; int64_t woff; int M, B, din, dout;
    const uint16_t *act;                                              // this layer's input (ReLU mask)
    float *out; uint16_t *out_bf16, *out_bf16_t;                      // [M][B][din], and [M][din][B]; each may be absent
    float *G; int64_t boff;                                           // bias of the layer below inside a gradient row
};

// dA = (dZ W^T) where A > 0, all batch rows (RT x 32 or fewer); both operands are contiguous along the contraction.  ALIGNED: an aligned layer, as
// dgrad_mfma_kernel computes it (its contraction starts elsewhere for every 128 columns and worker; column sums over 64 rows); otherwise as
// tile_dgrad_kernel does (column sums over 32 rows).  ZB: dZ is bfloat16 in memory.  V: pieces of W do not cross a layout tile.
template <bool ALIGNED, int RT, bool V, bool TAIL>
__global__ void __launch_bounds__(CH_THREADS) chain_dgrad_kernel(ChainDgrad p)
{
    constexpr bool ZB = ALIGNED;
    __shared__ __attribute__((aligned(16))) unsigned char smem[chain_lds<RT>()];
    __shared__ float red[RT][2][WF_COLS];
    tile_u32x4 *units = reinterpret_cast<tile_u32x4 *>(smem);
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const unsigned nblk = (unsigned)((p.din + WF_COLS - 1) / WF_COLS);
    int g;
    unsigned local;
    if (!decode_group(tile_block(), nblk, p.M, g, local)) return;
    const int n0 = (int)local * WF_COLS, K = p.dout, total = K / CH_STEP;
    const int shift = ALIGNED ? (int)(((unsigned)n0 / 128 * 5u + (unsigned)g * 3u) % (unsigned)total) : 0;
    // pieces that this lane brings into LDS: `pa` of rows pr and pr + 16 of every tile and of the 32 features; past the end the last one again
    const int pa = lane & 3, pr = lane >> 2;
    int64_t z_row[RT][2], w_row[2];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) z_row[i][h] = ((int64_t)g * p.B + min(32 * i + 16 * h + pr, p.B - 1)) * K;
#pragma unroll
    for (int h = 0; h < 2; ++h) w_row[h] = p.woff + (int64_t)min(n0 + 16 * h + pr, p.din - 1) * K;
    auto w4 = [&](int64_t j) { return load4_params<V>(p.X, p.M, g, j); };
    ChainRaw<!ZB> z[CH_SETS][RT][2];
    ChainRaw<true> w[CH_SETS][2];
    auto request = [&](int d, int s) {
        int at = s + shift;
        if (ALIGNED && at >= total) at -= total;
        const int k = at * CH_STEP + 8 * pa;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            w[d][h].v[0] = w4(w_row[h] + k);
            w[d][h].v[1] = w4(w_row[h] + k + 4);
        }
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if constexpr (ZB) z[d][i][h].v = *reinterpret_cast<const tile_u32x4_any *>((const uint16_t *)p.dz + z_row[i][h] + k);
                else {
#pragma unroll
                    for (int q = 0; q < 2; ++q) z[d][i][h].v[q] = *reinterpret_cast<const tile_f32x4_any *>((const float *)p.dz + z_row[i][h] + k + 4 * q);
                }
            }
    };
    auto put = [&](int d, tile_u32x4 *to) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int u = wave_unit(16 * h + pr, pa);
#pragma unroll
            for (int i = 0; i < RT; ++i) to[32 * 4 * i + u] = chain_piece(z[d][i][h]);
            to[32 * 4 * RT + u] = chain_piece(w[d][h]);
        }
    };
    // what is behind the last whole step: asked for first, a tile by each wave; what does not exist counts as zero
    float zt[2][8], wt[2][8];
    const int from = total * CH_STEP + 8 * pa, left = K - from;
    if constexpr (TAIL) {
        static_assert(!ALIGNED, "aligned layers have whole steps");
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int64_t r = z_row[0][h];
#pragma unroll
            for (int i = 1; i < RT; ++i) r = wave == i ? z_row[i][h] : r;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                wt[h][e] = p.X[tiled_offset_quick(p.M, g, w_row[h] + min(from + e, K - 1))];
                zt[h][e] = ((const float *)p.dz)[r + min(from + e, K - 1)];
            }
        }
    }
    tile_f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    chain_steps<RT>(total, wave, lane, units, acc, request, put);
    if constexpr (TAIL) {
        tile_u32x4 *buf = units + ((total + CH_WAVES - 1) / CH_WAVES & 1) * (CH_WAVES * chain_step_units<RT>());      // the other buffer's turn
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                zt[h][e] = e < left ? zt[h][e] : 0.0f;
                wt[h][e] = e < left ? wt[h][e] : 0.0f;
            }
            const int u = wave_unit(16 * h + pr, pa);
            if (wave < RT) buf[32 * 4 * wave + u] = chain_pack(f32x4{zt[h][0], zt[h][1], zt[h][2], zt[h][3]}, f32x4{zt[h][4], zt[h][5], zt[h][6], zt[h][7]});
            if (wave == 0) buf[32 * 4 * RT + u] = chain_pack(f32x4{wt[h][0], wt[h][1], wt[h][2], wt[h][3]}, f32x4{wt[h][4], wt[h][5], wt[h][6], wt[h][7]});
        }
        __syncthreads();
        if (wave < RT) chain_multiply<RT>(buf, wave, lane, acc);
    }
    __syncthreads();                                                  // the operands' space becomes the results
    float (*F)[CH_PITCH] = reinterpret_cast<float (*)[CH_PITCH]>(smem);
    if (wave < RT) {
        const int c = lane & 31, col = min(n0 + c, p.din - 1);
        uint16_t on[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) on[v] = p.act[((size_t)g * p.B + min(32 * wave + tile_row(lane, v), p.B - 1)) * p.din + col];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int r = 32 * wave + tile_row(lane, v);
            F[r][c] = bf16_positive(on[v]) && r < p.B ? acc[v] : 0.0f;
        }
    }
    __syncthreads();
    const int rows = p.B, cols = min(WF_COLS, p.din - n0);
    // column sums: the rows that a lane of the other kernels has, in its order; then these
    constexpr int TILES = ALIGNED && RT > 1 ? 2 : 1;                  // of 32 rows in a part
    if (t < 64 * (RT / TILES)) {
        const int c = t & 31, half = (t >> 5) & 1, part = t >> 6;
        float s = 0.0f;
#pragma unroll
        for (int i = 0; i < TILES; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) s += F[32 * (TILES * part + i) + tile_row(32 * half, v)][c];
        red[part][half][c] = s;
    }
    __syncthreads();
    if (t < cols) {
        float s = ALIGNED ? 0.0f : red[0][0][t] + red[0][1][t];
#pragma unroll
        for (int k = ALIGNED ? 0 : 1; k < RT / TILES; ++k) {
            if constexpr (ALIGNED) s = s + red[k][0][t] + red[k][1][t];
            else s += red[k][0][t] + red[k][1][t];
        }
        p.G[tiled_offset_quick(p.M, g, p.boff + n0 + t)] = s;
    }
    if (p.out)
        for (int e = t; e < 32 * RT * 32; e += CH_THREADS)
            if ((e >> 5) < rows && (e & 31) < cols) p.out[((size_t)g * p.B + (e >> 5)) * p.din + n0 + (e & 31)] = F[e >> 5][e & 31];
    chain_store<RT>(F, t, rows, cols, p.out_bf16 ? p.out_bf16 + ((size_t)g * p.B) * p.din + n0 : nullptr, p.din,
                    p.out_bf16_t ? p.out_bf16_t + ((size_t)g * p.din + n0) * p.B : nullptr, p.B);
}

// Whether chain_fwd_kernel takes a layer: few blocks of 32 columns (of all workers, times the batch's parts of 128 rows).  us, it and the other kernel, either
// side of each line:
//   aligned layers   batch <= 32   48 x 256-512 (768 blocks) 9.0 and 11.8, 64 x (1024) 13.1 and 12.6; of 1024 indices and more 64 x 1024-512 25 and 30, 32 x
//                                  3072-1024 (1024) 89 and 98, 48 x (1536) 138 and 114
//                    batch <= 64   32 x 256-512 (512) 8.5 and 11.5, 48 x (768) 13.2 and 13.0; long ones 32 x 3072-1024 (1024) 95 and 106, 48 x (1536) 151 and 124
//                    more          32 x 256-512, batch 128 (512) 13.3 and 13.4, 16 x 3072-1024 (512) 48 and 81, 24 x (768) 112 and 106
//   others           batch <= 64   30 x 784-516 (510) 18.8 and 20.9, 45 x (765) 25.4 and 22.1;  more  15 x 784-516, batch 128 (255) 16.6 and 19.4, 23 x (391)
//                                  29 and 22; fewer indices 15 x 252-516 12.6 and 10.2, batch <= 32 60 x 784-516 (1020) 26.3 and 26.2
bool chain_fwd_pays(const MlpPlan &p, int l)
{
    const int64_t din = p.dims[l], dout = p.dims[l + 1], step = (CH_STEP * dout + TILE) / TILE + 1;
    const int64_t blocks = p.M * ((dout + WF_COLS - 1) / WF_COLS) * ((p.B + 127) / 128);
    // 32-bit offsets inside a step's rows of W
    if (!p.bf16 || p.M > 2048 || step * p.M * (TILE * 4) >= (int64_t)1 << 32) return false;
    // an aligned last layer has no activations to keep and is a layer of any width for the other kernels, too
    if (mfma_layer_ok(p, l) && l + 1 < p.n_layers) return blocks <= (p.B > 64 ? 512 : din >= 1024 ? 1024 : p.B > 32 ? 512 : 768);
    return tile_fwd_one_chain(p, l) && din >= 640 && p.B > 32 && blocks <= (p.B > 64 ? 256 : 512);
}

void launch_chain_fwd(hipStream_t s, const MlpPlan &p, int l, const float *X, bool need_t)
{
    const bool last = l + 1 == p.n_layers;
    ChainFwd a;
    a.feats = l == 0 ? (const uint16_t *)p.feats : nullptr; a.row0 = p.row0; a.idx = p.idx; a.act = l == 0 ? nullptr : p.hb[l];
    a.X = X; a.woff = p.woff[l]; a.M = p.M; a.B = p.B; a.din = (int)p.dims[l]; a.dout = (int)p.dims[l + 1]; a.relu = !last;
    a.out = last ? p.act[l + 1] : nullptr;
    a.out_bf16 = last ? nullptr : p.hb[l + 1];
    a.out_bf16_t = !last && need_t ? p.ht[l + 1] : nullptr;
    auto go = [&](auto *kernel, int rt) {
        const unsigned n = (unsigned)((a.dout + WF_COLS - 1) / WF_COLS) * (unsigned)((a.B + 32 * rt - 1) / (32 * rt));
        hipLaunchKernelGGL(kernel, tile_grid(grouped_grid(a.M, n)), dim3(CH_THREADS), 0, s, a);
    };
    const bool tail = a.din % CH_STEP != 0;
    if (a.B <= 32) go(chain_fwd_kernel<1, false>, 1);                 // chain_fwd_pays(): aligned layers only
    else if (a.B <= 64) { if (tail) go(chain_fwd_kernel<2, true>, 2); else go(chain_fwd_kernel<2, false>, 2); }
    else { if (tail) go(chain_fwd_kernel<4, true>, 4); else go(chain_fwd_kernel<4, false>, 4); }
}

// The same of chain_dgrad_kernel:
//   aligned layers   batch <= 32   64 x 1024-1024 (2048 blocks) 54 and 57, 128 x 512-128 13.8 and 16.8;  <= 64  48 x 1024-1024 (1536) 42 and 51, 64 x (2048) 67 and 66;
//                    more  24 x 1024-1024, batch 128 (768) 38 and 39, 32 x (1024) 50 and 43
//   others, rows of W that start anywhere (which cost the other kernel a load a float): 51 x 301-1001 (510), batch 20 21 and 36, 60 28 and 40, 128 47 and 80; 128 x
//                    102-301 (512) 12.3 and 13.9, 15.3 and 16.0, 25 and 30
//   others, aligned rows: many outputs only, batch <= 32 16 x 1000-1000 (512) 16.4 and 19.0, 8 x 1000-300 8.0 and 7.4;  <= 64 8 x 1000-1000 (256) 14.6 and 15.7,
//                    12 x (384) 22 and 18;  more  8 x (256) 20.2 and 18.3
bool chain_dgrad_pays(const MlpPlan &p, int l)
{
    if (!p.bf16 || p.B > 128) return false;
    const int64_t K = p.dims[l + 1], blocks = p.M * ((p.dims[l] + WF_COLS - 1) / WF_COLS);
    if (mfma_layer_ok(p, l)) return blocks <= (p.B > 64 ? 768 : p.B > 32 ? 1536 : 2048);
    // tile_dgrad_kernel adds the columns of 32 rows at a time while its blocks are few; the last layer may have a kernel of its own
    if (p.M * ((p.dims[l] + 63) / 64) > 256 || (l + 1 == p.n_layers && mfma_small_last_ok(p))) return false;
    if (K % 4 != 0 || p.woff[l] % 4 != 0) return K >= 256 && blocks <= 512;
    return K >= 640 && p.B <= 64 && blocks <= (p.B > 32 ? 256 : 512);
}

void launch_chain_dgrad(hipStream_t s, const MlpPlan &p, int l, const float *X, float *G, int cur, bool below_fast)
{
    const bool aligned = mfma_layer_ok(p, l);
    ChainDgrad a;
    a.dz = aligned ? (const void *)p.dzb[cur] : (const void *)p.dz[cur]; a.X = X; a.woff = p.woff[l]; a.M = p.M; a.B = p.B; a.din = (int)p.dims[l]; a.dout = (int)p.dims[l + 1];
    a.act = p.hb[l];
    a.out = aligned && below_fast ? nullptr : p.dz[cur ^ 1];
    a.out_bf16 = aligned || below_fast ? p.dzb[cur ^ 1] : nullptr;
    a.out_bf16_t = aligned || below_fast ? p.dzt[cur ^ 1] : nullptr;
    a.G = G; a.boff = p.woff[l - 1] + p.dims[l - 1] * p.dims[l];
    const dim3 grid = tile_grid(grouped_grid(a.M, (unsigned)((a.din + WF_COLS - 1) / WF_COLS)));
    auto go = [&](auto *kernel) { hipLaunchKernelGGL(kernel, grid, dim3(CH_THREADS), 0, s, a); };
    const bool v = a.dout % 4 == 0 && a.woff % 4 == 0, tail = a.dout % CH_STEP != 0;
    if (aligned) {
        if (a.B <= 32) go(chain_dgrad_kernel<true, 1, true, false>);
        else if (a.B <= 64) go(chain_dgrad_kernel<true, 2, true, false>);
        else go(chain_dgrad_kernel<true, 4, true, false>);
        return;
    }
    auto rows = [&](auto rt) {
        constexpr int RT = decltype(rt)::value;
        if constexpr (RT < 4) {                                       // chain_dgrad_pays(): larger batches on other rows only
            if (v && tail) return go(chain_dgrad_kernel<false, RT, true, true>);
            if (v) return go(chain_dgrad_kernel<false, RT, true, false>);
        }
        if (tail) go(chain_dgrad_kernel<false, RT, false, true>);
        else go(chain_dgrad_kernel<false, RT, false, false>);
    };
    if (a.B <= 32) rows(std::integral_constant<int, 1>{});
    else if (a.B <= 64) rows(std::integral_constant<int, 2>{});
    else rows(std::integral_constant<int, 4>{});
}

}  // namespace netmax
