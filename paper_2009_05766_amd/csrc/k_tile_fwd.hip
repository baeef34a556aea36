// Forward pass of a layer of any shape, Z = A W + b with optional ReLU, for all workers (the stochastic gradient of
// Algorithm 2's first-step update): the tiled kernel for what the kernels of k_grad_mfma.hip and k_grad_f32.hip do not take.
//
// A workgroup takes BM batch rows and BN outputs of one worker.  A is contiguous along the contraction (gathered data rows
// or activations), W across it.  Pieces of A are one load whatever the length of its rows, W is read in pieces where its rows start
// at multiples of four and lane by lane elsewhere.  Element by element with the lanes four elements apart, and without the steps
// shared by four waves (launch_rows), odd shapes took two to three times as long, in us: 5 x 1227 -> 254, batch 128, 69 and now 19;
// 52 x 3072 -> 51, batch 42, 103 and 38; 47 x 1330 -> 184, batch 128, 134 and 61; bfloat16 5 x 3072 -> 82, batch 20, 81 and 29.
//
// Large layers on fp32 operands are bound by the fp32 matrix rate: 3072 -> 1024, batch 128, 32 workers
// 273 to 292 us, the matrix pipe busy 66 % of the time (64 x 64 blocks: 293 us; the 64 x 64 kernel with 4-byte loads and steps of 32
// before it: 367 us).  With the operands as three bfloat16 planes (split_fwd_kernel) 223 to 240 us on the same boxes, 3072-1024-10
// with it 679 instead of 716 us per iteration, 784-1024-10 with 64 workers 399 instead of 449 us; the hidden activations are then
// 8.6e-7 off their 64-bit values instead of 9.9e-7 (3072 terms; 1.5e-7 and 1.8e-7 with 100).  Bound there by the vector
// instructions of the split (55 % of a SIMD's cycles) beside the products (39 %); forcing the two into turns inside a wave, and eight
// waves instead of four, changed nothing.  Small bfloat16 layers are bound by the chain of steps: 784 -> 500 and 500 -> 300, batch
// 100, 16 workers 20 and 10 us (39 and 28 us with the earlier kernel, which multiplied the rounded operands by fp32 instructions).
#include "tile.h"

#include <type_traits>

namespace netmax {

struct TileFwd {
    const void *feats; const int64_t *row0; const int32_t *idx;      // first layer: gathered data rows
    const void *act;                                                  // else the activation below, [M][B][din]
    const float *X; int64_t woff; int M, B, din, dout, relu;
    float *out; uint16_t *out_bf16, *out_bf16_t;                      // [M][B][dout], and [M][dout][B]; each may be absent
};

// ReLU and the store of one element (bias added)
template <bool BF> __device__ __forceinline__ void tile_fwd_put(const TileFwd &p, int g, int row, int col, float z)
{
    if (p.relu) z = z > 0.0f ? z : 0.0f;
    if (col < p.dout && row < p.B) {
        const size_t q = ((size_t)g * p.B + row) * p.dout + col;
        if (p.out) p.out[q] = z;
        if constexpr (BF) {
            const uint16_t h = (uint16_t)bf16_bits(z);
            if (p.out_bf16) p.out_bf16[q] = h;
            if (p.out_bf16_t) p.out_bf16_t[((size_t)g * p.dout + col) * p.B + row] = h;
        }
    }
}
__device__ __forceinline__ float tile_fwd_bias(const TileFwd &p, int g, int col)
{
    return p.X[tiled_offset_quick(p.M, g, p.woff + (int64_t)p.din * p.dout + (col < p.dout ? col : p.dout - 1))];
}

// bias, ReLU and the store of a finished block
template <bool BF, int BM, int BN, int WM, int WN, int RI, int CJ>
__device__ __forceinline__ void tile_fwd_store(const TileFwd &p, int g, int m0, int n0, int wm, int wn, int lane, const tile_f32x16 (&acc)[RI][CJ])
{
#pragma unroll
    for (int j = 0; j < CJ; ++j) {
        const int col = n0 + wn * (BN / WN) + 32 * j + (lane & 31);
        const float bias = tile_fwd_bias(p, g, col);
#pragma unroll
        for (int i = 0; i < RI; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                tile_fwd_put<BF>(p, g, m0 + wm * (BM / WM) + 32 * i + tile_row(lane, v), col, acc[i][j][v] + bias);
    }
}

// The product of one block, operands as they are (BF: rounded to bfloat16).  smem: LDS for both.  Rows of A have four elements or
// more.  VW: rows of W start at multiples of four and four columns at a time are one load, otherwise a thread's loads are single
// floats, neighbouring lanes neighbouring columns.
template <bool BF, bool VW, int BM, int BN, int BK, int WM, int WN, int RI, int CJ>
__device__ __forceinline__ void tile_fwd_product(const TileFwd &p, int g, int m0, int n0, unsigned char *smem, tile_f32x16 (&acc)[RI][CJ])
{
    constexpr int NT = 64 * WM * WN, K4 = BK / 4;
    constexpr int NA = BM * K4 / NT, NB = BN * K4 / 4 / NT;           // pieces of A, 4 x 4 blocks of W per thread and step
    static_assert(NA * NT == BM * K4 && NB * NT == BN * K4 / 4, "every thread has the same share");
    static_assert(BK <= 128 && NT % BN == 0, "offsets inside a step; a column per thread");
    typedef TileLds<BF, BK> L;
    typedef typename L::elem elem;
    elem (*As)[L::PITCH] = reinterpret_cast<elem (*)[L::PITCH]>(smem);
    elem (*Bs)[L::PITCH] = reinterpret_cast<elem (*)[L::PITCH]>(smem + BM * L::PITCH * sizeof(elem));
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave / WN, wn = wave % WN;
    const int K = p.din;

    int64_t a_row[NA];                                                // element index of a piece at step 0 (row clamped)
    int a_m[NA], a_k[NA];
#pragma unroll
    for (int u = 0; u < NA; ++u) {
        const int c = t + u * NT;
        a_m[u] = c / K4;
        a_k[u] = c % K4 * 4;
        const int r = m0 + a_m[u] < p.B ? m0 + a_m[u] : p.B - 1;
        a_row[u] = p.feats ? (p.row0[g] + p.idx[(size_t)g * p.B + r]) * K : ((int64_t)g * p.B + r) * K;
    }
    // VW: a 4 x 4 block at rows b_k, columns b_n.  Otherwise four pieces of four rows of a column: 4 u + i at rows b_k[u] + i * NT / BN * 4
    constexpr int STRIPE = VW ? 0 : NT / BN * 4;
    int b_n[NB], b_k[NB], b_c[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        const int c = t + u * NT;
        b_n[u] = VW ? c % (BN / 4) * 4 : t % BN;
        b_k[u] = VW ? c / (BN / 4) * 4 : t / BN * 4 + u * 4 * STRIPE;
        const int want = n0 + b_n[u];                                 // columns past the end repeat the last one(s)
        b_c[u] = want < p.dout ? want : (VW ? p.dout - 4 : p.dout - 1);
    }
    Piece<BF> ra[NA];
    Piece<false> rb[NB][4];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            const int k = min(k0 + a_k[u], K - 4);
            if constexpr (BF) ra[u] = load_piece<true>((const uint16_t *)(p.feats ? p.feats : p.act) + a_row[u] + k, K - k);
            else ra[u] = load_piece<true>((const float *)(p.feats ? p.feats : p.act) + a_row[u] + k, K - k);
        }
        if constexpr (VW) {
#pragma unroll
            for (int u = 0; u < NB; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int k = k0 + b_k[u] + i < K ? k0 + b_k[u] + i : K - 1;
                    rb[u][i].v = load4(p.X + tiled_offset_quick(p.M, g, p.woff + (int64_t)k * p.dout + b_c[u]));
                }
        } else {
            const TileSpan w(p.M, g, p.woff + (int64_t)k0 * p.dout);
            const float *Xs = p.X + w.base;
            const uint32_t last = (uint32_t)min(K - 1 - k0, BK) * (uint32_t)p.dout;   // rows past the end repeat the last one
#pragma unroll
            for (int u = 0; u < NB; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        rb[u][i].v[e] = Xs[w.at(min((uint32_t)(b_k[u] + i * STRIPE + e) * (uint32_t)p.dout, last) + (uint32_t)b_c[u])];
        }
    };
    auto stash = [&](int k0) {
        // indices that exist from k on: 4 or more everywhere but in the last step
        const int left = K - k0;
#pragma unroll
        for (int u = 0; u < NA; ++u) put_piece(&As[a_m[u]][a_k[u]], piece_tail(ra[u], left - a_k[u]).v, 4);
#pragma unroll
        for (int u = 0; u < NB; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (VW) put_piece(&Bs[b_n[u] + e][b_k[u]], turned(rb[u], e), left - b_k[u]);
                else put_piece(&Bs[b_n[u]][b_k[u] + e * STRIPE], rb[u][e].v, left - b_k[u] - e * STRIPE);
            }
    };

    tile_clear(acc);
    fetch(0);
    for (int k0 = 0; k0 < K; k0 += BK) {
        __syncthreads();                                              // the previous step's reads of LDS are done
        stash(k0);
        __syncthreads();
        if (k0 + BK < K) fetch(k0 + BK);                              // travels while this step is multiplied
        tile_multiply<BK>(As, Bs, wm * (BM / WM), wn * (BN / WN), lane, acc);
    }
}

template <bool BF, int BM, int BN, int BK> constexpr int tile_fwd_lds()
{
    return (BM + BN) * TileLds<BF, BK>::PITCH * (int)sizeof(typename TileLds<BF, BK>::elem);
}

template <bool BF, bool VW, int BM, int BN, int BK, int WM, int WN>
__global__ void __launch_bounds__(64 * WM * WN) tile_fwd_kernel(TileFwd p)
{
    constexpr int RI = BM / WM / 32, CJ = BN / WN / 32;
    __shared__ __attribute__((aligned(16))) unsigned char smem[tile_fwd_lds<BF, BM, BN, BK>()];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wm = wave / WN, wn = wave % WN;
    const unsigned nblk = (unsigned)((p.dout + BN - 1) / BN), mblk = (unsigned)((p.B + BM - 1) / BM);
    int g;
    unsigned local;
    if (!decode_group(tile_block(), nblk * mblk, p.M, g, local)) return;
    const int n0 = (int)(local % nblk) * BN, m0 = (int)(local / nblk) * BM;
    tile_f32x16 acc[RI][CJ];
    tile_fwd_product<BF, VW, BM, BN, BK, WM, WN>(p, g, m0, n0, smem, acc);
    tile_fwd_store<BF, BM, BN, WM, WN>(p, g, m0, n0, wm, wn, lane, acc);
}

// Few blocks: 32 columns and RT x 32 batch rows, four waves that share the contraction, 32 indices of every 128 each.  A wave asks for both operands
// DEPTH steps of 64 bytes of a row of A (sixteen indices, bfloat16 32) ahead.  A crosses LDS by way of the wave's own buffer, so that four
// lanes read 64 neighbouring bytes of a row; a lane per row, in the layout of the matrix instruction, takes 64 turns of the cache a load instead of 16 (7 x
// 3072 -> 1024, batch 128, fp32 94 us, 71 with it).  A lane's operands of W are neighbouring rows of its column, each a load of a float (32
// lanes 128 bytes of a row).  No barrier until the waves' parts are added, in the order of the waves.  TAIL: indices behind the last
// whole step.  FAR: rows of W too far apart for 32-bit offsets.
// Bound by the chain of loads where there are few blocks, then by the fp32 matrix rate or the bytes of W.  Steps through LDS that all waves wait for
// twice (32 x 32 blocks, the same sums), and now, us: 5 x 3072 -> 858, batch 128, fp32 101 and 73; 28 x 768 -> 192, batch 23, 11.5 and 9.2; bfloat16 27 x
// 3072 -> 64, batch 32, 29 and 14; 37 x 3072 -> 192, batch 104, 44 and 30.
constexpr int SH_WAVES = 4, SH_THREADS = 64 * SH_WAVES;
template <bool BF, int RT, bool TAIL, int DEPTH, bool FAR = false>
__global__ void __launch_bounds__(SH_THREADS) wave_fwd_kernel(TileFwd p)
{
    constexpr int PE = BF ? 8 : 4, KS = 4 * PE, BM = 32 * RT, TP = BM + 8;     // elements of a piece; indices of a step
    typedef typename WaveOperand<BF>::piece piece;
    typedef typename WaveOperand<BF>::elem elem;
    constexpr int PART = SH_WAVES * 32 * WF_PITCH * 4, OPERAND = SH_WAVES * BM * 64;
    __shared__ __attribute__((aligned(16))) unsigned char smem[PART > OPERAND ? PART : OPERAND];
    __shared__ __attribute__((aligned(16))) uint16_t turn[BF ? WF_COLS : 1][TP];       // the block's activations, transposed
    const int t = threadIdx.x, lane = t & 63, row = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    piece *own = reinterpret_cast<piece *>(smem) + wave * (BM * 4);
    const unsigned nblk = (unsigned)((p.dout + WF_COLS - 1) / WF_COLS), mblk = (unsigned)((p.B + BM - 1) / BM);
    int g;
    unsigned local;
    if (!decode_group(tile_block(), nblk * mblk, p.M, g, local)) return;
    const int n0 = (int)(local % nblk) * WF_COLS, m0 = (int)(local / nblk) * BM, K = p.din;
    const float bias = tile_fwd_bias(p, g, n0 + (t & 31));            // for the end; requested first
    // this wave's steps, n-th of them: 32 indices of every 128
    constexpr int OF = 32 / KS;                                       // steps of 32 indices
    const int total = K / KS, n_mine = total / (4 * OF) * OF + min(max(total % (4 * OF) - OF * wave, 0), OF);
    auto step = [&](int n) {                                          // past the last one: that one again, never used
        n = min(n, n_mine - 1);
        return n / OF * (4 * OF) + OF * wave + n % OF;
    };
    const uint32_t skip = (uint32_t)(p.M - 1) << (TILE_SHIFT + 2), dout4 = (uint32_t)p.dout * 4u;
    const int col = min(n0 + row, p.dout - 1);                        // columns past the end repeat the last one
    const uint32_t w_first = (uint32_t)col * 4u + (uint32_t)(PE * half) * dout4;
    // index of a lane's element e of a step: pieces `half` and `half` + 2
    auto index = [&](int e) { return e < PE ? PE * half + e : PE * half + PE + e; };
    float w[DEPTH][2 * PE];
    piece a[DEPTH][RT][2];
    auto request_w = [&](int d, int s) {
        if constexpr (FAR) {
#pragma unroll
            for (int e = 0; e < 2 * PE; ++e) w[d][e] = p.X[tiled_offset_quick(p.M, g, p.woff + (int64_t)(s * KS + index(e)) * p.dout + col)];
            return;
        }
        const int64_t j0 = p.woff + (int64_t)s * KS * p.dout;
        const float *base = p.X + (((size_t)(j0 >> TILE_SHIFT) * p.M + g) << TILE_SHIFT);
        const uint32_t from = w_first + (uint32_t)(j0 & (TILE - 1)) * 4u;
#pragma unroll
        for (int e = 0; e < 2 * PE; ++e) {
            const uint32_t q = from + (uint32_t)(e < PE ? e : PE + e) * dout4;
            w[d][e] = *(const float *)((const char *)base + (__umul24(q >> (TILE_SHIFT + 2), skip) + q));
        }
    };
    if (n_mine > 0) {                                                 // these do not wait for the batch-row numbers
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) request_w(d, step(d));
    }
    // pieces that this lane brings into LDS: lane % 4 of rows lane / 4 and lane / 4 + 16 of every tile
    const int pa = lane & 3, pr = lane >> 2;
    const elem *a_row[RT][2];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int r = min(m0 + 32 * i + 16 * h + pr, p.B - 1);    // rows past the batch repeat the last one
            a_row[i][h] = (const elem *)(p.feats ? p.feats : p.act) + (p.feats ? p.row0[g] + p.idx[(size_t)g * p.B + r] : (int64_t)g * p.B + r) * K;
        }
    auto request_a = [&](int d, int s) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) a[d][i][h] = *reinterpret_cast<const typename WaveOperand<BF>::any *>(a_row[i][h] + (s * KS + PE * pa));
    };
    tile_f32x16 acc[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.0f;
    auto multiply = [&](const piece (&from)[RT][2], const float (&ws)[2 * PE]) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) own[32 * 4 * i + wave_unit(16 * h + pr, pa)] = from[i][h];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            piece x[RT];
#pragma unroll
            for (int i = 0; i < RT; ++i) x[i] = own[32 * 4 * i + wave_unit(row, 2 * j + half)];
            wave_multiply(x, ws + j * PE, acc);
        }
        __builtin_amdgcn_wave_barrier();
    };
    if (n_mine > 0) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) request_a(d, step(d));
    }
    if (n_mine > 0) {
        int done = 0;
        for (; done + DEPTH <= n_mine; done += DEPTH) {
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                multiply(a[d], w[d]);
                const int s = step(done + d + DEPTH);
                request_a(d, s);
                request_w(d, s);
            }
        }
#pragma unroll
        for (int d = 0; d < DEPTH - 1; ++d)
            if (done + d < n_mine) multiply(a[d], w[d]);
    }
    if (TAIL && wave == total % (4 * OF) / OF) {                      // what does not exist counts as zero
        const int from = total * KS, left = K - from;
        float wt[2 * PE];
        piece at[RT][2];
#pragma unroll
        for (int e = 0; e < 2 * PE; ++e) wt[e] = p.X[tiled_offset_quick(p.M, g, p.woff + (int64_t)min(from + index(e), K - 1) * p.dout + col)];
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                elem x[PE];
#pragma unroll
                for (int e = 0; e < PE; ++e) x[e] = a_row[i][h][min(from + PE * pa + e, K - 1)];
                if constexpr (BF) {
#pragma unroll
                    for (int e = 0; e < PE; e += 2)
                        at[i][h][e / 2] = (PE * pa + e < left ? (uint32_t)x[e] : 0u) | (PE * pa + e + 1 < left ? (uint32_t)x[e + 1] << 16 : 0u);
                } else {
#pragma unroll
                    for (int e = 0; e < PE; ++e) at[i][h][e] = PE * pa + e < left ? x[e] : 0.0f;
                }
            }
#pragma unroll
        for (int e = 0; e < 2 * PE; ++e) wt[e] = index(e) < left ? wt[e] : 0.0f;
        multiply(at, wt);
    }
    __syncthreads();                                                  // the operands' space becomes the parts
    float (*part)[32][WF_PITCH] = reinterpret_cast<float (*)[32][WF_PITCH]>(smem);
    const int c = t & 31;
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        if (i > 0) __syncthreads();                                   // the tile before has been read
#pragma unroll
        for (int v = 0; v < 16; ++v) part[wave][tile_row(lane, v)][row] = acc[i][v];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 16 / SH_WAVES; ++u) {
            const int r = (t >> 5) + 2 * SH_WAVES * u, b = m0 + 32 * i + r;
            float z = part[0][r][c];
#pragma unroll
            for (int k = 1; k < SH_WAVES; ++k) z += part[k][r][c];
            z += bias;
            if (p.relu) z = z > 0.0f ? z : 0.0f;
            const size_t at = ((size_t)g * p.B + b) * p.dout + n0 + c;
            const bool real = b < p.B && n0 + c < p.dout;
            if (real && p.out) p.out[at] = z;
            if constexpr (BF) {
                const uint16_t h = (uint16_t)bf16_bits(z);
                if (real && p.out_bf16) p.out_bf16[at] = h;
                turn[c][32 * i + r] = h;
            }
        }
    }
    if constexpr (BF) {
        if (!p.out_bf16_t) return;
        __syncthreads();
        const int rows = min(BM, p.B - m0), cols = min(WF_COLS, p.dout - n0);
        uint16_t *to = p.out_bf16_t + ((size_t)g * p.dout + n0) * p.B + m0;
        for (int e = t; e < cols * (BM / 8); e += SH_THREADS) {      // who asks for it has a batch of whole 32 rows
            const int c8 = e % (BM / 8) * 8, k = e / (BM / 8);
            if (c8 < rows) *reinterpret_cast<tile_u32x4 *>(to + (size_t)k * p.B + c8) = *reinterpret_cast<const tile_u32x4 *>(&turn[k][c8]);
        }
    }
}

// fp32 operands on the bfloat16 matrix instructions: 128 x 64 blocks, steps of 32, three planes of each operand in LDS, twice:
// the next step is split while this one is multiplied.
constexpr int SF_BM = 128, SF_BN = 64, SF_BK = 32, SF_WM = 2, SF_WN = 2, SF_THREADS = 256;
template <bool VW>
__global__ void __launch_bounds__(SF_THREADS, 2) split_fwd_kernel(TileFwd p)
{
    constexpr int BM = SF_BM, BN = SF_BN, BK = SF_BK, WM = SF_WM, WN = SF_WN, NT = SF_THREADS, RI = BM / WM / 32, CJ = BN / WN / 32, K4 = BK / 4;
    constexpr int NA = BM * K4 / NT;                                  // pieces of A per thread; of W two rows of four columns
    static_assert(NA * NT == BM * K4 && BN / 4 * (BK / 2) == NT && BK == 32, "every thread has the same share");
    constexpr int SA = BM * 32, SB = BN * SPLIT_PITCH, BUF = 3 * (SA + SB);      // elements
    constexpr int PLAIN = tile_fwd_lds<false, BM, BN, 64>();
    __shared__ __attribute__((aligned(16))) unsigned char smem[4 * BUF > PLAIN ? 4 * BUF : PLAIN];
    uint16_t *planes = reinterpret_cast<uint16_t *>(smem);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave / WN, wn = wave % WN;
    const unsigned nblk = (unsigned)((p.dout + BN - 1) / BN), mblk = (unsigned)((p.B + BM - 1) / BM);
    int g;
    unsigned local;
    if (!decode_group(tile_block(), nblk * mblk, p.M, g, local)) return;
    const int n0 = (int)(local % nblk) * BN, m0 = (int)(local / nblk) * BM;
    const int K = p.din;
    const float *in = (const float *)(p.feats ? p.feats : p.act);
    int64_t a_row[NA];                                                // element index of a piece at step 0 (row clamped)
    const int a_k = t % K4 * 4;                                       // NT is a multiple of K4: the same for all pieces of a thread
#pragma unroll
    for (int u = 0; u < NA; ++u) {
        const int m = m0 + (t + u * NT) / K4, r = m < p.B ? m : p.B - 1;
        a_row[u] = p.feats ? (p.row0[g] + p.idx[(size_t)g * p.B + r]) * K : ((int64_t)g * p.B + r) * K;
    }
    // VW: two rows of four columns.  Otherwise eight rows of a column: neighbouring lanes, neighbouring columns
    const int b_n = VW ? t / (BK / 2) * 4 : t % BN, b_k = VW ? t % (BK / 2) * 2 : t / BN * 8;
    static_assert(NT / BN * 8 == BK, "a column and eight rows per thread");
    const int b_c = n0 + b_n < p.dout ? n0 + b_n : (VW ? p.dout - 4 : p.dout - 1);     // columns past the end repeat the last one(s)
    Piece<false> ra[NA], rb[2];
    bool lost = false;                                                // an operand of this thread that its planes do not hold
    auto fetch = [&](int k0) {
        const int k = min(k0 + a_k, K - 4);
#pragma unroll
        for (int u = 0; u < NA; ++u) ra[u] = load_piece<true>(in + a_row[u] + k, 4);
        if constexpr (VW) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int kb = k0 + b_k + i < K ? k0 + b_k + i : K - 1;
                rb[i].v = load4(p.X + tiled_offset_quick(p.M, g, p.woff + (int64_t)kb * p.dout + b_c));
            }
        } else {
            const int from = k0 < K ? k0 : K - 1;                     // fetches past the end: the last row again
            const TileSpan w(p.M, g, p.woff + (int64_t)from * p.dout);
            const float *Xs = p.X + w.base;
            const uint32_t last = (uint32_t)min(K - 1 - from, BK) * (uint32_t)p.dout;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) rb[i].v[e] = Xs[w.at(min((uint32_t)(b_k + 4 * i + e) * (uint32_t)p.dout, last) + (uint32_t)b_c)];
        }
    };
    auto stash = [&](int k0, uint16_t *buf, auto whole) {             // whole: all indices of the step exist
        const int left = decltype(whole)::value ? BK : K - k0;
#pragma unroll
        for (int u = 0; u < NA; ++u)
            put_split(buf + split_at((t + u * NT) / K4, a_k), SA,
                      decltype(whole)::value ? ra[u].v : piece_tail(ra[u], left - a_k).v, lost);
        if constexpr (VW) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                put_split(buf + 3 * SA + (b_n + e) * SPLIT_PITCH + b_k, SB, left > b_k ? rb[0].v[e] : 0.0f, left > b_k + 1 ? rb[1].v[e] : 0.0f,
                          lost);
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i)
                put_split(buf + 3 * SA + b_n * SPLIT_PITCH + b_k + 4 * i, SB, first_of(rb[i].v, left - b_k - 4 * i), lost);
        }
    };
    tile_f32x16 acc[RI][CJ];
    tile_clear(acc);
    fetch(0);
    stash(0, planes, std::false_type{});
    fetch(BK);
    int k0 = 0, cur = 0;
    auto step = [&](auto whole) {
        __syncthreads();                                              // this step is in LDS, the step before has been read
        stash(k0 + BK, planes + (cur ^ 1) * BUF, whole);
        fetch(k0 + 2 * BK);                                           // past the end: the last index again
        const uint16_t *buf = planes + cur * BUF;
        split_multiply(buf, SA, buf + 3 * SA, SB, wm * (BM / WM), wn * (BN / WN), lane, acc);
        k0 += BK;
        cur ^= 1;
    };
    while (k0 + 2 * BK <= K) step(std::true_type{});                  // the step behind is whole
    while (k0 < K) step(std::false_type{});
    // again, in fp32: an operand that its planes do not hold, a sum that is not finite, or one so small that the products of the
    // lower planes come near the smallest number there is
    constexpr float FEW_BITS = 0x1p-100f;
    float watch = 0.0f;                                               // 0 or NaN
#pragma unroll
    for (int i = 0; i < RI; ++i)
#pragma unroll
        for (int j = 0; j < CJ; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                watch = fmaf(acc[i][j][v], 0.0f, watch);
                lost |= fabsf(acc[i][j][v]) < FEW_BITS && acc[i][j][v] != 0.0f;
            }
    if (__syncthreads_or(lost || !(watch == 0.0f)))
        tile_fwd_product<false, VW, BM, BN, 64, WM, WN>(p, g, m0, n0, smem, acc);
    tile_fwd_store<false, BM, BN, WM, WN>(p, g, m0, n0, wm, wn, lane, acc);
}

template <bool BF, bool VW, int BM, int BN, int BK, int WM, int WN>
static void launch_shape(hipStream_t s, const TileFwd &a)
{
    const unsigned blocks = (unsigned)((a.dout + BN - 1) / BN) * (unsigned)((a.B + BM - 1) / BM);
    hipLaunchKernelGGL((tile_fwd_kernel<BF, VW, BM, BN, BK, WM, WN>), tile_grid(grouped_grid(a.M, blocks)), dim3(64 * WM * WN), 0, s, a);
}

// Few workgroups are bound by the chain of steps: 32 x 32 blocks whose steps four waves share, until there are enough of the larger
// blocks.  Counted in 32 x 64 blocks; us per iteration, shared and the larger form, either side of each line (of the form with
// barriers that wave_fwd_kernel has replaced, which is slower throughout; the lines also separate two orders of sums and stay):
//   fp32, batch <= 32      96 x 784-515 (864) 287 and 304, 128 x 784-515 (1152) 381 and 385, 128 x 100-900 (1920) 104 and 104
//   fp32, batch <= 64      64 x 784-300 (640) 131 and 137, 96 x 784-300 (960) 190 and 178
//   fp32, more             24 x 784-512, batch 128 (768) 107 and 115, 48 x 784-512 (1536) 188 and 168; on the line (1024) 64 x 784-256
//                          135 and 131, 16 x 3072-1024 400 and 404, 8 x 3072-1024, batch 200 323 and 339
//   bfloat16               48 x 1227-254, batch 64 (384) 117 and 119, 31 x 3001-999, batch 20 (496) 577 and 590; 64 x 784-300, batch 50
//                          (640) 107 and 106, 48 x 784-515, batch 50 (864) 151 and 145
// Larger forms, bfloat16, batch > 64: 128 x 32 blocks while the 128 x 64 ones do not fill the chip: 31 x 784-500, batch 100 (248 of
// the latter) 97 and 102, 64 x 1000-300 (320) 145 and 143, 31 x 3001-999 (496) 755 and 710.
// 32-bit offsets do not reach over a step's rows of W.
static bool far_rows(const TileFwd &a) { return a.M > 2048 || ((32 * (int64_t)a.dout + TILE) / TILE + 1) * a.M * (TILE * 4) >= (int64_t)1 << 32; }
template <bool BF, int RT> static void launch_wave(hipStream_t s, const TileFwd &a)
{
    const unsigned n = (unsigned)((a.dout + WF_COLS - 1) / WF_COLS) * (unsigned)((a.B + 32 * RT - 1) / (32 * RT));
    const dim3 grid = tile_grid(grouped_grid(a.M, n)), block(SH_THREADS);
    const bool tail = a.din % (BF ? 32 : 16) != 0;
    if constexpr (RT == 1)
        if (far_rows(a)) {
            hipLaunchKernelGGL((wave_fwd_kernel<BF, 1, true, 2, true>), grid, block, 0, s, a);
            return;
        }
    // fp32, two steps ahead and three: 1330 indices 1.24 and 1.33 times as fast as the kernel before, 3072 1.22 and 1.48, 784 1.33 and 1.31
    if constexpr (!BF)
        if (a.din >= 1024) {
            if (tail) hipLaunchKernelGGL((wave_fwd_kernel<BF, RT, true, 3>), grid, block, 0, s, a);
            else hipLaunchKernelGGL((wave_fwd_kernel<BF, RT, false, 3>), grid, block, 0, s, a);
            return;
        }
    if (tail) hipLaunchKernelGGL((wave_fwd_kernel<BF, RT, true, 2>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((wave_fwd_kernel<BF, RT, false, 2>), grid, block, 0, s, a);
}
// Tiles of 32 batch rows in a workgroup: rounds of workgroups over the compute units times what one takes, in proportion to the tiles and a part that does
// not depend on them (of a tile's time fp32 0.3, bfloat16 1).  us, one, two and four tiles: bfloat16 48 x 3072 -> 256, batch 128 61, 53, 56, 64 x 101, 84,
// 70; fp32 12 x 3072 -> 1024, batch 60 62, 72, 16 x 87, 73, batch 128 12 x 126, 109.  fp32 never gains by four: 47 x 1330 -> 184, batch
// 128, 48, 52, 66.  Short contractions: one (124 indices, batch 128, 300 to 600 blocks 25 % faster than by that rule).
template <bool BF> static void launch_wave(hipStream_t s, const TileFwd &a)
{
    const int64_t cols = (int64_t)a.M * ((a.dout + WF_COLS - 1) / WF_COLS);
    auto cost = [&](int rt) { return (cols * ((a.B + 32 * rt - 1) / (32 * rt)) + MF_XCD * XCD_CUS - 1) / (MF_XCD * XCD_CUS) * (10 * rt + (BF ? 10 : 3)); };
    int rt = 1;
    for (int k = 2; k <= (BF ? 4 : 2) && a.din >= 384 && !far_rows(a); k *= 2)
        if (a.B > 16 * k && cost(k) < cost(rt)) rt = k;
    if (rt == 1) launch_wave<BF, 1>(s, a);
    else if (rt == 2) launch_wave<BF, 2>(s, a);
    else if constexpr (BF) launch_wave<BF, 4>(s, a);
}

static bool enough_blocks(int M, int B, int64_t din, int64_t dout, bool bf)
{
    return din >= 4 && M * ((dout + 63) / 64) * ((B + 31) / 32) >= (bf ? 512 : B > 32 && B <= 64 ? 641 : 1025);
}
bool tile_fwd_one_chain(const MlpPlan &p, int l) { return enough_blocks(p.M, p.B, p.dims[l], p.dims[l + 1], p.bf16 != 0); }

template <bool BF, bool VW> static void launch_rows(hipStream_t s, const TileFwd &a)
{
    const int64_t wide = (int64_t)a.M * ((a.dout + 63) / 64) * ((a.B + 127) / 128);
    if (!enough_blocks(a.M, a.B, a.din, a.dout, BF)) return launch_wave<BF>(s, a);
    if (a.B <= 32) launch_shape<BF, VW, 32, 64, 64, 1, 2>(s, a);
    else if (a.B <= 64) launch_shape<BF, VW, 64, 64, BF ? 128 : 64, 2, 2>(s, a);
    else if constexpr (!BF) {
        const unsigned n = (unsigned)((a.dout + SF_BN - 1) / SF_BN) * (unsigned)((a.B + SF_BM - 1) / SF_BM);
        hipLaunchKernelGGL((split_fwd_kernel<VW>), tile_grid(grouped_grid(a.M, n)), dim3(SF_THREADS), 0, s, a);
    }
    else if (wide <= MF_XCD * XCD_CUS) launch_shape<BF, VW, 128, 32, 128, 4, 1>(s, a);
    else launch_shape<BF, VW, 128, 64, 64, 2, 2>(s, a);
}

void launch_tile_fwd(hipStream_t s, const MlpPlan &p, int l, const float *X, bool need_t)
{
    const bool bf = p.bf16 != 0, last = l + 1 == p.n_layers;
    TileFwd a;
    a.feats = l == 0 ? p.feats : nullptr; a.row0 = p.row0; a.idx = p.idx;
    a.act = l == 0 ? nullptr : (bf ? (const void *)p.hb[l] : (const void *)p.act[l]);
    a.X = X; a.woff = p.woff[l]; a.M = p.M; a.B = p.B; a.din = (int)p.dims[l]; a.dout = (int)p.dims[l + 1]; a.relu = !last;
    a.out = (last || !bf) ? p.act[l + 1] : nullptr;
    a.out_bf16 = (bf && !last) ? p.hb[l + 1] : nullptr;
    a.out_bf16_t = (bf && !last && need_t) ? p.ht[l + 1] : nullptr;
    const bool vw = a.dout % 4 == 0 && a.woff % 4 == 0;               // pieces of W: four columns of a row that starts at a multiple of four
    if (bf) {
        if (vw) launch_rows<true, true>(s, a); else launch_rows<true, false>(s, a);
    } else {
        if (vw) launch_rows<false, true>(s, a); else launch_rows<false, false>(s, a);
    }
}

}  // namespace netmax
