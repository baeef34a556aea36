// Weight gradient dW = A^T dZ of a layer of any shape for all workers (the stochastic gradient of Algorithm 2's first-step
// update): the tiled kernel for what the kernels of k_grad_mfma.hip and k_grad_f32.hip do not take.
//
// A workgroup takes 64 input features and BN outputs of one worker; the contraction runs over the batch, both operands lie
// across it in memory.  The block is turned through LDS and leaves as row pieces of BN floats.
// 3072 x 1024, batch 128, 32 workers, fp32: 312 us (402 us with 64 x 64 blocks, 4-byte loads and 128-byte row pieces);
// 784 x 500 and 500 x 300, batch 100, 16 workers, bfloat16: 22 us together (54 us with fp32 instructions).
#include "tile.h"

namespace netmax {

struct TileWgrad {
    const void *feats; const int64_t *row0; const int32_t *idx;      // first layer: gathered data rows
    const void *act;                                                  // else the activation below, [M][B][din]
    const float *dz; int M, B, din, dout; int64_t woff; float *G;
};

constexpr int TW_BM = 64, TW_BK = 32, TW_THREADS = 256;

template <bool BF, bool VA, bool VZ, int BN>
__global__ void __launch_bounds__(TW_THREADS) tile_wgrad_kernel(TileWgrad p)
{
    constexpr int BM = TW_BM, BK = TW_BK, NT = TW_THREADS, CJ = BN / 64, K4 = BK / 4;
    constexpr int BLOCKS_A = BM / 4 * K4, NB = BN / 4 * K4 / NT;      // 4 x 4 blocks
    static_assert(BLOCKS_A == NT / 2 && NB * NT == BN / 4 * K4, "half a block of A per thread, whole ones of dZ");
    typedef TileLds<BF, BK> L;
    typedef typename L::elem elem;
    constexpr int TP = BN + 4;                                        // floats per row of the staged result
    constexpr int OPERANDS = (BM + BN) * L::PITCH * (int)sizeof(elem), RESULT = BM * TP * 4;
    __shared__ __attribute__((aligned(16))) unsigned char smem[OPERANDS > RESULT ? OPERANDS : RESULT];
    elem (*As)[L::PITCH] = reinterpret_cast<elem (*)[L::PITCH]>(smem);
    elem (*Bs)[L::PITCH] = reinterpret_cast<elem (*)[L::PITCH]>(smem + BM * L::PITCH * sizeof(elem));
    float (*T)[TP] = reinterpret_cast<float (*)[TP]>(smem);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 1, wn = wave & 1;
    const unsigned nblk = (unsigned)((p.dout + BN - 1) / BN), mblk = (unsigned)((p.din + BM - 1) / BM);
    int g;
    unsigned local;
    if (!decode_group(blockIdx.x, nblk * mblk, p.M, g, local)) return;
    const int n0 = (int)(local % nblk) * BN, f0 = (int)(local / nblk) * BM;
    const int K = p.B;

    // A: half a 4 x 4 block per thread (two batch rows of four features); lanes l and l + 32 of a wave share a block's features
    const int a_m = (t & 15) * 4, a_k = (t >> 4) * 2;                 // 16 lanes along the 64 features, 16 pairs of batch rows
    int a_f = f0 + a_m;
    a_f = a_f < p.din ? a_f : (VA ? p.din - 4 : p.din - 1);
    const int a_have = p.din - a_f;
    const int64_t base_row = p.feats ? p.row0[g] : (int64_t)g * K;
    const int32_t *rows = p.feats ? p.idx + (size_t)g * K : nullptr;
    int b_n[NB], b_k[NB], b_c[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        const int c = t + u * NT;
        b_n[u] = c % (BN / 4) * 4;
        b_k[u] = c / (BN / 4) * 4;
        const int want = n0 + b_n[u];
        b_c[u] = want < p.dout ? want : (VZ ? p.dout - 4 : p.dout - 1);
    }
    const float *zg = p.dz + (size_t)g * K * p.dout;
    int32_t row_of[2];                                                // batch rows of the coming step, asked for a step ahead
    auto fetch_rows = [&](int k0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int b = k0 + a_k + i < K ? k0 + a_k + i : K - 1;
            row_of[i] = rows ? rows[b] : b;
        }
    };
    Piece<BF> ra[2];
    Piece<false> rb[NB][4];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < NB; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int b = k0 + b_k[u] + i < K ? k0 + b_k[u] + i : K - 1;
                rb[u][i] = load_piece<VZ>(zg + (size_t)b * p.dout + b_c[u], p.dout - b_c[u]);
            }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int64_t q = (base_row + row_of[i]) * p.din + a_f;
            if constexpr (BF) ra[i] = load_piece<VA>((const uint16_t *)(p.feats ? p.feats : p.act) + q, a_have);
            else ra[i] = load_piece<VA>((const float *)(p.feats ? p.feats : p.act) + q, a_have);
        }
    };
    auto stash = [&](int k0) {
        const int left = K - k0;
        // two neighbouring k of a feature: one 64-bit (32-bit) word of its row
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (BF) {
                uint32_t h = piece_bits(ra[0], e) | (piece_bits(ra[1], e) << 16);
                h = left - a_k >= 2 ? h : (left - a_k == 1 ? h & 0xFFFFu : 0u);
                *reinterpret_cast<uint32_t *>(&As[a_m + e][a_k]) = h;
            } else {
                typedef float f32x2 __attribute__((ext_vector_type(2)));
                f32x2 v = {left - a_k >= 1 ? piece_f32(ra[0], e) : 0.0f, left - a_k >= 2 ? piece_f32(ra[1], e) : 0.0f};
                *reinterpret_cast<f32x2 *>(&As[a_m + e][a_k]) = v;
            }
        }
#pragma unroll
        for (int u = 0; u < NB; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) put_piece(&Bs[b_n[u] + e][b_k[u]], turned(rb[u], e), left - b_k[u]);
    };
    tile_f32x16 acc[1][CJ];
    tile_clear(acc);
    fetch_rows(0);
    fetch(0);
    fetch_rows(BK);
    for (int k0 = 0; k0 < K; k0 += BK) {
        __syncthreads();                                              // the previous step's reads of LDS are done
        stash(k0);
        __syncthreads();
        if (k0 + BK < K) {                                            // travels while this step is multiplied
            fetch(k0 + BK);
            fetch_rows(k0 + 2 * BK);
        }
        tile_multiply<BK>(As, Bs, 32 * wm, (BN / 2) * wn, lane, acc);
    }
    __syncthreads();                                                  // the operands' space becomes the staged result
#pragma unroll
    for (int j = 0; j < CJ; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) T[32 * wm + tile_row(lane, v)][(BN / 2) * wn + 32 * j + (lane & 31)] = acc[0][j][v];
    __syncthreads();
    if constexpr (VZ) {
        constexpr int PER_ROW = BN / 4, ROWS = NT / PER_ROW;
        const int c = (t % PER_ROW) * 4, r_in = t / PER_ROW;
        if (n0 + c < p.dout) {
#pragma unroll
            for (int pass = 0; pass < BM / ROWS; ++pass) {
                const int r = pass * ROWS + r_in;
                if (f0 + r < p.din)
                    store4_stream(p.G + tiled_offset_quick(p.M, g, p.woff + (int64_t)(f0 + r) * p.dout + n0 + c),
                                  *reinterpret_cast<const f32x4 *>(&T[r][c]));
            }
        }
    } else {
        constexpr int ROWS = NT / BN;
        const int c = t % BN, r_in = t / BN;
        if (n0 + c < p.dout) {
#pragma unroll 8
            for (int pass = 0; pass < BM / ROWS; ++pass) {
                const int r = pass * ROWS + r_in;
                if (f0 + r < p.din)
                    __builtin_nontemporal_store(T[r][c], p.G + tiled_offset_quick(p.M, g, p.woff + (int64_t)(f0 + r) * p.dout + n0 + c));
            }
        }
    }
}

template <bool BF, bool VA, bool VZ> static void launch_cols(hipStream_t s, const TileWgrad &a)
{
    const unsigned mblk = (unsigned)((a.din + TW_BM - 1) / TW_BM);
    const unsigned blocks = (unsigned)((a.dout + 127) / 128) * mblk;
    hipLaunchKernelGGL((tile_wgrad_kernel<BF, VA, VZ, 128>), dim3(grouped_grid(a.M, blocks)), dim3(TW_THREADS), 0, s, a);
}

void launch_tile_wgrad(hipStream_t s, const MlpPlan &p, int l, float *G, int cur)
{
    const bool bf = p.bf16 != 0;
    TileWgrad a;
    a.feats = l == 0 ? p.feats : nullptr; a.row0 = p.row0; a.idx = p.idx;
    a.act = l == 0 ? nullptr : (bf ? (const void *)p.hb[l] : (const void *)p.act[l]);
    a.dz = p.dz[cur]; a.M = p.M; a.B = p.B; a.din = (int)p.dims[l]; a.dout = (int)p.dims[l + 1]; a.woff = p.woff[l]; a.G = G;
    const bool va = a.din % 4 == 0 && reinterpret_cast<uintptr_t>(a.feats ? a.feats : a.act) % (bf ? 8 : 16) == 0;
    const bool vz = a.dout % 4 == 0 && a.woff % 4 == 0;              // rows of dZ and of dW start at multiples of 16 bytes
    if (bf) {
        if (va) { if (vz) launch_cols<true, true, true>(s, a); else launch_cols<true, true, false>(s, a); }
        else { if (vz) launch_cols<true, false, true>(s, a); else launch_cols<true, false, false>(s, a); }
    } else {
        if (va) { if (vz) launch_cols<false, true, true>(s, a); else launch_cols<false, true, false>(s, a); }
        else { if (vz) launch_cols<false, false, true>(s, a); else launch_cols<false, false, false>(s, a); }
    }
}

}  // namespace netmax
