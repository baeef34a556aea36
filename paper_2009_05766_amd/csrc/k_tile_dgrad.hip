// Error of the layer below, dA = (dZ W^T) where A > 0, of a layer of any shape for all workers (the stochastic gradient of
// Algorithm 2's first-step update): the tiled kernel for what the kernels of k_grad_mfma.hip do not take.
//
// A workgroup takes BM batch rows and BN input features of one worker; both operands are contiguous along the contraction
// (rows of dZ, rows of W).  If its rows are the whole batch it also adds up the columns of dA, the bias gradient of the layer
// below, in a fixed order.
#include "tile.h"

namespace netmax {

struct TileDgrad {
    const float *dz, *X; int64_t woff; int M, B, din, dout;
    const float *act; const uint16_t *act_bf16;                       // this layer's input (ReLU mask), one of the two
    float *out; uint16_t *out_bf16, *out_bf16_t;                      // [M][B][din], and [M][din][B]; the latter two may be absent
    float *G; int64_t boff;                                           // bias of the layer below inside a gradient row
};

template <bool BF, bool V, int BM, int BN, int BK, int WM, int WN>
__global__ void __launch_bounds__(64 * WM * WN) tile_dgrad_kernel(TileDgrad p)
{
    constexpr int NT = 64 * WM * WN, RI = BM / WM / 32, CJ = BN / WN / 32, K4 = BK / 4;
    constexpr int NA = BM * K4 / NT, NB = BN * K4 / NT;               // pieces per thread and step
    static_assert(NA * NT == BM * K4 && NB * NT == BN * K4, "every thread has the same share");
    typedef TileLds<BF, BK> L;
    typedef typename L::elem elem;
    __shared__ __attribute__((aligned(16))) elem As[BM][L::PITCH];
    __shared__ __attribute__((aligned(16))) elem Bs[BN][L::PITCH];
    __shared__ float red[WM][BN];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave / WN, wn = wave % WN;
    const unsigned nblk = (unsigned)((p.din + BN - 1) / BN), mblk = (unsigned)((p.B + BM - 1) / BM);
    int g;
    unsigned local;
    if (!decode_group(tile_block(), nblk * mblk, p.M, g, local)) return;
    const int n0 = (int)(local % nblk) * BN, m0 = (int)(local / nblk) * BM;
    const int K = p.dout;

    const float *a_row[NA];
    int64_t b_row[NB];
#pragma unroll
    for (int u = 0; u < NA; ++u) {
        const int m = m0 + (t + u * NT) / K4;
        a_row[u] = p.dz + ((size_t)g * p.B + (m < p.B ? m : p.B - 1)) * K;
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        const int c = n0 + (t + u * NT) / K4;
        b_row[u] = p.woff + (int64_t)(c < p.din ? c : p.din - 1) * K;
    }
    const int k_own = t % K4 * 4;                                     // NT is a multiple of K4: the same for all pieces of a thread
    static_assert(NT % K4 == 0, "one contraction offset per thread");
    Piece<false> ra[NA], rb[NB];
    auto fetch = [&](int k0) {
        int k = k0 + k_own;
        k = k < K ? k : (V ? K - 4 : K - 1);
#pragma unroll
        for (int u = 0; u < NA; ++u) ra[u] = load_piece<V>(a_row[u] + k, K - k);
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            if constexpr (V) rb[u] = load_piece<true>(p.X + tiled_offset_quick(p.M, g, b_row[u] + k), 4);
            else {
#pragma unroll
                for (int e = 0; e < 4; ++e) rb[u].v[e] = p.X[tiled_offset_quick(p.M, g, b_row[u] + (k + e < K ? k + e : K - 1))];
            }
        }
    };
    auto stash = [&](int k0) {
        const int left = K - k0 - k_own;
#pragma unroll
        for (int u = 0; u < NA; ++u) put_piece(&As[(t + u * NT) / K4][k_own], ra[u].v, left);
#pragma unroll
        for (int u = 0; u < NB; ++u) put_piece(&Bs[(t + u * NT) / K4][k_own], rb[u].v, left);
    };
    tile_f32x16 acc[RI][CJ];
    tile_clear(acc);
    fetch(0);
    for (int k0 = 0; k0 < K; k0 += BK) {
        __syncthreads();                                              // the previous step's reads of LDS are done
        stash(k0);
        __syncthreads();
        if (k0 + BK < K) fetch(k0 + BK);                              // travels while this step is multiplied
        tile_multiply<BK>(As, Bs, wm * (BM / WM), wn * (BN / WN), lane, acc);
    }
#pragma unroll
    for (int j = 0; j < CJ; ++j) {
        const int nl = wn * (BN / WN) + 32 * j + (lane & 31), col = n0 + nl;
        const int cc = col < p.din ? col : p.din - 1;
        float csum = 0.0f;
#pragma unroll
        for (int i = 0; i < RI; ++i) {
            bool on[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {                            // all masks requested before the first is used
                const int row = m0 + wm * (BM / WM) + 32 * i + tile_row(lane, v);
                const size_t q = ((size_t)g * p.B + (row < p.B ? row : p.B - 1)) * p.din + cc;
                on[v] = BF ? bf16_positive(p.act_bf16[q]) : p.act[q] > 0.0f;
                on[v] = on[v] && row < p.B;
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = m0 + wm * (BM / WM) + 32 * i + tile_row(lane, v);
                const float d = on[v] ? acc[i][j][v] : 0.0f;
                csum += d;
                if (col < p.din && row < p.B) {
                    const size_t q = ((size_t)g * p.B + row) * p.din + col;
                    p.out[q] = d;
                    if (BF && p.out_bf16) {
                        const uint16_t h = (uint16_t)bf16_bits(d);
                        p.out_bf16[q] = h;
                        p.out_bf16_t[((size_t)g * p.din + col) * p.B + row] = h;
                    }
                }
            }
        }
        csum += __shfl_xor(csum, 32);
        if (lane < 32) red[wm][nl] = csum;
    }
    if (mblk == 1) {
        __syncthreads();
        if (t < BN && n0 + t < p.din) {
            float s = red[0][t];
#pragma unroll
            for (int w = 1; w < WM; ++w) s += red[w][t];
            p.G[tiled_offset_quick(p.M, g, p.boff + n0 + t)] = s;
        }
    }
}

template <bool BF, bool V, int BM, int BN, int BK, int WM, int WN>
static bool launch_shape(hipStream_t s, const TileDgrad &a)
{
    const unsigned mblk = (unsigned)((a.B + BM - 1) / BM), blocks = (unsigned)((a.din + BN - 1) / BN) * mblk;
    hipLaunchKernelGGL((tile_dgrad_kernel<BF, V, BM, BN, BK, WM, WN>), tile_grid(grouped_grid(a.M, blocks)), dim3(64 * WM * WN), 0, s, a);
    return mblk == 1;
}

// Few workgroups are bound by the chain of steps, not by what a step costs: longer steps, narrower blocks, until there are about as
// many of the wider blocks as half the compute units (bfloat16: as all of them).  us per iteration, 128 x 32 and 128 x 64 blocks,
// number of the latter: fp32 16 x 784-500-300, batch 100 (128) 134.5 and 135.7, 24 x 784-500-300 (192) 188 and 182, 31 x 300-1000-300,
// batch 128 (496) 261 and 243; bfloat16 32 x 784-500-300 (256) 147.5 and 149, 40 x (320) 180 and 177, 56 x (448) 236 and 230.
template <bool BF, bool V> static bool launch_rows(hipStream_t s, const TileDgrad &a)
{
    static_assert(TILE_DGRAD_BATCH == 128, "the rows of the largest block below");
    constexpr int LONG = BF ? 128 : 64;
    const int64_t wide = (int64_t)a.M * ((a.din + 63) / 64) * ((a.B + 127) / 128);
    if (a.B <= 32) return launch_shape<BF, V, 32, 64, 64, 1, 2>(s, a);
    if (a.B <= 64) return launch_shape<BF, V, 64, 64, LONG, 2, 2>(s, a);
    if (wide <= (BF ? 256 : 128)) return launch_shape<BF, V, 128, 32, 128, 4, 1>(s, a);
    return launch_shape<BF, V, 128, 64, 64, 2, 2>(s, a);
}

bool launch_tile_dgrad(hipStream_t s, const MlpPlan &p, int l, const float *X, float *G, int cur, bool below_fast)
{
    const bool bf = p.bf16 != 0;
    TileDgrad a;
    a.dz = p.dz[cur]; a.X = X; a.woff = p.woff[l]; a.M = p.M; a.B = p.B; a.din = (int)p.dims[l]; a.dout = (int)p.dims[l + 1];
    a.act = bf ? nullptr : p.act[l]; a.act_bf16 = bf ? p.hb[l] : nullptr;
    a.out = p.dz[cur ^ 1];
    a.out_bf16 = (bf && below_fast) ? p.dzb[cur ^ 1] : nullptr;
    a.out_bf16_t = (bf && below_fast) ? p.dzt[cur ^ 1] : nullptr;
    a.G = G; a.boff = p.woff[l - 1] + p.dims[l - 1] * p.dims[l];
    const bool v = a.dout % 4 == 0 && a.woff % 4 == 0;               // pieces of rows of dZ and W: aligned, none past the end of a row
    if (bf) return v ? launch_rows<true, true>(s, a) : launch_rows<true, false>(s, a);
    return v ? launch_rows<false, true>(s, a) : launch_rows<false, false>(s, a);
}

}  // namespace netmax
