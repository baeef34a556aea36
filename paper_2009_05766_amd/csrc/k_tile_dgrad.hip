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

// fp32 operands, few blocks: 32 columns (input features) and RT x 32 batch rows, eight waves that share the contraction.  Wave w takes the steps w, w + 8, ... of
// sixteen indices; rows of dZ and of W come in as 16-byte pieces, four lanes along a row, two steps ahead, and go through the wave's own LDS
// into the layout of the matrix instruction; the parts are added in the order of the waves.  V: pieces of W do not cross a layout tile.
// TAIL: indices behind the last whole step.
// Bound by one or two chains of loads where the other kernel waits for one at every step: 4 x 1000-1000, batch 20, 9.3 us (tile_dgrad_kernel 27), 13 x
// 301-1001, batch 60, 18 us (43).  (bfloat16 operands: k_chain.hip.)
constexpr int WD_DEPTH = 2, WF_WAVES = 8, WF_THREADS = 64 * WF_WAVES;
template <int RT, bool V, bool TAIL>
__global__ void __launch_bounds__(WF_THREADS) wave_dgrad_kernel(TileDgrad p)
{
    constexpr int KS = 16, BM = 32 * RT;
    constexpr int PART = WF_WAVES * 32 * WF_PITCH * 4, OPERAND = WF_WAVES * (BM + 32) * 64;
    __shared__ __attribute__((aligned(16))) unsigned char smem[PART > OPERAND ? PART : OPERAND];
    __shared__ float red[2 * WF_WAVES][WF_COLS];
    const int t = threadIdx.x, lane = t & 63, row = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    f32x4 *own = reinterpret_cast<f32x4 *>(smem) + wave * ((BM + 32) * 4);            // rows of dZ, then of W
    const unsigned nblk = (unsigned)((p.din + WF_COLS - 1) / WF_COLS), mblk = (unsigned)((p.B + BM - 1) / BM);
    int g;
    unsigned local;
    if (!decode_group(tile_block(), nblk * mblk, p.M, g, local)) return;
    const int n0 = (int)(local % nblk) * WF_COLS, m0 = (int)(local / nblk) * BM, K = p.dout;
    const int total = K / KS, n_mine = wave < total ? (total - wave + WF_WAVES - 1) / WF_WAVES : 0, s_last = wave + WF_WAVES * (n_mine - 1);
    // pieces that this lane brings into LDS: `pa` of rows pr and pr + 16 of every tile; rows and features past the end repeat the last one
    const int pa = lane & 3, pr = lane >> 2;
    int64_t z_row[RT][2], w_row[2];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) z_row[i][h] = ((int64_t)g * p.B + min(m0 + 32 * i + 16 * h + pr, p.B - 1)) * K;
#pragma unroll
    for (int h = 0; h < 2; ++h) w_row[h] = p.woff + (int64_t)min(n0 + 16 * h + pr, p.din - 1) * K;
    auto w4 = [&](int64_t j) { return load4_params<V>(p.X, p.M, g, j); };
    f32x4 z[WD_DEPTH][RT][2], w[WD_DEPTH][2];
    auto request = [&](int d, int s) {
        const int k = s * KS + 4 * pa;
#pragma unroll
        for (int h = 0; h < 2; ++h) w[d][h] = w4(w_row[h] + k);
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) z[d][i][h] = *reinterpret_cast<const tile_f32x4_any *>(p.dz + z_row[i][h] + k);
    };
    auto clamped = [&](int s) { return s < s_last ? s : s_last; };    // past the last step: that one again, never used
    if (n_mine > 0) {
#pragma unroll
        for (int d = 0; d < WD_DEPTH; ++d) request(d, clamped(wave + WF_WAVES * d));
    }
    // the input: this thread's rows t / 32 and 16 more of every tile, column t % 32
    const int c = t & 31, col = min(n0 + c, p.din - 1);
    float on[RT][2];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int u = 0; u < 2; ++u) on[i][u] = p.act[((size_t)g * p.B + min(m0 + 32 * i + (t >> 5) + 16 * u, p.B - 1)) * p.din + col];
    tile_f32x16 acc[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.0f;
    auto multiply = [&](const f32x4 (&zs)[RT][2], const f32x4 (&ws)[2]) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int i = 0; i < RT; ++i) own[32 * 4 * i + wave_unit(16 * h + pr, pa)] = zs[i][h];
            own[BM * 4 + wave_unit(16 * h + pr, pa)] = ws[h];
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int at = wave_unit(row, 2 * j + half);
            const f32x4 b = own[BM * 4 + at];
            f32x4 a[RT];
#pragma unroll
            for (int i = 0; i < RT; ++i) a[i] = own[32 * 4 * i + at];
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < RT; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[e], acc[i], 0, 0, 0);
        }
        __builtin_amdgcn_wave_barrier();
    };
    if (TAIL && wave == total % WF_WAVES) {                           // the wave whose turn it would be; what does not exist counts as zero
        const int k = total * KS + 4 * pa, left = K - k;
        f32x4 zt[RT][2], wt[2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x = p.X[tiled_offset_quick(p.M, g, w_row[h] + min(k + e, K - 1))];
                wt[h][e] = e < left ? x : 0.0f;
#pragma unroll
                for (int i = 0; i < RT; ++i) {
                    const float y = p.dz[z_row[i][h] + min(k + e, K - 1)];
                    zt[i][h][e] = e < left ? y : 0.0f;
                }
            }
        multiply(zt, wt);
    }
    if (n_mine > 0) {
        int done = 0;
        for (; done + WD_DEPTH <= n_mine; done += WD_DEPTH) {
#pragma unroll
            for (int d = 0; d < WD_DEPTH; ++d) {
                multiply(z[d], w[d]);
                request(d, clamped(wave + WF_WAVES * (done + d + WD_DEPTH)));
            }
        }
#pragma unroll
        for (int d = 0; d < WD_DEPTH - 1; ++d)
            if (done + d < n_mine) multiply(z[d], w[d]);
    }
    __syncthreads();                                                  // the operands' space becomes the parts
    float (*part)[32][WF_PITCH] = reinterpret_cast<float (*)[32][WF_PITCH]>(smem);
    float csum = 0.0f;
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        if (i > 0) __syncthreads();                                   // the tile before has been read
#pragma unroll
        for (int v = 0; v < 16; ++v) part[wave][tile_row(lane, v)][row] = acc[i][v];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int r = (t >> 5) + 16 * u, b = m0 + 32 * i + r;
            float d = part[0][r][c];
#pragma unroll
            for (int k = 1; k < WF_WAVES; ++k) d += part[k][r][c];
            d = on[i][u] > 0.0f && b < p.B ? d : 0.0f;
            csum += d;
            if (b < p.B && n0 + c < p.din) p.out[((size_t)g * p.B + b) * p.din + n0 + c] = d;
        }
    }
    red[t >> 5][c] = csum;
    __syncthreads();
    if (mblk == 1 && t < WF_COLS && n0 + t < p.din) {
        float s = red[0][t];
#pragma unroll
        for (int k = 1; k < 2 * WF_WAVES; ++k) s += red[k][t];
        p.G[tiled_offset_quick(p.M, g, p.boff + n0 + t)] = s;
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

template <int RT> static bool launch_wave(hipStream_t s, const TileDgrad &a)
{
    const unsigned mblk = (unsigned)((a.B + 32 * RT - 1) / (32 * RT)), blocks = (unsigned)((a.din + WF_COLS - 1) / WF_COLS) * mblk;
    const dim3 grid = tile_grid(grouped_grid(a.M, blocks)), block(WF_THREADS);
    const bool v = a.dout % 4 == 0 && a.woff % 4 == 0, tail = a.dout % 16 != 0;
    if (v && tail) hipLaunchKernelGGL((wave_dgrad_kernel<RT, true, true>), grid, block, 0, s, a);
    else if (v) hipLaunchKernelGGL((wave_dgrad_kernel<RT, true, false>), grid, block, 0, s, a);
    else if (tail) hipLaunchKernelGGL((wave_dgrad_kernel<RT, false, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((wave_dgrad_kernel<RT, false, false>), grid, block, 0, s, a);
    return mblk == 1;
}

// Whether wave_dgrad_kernel takes a layer: few blocks of 32 columns (of all workers, times the batch's parts of 128 rows).  The two kernels add in
// different orders: batches of asynchronous steps go by one number of workers whatever their own, so that a step's errors don't depend on the
// steps beside it.  us, it and the other kernel, either side of each line:
//   batch <= 32    48 x 1000-300 (1536 blocks) 21.6 and 24.6, 64 x (2048) 27.2 and 27.1
//   batch <= 64    8 x 1000-300 (256) 8.8 and 11.7, 12 x (384) 12.9 and 12.0; many outputs 16 x 1000-1000 (512) 28.1 and 29.3, 32 x (1024) 56 and 52
//   more           many outputs 8 x 1000-1000 (256) 29.6 and 31.1, 12 x (384) 53 and 52
// Rows of W that start anywhere cost the other kernel a load a float:
//   batch <= 64    102 x 301-1001 (1020) 76 and 81, 51 x 301-102 (510) 11.2 and 10.4
//   more           128 x 102-602 (512) 43 and 51, 128 x 102-301 30.2 and 29.4, 64 x 102-301 (256) 16 and 23
static bool wave_dgrad_pays(const TileDgrad &a, int M)
{
    const int64_t K = a.dout, blocks = (int64_t)M * ((a.din + WF_COLS - 1) / WF_COLS) * ((a.B + 127) / 128);
    const bool any = K % 4 != 0 || a.woff % 4 != 0, deep = K >= (any ? 256 : 640);
    if (a.B <= 32) return blocks <= 1536;
    if (a.B <= 64) return blocks <= (!deep ? 256 : any ? 1024 : 512);
    return any ? blocks <= (K >= 480 ? 512 : 256) : deep && blocks <= 256;
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
    if (!bf && wave_dgrad_pays(a, p.M_rule)) {
        if (a.B <= 32) return launch_wave<1>(s, a);
        return a.B <= 64 ? launch_wave<2>(s, a) : launch_wave<4>(s, a);
    }
    const bool v = a.dout % 4 == 0 && a.woff % 4 == 0;               // pieces of rows of dZ and W: aligned, none past the end of a row
    if (bf) return v ? launch_rows<true, true>(s, a) : launch_rows<true, false>(s, a);
    return v ? launch_rows<false, true>(s, a) : launch_rows<false, false>(s, a);
}

}  // namespace netmax
