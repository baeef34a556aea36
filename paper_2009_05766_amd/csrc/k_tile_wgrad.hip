// Weight gradient dW = A^T dZ of a layer of any shape for all workers (the stochastic gradient of Algorithm 2's first-step
// update): the tiled kernel for what the kernels of k_grad_mfma.hip and k_grad_f32.hip do not take.
//
// A workgroup takes 64 input features and 64 or 128 outputs of one worker; the contraction runs over the batch, both operands lie
// across it in memory.  The block is turned through LDS and leaves as pieces of rows.
// Rows of any length are read in pieces of four elements: 52 workers 3072 x 51, batch 42, fp32 25 us (50 us element by element, the
// lanes four apart, in blocks of 128 columns; 32 us with the 64 x 64 blocks and 4-byte loads before that).
// 3072 x 1024, batch 128, 32 workers, fp32: 311 us (402 us with 64 x 64 blocks, 4-byte loads and 128-byte row pieces);
// 784 x 500 and 500 x 300, batch 100, 16 workers, bfloat16: 21 us together (54 us with fp32 instructions).
//
// UPDATE (fp32 operands, aligned rows): the block's columns also get the momentum step and the mix (Eq. (c0), (c1)).  480 us
// at the first shape (median of 30 calls in a row; 509 us of the first six), 2.46 GB moved, 5.1 TB/s, against 311 us and 314 us for
// the separate mix.  Bound by how well the fp32 matrix
// instructions (180 us) and the memory traffic (390 us at the mix kernel's rate) overlap.  What mattered, per iteration of that
// network: blocks worker by worker (block by block over the workers, as the mix orders its tiles, fetches 2.0 instead of 1.25 GB:
// every block's operands again); the blocks of a strip side by side and not one after the other in a workgroup (755 against 880
// us: the pieces of a layout tile should leave together); x and v asked for behind the last operands, the peer's x behind the
// products (716 us; all ahead of the operands of the second step 817 us, all behind the last operands 722 us).
#include "mix_subset.h"
#include "tile.h"

namespace netmax {

struct TileWgrad {
    const void *feats; const int64_t *row0; const int32_t *idx;      // first layer: gathered data rows
    const void *act;                                                  // else the activation below, [M][B][din]
    const float *dz; int M, B, din, dout; int64_t woff; float *G;
    MixArgs mix;                                                      // UPDATE
    // and the other columns, by the first `other_blocks` workgroups (a multiple of the XCDs)
    const int32_t *tiles; int n_tiles; unsigned other_blocks; MixSkip skip;
};

// Rows of dZ and dW that start at multiples of 16 bytes; rows of at least four elements at any address; anything.  The first two read
// pieces of four elements, the first one writes them.
enum : int { TW_ALIGNED = 0, TW_PIECES = 1, TW_SINGLE = 2 };
constexpr int tw_threads(int BM, int BN, int WK) { return BM * BN * WK / 16; }        // waves of 32 x 32 blocks, WK of them share a step's batch rows
// (Four waves per SIMD; the narrow block with update would spill its pieces of x and v at that.)
template <bool BF, int MODE, bool UPDATE, int BM, int BN, int WK>
__global__ void __launch_bounds__(tw_threads(BM, BN, WK), UPDATE && BN == 64 ? 3 : 4) tile_wgrad_kernel(TileWgrad p)
{
    constexpr bool V = MODE != TW_SINGLE, VZ = MODE == TW_ALIGNED;
    static_assert(!UPDATE || VZ, "the update works on 128-bit pieces");
    constexpr int KW = WK > 1 ? 32 : 64, BK = KW * WK, NT = tw_threads(BM, BN, WK), RW = BM / 32, CW = BN / 32;
    constexpr int AR = BM * BK / 4 / NT;                              // batch rows of four features of A per step and thread
    static_assert((AR == 2 || AR == 4) && BN / 4 * (BK / 4) == NT, "half a 4 x 4 block of A or a whole one, and one of dZ");
    typedef TileLds<BF, BK> L;
    typedef typename L::elem elem;
    constexpr int TP = BN + 4;                                        // floats per row of the staged result
    constexpr int OPERANDS = (BM + BN) * L::PITCH * (int)sizeof(elem), RESULT = BM * TP * 4;
    __shared__ __attribute__((aligned(16))) unsigned char smem[OPERANDS > RESULT ? OPERANDS : RESULT];
    elem (*As)[L::PITCH] = reinterpret_cast<elem (*)[L::PITCH]>(smem);
    elem (*Zs)[L::PITCH] = reinterpret_cast<elem (*)[L::PITCH]>(smem + BM * L::PITCH * sizeof(elem));
    float (*T)[TP] = reinterpret_cast<float (*)[TP]>(smem);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave / CW % RW, wn = wave % CW;
    const int wk = __builtin_amdgcn_readfirstlane(wave / (RW * CW));
    const int nblk = (p.dout + BN - 1) / BN, mblk = (p.din + BM - 1) / BM;
    unsigned bid = tile_block();
    if constexpr (UPDATE) {
        if (bid < p.other_blocks) {
            const unsigned tile = bid / (unsigned)p.M;
            constexpr int OT = NT < TILE / 4 ? NT : TILE / 4;
            if (tile < (unsigned)p.n_tiles && t < OT) mix_subset_block<OT>(p.M, p.tiles[tile], (int)(bid - tile * (unsigned)p.M), (int)(bid - tile * (unsigned)p.M), p.skip, p.G, p.mix);
            return;
        }
        bid -= p.other_blocks;
    }
    int g;
    unsigned local;
    // worker by worker, the blocks of a strip side by side: the operands are read once, into one XCD's L2, and the pieces of a
    // layout tile leave at about the same time
    if (!decode_group(bid, (unsigned)(nblk * mblk), p.M, g, local)) return;
    const int f0 = (int)(local / (unsigned)nblk) * BM, n0 = (int)(local % (unsigned)nblk) * BN;
    const int K = p.B;

    // A: AR batch rows of four features per thread.  Pieces that reach over the end are read from four elements before it and
    // turned to their place; what is past the end is never stored
    const int a_m = t % (BM / 4) * 4, a_k = t / (BM / 4) * AR;
    const int a_left = p.din - f0 - a_m, a_f = V ? min(f0 + a_m, p.din - 4) : min(f0 + a_m, p.din - 1);
    const int64_t base_row = p.feats ? p.row0[g] : (int64_t)g * K;
    const int32_t *rows = p.feats ? p.idx + (size_t)g * K : nullptr;
    const int z_n = t % (BN / 4) * 4, z_k = t / (BN / 4) * 4;
    const int z_left = p.dout - n0 - z_n, z_c = V ? min(n0 + z_n, p.dout - 4) : min(n0 + z_n, p.dout - 1);
    const float *zg = p.dz + (size_t)g * K * p.dout + z_c;
    int32_t row_of[AR];                                               // batch rows of the coming step, asked for a step ahead
    auto fetch_rows = [&](int k0) {
#pragma unroll
        for (int i = 0; i < AR; ++i) {
            const int k = k0 + a_k + i < K ? k0 + a_k + i : K - 1;
            row_of[i] = rows ? rows[k] : k;
        }
    };
    Piece<BF> ra[AR];
    Piece<false> rz[4];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = k0 + z_k + i < K ? k0 + z_k + i : K - 1;
            rz[i] = load_piece<V>(zg + (size_t)k * p.dout, p.dout - z_c);
        }
#pragma unroll
        for (int i = 0; i < AR; ++i) {
            const int64_t q = (base_row + row_of[i]) * p.din + a_f;
            if constexpr (BF) ra[i] = load_piece<V>((const uint16_t *)(p.feats ? p.feats : p.act) + q, p.din - a_f);
            else ra[i] = load_piece<V>((const float *)(p.feats ? p.feats : p.act) + q, p.din - a_f);
        }
    };
    auto stash = [&](int k0) {
        const int left = K - k0;
        if constexpr (V) {
            if (a_left < 4) {
#pragma unroll
                for (int i = 0; i < AR; ++i) ra[i] = piece_tail(ra[i], a_left);
            }
            if (MODE == TW_PIECES && z_left < 4) {
#pragma unroll
                for (int i = 0; i < 4; ++i) rz[i] = piece_tail(rz[i], z_left);
            }
        }
        // neighbouring k of a feature: one word of its row, of two or four elements
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (AR == 4) {
                put_piece(&As[a_m + e][a_k], turned(ra, e), left - a_k);
            } else if constexpr (BF) {
                uint32_t h = piece_bits(ra[0], e) | (piece_bits(ra[1], e) << 16);
                h = left - a_k >= 2 ? h : (left - a_k == 1 ? h & 0xFFFFu : 0u);
                *reinterpret_cast<uint32_t *>(&As[a_m + e][a_k]) = h;
            } else {
                typedef float f32x2 __attribute__((ext_vector_type(2)));
                const f32x2 v = {left - a_k >= 1 ? ra[0].v[e] : 0.0f, left - a_k >= 2 ? ra[1].v[e] : 0.0f};
                *reinterpret_cast<f32x2 *>(&As[a_m + e][a_k]) = v;
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) put_piece(&Zs[z_n + e][z_k], turned(rz, e), left - z_k);
    };
    int m = g;
    float wi = 0.0f;
    if constexpr (UPDATE) {
        m = p.mix.peer[g];
        if ((unsigned)m >= (unsigned)p.M) m = g;                      // an index outside [0, M) is treated as a self draw
        wi = p.mix.w[(size_t)g * p.M + m];
    }
    const size_t peer_shift = ((size_t)m - (size_t)g) << TILE_SHIFT;  // from a worker's element to its peer's
    // the finished block by rows: 128-bit pieces (VZ) or single floats
    constexpr int W = VZ ? 4 : 1, PER_ROW = BN / W, ROWS = NT / PER_ROW, PASSES = BM / ROWS;
    const int oc = t % PER_ROW * W, orow = t / PER_ROW;
    const bool col_ok = n0 + oc < p.dout;
    const int64_t j0 = p.woff + (int64_t)f0 * p.dout + (col_ok ? n0 + oc : 0);
    const TileSpan rows_of_g(p.M, g, p.woff + (int64_t)f0 * p.dout);
    float *Gs = p.G + rows_of_g.base;
    auto own_of = [&](int u) {
        const int r = tile_opaque(u * ROWS + orow);
        return tiled_offset_quick(p.M, g, j0 + (int64_t)(f0 + r < p.din ? r : 0) * p.dout);
    };
    f32x4 ux[UPDATE ? PASSES : 1], uv[UPDATE ? PASSES : 1], up[UPDATE ? PASSES : 1];

    tile_f32x16 acc[1][1];
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
        if (UPDATE && k0 + BK >= K) {                                 // so do x and v of the block, behind the last operands
#pragma unroll
            for (int u = 0; u < PASSES; ++u) {
                const size_t own = own_of(u);
                ux[u] = load4(p.mix.Xcur + own);
                uv[u] = load4_stream(p.mix.V + own);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (WK == 1 || k0 + KW * wk < K) tile_multiply<KW>(As, Zs, 32 * wm, 32 * wn, lane, acc, K - k0 - KW * wk, KW * wk);
    }
    if constexpr (UPDATE) {
#pragma unroll
        for (int u = 0; u < PASSES; ++u) up[u] = load4(p.mix.Xcur + own_of(u) + peer_shift);
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();                                                  // the operands' space becomes the staged result
    if (wk == 0) {
#pragma unroll
        for (int v = 0; v < 16; ++v) T[32 * wm + tile_row(lane, v)][32 * wn + (lane & 31)] = acc[0][0][v];
    }
    __syncthreads();
    for (int w = 1; w < WK; ++w) {                                    // the other waves' parts, in their order
        if (wk == w) {
#pragma unroll
            for (int v = 0; v < 16; ++v) T[32 * wm + tile_row(lane, v)][32 * wn + (lane & 31)] += acc[0][0][v];
        }
        __syncthreads();
    }
    if (!col_ok) return;
#pragma unroll
    for (int u = 0; u < PASSES; ++u) {
        const int r = u * ROWS + orow;
        if (f0 + r < p.din) {
            if constexpr (VZ) {
                const size_t own = own_of(u);
                const f32x4 gr = *reinterpret_cast<const f32x4 *>(&T[r][oc]);
                if (!UPDATE || p.mix.keep_g) store4_stream(p.G + own, gr);
                if constexpr (UPDATE) {
                    f32x4 xn, vn;
                    momentum_mix4(ux[u], uv[u], gr, up[u], wi, p.mix.alpha, p.mix.mu, p.mix.wd, xn, vn);
                    store4_stream(p.mix.Xnext + own, xn);
                    store4_stream(p.mix.V + own, vn);
                }
            } else {
                Gs[rows_of_g.at((uint32_t)r * (uint32_t)p.dout + (uint32_t)(n0 + oc))] = T[r][oc];
            }
        }
    }
}

template <bool BF, int MODE, int BM, int BN, int WK> static void launch_block(hipStream_t s, TileWgrad &a, bool update)
{
    const dim3 grid = tile_grid(a.other_blocks + grouped_grid(a.M, (unsigned)((a.dout + BN - 1) / BN) * (unsigned)((a.din + BM - 1) / BM)));
    const dim3 block(tw_threads(BM, BN, WK));
    if constexpr (MODE == TW_ALIGNED && !BF)
        if (update) {
            hipLaunchKernelGGL((tile_wgrad_kernel<BF, MODE, true, BM, BN, WK>), grid, block, 0, s, a);
            return;
        }
    hipLaunchKernelGGL((tile_wgrad_kernel<BF, MODE, false, BM, BN, WK>), grid, block, 0, s, a);
}

// From a batch of 128 on and with few blocks, 32 x 32 blocks whose batch rows four waves share: four times as many compute units at
// work.  us per iteration, shared and 64 x 64 blocks, number of the latter: fp32 2 x 784-100 (26), batch 128 30 and 36, batch 785 82
// and 131; 9 x 784-100 (234) 35 and 37, 122 and 152; 16 x 784-100 (416) 40 and 37.5; bfloat16 2 x 1227-254 (160), batch 128 39.9 and
// 40.8; 9 x 784-100 34.5 and 33.8.
// Blocks of 64 columns where they leave less of a narrow layer empty (up to 64 columns, 129 to 192), and on fp32 rows that are not
// aligned, whose results leave as single floats either way.  us per iteration, 52 workers, with 64 and with 128 columns:
//   784-64, batch 100 49 and 59, 784-192 92 and 101, 784-150 bfloat16, batch 200 104 and 106; but 784-100, batch 42 57 and 51,
//   784-300 124 and 115, batch 200 216 and 226
//   rows not aligned, batch 200: 3072-51 190 and 249, 1227-254 262 and 273, 784-515 350 and 379; bfloat16 126 and 141, 173 and 169,
//   227 and 226
template <bool BF, int MODE> static void launch_cols(hipStream_t s, TileWgrad &a, bool update)
{
    const int64_t blocks = (int64_t)a.M * ((a.dout + 63) / 64) * ((a.din + 63) / 64);
    if (a.B >= 128 && blocks <= (BF ? 160 : 256)) launch_block<BF, MODE, 32, 32, 4>(s, a, update);
    else if ((a.dout <= 192 && (a.dout + 63) / 64 % 2) || (!BF && MODE != TW_ALIGNED)) launch_block<BF, MODE, 64, 64, 1>(s, a, update);
    else launch_block<BF, MODE, 64, 128, 1>(s, a, update);
}

// Rows of dZ and of dW start at multiples of 16 bytes.
static bool rows_in_pieces(const MlpPlan &p, int l) { return p.dims[l + 1] % 4 == 0 && p.woff[l] % 4 == 0; }

bool tile_wgrad_update_ok(const MlpPlan &p, int l) { return !p.bf16 && rows_in_pieces(p, l) && p.dims[l] >= 4; }

void launch_tile_wgrad(hipStream_t s, const MlpPlan &p, int l, float *G, int cur, const TailArgs *tail, bool others)
{
    const bool bf = p.bf16 != 0, u = tail != nullptr;
    TileWgrad a{};
    if (u) a.mix = tail->mix;
    if (others) {
        a.tiles = tail->tiles; a.n_tiles = tail->n_tiles; a.skip = tail->skip;
        a.other_blocks = grouped_blocks((unsigned)a.n_tiles * (unsigned)p.M);
    }
    a.feats = l == 0 ? p.feats : nullptr; a.row0 = p.row0; a.idx = p.idx;
    a.act = l == 0 ? nullptr : (bf ? (const void *)p.hb[l] : (const void *)p.act[l]);
    a.dz = p.dz[cur]; a.M = p.M; a.B = p.B; a.din = (int)p.dims[l]; a.dout = (int)p.dims[l + 1]; a.woff = p.woff[l]; a.G = G;
    const bool pieces = a.din >= 4 && a.dout >= 4;
    if (bf) {
        if (!pieces) launch_cols<true, TW_SINGLE>(s, a, u);
        else if (rows_in_pieces(p, l)) launch_cols<true, TW_ALIGNED>(s, a, u);
        else launch_cols<true, TW_PIECES>(s, a, u);
    } else {
        if (!pieces) launch_cols<false, TW_SINGLE>(s, a, u);
        else if (rows_in_pieces(p, l)) launch_cols<false, TW_ALIGNED>(s, a, u);
        else launch_cols<false, TW_PIECES>(s, a, u);
    }
}

}  // namespace netmax
