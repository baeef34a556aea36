// Weight gradient dW = A^T dZ of a layer of any shape for all workers (the stochastic gradient of Algorithm 2's first-step
// update): the tiled kernel for what the kernels of k_grad_mfma.hip and k_grad_f32.hip do not take.
//
// A workgroup takes 64 input features and 128 outputs of one worker; the contraction runs over the batch, both operands lie
// across it in memory.  The block is turned through LDS and leaves as row pieces of 128 floats.
// 3072 x 1024, batch 128, 32 workers, fp32: 311 us (402 us with 64 x 64 blocks, 4-byte loads and 128-byte row pieces);
// 784 x 500 and 500 x 300, batch 100, 16 workers, bfloat16: 21 us together (54 us with fp32 instructions).
//
// UPDATE (fp32 operands, aligned rows): the block's columns also get the momentum step and the mix (Eq. (c0), (c1)).  460 to 480
// us at the first shape, 2.46 GB moved, against 311 us and 314 us for the separate mix.  Bound by how well the fp32 matrix
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

constexpr int TW_BM = 64, TW_BN = 128, TW_BK = 64, TW_THREADS = 512;

template <bool BF, bool VA, bool VZ, bool UPDATE>
__global__ void __launch_bounds__(TW_THREADS, 4) tile_wgrad_kernel(TileWgrad p)
{
    static_assert(!UPDATE || VZ, "the update works on 128-bit pieces");
    constexpr int BM = TW_BM, BN = TW_BN, BK = TW_BK, NT = TW_THREADS;
    constexpr int A_BLOCKS = BM / 4 * (BK / 4);                       // 4 x 4 blocks of A per step: half a block per thread
    static_assert(2 * A_BLOCKS == NT && BN / 4 * (BK / 4) == NT, "half a block of A and one of dZ per step and thread");
    typedef TileLds<BF, BK> L;
    typedef typename L::elem elem;
    constexpr int TP = BN + 4;                                        // floats per row of the staged result
    constexpr int OPERANDS = (BM + BN) * L::PITCH * (int)sizeof(elem), RESULT = BM * TP * 4;
    __shared__ __attribute__((aligned(16))) unsigned char smem[OPERANDS > RESULT ? OPERANDS : RESULT];
    elem (*As)[L::PITCH] = reinterpret_cast<elem (*)[L::PITCH]>(smem);
    elem (*Zs)[L::PITCH] = reinterpret_cast<elem (*)[L::PITCH]>(smem + BM * L::PITCH * sizeof(elem));
    float (*T)[TP] = reinterpret_cast<float (*)[TP]>(smem);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave >> 2, wn = wave & 3;
    const int nblk = (p.dout + BN - 1) / BN, mblk = (p.din + BM - 1) / BM;
    unsigned bid = tile_block();
    if constexpr (UPDATE) {
        if (bid < p.other_blocks) {
            const unsigned tile = bid / (unsigned)p.M;
            if (tile < (unsigned)p.n_tiles) mix_subset_block<TW_THREADS>(p.M, p.tiles[tile], (int)(bid - tile * (unsigned)p.M), p.skip, p.G, p.mix);
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

    // A: two batch rows of four features per thread
    const int a_m = t % (BM / 4) * 4, a_k = t / (BM / 4) * 2;
    int a_f = f0 + a_m;
    a_f = a_f < p.din ? a_f : (VA ? p.din - 4 : p.din - 1);
    const int a_have = p.din - a_f;
    const int64_t base_row = p.feats ? p.row0[g] : (int64_t)g * K;
    const int32_t *rows = p.feats ? p.idx + (size_t)g * K : nullptr;
    const int z_n = t % (BN / 4) * 4, z_k = t / (BN / 4) * 4;
    int z_c = n0 + z_n;
    z_c = z_c < p.dout ? z_c : (VZ ? p.dout - 4 : p.dout - 1);
    const float *zg = p.dz + (size_t)g * K * p.dout + z_c;
    int32_t row_of[2];                                                // batch rows of the coming step, asked for a step ahead
    auto fetch_rows = [&](int k0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int k = k0 + a_k + i < K ? k0 + a_k + i : K - 1;
            row_of[i] = rows ? rows[k] : k;
        }
    };
    Piece<BF> ra[2];
    Piece<false> rz[4];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = k0 + z_k + i < K ? k0 + z_k + i : K - 1;
            rz[i] = load_piece<VZ>(zg + (size_t)k * p.dout, p.dout - z_c);
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
        tile_multiply<BK>(As, Zs, 32 * wm, 32 * wn, lane, acc, K - k0);
    }
    if constexpr (UPDATE) {
#pragma unroll
        for (int u = 0; u < PASSES; ++u) up[u] = load4(p.mix.Xcur + own_of(u) + peer_shift);
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();                                                  // the operands' space becomes the staged result
#pragma unroll
    for (int v = 0; v < 16; ++v) T[32 * wm + tile_row(lane, v)][32 * wn + (lane & 31)] = acc[0][0][v];
    __syncthreads();
    if (!col_ok) return;
#pragma unroll
    for (int u = 0; u < PASSES; ++u) {
        const int r = u * ROWS + orow;
        if (f0 + r < p.din) {
            const size_t own = own_of(u);
            if constexpr (VZ) {
                const f32x4 gr = *reinterpret_cast<const f32x4 *>(&T[r][oc]);
                store4_stream(p.G + own, gr);
                if constexpr (UPDATE) {
                    f32x4 xn, vn;
                    momentum_mix4(ux[u], uv[u], gr, up[u], wi, p.mix.alpha, p.mix.mu, p.mix.wd, xn, vn);
                    store4_stream(p.mix.Xnext + own, xn);
                    store4_stream(p.mix.V + own, vn);
                }
            } else {
                p.G[own] = T[r][oc];
            }
        }
    }
}

template <bool BF, bool VA, bool VZ> static void launch_cols(hipStream_t s, const TileWgrad &a, bool update)
{
    const dim3 grid = tile_grid(a.other_blocks + grouped_grid(a.M, (unsigned)((a.dout + TW_BN - 1) / TW_BN) * (unsigned)((a.din + TW_BM - 1) / TW_BM))), block(TW_THREADS);
    if constexpr (VZ && !BF)
        if (update) {
            hipLaunchKernelGGL((tile_wgrad_kernel<BF, VA, VZ, true>), grid, block, 0, s, a);
            return;
        }
    hipLaunchKernelGGL((tile_wgrad_kernel<BF, VA, VZ, false>), grid, block, 0, s, a);
}

// Rows of dZ and of dW start at multiples of 16 bytes.
static bool rows_in_pieces(const MlpPlan &p, int l) { return p.dims[l + 1] % 4 == 0 && p.woff[l] % 4 == 0; }

bool tile_wgrad_update_ok(const MlpPlan &p, int l) { return !p.bf16 && rows_in_pieces(p, l); }

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
    const bool va = a.din % 4 == 0 && reinterpret_cast<uintptr_t>(a.feats ? a.feats : a.act) % (bf ? 8 : 16) == 0;
    const bool vz = rows_in_pieces(p, l);
    if (bf) {
        if (va) { if (vz) launch_cols<true, true, true>(s, a, u); else launch_cols<true, true, false>(s, a, u); }
        else { if (vz) launch_cols<true, false, true>(s, a, u); else launch_cols<true, false, false>(s, a, u); }
    } else {
        if (va) { if (vz) launch_cols<false, true, true>(s, a, u); else launch_cols<false, true, false>(s, a, u); }
        else { if (vz) launch_cols<false, false, true>(s, a, u); else launch_cols<false, false, false>(s, a, u); }
    }
}

}  // namespace netmax
