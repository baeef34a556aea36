// Forward pass of a layer of any shape, Z = A W + b with optional ReLU, for all workers (the stochastic gradient of
// Algorithm 2's first-step update): the tiled kernel for what the kernels of k_grad_mfma.hip and k_grad_f32.hip do not take.
//
// A workgroup takes BM batch rows and BN outputs of one worker.  A is contiguous along the contraction (gathered data rows
// or activations), W across it.  Large layers on fp32 operands are bound by the fp32 matrix rate: 3072 -> 1024, batch 128, 32 workers
// 273 to 292 us, the matrix pipe busy 66 % of the time (64 x 64 blocks: 293 us; the 64 x 64 kernel with 4-byte loads and steps of 32
// before it: 367 us).  With the operands as three bfloat16 planes (split_fwd_kernel) 223 to 233 us on the same boxes, 3072-1024-10
// with it 679 instead of 716 us per iteration, 784-1024-10 with 64 workers 399 instead of 449 us; the hidden activations are then
// 8.6e-7 off their 64-bit values instead of 9.9e-7 (3072 terms; 1.5e-7 and 1.8e-7 with 100).  Bound there by the vector
// instructions of the split (55 % of a SIMD's cycles) beside the products (39 %); forcing the two into turns inside a wave, and eight
// waves instead of four, changed nothing.  Small bfloat16 layers are bound by the chain of steps: 784 -> 500 and 500 -> 300, batch
// 100, 16 workers 33 us together (66 us with the earlier kernel, which multiplied the rounded operands by fp32 instructions).
#include "tile.h"

#include <type_traits>

namespace netmax {

struct TileFwd {
    const void *feats; const int64_t *row0; const int32_t *idx;      // first layer: gathered data rows
    const void *act;                                                  // else the activation below, [M][B][din]
    const float *X; int64_t woff; int M, B, din, dout, relu;
    float *out; uint16_t *out_bf16, *out_bf16_t;                      // [M][B][dout], and [M][dout][B]; each may be absent
};

// bias, ReLU and the store of a finished block
template <bool BF, int BM, int BN, int WM, int WN, int RI, int CJ>
__device__ __forceinline__ void tile_fwd_store(const TileFwd &p, int g, int m0, int n0, int wm, int wn, int lane, const tile_f32x16 (&acc)[RI][CJ])
{
#pragma unroll
    for (int j = 0; j < CJ; ++j) {
        const int col = n0 + wn * (BN / WN) + 32 * j + (lane & 31);
        const int cc = col < p.dout ? col : p.dout - 1;
        const float bias = p.X[tiled_offset_quick(p.M, g, p.woff + (int64_t)p.din * p.dout + cc)];
#pragma unroll
        for (int i = 0; i < RI; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = m0 + wm * (BM / WM) + 32 * i + tile_row(lane, v);
                float z = acc[i][j][v] + bias;
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
    }
}

// The product of one block, operands as they are (BF: rounded to bfloat16).  smem: LDS for both.
template <bool BF, bool VA, bool VW, int BM, int BN, int BK, int WM, int WN, int RI, int CJ>
__device__ __forceinline__ void tile_fwd_product(const TileFwd &p, int g, int m0, int n0, unsigned char *smem, tile_f32x16 (&acc)[RI][CJ])
{
    constexpr int NT = 64 * WM * WN, K4 = BK / 4;
    constexpr int NA = BM * K4 / NT, NB = BN * K4 / 4 / NT;           // pieces of A, 4 x 4 blocks of W per thread and step
    static_assert(NA * NT == BM * K4 && NB * NT == BN * K4 / 4, "every thread has the same share");
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
    int b_n[NB], b_k[NB], b_c[NB], b_have[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        const int c = t + u * NT;
        b_n[u] = c % (BN / 4) * 4;
        b_k[u] = c / (BN / 4) * 4;
        const int want = n0 + b_n[u];                                 // columns past the end repeat the last one(s)
        b_c[u] = want < p.dout ? want : (VW ? p.dout - 4 : p.dout - 1);
        b_have[u] = p.dout - b_c[u];
    }
    Piece<BF> ra[NA];
    Piece<false> rb[NB][4];
    const float *Xg = p.X;
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            int k = k0 + a_k[u];
            k = k < K ? k : (VA ? K - 4 : K - 1);
            if constexpr (BF) ra[u] = load_piece<VA>((const uint16_t *)(p.feats ? p.feats : p.act) + a_row[u] + k, K - k);
            else ra[u] = load_piece<VA>((const float *)(p.feats ? p.feats : p.act) + a_row[u] + k, K - k);
        }
#pragma unroll
        for (int u = 0; u < NB; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int k = k0 + b_k[u] + i < K ? k0 + b_k[u] + i : K - 1;
                const int64_t j = p.woff + (int64_t)k * p.dout + b_c[u];
                if constexpr (VW) rb[u][i] = load_piece<true>(Xg + tiled_offset_quick(p.M, g, j), 4);
                else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        rb[u][i].v[e] = Xg[tiled_offset_quick(p.M, g, j + (e < b_have[u] ? e : b_have[u] - 1))];
                }
            }
    };
    auto stash = [&](int k0) {
        // indices that exist from k on: 4 or more everywhere but in the last step
        const int left = K - k0;
#pragma unroll
        for (int u = 0; u < NA; ++u) put_piece(&As[a_m[u]][a_k[u]], ra[u].v, left - a_k[u]);
#pragma unroll
        for (int u = 0; u < NB; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) put_piece(&Bs[b_n[u] + e][b_k[u]], turned(rb[u], e), left - b_k[u]);
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

template <bool BF, bool VA, bool VW, int BM, int BN, int BK, int WM, int WN>
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
    tile_fwd_product<BF, VA, VW, BM, BN, BK, WM, WN>(p, g, m0, n0, smem, acc);
    tile_fwd_store<BF, BM, BN, WM, WN>(p, g, m0, n0, wm, wn, lane, acc);
}

// fp32 operands on the bfloat16 matrix instructions: 128 x 64 blocks, steps of 32, three planes of each operand in LDS, twice:
// the next step is split while this one is multiplied.
constexpr int SF_BM = 128, SF_BN = 64, SF_BK = 32, SF_WM = 2, SF_WN = 2, SF_THREADS = 256;
template <bool VA, bool VW>
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
    const int b_n = t / (BK / 2) * 4, b_k = t % (BK / 2) * 2;
    const int b_c = n0 + b_n < p.dout ? n0 + b_n : (VW ? p.dout - 4 : p.dout - 1);     // columns past the end repeat the last one(s)
    const int b_have = p.dout - b_c;
    Piece<false> ra[NA], rb[2];
    bool lost = false;                                                // an operand of this thread that its planes do not hold
    auto fetch = [&](int k0) {
        int k = k0 + a_k;
        k = k < K ? k : (VA ? K - 4 : K - 1);
#pragma unroll
        for (int u = 0; u < NA; ++u) ra[u] = load_piece<VA>(in + a_row[u] + k, K - k);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int kb = k0 + b_k + i < K ? k0 + b_k + i : K - 1;
            const int64_t j = p.woff + (int64_t)kb * p.dout + b_c;
            if constexpr (VW) rb[i] = load_piece<true>(p.X + tiled_offset_quick(p.M, g, j), 4);
            else {
#pragma unroll
                for (int e = 0; e < 4; ++e) rb[i].v[e] = p.X[tiled_offset_quick(p.M, g, j + (e < b_have ? e : b_have - 1))];
            }
        }
    };
    auto stash = [&](int k0, uint16_t *buf, auto whole) {             // whole: all indices of the step exist
        const int left = decltype(whole)::value ? BK : K - k0;
#pragma unroll
        for (int u = 0; u < NA; ++u)
            put_split(buf + split_at((t + u * NT) / K4, a_k), SA, decltype(whole)::value ? ra[u].v : first_of(ra[u].v, left - a_k), lost);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            put_split(buf + 3 * SA + (b_n + e) * SPLIT_PITCH + b_k, SB, left > b_k ? rb[0].v[e] : 0.0f, left > b_k + 1 ? rb[1].v[e] : 0.0f,
                      lost);
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
        tile_fwd_product<false, VA, VW, BM, BN, 64, WM, WN>(p, g, m0, n0, smem, acc);
    tile_fwd_store<false, BM, BN, WM, WN>(p, g, m0, n0, wm, wn, lane, acc);
}

template <bool BF, bool VA, bool VW, int BM, int BN, int BK, int WM, int WN>
static void launch_shape(hipStream_t s, const TileFwd &a)
{
    const unsigned blocks = (unsigned)((a.dout + BN - 1) / BN) * (unsigned)((a.B + BM - 1) / BM);
    hipLaunchKernelGGL((tile_fwd_kernel<BF, VA, VW, BM, BN, BK, WM, WN>), tile_grid(grouped_grid(a.M, blocks)), dim3(64 * WM * WN), 0, s, a);
}

// Few workgroups are bound by the chain of steps, not by what a step costs: longer steps, narrower blocks.  Only full chips of
// more than 64 batch rows are bound by the fp32 matrix rate.
template <bool BF, bool VA, bool VW> static void launch_rows(hipStream_t s, const TileFwd &a)
{
    constexpr int LONG = BF ? 128 : 64;
    const int64_t wide = (int64_t)a.M * ((a.dout + 63) / 64) * ((a.B + 127) / 128);
    if (a.B <= 32) launch_shape<BF, VA, VW, 32, 64, 64, 1, 2>(s, a);
    else if (a.B <= 64) launch_shape<BF, VA, VW, 64, 64, LONG, 2, 2>(s, a);
    else if (wide < 512) launch_shape<BF, VA, VW, 128, 32, 128, 4, 1>(s, a);
    else if constexpr (BF) launch_shape<BF, VA, VW, 128, 64, 64, 2, 2>(s, a);
    else {
        const unsigned blocks = (unsigned)((a.dout + SF_BN - 1) / SF_BN) * (unsigned)((a.B + SF_BM - 1) / SF_BM);
        hipLaunchKernelGGL((split_fwd_kernel<VA, VW>), tile_grid(grouped_grid(a.M, blocks)), dim3(SF_THREADS), 0, s, a);
    }
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
    // pieces of A: four elements, aligned to their size; pieces of W: four columns of a row that starts at a multiple of four
    const bool va = a.din % 4 == 0 && reinterpret_cast<uintptr_t>(a.feats ? a.feats : a.act) % (bf ? 8 : 16) == 0;
    const bool vw = a.dout % 4 == 0 && a.woff % 4 == 0;
    if (bf) {
        if (va) { if (vw) launch_rows<true, true, true>(s, a); else launch_rows<true, true, false>(s, a); }
        else { if (vw) launch_rows<true, false, true>(s, a); else launch_rows<true, false, false>(s, a); }
    } else {
        if (va) { if (vw) launch_rows<false, true, true>(s, a); else launch_rows<false, true, false>(s, a); }
        else { if (vw) launch_rows<false, false, true>(s, a); else launch_rows<false, false, false>(s, a); }
    }
}

}  // namespace netmax
