// Per-worker gradient of a ReLU perceptron with softmax cross-entropy (one layer = softmax regression):
// the stochastic gradient of Algorithm 2's first-step update, for all workers at once.  Every GEMM is
// grouped, one group per worker, because each worker multiplies its own batch with its own weights.
//
// This file holds the sequence of a gradient's launches, the forward pass of layers with few outputs, and the loss and bias
// gradients of what the more specialised kernels leave.  With bf16 operands the inputs of every product are rounded to
// bfloat16 first and accumulated in fp32.
#include "softmax_xent.h"
#include "tile.h"

namespace netmax {

// Where the input of a layer comes from: the gathered data rows (fp32 or bfloat16 storage) for the first
// layer, else the previous layer's activation (fp32, or its stored bfloat16 copy when the operands are bf16).
enum : int { IN_GATHER_F32 = 0, IN_GATHER_BF16 = 1, IN_ACT_F32 = 2, IN_ACT_BF16 = 3 };

__device__ __forceinline__ float as_float(uint32_t u) { return __builtin_bit_cast(float, u); }
// Operands are rounded to bfloat16 exactly when the layer inputs are stored as bfloat16 (the odd kinds): a property
// of the instantiation, so the fp32 kernels carry no rounding code.
template <int KIND> __device__ __forceinline__ float operand(float x)
{
    if constexpr ((KIND & 1) != 0) return round_bf16(x);
    else return x;
}

// Input of a layer: element `index` of it as loaded, and as the multiplicand.
struct LayerInput {
    const void *feats; const int64_t *row0; const int32_t *idx; const float *act_prev;
    const uint16_t *act_prev_bf16;
    int B; int64_t din; int kind;
    template <int KIND> __device__ __forceinline__ float value(uint32_t u) const
    {
        if constexpr (KIND == IN_GATHER_BF16 || KIND == IN_ACT_BF16) return as_float(u << 16);
        else return as_float(u);
    }
    template <int KIND> __device__ __forceinline__ uint32_t load_index(int64_t index) const
    {
        if constexpr (KIND == IN_GATHER_F32) return ((const uint32_t *)feats)[index];
        else if constexpr (KIND == IN_GATHER_BF16) return ((const uint16_t *)feats)[index];
        else if constexpr (KIND == IN_ACT_F32) return ((const uint32_t *)act_prev)[index];
        else return act_prev_bf16[index];
    }
};

// Z = A W + b, optional ReLU.
struct FwdProblem {
    LayerInput in; const float *X; int64_t woff, din, dout; int M, B, relu; float *out;
    uint16_t *out_bf16, *out_bf16_t;     // optional bfloat16 copies: [B][dout] and transposed [dout][B]
    template <int AK> __device__ float a_val(uint32_t u) const { return in.value<AK>(u); }
    template <int AK> __device__ float b_val(uint32_t u) const { return operand<AK>(as_float(u)); }
    __device__ void store(int g, int64_t r, int64_t c, float acc) const
    {
        float z = acc + X[tiled_offset(M, g, woff + din * dout + c)];
        if (relu) z = z > 0.0f ? z : 0.0f;
        if (out) out[((size_t)g * B + r) * dout + c] = z;
        if (out_bf16) {
            const uint16_t h = (uint16_t)bf16_bits(z);
            out_bf16[((size_t)g * B + r) * dout + c] = h;
            out_bf16_t[((size_t)g * dout + c) * B + r] = h;
        }
    }
};

// Forward pass of a layer with few outputs (at most 32: the classifier layer), any input width and kind.  The tiled
// kernels would use one 64-column tile per worker for it, most of it padding, on few workgroups.  Here a
// workgroup takes 16 batch rows of one worker; 16 threads share a row and split the contraction index between them
// (thread q takes k = q, q + 16, ...).  The weights of a chunk of the contraction are a run of consecutive
// parameters (rows of W are dout long), copied to LDS as they lie; all loads of a chunk are requested before the
// first is used.  The 16 partial sums of a row are added in a fixed butterfly order.  Products and sums in fp32.
constexpr int NARROW_ROWS = 16, NARROW_SPLIT = 16, NARROW_THREADS = NARROW_ROWS * NARROW_SPLIT, NARROW_WEIGHTS = 2048;
template <int AK, int CP>       // CP: outputs padded to 16 or 32
__global__ void __launch_bounds__(NARROW_THREADS) fwd_narrow_kernel(FwdProblem p)
{
    constexpr int CHUNK = NARROW_WEIGHTS / CP;                 // contraction indices per chunk
    constexpr int PER = CHUNK / NARROW_SPLIT, W_PER = NARROW_WEIGHTS / NARROW_THREADS;
    __shared__ float Wl[NARROW_WEIGHTS + CP];                   // CP more: the padded columns of the last row read on
    __shared__ int64_t s_row[NARROW_ROWS];
    const int g = blockIdx.y, tid = threadIdx.x, r = tid / NARROW_SPLIT, q = tid % NARROW_SPLIT;
    const int b = blockIdx.x * NARROW_ROWS + r;
    const int C = (int)p.dout;
    if (tid < NARROW_ROWS) {
        const int bb = blockIdx.x * NARROW_ROWS + tid;
        const int bq = bb < p.B ? bb : p.B - 1;              // rows beyond the batch repeat the last one and are not stored
        const LayerInput &in = p.in;
        s_row[tid] = (AK == IN_GATHER_F32 || AK == IN_GATHER_BF16) ? (in.row0[g] + in.idx[(size_t)g * in.B + bq]) * in.din
                                                                   : ((int64_t)g * in.B + bq) * in.din;
    }
    if (tid < CP) Wl[NARROW_WEIGHTS + tid] = 0.0f;
    __syncthreads();
    const int64_t a_row = s_row[r];
    float acc[CP];
#pragma unroll
    for (int c = 0; c < CP; ++c) acc[c] = 0.0f;
    // Chunks are small (8 loads of each kind per thread) and every loop over them is unrolled completely, so that the
    // staged values stay in registers; clamped unconditional loads, no predicates.
    for (int64_t k0 = 0; k0 < p.din; k0 += CHUNK) {
        const int n = (int)(p.din - k0 < CHUNK ? p.din - k0 : CHUNK), n_w = n * C;
        uint32_t av[PER], wv[W_PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int kk = q + u * NARROW_SPLIT;
            av[u] = p.in.template load_index<AK>(a_row + k0 + (kk < n ? kk : n - 1));
        }
        const int64_t w0 = p.woff + k0 * p.dout;               // first parameter of the chunk
#pragma unroll
        for (int u = 0; u < W_PER; ++u) {
            const int e = tid + u * NARROW_THREADS;
            wv[u] = ((const uint32_t *)p.X)[tiled_offset_quick(p.M, g, w0 + (e < n_w ? e : n_w - 1))];
        }
        __syncthreads();                                       // the previous chunk has been used
#pragma unroll
        for (int u = 0; u < W_PER; ++u) {
            const int e = tid + u * NARROW_THREADS;
            Wl[e < n_w ? e : n_w - 1] = p.template b_val<AK>(wv[u]);     // clamped slots all hold the last weight
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int kk = q + u * NARROW_SPLIT;
            const float a = kk < n ? p.template a_val<AK>(av[u]) : 0.0f;
            const float *wk = Wl + (kk < n ? kk : 0) * C;
            // columns from C on multiply whatever follows the row (finite numbers); those sums are never stored
#pragma unroll
            for (int c = 0; c < CP; ++c) acc[c] = fmaf(a, wk[c], acc[c]);
        }
    }
    // the 16 partial sums of a row sit in 16 neighbouring lanes: butterfly over lane distances 8, 4, 2, 1
#pragma unroll
    for (int c = 0; c < CP; ++c)
#pragma unroll
        for (int d = NARROW_SPLIT / 2; d > 0; d >>= 1) acc[c] += __shfl_xor(acc[c], d, 64);
    if (b < p.B) {
#pragma unroll
        for (int c0 = 0; c0 < CP; c0 += NARROW_SPLIT) {        // thread q stores columns q, q + 16
            float v = 0.0f;
#pragma unroll
            for (int c = 0; c < NARROW_SPLIT; ++c) v = (c == q) ? acc[c0 + c] : v;
            if (c0 + q < C) p.store(g, b, c0 + q, v);
        }
    }
}

template <int CP> static void launch_fwd_narrow_kind(hipStream_t s, const FwdProblem &p, int kind, dim3 grid)
{
    const dim3 block(NARROW_THREADS);
    switch (kind) {
    case IN_GATHER_F32: hipLaunchKernelGGL((fwd_narrow_kernel<IN_GATHER_F32, CP>), grid, block, 0, s, p); break;
    case IN_GATHER_BF16: hipLaunchKernelGGL((fwd_narrow_kernel<IN_GATHER_BF16, CP>), grid, block, 0, s, p); break;
    case IN_ACT_F32: hipLaunchKernelGGL((fwd_narrow_kernel<IN_ACT_F32, CP>), grid, block, 0, s, p); break;
    default: hipLaunchKernelGGL((fwd_narrow_kernel<IN_ACT_BF16, CP>), grid, block, 0, s, p); break;
    }
}
static void launch_fwd_narrow(hipStream_t s, const FwdProblem &p, int kind, int groups)
{
    const dim3 grid((unsigned)((p.B + NARROW_ROWS - 1) / NARROW_ROWS), (unsigned)groups);
    if (p.dout <= 16) launch_fwd_narrow_kind<16>(s, p, kind, grid);
    else launch_fwd_narrow_kind<32>(s, p, kind, grid);
}

// Softmax cross-entropy on the logits (softmax_xent.h): one workgroup per worker.
__global__ void __launch_bounds__(1024) softmax_xent_kernel(SoftmaxArgs a) { softmax_xent_block(a, blockIdx.x, softmax_label(a, blockIdx.x)); }

// db = column sums of dZ.  One workgroup = one worker x 64 outputs; the batch rows are dealt to four groups of
// threads (rows r, r + 4, ...), whose partial sums are added in the order of the groups.  Eight rows of a group are asked for
// before the first is added (batch 785, 2 workers 12 us; one by one 49 us).
__global__ void __launch_bounds__(256)
bias_grad_kernel(int M, int B, int64_t dout, const float *__restrict__ dz, int64_t boff,
                 float *__restrict__ G)
{
    __shared__ float part[4][64];
    const int g = blockIdx.y, lane_c = threadIdx.x & 63, rg = threadIdx.x >> 6;
    const int64_t c = (int64_t)blockIdx.x * 64 + lane_c;
    float s = 0.0f;
    if (c < dout) {
#pragma unroll 8
        for (int b = rg; b < B; b += 4) s += dz[((size_t)g * B + b) * dout + c];
    }
    part[rg][lane_c] = s;
    __syncthreads();
    if (rg == 0 && c < dout) G[tiled_offset(M, g, boff + c)] = ((part[0][lane_c] + part[1][lane_c]) + part[2][lane_c]) + part[3][lane_c];
}

// A weight gradient on fp32 operands holds dW of most columns on its way to memory; applying the update there saves the read of g
// and, for middling models, most of a launch.  x' goes to the other buffer and nobody else looks at these columns of v, so a
// layer's update need not wait for the layers below.  Per iteration, with the separate mix and with the update in the kernels:
// 3072-1024-10, batch 128, 32 workers 873 and 716 us, 64 workers 1725 and 1420 us; 784-512-10, 16 workers, batch 128 95 and 89 us,
// batch 64 71 and 63 us.  The first layer's kernel, if it is the last of the iteration, also updates the columns that no kernel
// has, which saves the mix's launch: batch 64 63 and 58 us.
// The line lies where x, v, g and the new x no longer fit the 32 MB of L2 together.  Per iteration, update in the first layer only
// and in every one: 256-256-256-10, batch 64, 11 workers (1.5 M floats) 47.8 and 47.9 us, 15 workers (2.0 M) 57.3 and 48.8 us;
// 128-wide 100-128-128-128-10, batch 32, 32 workers (1.5 M) 51.2 and 51.5 us, 43 workers (2.1 M) 58.4 and 53.4 us;
// 300-60-60-60-10, batch 60, 58 workers (1.6 M) 57.5 and 59.4 us, 116 workers (3.1 M) 71.1 and 70.2 us.
// Smaller models have the first layer update and take the other columns as those that are
// left, if that does save the launch: 256-256-10, 8 workers, batch 32 27.0 us with the mix and 23.0 us, 784-512-10, 4 workers
// 45.0 and 39.6 us; every layer for itself lengthens the chain (300-60-60-60-10, 8 workers 64.7 and 66.5 us).
// Where it loses: rows of W that do not start at multiples of 16 bytes (3001-999-10: 1118 and 1519 us); bfloat16 operands, whose
// products leave little to hide (784-500-300-10, 16 workers 106 and 113 us, 3000-1000-10, 128 workers 2354 and 2644 us).  The
// matrix-core layers have a kernel in the mix's order for it, which they take where it saves bytes (wgrad_mix_saves()): batch 128, 3072-1024-1024-10, 48 workers 1159 and 1070 us, 128 workers,
// two iterations 5668 and 5259 us (the first need not write g); batch 64, 1024-1024-10, 32 workers 2 x 221 and
// 2 x 181 us, 512-512-256-10, 16 workers 2 x 88 and 2 x 81 us, 1024-512-10, 4 workers (2.1 M floats) 2 x 68 and 2 x 63 us, but
// 512-128-128-10, 2 workers 4 x 57.5 and 4 x 60 us.
constexpr int64_t UPDATE_MIN_FLOATS = 7 << 18;       // M x ld
constexpr double UPDATE_MIN_SAVED = -0.5, UPDATE_MIN_SAVED_G = -0.1;       // bytes a parameter, of wgrad_mix_saves(): of 4400 drawn networks 13 lost more than 2 % (at most 7) from there on and 11 below would have gained as much; with g 31 (at most 7) and 25 of 3000
static bool first_layer_last(const MlpPlan &p) { return p.n_layers == 1 || (p.n_layers == 2 && head_ok(p)) || p.B <= TILE_DGRAD_BATCH; }

int64_t update_end(const MlpPlan &p, int l)
{
    const bool head = head_ok(p);
    if (p.n_layers == 1 && head) return p.ld;                        // the last-layer kernel updates everything
    if (mfma_layer_ok(p, l)) return p.M * p.ld < UPDATE_MIN_FLOATS || wgrad_mix_saves(p, false) < UPDATE_MIN_SAVED ? 0 : p.woff[l] + p.dims[l] * p.dims[l + 1];
    if (p.bf16 || (l == p.n_layers - 1 && head) || p.woff[l] % 4 != 0) return 0;
    if (p.M * p.ld < UPDATE_MIN_FLOATS && (l > 0 || !first_layer_last(p))) return 0;
    if (!wgrad_f32_ok(p, l) && !tile_wgrad_update_ok(p, l)) return 0;
    return p.woff[l] + p.dims[l] * p.dims[l + 1];
}

// Iterations that keep g.  An XCD holds 96 workers of a block at a time; beyond, a good part of the peers' columns comes from memory, the more the further the workers drift
// apart along their walks, and the time depends on where the buffers lie: 128 workers 3072-1024-1024-10, batch 128, 2804 to 2946 us with the update in the weight
// gradients and 2824 to 2862 with the separate mix, 112 workers 2371 to 2594 and 2487.  So from 128 workers on only walks of one strip (batches of up to 64) that save
// a byte and a half a parameter: batch 32, 128 workers 3072-1024-1024-10 2425 to 2560 and 2676, 1024-1024-10 633 to 650 and 692, 160 workers 776 to 834 and 866.  From two
// rounds of 96 on none: 300 workers 3072-1024-1024-10, batch 128 7090 and 6650, 256 workers 1024-1024-10, batch 64 1466 and 1421, batch 32 1359 and 1360.
bool update_beside_g(const MlpPlan &p)
{
    bool any = false;
    for (int l = 0; l < p.n_layers; ++l) any |= mfma_layer_ok(p, l) && update_end(p, l) > 0;
    if (!any) return true;
    return p.M < 128 ? wgrad_mix_saves(p, true) >= UPDATE_MIN_SAVED_G : p.M < 192 && p.B <= 64 && wgrad_mix_saves(p, true) >= 1.5;
}

// One fp32 hidden layer on the kernels of k_grad_f32.hip, or none: forward, the last layer's two kernels, weight gradient with the
// update of everything.
bool layer_list_ok(const MlpPlan &p)
{
    if (p.bf16 || !head_ok(p) || update_end(p, 0) <= 0) return false;
    return p.n_layers == 1 || (p.n_layers == 2 && fwd_f32_ok(p, 0) && wgrad_f32_ok(p, 0));
}

bool launch_mlp_grad(hipStream_t s, const MlpPlan &p, const float *X, float *G, const MixArgs *fuse, const TailArgs *tail)
{
    const int L = p.n_layers;
    const bool bf = p.bf16 != 0;
    bool fast[8] = {};
    for (int l = 0; l < L; ++l) fast[l] = mfma_layer_ok(p, l);
    const bool small_last = mfma_small_last_ok(p);
    const bool head = head_ok(p);
    auto tail_of = [&](int l) { return tail && update_end(p, l) > 0 ? tail : nullptr; };
    auto input_of = [&](int l) {
        LayerInput in;
        in.feats = p.feats; in.row0 = p.row0; in.idx = p.idx;
        in.act_prev = (l > 0 && !bf) ? p.act[l] : nullptr;
        in.act_prev_bf16 = (l > 0 && bf) ? p.hb[l] : nullptr;
        in.B = p.B; in.din = p.dims[l];
        in.kind = l == 0 ? (bf ? IN_GATHER_BF16 : IN_GATHER_F32) : (bf ? IN_ACT_BF16 : IN_ACT_F32);
        return in;
    };
    // forward.  With bf16 operands the hidden activations are kept as bfloat16 only (both orientations).
    for (int l = 0; l < L; ++l) {
        const bool last = (l + 1 == L);
        if (fast[l] && !last) {
            if (chain_fwd_pays(p, l)) launch_chain_fwd(s, p, l, X, true);
            else launch_fwd_mfma(s, p, l, X);
            continue;
        }
        if (last && small_last) {
            launch_fwd_small(s, p, X, G);
            continue;
        }
        if (last && head) break;         // the head kernel below starts from the last hidden activation
        if (fwd_f32_ok(p, l)) {
            launch_fwd_f32(s, p, l, X);
            continue;
        }
        if (p.dims[l + 1] > 32) {
            // the transposed bfloat16 activation is read by the matrix-core weight gradients only
            const bool need_t = !last && (fast[l + 1] || (l + 2 == L && small_last));
            if (chain_fwd_pays(p, l)) launch_chain_fwd(s, p, l, X, need_t);
            else launch_tile_fwd(s, p, l, X, need_t);
            continue;
        }
        FwdProblem f;
        f.in = input_of(l); f.X = X; f.M = p.M; f.woff = p.woff[l]; f.din = p.dims[l]; f.dout = p.dims[l + 1];
        f.B = p.B; f.relu = !last;
        f.out = (last || !bf) ? p.act[l + 1] : nullptr;
        f.out_bf16 = (bf && !last) ? p.hb[l + 1] : nullptr;
        f.out_bf16_t = (bf && !last) ? p.ht[l + 1] : nullptr;
        // few outputs: the tiled kernel would pad them to a 64-column tile on one workgroup per worker
        launch_fwd_narrow(s, f, f.in.kind, p.M);
    }
    bool bias_done[8] = {}, all_updated = L == 1 && head && tail_of(0);
    int cur = 0, l_top = L - 1;
    if (head) {
        // logits, loss, the last layer's gradient and the error of the last hidden layer (with its column sums)
        launch_head(s, p, X, G, L == 1 && tail_of(0) ? &tail->mix : nullptr);
        bias_done[L - 1] = true;
        if (L > 1) bias_done[L - 2] = true;
        l_top = L - 2;
        cur = 1;
    } else {
        // loss and dZ of the last layer
        const int sm_threads = p.B <= 64 ? 64 : (p.B <= 256 ? 256 : 1024);
        if (!small_last)             // (the last-layer forward kernel of the matrix-core path ends with it)
            hipLaunchKernelGGL(softmax_xent_kernel, dim3(p.M), dim3(sm_threads), 0, s, softmax_args(p, G));
        bias_done[L - 1] = true;     // by the kernel above
    }
    // backward
    for (int l = l_top; l >= 0; --l) {
        const int64_t din = p.dims[l], dout = p.dims[l + 1];
        const bool others = l == 0 && !fast[0] && bias_done[0] && tail_of(0) != nullptr;       // the last launch: it can update what is left
        all_updated |= others;
        if (fast[l]) {
            if (fuse) launch_wgrad_mix_mfma(s, p, l, G, cur, *fuse);
            else if (const TailArgs *u = tail_of(l)) launch_wgrad_mix_mfma(s, p, l, G, cur, u->mix);
            else launch_wgrad_mfma(s, p, l, G, cur);
        } else if (l == L - 1 && small_last) {
            launch_wgrad_small(s, p, G, cur);
        } else if (wgrad_f32_ok(p, l)) {
            launch_wgrad_f32(s, p, l, G, p.dz[cur], tail_of(l), others);
        } else {
            launch_tile_wgrad(s, p, l, G, cur, tail_of(l), others);
        }
        if (!bias_done[l]) {
            hipLaunchKernelGGL(bias_grad_kernel, dim3((unsigned)((dout + 63) / 64), (unsigned)p.M), dim3(256), 0, s, p.M, p.B,
                               dout, p.dz[cur], p.woff[l] + din * dout, G);
        }
        if (l > 0) {
            if (chain_dgrad_pays(p, l)) {
                launch_chain_dgrad(s, p, l, X, G, cur, fast[l - 1]);
                bias_done[l - 1] = true;
            } else if (fast[l]) {
                launch_dgrad_mfma(s, p, l, X, G, cur, !fast[l - 1]);
                bias_done[l - 1] = true;
            } else if (l == L - 1 && small_last) {
                launch_dgrad_small(s, p, X, G, cur, !fast[l - 1]);
                bias_done[l - 1] = true;
            } else {
                bias_done[l - 1] = launch_tile_dgrad(s, p, l, X, G, cur, fast[l - 1]);
            }
            cur ^= 1;
        }
    }
    return all_updated;
}

}  // namespace netmax
