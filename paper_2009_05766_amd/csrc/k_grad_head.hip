// Last layer of a perceptron with at most 32 classes, from its input h (the last hidden activation, or the gathered data rows of
// a softmax regression) to the error handed to the layer below (the stochastic gradient of Algorithm 2's first-step
// update, its part above the last hidden layer): logits = h W + b, softmax cross-entropy (mean loss, dZ = (softmax - onehot) / B),
// dW = h^T dZ, db = column sums of dZ, dH = (dZ W^T) masked by h > 0, and the column sums of dH = the bias gradient of the layer
// below.  Kernels of one purpose each take three to five dependent launches of a few microseconds for this; small models are
// bound by exactly that latency.  Here it is two:
//
//   head_logits_kernel  one workgroup per worker and 16 batch rows; its waves split the features, add their
//                       partial logits through LDS in wave order, then sixteen lanes per row do the softmax
//   head_grads_kernel   one workgroup per worker and 64 features; a wave takes sixteen of them: sixteen rows of
//                       dW and sixteen columns of dH from one set of loads of h (the order of the contraction over
//                       the batch in dW is chosen so that the lanes hold the 16 x B block of h exactly as the result
//                       block of dH, which needs it for the ReLU mask)
//
// so that h is read once by each, by many compute units (one kernel that did everything per worker had a single
// compute unit pull 200 KB and took 14.6 us at 16 workers, 512 hidden units; these take 4.6 and 4.8 us).  Softmax regression on
// 784 features, 16 workers, batch 64: 6.2 and 4.2 us (5.2 us with the update of all columns, which
// saves the mix kernel's 3.1 us and its launch) in place of three kernels of 15.0, 9.3 and 6.2 us; 1024 hidden units, 32
// workers, batch 128: 10 and 14 us in place of five kernels of 16, 12, 12, 17 and 16 us.
// The products run on v_mfma_f32_16x16x4_f32 with the classes padded to one or two 16-wide tiles (lane l
// supplies A[l % 16][l / 16] and B[l / 16][l % 16] and receives D[4 (l / 16) + v][l % 16], v = 0..3); bfloat16 operands are
// rounded first, their products are exact there.  The operands from W are loaded straight into that layout (a wave's load is 4
// rows of W = 4 C contiguous floats).
// No load sits under a branch: where a bound has to be respected the index is clamped and the value discarded; numbers of
// features that fill the steps of sixteen have a form without any bound (7.7 -> 6.2 us at 784 features).
#include "tile.h"

namespace netmax {

constexpr int HD_THREADS = 256, HD_WAVES = HD_THREADS / 64;          // gradients kernel
// logits kernel: steps of sixteen features of a wave's part whose loads are in flight together.  Up to 32 steps four waves
// take them (a wave with fewer than eight steps asks for its first one again instead), more are dealt to eight waves.
constexpr int HD_STEPS = 8, HL_FEW = 4, HL_MANY = 8;
constexpr int HD_MAX_B = 256, HD_MAX_C = 32;

struct HeadArgs {
    const void *in;                 // [M][B][H] activation of the last hidden layer
    int gather;                     // (or the data rows)
    const int64_t *row0; const int32_t *idx;                         // batch rows of every worker [M][B]
    const float *X; float *G;       // parameters and gradient, tile layout
    const int32_t *labels;
    float *dz;                      // [M][B][C]
    float *row_loss;                // [M][B] loss of every batch row (between the two kernels)
    float *dh;                      // [M][B][H]
    float *loss;                    // [M]
    int M, B, H, C;
    int64_t woff;                   // W [H][C] of the last layer inside a parameter row, its bias behind it
    int64_t boff_below;             // bias of the layer below
    int64_t D, ld;
    MixArgs mix;                    // UPDATE
    int Mx; const int32_t *worker;  // LIST: see MlpPlan
    int pairs;                      // host: logits by pairs of steps
};

__device__ __forceinline__ f32x4 mfma_16x16x4(float a, float b, f32x4 acc) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0); }

// Operands: fp32 as they are, bfloat16 (BF) rounded; inputs are stored as bfloat16 then.
template <bool BF> __device__ __forceinline__ float head_operand(float x) { return BF ? round_bf16(x) : x; }
template <bool BF> __device__ __forceinline__ float head_input(const void *in, int64_t index)
{
    if constexpr (BF) return bf16_bits_to_float(((const uint16_t *)in)[index]);
    else return ((const float *)in)[index];
}
template <bool BF> struct HeadElem { typedef float type; };
template <> struct HeadElem<true> { typedef uint16_t type; };
// A worker's last layer inside the tile layout: parameter u of it (u = k C + c, bias behind) counted from the start of the tile
// that holds its first one.  32-bit: head_ok() has checked that the layer's span fits.
struct HeadParams {
    size_t base; uint32_t skip, first;
    __device__ __forceinline__ HeadParams(int M, int g, int64_t woff)
        : base(((size_t)(woff >> TILE_SHIFT) * M + g) << TILE_SHIFT), skip((uint32_t)(M - 1) << TILE_SHIFT), first((uint32_t)(woff & (TILE - 1))) {}
    __device__ __forceinline__ uint32_t at(uint32_t u) const { return u + first + ((u + first) >> TILE_SHIFT) * skip; }
};
// Element index of feature 0 of batch row b.
__device__ __forceinline__ int64_t head_row(const HeadArgs &p, int g, int wk, int b)
{
    return (p.gather ? p.row0[wk] + p.idx[(size_t)g * p.B + b] : (int64_t)g * p.B + b) * p.H;
}

// Grid: (ceil(B / 16), workers).  CT: tiles of sixteen classes.  How the input's rows are read: feature by feature, in pieces of
// four features, in pieces of a number of features that fills the steps of sixteen (no bounds to respect).
// LIST: p.worker (see k_grad_f32.hip).  TWO: a wave's run is summed in pairs of steps, the parts that resident_mlp_kernel's workgroups have, these
// and then the waves' sums two by two; eight steps per wave at most then.
enum : int { HL_SINGLE = 0, HL_PIECES = 1, HL_WHOLE = 2 };
template <bool BF, int MODE, int CT, int NW, bool TWO = false, bool LIST = false>
__global__ void __launch_bounds__(64 * NW) head_logits_kernel(HeadArgs p)
{
    constexpr int PER_WAVE = TWO ? HD_STEPS / 2 : 1;         // sums
    static_assert(!TWO || PER_WAVE == 4, "the sums are added two by two");
    __shared__ float part[NW][16][16 * CT];
    const int B = p.B, H = p.H, C = p.C;
    const int g = blockIdx.y, rt = blockIdx.x, t = threadIdx.x, lane = t & 63, r = lane & 15, q = lane >> 4;
    const int kp = __builtin_amdgcn_readfirstlane(t >> 6);
    // each wave takes a run of steps of sixteen features; rows past the batch and features past the end are clamped, the
    // features' products then masked
    const int steps = (H + 15) / 16, per = TWO ? (steps / 2 + NW - 1) / NW * 2 : (steps + NW - 1) / NW;
    const int s_begin = kp * per, s_end = s_begin + per < steps ? s_begin + per : steps;
    const int wk = LIST ? p.worker[g] : g, Mx = LIST ? p.Mx : p.M;
    const int64_t a_row = head_row(p, g, wk, 16 * rt + r < B ? 16 * rt + r : B - 1);
    const HeadParams at(Mx, wk, p.woff);
    const float *Xg = p.X + at.base;
    uint32_t wcol[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) wcol[c] = min(16 * c + r, C - 1);
    f32x4 acc[PER_WAVE][CT];
#pragma unroll
    for (int u = 0; u < PER_WAVE; ++u)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[u][c] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    float a[HD_STEPS][4], b[HD_STEPS][4][CT];
    auto request = [&](int s0) {
#pragma unroll
        for (int i = 0; i < HD_STEPS; ++i) {
            const int k0 = 16 * (s0 + i < s_end ? s0 + i : s_begin) + 4 * q;        // past the part: its first step again, unused
            if constexpr (MODE != HL_SINGLE) {
                const Piece<BF> x = load_piece<true>((const typename HeadElem<BF>::type *)p.in + a_row + (MODE == HL_WHOLE ? k0 : min(k0, H - 4)), 4);
#pragma unroll
                for (int j = 0; j < 4; ++j) a[i][j] = piece_value(x, j);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) a[i][j] = head_input<BF>(p.in, a_row + min(k0 + j, H - 1));
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int c = 0; c < CT; ++c) b[i][j][c] = Xg[at.at((uint32_t)(MODE == HL_WHOLE ? k0 + j : min(k0 + j, H - 1)) * (uint32_t)C + wcol[c])];
        }
    };
    // what the softmax needs is asked for behind the first requests and waited for after the products: sixteen lanes per row
    const int row = (t >> 4) & 15, l16 = t & 15, b_row = 16 * rt + row;
    const int32_t drawn = p.idx[(size_t)g * B + min(b_row, B - 1)];
    if (s_begin < s_end) request(s_begin);
    __builtin_amdgcn_sched_barrier(0);
    const int y = p.labels[p.row0[wk] + drawn];
    float bias[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) bias[c] = Xg[at.at((uint32_t)(H * C + min(16 * c + l16, C - 1)))];
    __builtin_amdgcn_sched_barrier(0);
    for (int s0 = s_begin; s0 < s_end; s0 += HD_STEPS) {
#pragma unroll
        for (int i = 0; i < HD_STEPS; ++i)
            if (s0 + i < s_end) {
                const int left = MODE == HL_WHOLE ? 4 : H - 16 * (s0 + i) - 4 * q;      // columns of W past the classes are never looked at
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int c = 0; c < CT; ++c)
                    {
                        f32x4 &sum = acc[TWO ? i / 2 : 0][c];
                        sum = mfma_16x16x4(j < left ? a[i][j] : 0.0f, j < left ? head_operand<BF>(b[i][j][c]) : 0.0f, sum);
                    }
            }
        __builtin_amdgcn_sched_barrier(0);
        if (s0 + HD_STEPS < s_end) request(s0 + HD_STEPS);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float sum = acc[0][c][v];
            if constexpr (TWO) sum = (sum + acc[1][c][v]) + (acc[2][c][v] + acc[3][c][v]);       // pairs past the wave's run are zeros
            part[kp][4 * q + v][16 * c + r] = sum;
        }
    __syncthreads();
    // the parts added in order, bias, softmax cross-entropy: sixteen lanes per batch row, CT classes each
    if (t >= 256) return;
    float z[CT], mx = -INFINITY;
    bool cls[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const int k = 16 * c + l16;
        cls[c] = k < C;
        float sum = part[0][row][k];
        if constexpr (TWO) {
            sum = (sum + part[1][row][k]) + (part[2][row][k] + part[3][row][k]);
            if constexpr (NW == 8) sum += (part[4][row][k] + part[5][row][k]) + (part[6][row][k] + part[7][row][k]);
        } else {
#pragma unroll
            for (int w = 1; w < NW; ++w) sum += part[w][row][k];
        }
        z[c] = cls[c] ? sum + bias[c] : -INFINITY;
        mx = fmaxf(mx, z[c]);
    }
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) mx = fmaxf(mx, __shfl_xor(mx, m, 16));
    float ex[CT], sum = 0.0f;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        ex[c] = cls[c] ? expf(z[c] - mx) : 0.0f;
        sum += ex[c];
    }
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) sum += __shfl_xor(sum, m, 16);
    if (b_row >= B) return;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const int k = 16 * c + l16;
        if (cls[c]) p.dz[((size_t)g * B + b_row) * C + k] = (ex[c] * (1.0f / sum) - (k == y ? 1.0f : 0.0f)) * (1.0f / (float)B);
        if (k == y) p.row_loss[(size_t)g * B + b_row] = logf(sum) - (z[c] - mx);
    }
}

// RT: 16-row tiles of the batch (1, 2, 4, 8 or 16; rows past the batch count as zeros).  CT: tiles of sixteen classes.  FIRST: the
// only layer (softmax regression): no error for a layer below.  UPDATE (then it is
// the only layer): the momentum step and the mix (Eq. (c0), (c1)) are applied to every column of the worker.  Grid: (ceil(H / 64), workers).
template <bool BF, int RT, int CT, bool FIRST, bool UPDATE, bool LIST>
__global__ void __launch_bounds__(HD_THREADS) head_grads_kernel(HeadArgs p)
{
    constexpr int BP = 16 * RT, CP = 16 * CT, tp = BP + 16;      // tp: pitch of the transposed dZ, rows 16 apart in banks
    constexpr int ZP = CP + 4;                   // floats per row of dZ: the four row groups that a wave reads at once differ in banks
    __shared__ float dzs[BP][ZP];                // dZ, columns C .. and rows B .. zero
    __shared__ float dzt[FIRST ? 1 : CP][tp];    // its transpose
    const int B = p.B, H = p.H, C = p.C;
    const int g = blockIdx.y, t = threadIdx.x, lane = t & 63, r = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wk = LIST ? p.worker[g] : g, Mx = LIST ? p.Mx : p.M;
    const bool first = blockIdx.x == 0;          // the workgroup that also writes what does not split by hidden units
    const int KT = (H + 15) / 16, kt = (int)blockIdx.x * HD_WAVES + wave;
    const int ktc = kt < KT ? kt : 0;            // waves past the end repeat the first block and store nothing
    const int hc = 16 * ktc + r < H ? 16 * ktc + r : H - 1;
    const HeadParams at(Mx, wk, p.woff);
    const float *Xg = p.X + at.base;
    // requests: this wave's 16 columns of the input (all batch rows; gathered rows by number first), its 16 rows of W, and dZ.
    // Rows past the batch repeat the last one and count as zeros.
    float hv[RT][4];                             // in[16 i + 4 q + v][16 kt + r]
    int32_t rows[RT][4];
    const int32_t *row_of = p.idx + (size_t)g * B;
    if (FIRST) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) rows[i][v] = row_of[min(16 * i + 4 * q + v, B - 1)];
    } else {
        const int64_t base = (int64_t)g * B * H;
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) hv[i][v] = head_input<BF>(p.in, base + (uint32_t)(min(16 * i + 4 * q + v, B - 1) * H + hc));
    }
    float wv[4 * CT];                            // W[16 kt + r][4 s + q]
    if constexpr (!FIRST) {
#pragma unroll
        for (int s = 0; s < 4 * CT; ++s) wv[s] = Xg[at.at((uint32_t)(hc * C + (4 * s + q < C ? 4 * s + q : 0)))];
    }
    float zv[BP * CP / HD_THREADS];
    const float *zg = p.dz + (size_t)g * B * C;
#pragma unroll
    for (int u = 0; u < BP * CP / HD_THREADS; ++u) {
        const int e = t + u * HD_THREADS, row = e / CP, c = e % CP;
        zv[u] = zg[min(row, B - 1) * C + (c < C ? c : 0)];
    }
    if (FIRST) {
        const int64_t base = p.row0[wk] * H + hc;
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) hv[i][v] = head_input<BF>(p.in, base + (int64_t)rows[i][v] * H);
    }
    // UPDATE: what it needs of this lane's parameters is asked for behind the operands and used after the products
    int m = g;
    float wi = 0.0f;
    size_t peer_shift = 0;
    float ux[CT][4], up[CT][4], uv[CT][4];
    auto update = [&](size_t own, float x, float v, float d, float xp) {
        float xn, vn;
        momentum_mix1(x, v, d, xp, wi, p.mix.alpha, p.mix.mu, p.mix.wd, xn, vn);
        p.mix.Xnext[own] = xn;
        p.mix.V[own] = vn;
    };
    if constexpr (UPDATE) {
        m = p.mix.peer[g];
        if ((unsigned)m >= (unsigned)Mx) m = wk;            // an index outside [0, M) is treated as a self draw
        wi = p.mix.w[(size_t)wk * Mx + m];
        peer_shift = ((size_t)m - (size_t)wk) << TILE_SHIFT;   // from a worker's element to its peer's
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const size_t own = at.base + at.at((uint32_t)(min(16 * ktc + 4 * q + v, H - 1) * C + min(16 * c + r, C - 1)));
                ux[c][v] = p.mix.Xcur[own];
                up[c][v] = p.mix.Xcur[own + peer_shift];
                uv[c][v] = p.mix.V[own];
            }
    }
    float lrow = 0.0f;
    if (first && wave == 0) {
#pragma unroll
        for (int u = 0; u < (BP + 63) / 64; ++u) {
            const int b = 64 * u + lane;
            const float l = p.row_loss[(size_t)g * B + (b < B ? b : B - 1)];
            lrow += b < B ? l : 0.0f;
        }
    }
#pragma unroll
    for (int u = 0; u < BP * CP / HD_THREADS; ++u) {
        const int e = t + u * HD_THREADS, row = e / CP, c = e % CP;
        const float d = c < C && row < B ? zv[u] : 0.0f;
        dzs[row][c] = d;
        if constexpr (!FIRST) dzt[c][row] = head_operand<BF>(d);
    }
    __syncthreads();
    if (first) {
        if (wave == 0) {
#pragma unroll
            for (int m = 32; m > 0; m >>= 1) lrow += __shfl_xor(lrow, m);
            if (lane == 0) p.loss[wk] = lrow / (float)B;
        }
        for (int64_t e = t; e < p.ld - p.D; e += HD_THREADS) {
            const size_t own = tiled_offset_quick(Mx, wk, p.D + e);
            p.G[own] = 0.0f;
            if constexpr (UPDATE) update(own, p.mix.Xcur[own], p.mix.V[own], 0.0f, p.mix.Xcur[own + peer_shift]);
        }
        // db = column sums of dZ: the product below with a row of ones in place of h^T (never rounded)
        if (wave == HD_WAVES - 1) {
            const float one = r == 0 ? 1.0f : 0.0f;
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int s = 0; s < BP / 4; ++s) acc = mfma_16x16x4(one, dzs[4 * s + q][16 * c + r], acc);
                if (q == 0 && 16 * c + r < C) {
                    const size_t own = at.base + at.at((uint32_t)(H * C + 16 * c + r));
                    p.G[own] = acc[0];
                    if constexpr (UPDATE) update(own, p.mix.Xcur[own], p.mix.V[own], acc[0], p.mix.Xcur[own + peer_shift]);
                }
            }
        }
    }
    if (kt >= KT) return;
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) hv[i][v] = 16 * i + 4 * q + v < B ? hv[i][v] : 0.0f;
    // ---- dW = h^T dZ, rows 16 kt .. 16 kt + 15: the batch is the contraction, taken in the order in which the lanes hold h
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc = mfma_16x16x4(hv[i][v], head_operand<BF>(dzs[16 * i + 4 * q + v][16 * c + r]), acc);
        if (16 * c + r < C) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (16 * kt + 4 * q + v < H) {
                    const size_t own = at.base + at.at((uint32_t)((16 * kt + 4 * q + v) * C + 16 * c + r));
                    p.G[own] = acc[v];
                    if constexpr (UPDATE) update(own, ux[c][v], uv[c][v], acc[v], up[c][v]);
                }
        }
    }
    // ---- dH = (dZ W^T) where h > 0, columns 16 kt .. 16 kt + 15 of all batch rows, and its column sums
    if constexpr (!FIRST) {
#pragma unroll
        for (int s = 0; s < 4 * CT; ++s) wv[s] = 4 * s + q < C ? head_operand<BF>(wv[s]) : 0.0f;
        const bool col_ok = 16 * kt + r < H;
        float *dhg = p.dh + (size_t)g * B * H;
        float colsum = 0.0f;
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int s = 0; s < 4 * CT; ++s) acc = mfma_16x16x4(dzt[4 * s + q][16 * i + r], wv[s], acc);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int b = 16 * i + 4 * q + v;
                const float d = hv[i][v] > 0.0f ? acc[v] : 0.0f;
                if (col_ok && b < B) dhg[(uint32_t)(b * H + 16 * kt + r)] = d;
                colsum += d;
            }
        }
        colsum += __shfl_xor(colsum, 16);
        colsum += __shfl_xor(colsum, 32);
        if (q == 0 && col_ok) p.G[tiled_offset_quick(Mx, wk, p.boff_below + 16 * kt + r)] = colsum;
    }
}

// At most 32 classes and 256 batch rows.  With bfloat16 operands the matrix-core kernels go first where they fit, and a
// matrix-core layer below wants the error as bfloat16 in both orientations, which these kernels do not write.
bool head_ok(const MlpPlan &p)
{
    const int L = p.n_layers;
    if (p.dims[L] > HD_MAX_C || p.B > HD_MAX_B) return false;
    // 32-bit element numbers inside the layer's span of the tile layout and inside a worker's activations
    const int64_t H = p.dims[L - 1], tiles = (H * p.dims[L] + p.dims[L]) / TILE + 2;
    if (tiles * p.Mx * TILE >= (int64_t)1 << 32 || H * p.B >= (int64_t)1 << 31) return false;
    return !p.bf16 || !(mfma_small_last_ok(p) || (L > 1 && mfma_layer_ok(p, L - 2)));
}

int head_pairs_per_wave(const MlpPlan &p)
{
    const int pairs = (int)(p.dims[p.n_layers - 1] / 32), waves = 2 * pairs <= HL_FEW * HD_STEPS ? HL_FEW : HL_MANY;
    return (pairs + waves - 1) / waves;
}
// Hidden units in pairs of steps of sixteen, not more than the waves' first ones.
bool head_parts_of_two(const MlpPlan &p)
{
    const int64_t H = p.dims[p.n_layers - 1], C = p.dims[p.n_layers];
    return p.n_layers > 1 && head_ok(p) && !p.bf16 && C <= 16 && H % 32 == 0 && H <= 16 * HD_STEPS * HL_MANY;
}

template <bool BF, int CT, int NW, bool LIST> static void launch_logits_waves(hipStream_t s, const HeadArgs &a)
{
    const dim3 grid((unsigned)((a.B + 15) / 16), (unsigned)a.M), block(64 * NW);
    // pieces of four features need rows that start at multiples of their size
    const bool pieces = a.H % 4 == 0 && reinterpret_cast<uintptr_t>(a.in) % (BF ? 8 : 16) == 0;
    if constexpr (!BF && CT == 1 && !LIST)
        if (a.pairs && pieces) {
            hipLaunchKernelGGL((head_logits_kernel<BF, HL_WHOLE, CT, NW, true>), grid, block, 0, s, a);
            return;
        }
    if (pieces && a.H % 16 == 0) hipLaunchKernelGGL((head_logits_kernel<BF, HL_WHOLE, CT, NW, false, LIST>), grid, block, 0, s, a);
    else if (pieces) hipLaunchKernelGGL((head_logits_kernel<BF, HL_PIECES, CT, NW, false, LIST>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((head_logits_kernel<BF, HL_SINGLE, CT, NW, false, LIST>), grid, block, 0, s, a);
}
template <bool BF, int CT, bool LIST> static void launch_logits(hipStream_t s, const HeadArgs &a)
{
    if ((a.H + 15) / 16 <= HL_FEW * HD_STEPS) launch_logits_waves<BF, CT, HL_FEW, LIST>(s, a);
    else launch_logits_waves<BF, CT, HL_MANY, LIST>(s, a);
}

template <bool BF, int CT, bool FIRST, bool UPDATE, bool LIST> static void launch_grads(hipStream_t s, const HeadArgs &a)
{
    const dim3 grid((unsigned)(((a.H + 15) / 16 + HD_WAVES - 1) / HD_WAVES), (unsigned)a.M), block(HD_THREADS);
    if (a.B <= 16) hipLaunchKernelGGL((head_grads_kernel<BF, 1, CT, FIRST, UPDATE, LIST>), grid, block, 0, s, a);
    else if (a.B <= 32) hipLaunchKernelGGL((head_grads_kernel<BF, 2, CT, FIRST, UPDATE, LIST>), grid, block, 0, s, a);
    else if (a.B <= 64) hipLaunchKernelGGL((head_grads_kernel<BF, 4, CT, FIRST, UPDATE, LIST>), grid, block, 0, s, a);
    else if (a.B <= 128) hipLaunchKernelGGL((head_grads_kernel<BF, 8, CT, FIRST, UPDATE, LIST>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((head_grads_kernel<BF, 16, CT, FIRST, UPDATE, LIST>), grid, block, 0, s, a);
}

template <bool BF, int CT> static void launch_both(hipStream_t s, const HeadArgs &a, bool only_layer, bool update)
{
    if constexpr (!BF)
        if (a.worker) {                          // layer_list_ok(): fp32, a single layer with its update
            launch_logits<BF, CT, true>(s, a);
            if (!only_layer) launch_grads<BF, CT, false, false, true>(s, a);
            else launch_grads<BF, CT, true, true, true>(s, a);
            return;
        }
    launch_logits<BF, CT, false>(s, a);
    if (!only_layer) launch_grads<BF, CT, false, false, false>(s, a);
    else if (update) launch_grads<BF, CT, true, true, false>(s, a);
    else launch_grads<BF, CT, true, false, false>(s, a);
}

void launch_head(hipStream_t s, const MlpPlan &p, const float *X, float *G, const MixArgs *tail)
{
    const int L = p.n_layers;
    HeadArgs a;
    a.mix = tail ? *tail : MixArgs{};
    a.in = L == 1 ? p.feats : (p.bf16 ? (const void *)p.hb[L - 1] : (const void *)p.act[L - 1]);
    a.row0 = p.row0; a.idx = p.idx; a.gather = L == 1;
    a.X = X; a.G = G; a.labels = p.labels;
    a.dz = p.dz[0]; a.dh = p.dz[1]; a.loss = p.loss;
    a.row_loss = p.act[L];          // [M][B][C], not used for the logits on this path
    a.M = p.M; a.B = p.B; a.H = (int)p.dims[L - 1]; a.C = (int)p.dims[L];
    a.Mx = p.Mx; a.worker = p.worker;
    a.pairs = p.head_pairs && head_parts_of_two(p);
    a.woff = p.woff[L - 1];
    a.boff_below = L == 1 ? 0 : p.woff[L - 2] + p.dims[L - 2] * p.dims[L - 1];
    a.D = p.woff[L - 1] + p.dims[L - 1] * p.dims[L] + p.dims[L]; a.ld = p.ld;
    if (p.bf16) {
        if (a.C <= 16) launch_both<true, 1>(s, a, L == 1, tail != nullptr);
        else launch_both<true, 2>(s, a, L == 1, tail != nullptr);
    } else {
        if (a.C <= 16) launch_both<false, 1>(s, a, L == 1, tail != nullptr);
        else launch_both<false, 2>(s, a, L == 1, tail != nullptr);
    }
}

}  // namespace netmax
