// Whole NetMax iterations of softmax-regression models that one workgroup cannot hold, in one kernel (Algorithm 2, all of its steps):
// a worker's features are cut into slices, one workgroup keeps a slice of the parameters, of the momentum and of the batch rows in LDS.
// An iteration needs two exchanges: the slices of a worker add up their partial logits, and a slice pulls the peer's same slice.
// The logits cross the chip once per iteration (stored, counted, polled, read: about 2 us); the peer's row was stored half an iteration
// before it is asked for.  784-10, batch 64, 16 workers, eight iterations 75 us, 21 of them outside the kernel (a cooperative launch), where the draws and
// the two kernels of k_grad_head.hip take 89 to 94.  The matrix units are busy 12 % of the time; the waves wait for memory, LDS or each other 51 % of theirs.
// An iteration in 6.6 us (time stamps in a copy of the kernel): logits 1.2, their
// exchange 1.5, softmax and waiting 1.1, gradient and update 1.8, the rest draws, row addresses and barriers.
//
// The slices are the runs of features that the waves of head_logits_kernel take, and all sums are made in that kernel's and in
// head_grads_kernel's order: the results are theirs bit for bit.
#include "kernels.h"
#include "layout.h"
#include "philox.h"
#include "resident.h"
#include "tile.h"

#include <type_traits>

namespace netmax {

constexpr int SL_THREADS = 1024, SL_WAVES = SL_THREADS / 64, SL_AHEAD = 16;
constexpr int SL_MAX_C = 16, SL_MAX_B = 64, SL_MAX_PAD = 4096, SL_LDS_LIMIT = 150 * 1024;
constexpr int SL_P16 = SL_MAX_C + 4;            // floats per row of W and of dZ in LDS, sixteen classes: four rows apart half a round over the banks
constexpr int SL_STEPS = 8;                     // steps of sixteen features in a slice, at most
constexpr int SL_PITCH = 16 * SL_STEPS + 20;    // floats per batch row in LDS: 20 more than whole rounds over the banks

struct SlicedArgs {
    int M, B, H, C, P, per;                     // P slices of `per` steps of sixteen features
    int64_t D, ld;
    const float *feats; const int32_t *labels; const int64_t *row0; const int32_t *n_rows;
    const uint32_t *thr; const int32_t *last; const float *w;
    float *x_first, *x_second, *V, *G, *loss; int32_t *peers;
    float alpha, mu, wd; uint64_t seed; IterRef iter; int n_iters;
    unsigned long long *parts;                  // [2][M][P][row tiles][256] partial logits, each with the ticket of its iteration above it
    float *biases;                              // [2][M][P][16] every slice's copy of the new bias
    unsigned ticket;                            // of the first iteration
    unsigned *rows_count; unsigned rows_base;   // [P], a line apart: arrivals with new rows, M per iteration but the last
    int *fault; long long patience;
};

static int sl_parts_of(int64_t H) { return (H + 15) / 16 <= 32 ? 4 : 8; }          // the waves of head_logits_kernel
static int sl_per(int64_t H) { return (int)(((H + 15) / 16 + sl_parts_of(H) - 1) / sl_parts_of(H)); }
static int sl_slices(int64_t H) { return (int)(((H + 15) / 16 + sl_per(H) - 1) / sl_per(H)); }
static __device__ __host__ __forceinline__ int sl_ahead(int B) { return 1024 / B < SL_AHEAD ? 1024 / B : SL_AHEAD; }
static size_t sl_lds(int B, int64_t pad)
{
    const int rows = B <= 16 ? 16 : B <= 32 ? 32 : 64;
    return sizeof(float) * ((size_t)rows * SL_PITCH + (size_t)(16 * SL_STEPS + rows) * SL_P16 + 64 + 16 + 2 * (size_t)pad) +
           sizeof(int32_t) * ((size_t)sl_ahead(B) * B + 2 * (size_t)B + 2 * SL_AHEAD * SL_WAVES);
}

// RT: 16-row tiles of the batch (1, 2 or 4; rows past the batch count as zeros): a wave each for the logits, four for the softmax.
// Sixteen features of the slice belong to a wave: it computes their dW, whose result layout (a lane has four rows of one class) also is
// the one in which it keeps their parameters and momentum in registers and updates them; LDS has a copy of W for the forward pass.
// (A thread per vector of four parameters, with dW turned through LDS, spends its time on addresses: 62 instead of 55 us for those, launched
// plainly.  256 threads with four rows of the softmax each: 69 us.  Counted arrivals instead of tickets, four round trips to memory instead of two: 126 us.)
// The last iteration asks for its own rows again (no load under a branch).
template <int RT>
__global__ void __launch_bounds__(SL_THREADS) sliced_softmax_kernel(SlicedArgs p)
{
    extern __shared__ __attribute__((aligned(16))) float sl_smem[];
    constexpr int BP = 16 * RT;
    constexpr int BURST = (BP * SL_STEPS * 4 + SL_THREADS - 1) / SL_THREADS;      // all of a slice's batch rows
    const int t = threadIdx.x, lane = t & 63, r = lane & 15, q = lane >> 4, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int i = (int)blockIdx.x / p.P, s = (int)blockIdx.x - i * p.P;
    const int F = 16 * p.per, f0 = s * F, Fs = min(F, p.H - f0);       // Fs: a multiple of four
    const bool tail = s == p.P - 1;                           // this slice also owns the bias and the padding
    const int pad = tail ? (int)(p.ld - p.D) : 0;
    float *xs = sl_smem;                                      // [BP][SL_PITCH] batch rows, zeros where there is none
    float *wl = xs + BP * SL_PITCH;                              // [16 STEPS][SL_P16] W, zeros beyond the slice and the classes
    float *dzs = wl + 16 * SL_STEPS * SL_P16;                    // [BP][SL_P16] dZ, zeros beyond the batch and the classes
    float *lr = dzs + BP * SL_P16;                            // [64] loss of every batch row
    float *xb = lr + 64;                                      // [16] the bias: every slice keeps it up to date
    float *px = xb + 16, *pv = px + pad;                      // the padding columns and their momentum
    int32_t *ib = reinterpret_cast<int32_t *>(px + 2 * (p.ld - p.D));      // [ahead][B] batch rows of the iterations drawn together
    const int ahead = sl_ahead(p.B);
    int32_t *yl = ib + ahead * p.B;                           // [2][B] labels of this and the next iteration
    int32_t *cnt = yl + 2 * p.B;                              // [2][SL_AHEAD][waves] thresholds of the peer draws that are <= u
    const uint64_t iter0 = iteration_of(p.iter);
    const uint32_t n_i = (uint32_t)p.n_rows[i];
    const int64_t r0 = p.row0[i];
    const int last_i = p.last[i];
    const float *shard = p.feats + (size_t)r0 * p.H + f0;
    const uint32_t thr_own = p.thr[(size_t)i * p.M + min(t, p.M - 1)];

    auto draw_group = [&](int it0, int group) {
        const int n = p.n_iters - it0 < ahead ? p.n_iters - it0 : ahead, blocks = (p.B + 3) >> 2;
        for (int e = SL_THREADS - 1 - t; e < n * blocks; e += SL_THREADS) {
            const int k = e / blocks, b4 = e - k * blocks;
            const Words4 d = draw_block(p.seed, STREAM_BATCH, (uint32_t)b4, (uint32_t)i, iter0 + (uint64_t)(it0 + k));
            const uint32_t word[4] = {d.a, d.b, d.c, d.d};
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (4 * b4 + c < p.B) ib[k * p.B + 4 * b4 + c] = (int32_t)__umulhi(word[c], n_i);
        }
        if (64 * wave >= p.M) return;
        const uint32_t us = draw_block(p.seed, STREAM_PEER, 0u, (uint32_t)i, iter0 + (uint64_t)(it0 + (lane < n ? lane : 0))).a;
        int32_t *to = cnt + group * (SL_AHEAD * SL_WAVES) + wave;
        for (int k = 0; k < n; ++k) {
            const uint32_t u = (uint32_t)__builtin_amdgcn_readlane((int)us, k);
            const int hits = (int)__popcll(__ballot(t < p.M && thr_own <= u));
            if (lane == 0) to[k * SL_WAVES] = hits;
        }
    };
    auto drawn_peer = [&](int group, int at) {
        const int32_t *counts = cnt + group * (SL_AHEAD * SL_WAVES) + at * SL_WAVES;
        int hits = counts[0];
        for (int w = 1; w < SL_WAVES && 64 * w < p.M; ++w) hits += counts[w];
        return __builtin_amdgcn_readfirstlane(hits < last_i ? hits : last_i);
    };
    // this thread's pieces of the batch rows: row of the batch, first feature (past the end the first piece again, unused)
    const int row_units = Fs >> 2, feat_units = p.B * row_units;
    int piece_row[BURST], piece_at[BURST];
#pragma unroll
    for (int e = 0; e < BURST; ++e) {
        const int u = e * SL_THREADS + t, uc = u < feat_units ? u : 0;
        piece_row[e] = uc / row_units;
        piece_at[e] = 4 * (uc - piece_row[e] * row_units);
    }
    f32x4 rf[BURST];
    const float *src[BURST];
    auto find_rows = [&](const int32_t *rows) {
#pragma unroll
        for (int e = 0; e < BURST; ++e) src[e] = shard + (size_t)rows[piece_row[e]] * p.H + piece_at[e];
    };
    auto request_rows = [&]() {
#pragma unroll
        for (int e = 0; e < BURST; ++e) rf[e] = *reinterpret_cast<const tile_f32x4_any *>(src[e]);
    };

    // ---- before the first iteration
    // this lane's parameters: rows 16 wave + 4 q + v, class r; and, each slice's copy, lanes 0 .. 15 of the last wave: the bias
    uint32_t own[4];                                          // bytes
    float x[4], vel[4];
    bool mine[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int k = 16 * wave + 4 * q + v;
        mine[v] = k < Fs && r < p.C;
        own[v] = (uint32_t)tiled_offset(p.M, i, (int64_t)(f0 + min(k, Fs - 1)) * p.C + min(r, p.C - 1)) * 4u;
        x[v] = *at_bytes(p.x_first, own[v]);
        vel[v] = *at_bytes(p.V, own[v]);
    }
    const bool bias_lane = wave == SL_WAVES - 1 && lane < 16;
    const uint32_t bias_own = (uint32_t)tiled_offset(p.M, i, (int64_t)p.H * p.C + min(r, p.C - 1));
    float bias_x = p.x_first[bias_own], bias_v = p.V[bias_own];
    draw_group(0, 0);
    for (int e = t; e < BP * SL_PITCH + 16 * SL_STEPS * SL_P16 + BP * SL_P16 + 64; e += SL_THREADS) xs[e] = 0.0f;
    __syncthreads();
    const int t_row = min(t, p.B - 1);
    int32_t label = p.labels[r0 + ib[t_row]];
    find_rows(ib);
    request_rows();
#pragma unroll
    for (int v = 0; v < 4; ++v)
        if (mine[v]) wl[(16 * wave + 4 * q + v) * SL_P16 + r] = x[v];
    if (bias_lane) {
        xb[r] = bias_x;
        // The peer's bias of the first iteration.  All slices read the one that the peer's last slice replaces in the second, so it is in LDS (behind
        // a class row of W) before this slice sends its first partial logits: the peer's last slice writes behind the arrivals of all
        // last slices, and the one of this worker arrives behind the logits of all of its slices.  What else a slice reads of a peer comes from
        // the same slice, whose arrival it has waited for.
        wl[r * SL_P16 + SL_MAX_C] = p.x_first[tiled_offset(p.M, drawn_peer(0, 0), (int64_t)p.H * p.C + min(r, p.C - 1))];
    }
    for (int e = t; e < pad; e += SL_THREADS) {
        const size_t at = tiled_offset(p.M, i, p.D + e);
        px[e] = p.x_first[at];
        pv[e] = p.V[at];
    }
    if (t < p.B) yl[t] = label;

    int at = 0, group = 0;                                    // the iteration's place in its group of draws, the group's parity
    for (int it = 0; it < p.n_iters; ++it) {
        const int cur = it & 1, nxt = cur ^ 1;
        const bool more = it + 1 < p.n_iters;
        float *Xcur = cur ? p.x_second : p.x_first, *Xnext = cur ? p.x_first : p.x_second;
        // ---- this iteration's batch rows into LDS
#pragma unroll
        for (int e = 0; e < BURST; ++e)
            if (e * SL_THREADS + t < feat_units) *reinterpret_cast<f32x4 *>(xs + piece_row[e] * SL_PITCH + piece_at[e]) = rf[e];
        if (it > 0) stores_arrived();                         // this wave's new parameters, on their way since the update
        __syncthreads();
        if (it > 0 && t == 0) __hip_atomic_fetch_add(p.rows_count + 32 * s, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned ticket = p.ticket + (unsigned)it;
        unsigned long long *words = p.parts + (((size_t)cur * p.M + i) * p.P * RT + wave % RT) * 256 + lane;      // slice k at k RT 256, element v at 64 v
        if (wave < RT) {
            // ---- partial logits of sixteen batch rows
            __builtin_amdgcn_s_setprio(3);                    // everybody waits for these
            f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
            const float *xrow = xs + (16 * wave + r) * SL_PITCH + 4 * q, *wcol = wl + 4 * q * SL_P16 + r;
            auto steps = [&](int u0, auto n) {
                constexpr int N = decltype(n)::value;
                f32x4 a[N];
                float b[N][4];
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    a[u] = *reinterpret_cast<const f32x4 *>(xrow + 16 * (u0 + u));
#pragma unroll
                    for (int j = 0; j < 4; ++j) b[u][j] = wcol[(16 * (u0 + u) + j) * SL_P16];
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < N; ++u)
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][j], b[u][j], acc, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            };
            const int n_steps = (Fs + 15) / 16;
            int u0 = 0;
            for (; u0 + 4 <= n_steps; u0 += 4) steps(u0, std::integral_constant<int, 4>{});
            if (n_steps - u0 == 3) steps(u0, std::integral_constant<int, 3>{});
            else if (n_steps - u0 == 2) steps(u0, std::integral_constant<int, 2>{});
            else if (n_steps - u0 == 1) steps(u0, std::integral_constant<int, 1>{});
            // A sum and its ticket are one word: who finds the ticket has the sum, and no store is waited for.  Two sets of words take turns: a
            // slice that writes the next set's has seen every slice of its worker past the one before.
            if (r < p.C) {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    __hip_atomic_store(words + (size_t)s * RT * 256 + 64 * v, ((unsigned long long)ticket << 32) | __float_as_uint(acc[v]), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            }
            __builtin_amdgcn_s_setprio(0);
        }
        const int m = drawn_peer(group, at);
        const float wi = p.w[(size_t)i * p.M + m];
        const ptrdiff_t shift = ((ptrdiff_t)m - i) * TILE;    // from a worker's element to its peer's
        if (t == 0 && s == 0 && !more) p.peers[i] = m;
        const bool fresh = more && at + 1 == ahead;
        const int next_at = fresh ? 0 : more ? at + 1 : at;
        if (fresh) {
            draw_group(it + 1, group ^ 1);
            __syncthreads();                                  // its rows are looked up before the next barrier
        }
        find_rows(ib + next_at * p.B);
        unsigned seen = 0;
        if (wave < 4 * RT) {
            // ---- the parts of one element of every lane's four: sixteen lanes have a batch row's classes
            const int v = wave / RT, b = 16 * (wave % RT) + 4 * q + v;
            words += 64 * v;
            unsigned long long word[8];
            long long polls = 0;
            bool here;
            do {
                here = true;
#pragma unroll
                for (int k = 0; k < 8; ++k) word[k] = __hip_atomic_load(words + (size_t)(k < p.P ? k : 0) * RT * 256, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int k = 0; k < 8; ++k) here &= (unsigned)(word[k] >> 32) == ticket;
            } while ((p.patience == 0 || __any(!here && r < p.C)) && !gives_up(++polls, p.fault, p.patience));
            if (wave == 0) seen = arrivals(p.rows_count + 32 * s);
            // ---- added in order, bias, softmax cross-entropy
            const bool real = r < p.C;
            float z = __uint_as_float((unsigned)word[0]);
#pragma unroll
            for (int k = 1; k < 8; ++k) z += k < p.P ? __uint_as_float((unsigned)word[k]) : 0.0f;
            z = real ? z + xb[r] : -INFINITY;
            float mx = z;
            mx = fmaxf(mx, xor_lane<1>(mx));
            mx = fmaxf(mx, xor_lane<2>(mx));
            mx = fmaxf(mx, xor_lane<4>(mx));
            mx = fmaxf(mx, xor_lane<8>(mx));
            const float ex = real ? expf(z - mx) : 0.0f;
            float sum = ex;
            sum += xor_lane<1>(sum);
            sum += xor_lane<2>(sum);
            sum += xor_lane<4>(sum);
            sum += xor_lane<8>(sum);
            const int y = yl[cur * p.B + min(b, p.B - 1)];
            const float d = (ex * (1.0f / sum) - (r == y ? 1.0f : 0.0f)) * (1.0f / (float)p.B);
            dzs[b * SL_P16 + r] = real && b < p.B ? d : 0.0f;
            if (!more && r == y && b < p.B) lr[b] = logf(sum) - (z - mx);
        }
        if (it > 0 && t == 0) await_arrivals(p.rows_count + 32 * s, seen, p.rows_base + (unsigned)it * (unsigned)p.M, p.fault, p.patience);
        __syncthreads();
        // ---- the peer's parameters, the next iteration's labels and batch rows: asked for here, used behind the products
        float xp[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) xp[v] = __hip_atomic_load(at_bytes(Xcur + shift, own[v]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const float bias_p = __hip_atomic_load(p.biases + (((size_t)cur * p.M + m) * p.P + s) * 16 + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        label = p.labels[r0 + ib[next_at * p.B + t_row]];
        request_rows();
        // ---- dW = X^T dZ: the batch is the contraction, taken in the order of head_grads_kernel; momentum step and mix (Eq. (c0), (c1))
        if (16 * wave < Fs) {
            float av[RT][4], bz[RT][4];
#pragma unroll
            for (int k = 0; k < RT; ++k)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    av[k][v] = xs[(16 * k + 4 * q + v) * SL_PITCH + 16 * wave + r];
                    bz[k][v] = dzs[(16 * k + 4 * q + v) * SL_P16 + r];
                }
            __builtin_amdgcn_sched_barrier(0);
            f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < RT; ++k)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[k][v], bz[k][v], acc, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float xn, vn;
                momentum_mix1(x[v], vel[v], acc[v], xp[v], wi, p.alpha, p.mu, p.wd, xn, vn);
                x[v] = xn;
                vel[v] = vn;
                if (mine[v]) {
                    store_row(at_bytes(Xnext, own[v]), xn, more);
                    wl[(16 * wave + 4 * q + v) * SL_P16 + r] = xn;
                    if (!more) { *at_bytes(p.V, own[v]) = vn; *at_bytes(p.G, own[v]) = acc[v]; }
                }
            }
        }
        if (wave == SL_WAVES - 1) {
            // db = column sums of dZ: the product with a row of ones, rows 4 s + q in step s
            f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
            const float one = r == 0 ? 1.0f : 0.0f;
#pragma unroll
            for (int k = 0; k < 4 * RT; ++k) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(one, dzs[(4 * k + q) * SL_P16 + r], acc, 0, 0, 0);
            if (bias_lane) {
                float xn, vn;
                momentum_mix1(bias_x, bias_v, acc[0], it == 0 ? wl[r * SL_P16 + SL_MAX_C] : bias_p, wi, p.alpha, p.mu, p.wd, xn, vn);
                bias_x = xn;
                bias_v = vn;
                xb[r] = xn;
                __hip_atomic_store(p.biases + (((size_t)nxt * p.M + i) * p.P + s) * 16 + r, xn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (tail && r < p.C) {
                    store_row(Xnext + bias_own, xn, more);
                    if (!more) { p.V[bias_own] = vn; p.G[bias_own] = acc[0]; }
                }
            }
        }
        for (int e = SL_THREADS - 1 - t; e < pad; e += SL_THREADS) {       // from the last wave down: the first ones have the tiles
            const size_t to = tiled_offset(p.M, i, p.D + e);
            float xn, vn;
            momentum_mix1(px[e], pv[e], 0.0f, __hip_atomic_load(Xcur + shift + to, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), wi, p.alpha, p.mu, p.wd, xn, vn);
            px[e] = xn;
            pv[e] = vn;
            store_row(Xnext + to, xn, more);
            if (!more) { p.V[to] = vn; p.G[to] = 0.0f; }
        }
        if (wave == 0 && s == 0 && !more) {
            float l = lane < p.B ? lr[lane] : 0.0f;
#pragma unroll
            for (int k = 32; k > 0; k >>= 1) l += __shfl_xor(l, k);
            if (lane == 0) p.loss[i] = l / (float)p.B;
        }
        if (more && t < p.B) yl[nxt * p.B + t] = label;
        at = next_at;
        group ^= fresh;
        __syncthreads();                                      // batch rows and dZ have been read
    }
}

typedef void (*SlicedKernel)(SlicedArgs);
static SlicedKernel sliced_kernel(int B) { return B <= 16 ? sliced_softmax_kernel<1> : B <= 32 ? sliced_softmax_kernel<2> : sliced_softmax_kernel<4>; }
static int64_t sl_padding(const MlpPlan &p) { return p.ld - (p.dims[0] * p.dims[1] + p.dims[1]); }

// Rows of four features at a time, slices that fit LDS and their waves, their padding with them.
bool sliced_iter_ok(const MlpPlan &p)
{
    return p.n_layers == 1 && !p.bf16 && p.M <= SL_THREADS && head_ok(p) && p.dims[1] <= SL_MAX_C && p.B <= SL_MAX_B && p.dims[0] % 4 == 0 &&
           sl_per(p.dims[0]) <= SL_STEPS && p.ld * p.M < (int64_t)1 << 30 && sl_padding(p) <= SL_MAX_PAD &&
           sl_lds(p.B, sl_padding(p)) <= (size_t)SL_LDS_LIMIT;
}

// What the context keeps for it: words of `parts` (cleared), floats of `biases`, counters (cleared).
void sliced_iter_scratch(const MlpPlan &p, size_t &parts, size_t &biases, size_t &counters)
{
    const size_t slices = (size_t)p.M * sl_slices(p.dims[0]);
    parts = 2 * slices * 4 * 256;
    biases = 2 * slices * 16;
    counters = 8 * 32;
}
int sliced_iter_slices(const MlpPlan &p) { return sl_slices(p.dims[0]); }

// A cooperative launch costs about 20 us more than a plain one.  The separate kernels and this one, us: 784-10, batch 64, 16 workers, 3 iterations 37.8 and 45.2,
// 4 49.0 and 50.8, 5 60.1 and 56.4, 8 88.9 and 72.9; 1024-16, 4 workers, 4 iterations 52.0 and 50.8, 5 63.8 and 57.3; 512-10, batch 32, 8 workers, 4
// iterations 43.8 and 45.2, 5 53.3 and 49.8.
bool sliced_iter_pays(int n_iters) { return n_iters >= 5; }

// Workgroups of the kernel that the device holds at once (0: it has no cooperative launches); raises its LDS limit.
hipError_t prepare_sliced_iter(const MlpPlan &p, int *resident)
{
    int dev = 0, cus = 0, cooperative = 0;
    *resident = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cooperative, hipDeviceAttributeCooperativeLaunch, dev);
    const void *kernel = reinterpret_cast<const void *>(sliced_kernel(p.B));
    int per_cu = 0;
    if (e == hipSuccess) e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, SL_LDS_LIMIT);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, SL_THREADS, sl_lds(p.B, sl_padding(p)));
    if (e == hipSuccess && cooperative) *resident = per_cu * cus;
    return e;
}

hipError_t launch_sliced_iter(hipStream_t s, const MlpPlan &p, const SlicedIterLaunch &a)
{
    SlicedArgs k{};
    k.M = p.M; k.B = p.B; k.H = (int)p.dims[0]; k.C = (int)p.dims[1]; k.P = sl_slices(p.dims[0]); k.per = sl_per(p.dims[0]);
    k.D = p.dims[0] * p.dims[1] + p.dims[1]; k.ld = p.ld;
    k.feats = (const float *)p.feats; k.labels = p.labels; k.row0 = p.row0; k.n_rows = a.n_rows;
    k.thr = a.thr; k.last = a.last; k.w = a.mix.w;
    k.x_first = const_cast<float *>(a.mix.Xcur); k.x_second = a.mix.Xnext; k.V = a.mix.V; k.G = a.G; k.loss = p.loss; k.peers = a.peers;
    k.alpha = a.mix.alpha; k.mu = a.mix.mu; k.wd = a.mix.wd; k.seed = a.seed; k.iter = a.iter; k.n_iters = a.n_iters;
    k.parts = a.parts; k.biases = a.biases;
    k.ticket = a.ticket; k.rows_count = a.counters; k.rows_base = a.rows_base;
    k.fault = a.fault; k.patience = a.patience;
    const dim3 grid((unsigned)(p.M * k.P)), block(SL_THREADS);
    void *args[] = {&k};
    return hipLaunchCooperativeKernel(reinterpret_cast<const void *>(sliced_kernel(p.B)), grid, block, args, (unsigned)sl_lds(p.B, sl_padding(p)), s);
}

}  // namespace netmax
