// Whole NetMax iterations of a perceptron with one hidden layer on fp32 operands in one kernel (Algorithm 2, all of its steps), for
// models whose first weight matrices fit the chip's LDS together: a workgroup keeps 32 hidden units of one worker for the whole
// launch: their columns of W1 in LDS, the momentum of these in registers, their rows of W2.  An iteration then reads the batch rows (twice), the
// peer's columns, and writes the new ones for those who pull them; x, v and g of the separate kernels' 20 bytes per parameter stay on the chip.
//
// The units of a worker meet once per iteration: every workgroup multiplies its 32 activations with its rows of W2 and sends the
// partial logits as words that carry the iteration's ticket; all add up all of them and make the softmax for themselves.  Everything
// below needs no other unit: dZ2 gives dW2's rows, the error of the units and their columns of dW1, which are updated where the product leaves
// them.  The peer's columns come from the workgroup of the same units, which wrote them half an iteration before.
//
// 784-512-10, batch 64, 16 workers (all 256 compute units), four iterations: 157 us, 17 of them outside the kernel (a cooperative launch), the separate
// kernels 211.  The matrix units are busy 36 % of the time; the waves wait for memory, LDS or each other 40 % and for their turn to issue 41 % of theirs.  An
// iteration takes 27 us (this and what follows: time stamps in a copy of the kernel):
// forward 7.3 (its matrix instructions 5.3), the waves' tiles added 1.9, exchange and softmax 4.5, error 1.1, dW1 and its update the rest, beside
// them the rows of W2 (3, two waves).  The strips of dW1 are bound by addresses and waiting, not by their matrix instructions (5.4).  What it
// is made of (four iterations, launched plainly): loads in global and not in flat address space (169 -> 143 us), the next strip's batch rows asked for before this one's stores, the
// peer's parameters only ahead of the strip's own products (12 registers spilled instead of 74: 148 -> 135 us), addresses as 32-bit byte
// offsets from a strip's first row, one path for all features of a strip.
//
// The sums are those of fwd_f32_kernel, head_logits_kernel, head_grads_kernel and wgrad_f32_kernel, in their order: the results are theirs bit
// for bit.
#include "kernels.h"
#include "layout.h"
#include "philox.h"
#include "resident.h"
#include "tile.h"

#include <cmath>
#include <type_traits>

namespace netmax {

constexpr int RM_THREADS = 512, RM_WAVES = RM_THREADS / 64, RM_COLS = 32, RM_KS = 8, RM_DEPTH = 4, RM_AHEAD = 16;
constexpr int RM_STRIPS = 4;                    // strips of 32 features per wave: up to 1024 features
constexpr int RM_MAX_C = 16, RM_P16 = RM_MAX_C + 4, RM_HP = RM_COLS + 4, RM_PP = RM_COLS + 1, RM_MAX_PAD = 2048;
constexpr int RM_WORDS = 16;                    // partial logits asked for together: those of four runs of at most four
constexpr int RM_LDS_LIMIT = 160 * 1024 - 512;

struct ResidentArgs {
    int M, B, din, H, C, NB, run;               // NB = H / 32 workgroups per worker; run: partial logits that are added up first
    int64_t D, ld;
    const float *feats; const int32_t *labels; const int64_t *row0; const int32_t *n_rows;
    const uint32_t *thr; const int32_t *last; const float *w;
    float *x_first, *x_second, *V, *G, *loss, *hidden; int32_t *peers;
    float alpha, mu, wd; uint64_t seed; IterRef iter; int n_iters;
    unsigned long long *words;                  // [2][M][NB][row tiles of sixteen][256] partial logits, each with its iteration's ticket above it
    float *biases;                              // [2][M][NB][16] every workgroup's copy of the new output bias
    unsigned ticket;                            // of the first iteration
    unsigned *rows_count; unsigned rows_base;   // [NB], a line apart: arrivals with new parameters, M per iteration but the last
    int *fault; long long patience;
};

static __device__ __host__ __forceinline__ int rm_ahead(int B) { return 1024 / B < RM_AHEAD ? 1024 / B : RM_AHEAD; }
static size_t rm_lds(int B, int64_t din, int64_t pad)
{
    return sizeof(float) * ((size_t)din * RM_COLS + RM_WAVES * 32 * RM_PP + (size_t)B * RM_HP + RM_COLS * RM_P16 + 32 + 16 + 64 + 2 * (size_t)pad) +
           sizeof(int32_t) * ((size_t)rm_ahead(B) * B + 3 * (size_t)B + 2 * RM_AHEAD * RM_WAVES);
}

typedef float rm_f32x16 __attribute__((ext_vector_type(16)));

// Byte offset of parameter j (4 j = j4) of a worker from its first one in the tile layout: skip = 8192 (M - 1) < 2^24.
__device__ __forceinline__ uint32_t tile_bytes(uint32_t j4, uint32_t skip) { return __umul24(j4 >> (TILE_SHIFT + 2), skip) + j4; }

// RT: batch / 32.
template <int RT>
__global__ void __launch_bounds__(RM_THREADS) resident_mlp_kernel(ResidentArgs p)
{
    extern __shared__ __attribute__((aligned(16))) float rm_smem[];
    constexpr int B = 32 * RT, T16 = 2 * RT, HB = B / 2;
    int i;
    unsigned nb;
    if (!decode_group(blockIdx.x, (unsigned)p.NB, p.M, i, nb)) return;          // a worker's workgroups share an XCD (its batch rows)
    const int t0 = threadIdx.x, t = t0, lane = t & 63, col = lane & 31, half = lane >> 5, r = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const bool tail = (int)nb == p.NB - 1;                    // also owns the output bias and the padding
    const int max_pad = (int)(p.ld - p.D), pad = tail ? max_pad : 0;
    float *wl = rm_smem;                                      // [din][32] this workgroup's columns of W1
    float *part = wl + p.din * RM_COLS;                       // [waves][32][33] partial tiles of the forward pass; then:
    float *dhs = part, *dzs = dhs + B * RM_HP;                //   [B][36] error of the units, [B][20] dZ2
    float *hs = part + RM_WAVES * 32 * RM_PP;                 // [B][36] activations
    float *w2l = hs + B * RM_HP;                              // [32][20] rows of W2, zeros beyond the classes
    float *b1l = w2l + RM_COLS * RM_P16, *b2l = b1l + 32, *lr = b2l + 16;       // biases; loss of every batch row
    float *px = lr + 64, *pv = px + pad;                      // the padding columns and their momentum
    int32_t *ib = reinterpret_cast<int32_t *>(px + 2 * max_pad);      // [ahead][B] batch rows of the iterations drawn together
    const int ahead = rm_ahead(B);
    int32_t *yl = ib + ahead * B;                             // [2][B] labels of this and the next iteration
    uint32_t *ro = reinterpret_cast<uint32_t *>(yl + 2 * B);  // [B] byte offsets of this iteration's rows inside the shard
    int32_t *cnt = yl + 3 * B;                                // [2][RM_AHEAD][waves] thresholds of the peer draws that are <= u
    const uint64_t iter0 = iteration_of(p.iter);
    const uint32_t n_i = (uint32_t)p.n_rows[i];
    const int64_t r0 = p.row0[i];
    const int last_i = p.last[i];
    const float *shard = p.feats + (size_t)r0 * p.din;
    const uint32_t thr_own = p.thr[(size_t)i * p.M + min(t, p.M - 1)];
    const uint32_t skip = (uint32_t)(p.M - 1) << (TILE_SHIFT + 2);
    const size_t first = (size_t)i << TILE_SHIFT;             // a worker's parameter 0 in the tile layout
    const int n_strips = (p.din + 31) / 32, strip0 = (wave + RM_WAVES - 2) % RM_WAVES;     // waves 0 and 1, which have other work, take the last of every round

    auto draw_group = [&](int it0, int group) {
        const int n = p.n_iters - it0 < ahead ? p.n_iters - it0 : ahead;
        for (int e = RM_THREADS - 1 - t; e < n * (B / 4); e += RM_THREADS) {
            const int k = e / (B / 4), b4 = e % (B / 4);
            const Words4 d = draw_block(p.seed, STREAM_BATCH, (uint32_t)b4, (uint32_t)i, iter0 + (uint64_t)(it0 + k));
            const uint32_t word[4] = {d.a, d.b, d.c, d.d};
#pragma unroll
            for (int c = 0; c < 4; ++c) ib[k * B + 4 * b4 + c] = (int32_t)__umulhi(word[c], n_i);
        }
        if (64 * wave >= p.M) return;
        const uint32_t us = draw_block(p.seed, STREAM_PEER, 0u, (uint32_t)i, iter0 + (uint64_t)(it0 + (lane < n ? lane : 0))).a;
        int32_t *to = cnt + group * (RM_AHEAD * RM_WAVES) + wave;
        for (int k = 0; k < n; ++k) {
            const uint32_t u = (uint32_t)__builtin_amdgcn_readlane((int)us, k);
            const int hits = (int)__popcll(__ballot(t < p.M && thr_own <= u));
            if (lane == 0) to[k * RM_WAVES] = hits;
        }
    };
    auto drawn_peer = [&](int group, int at) {
        const int32_t *counts = cnt + group * (RM_AHEAD * RM_WAVES) + at * RM_WAVES;
        int hits = counts[0];
        for (int w = 1; w < RM_WAVES && 64 * w < p.M; ++w) hits += counts[w];
        return __builtin_amdgcn_readfirstlane(hits < last_i ? hits : last_i);
    };
    // rows 8 (v / 4) + 4 half + v % 4 of a strip, column `col`: where the 32 x 32 product leaves a lane's values
    const uint32_t w1_row4 = (uint32_t)p.H * 4u;
    auto w1_row = [](int half, int strip, int v) { return 32 * strip + 8 * (v >> 2) + 4 * half + (v & 3); };
    auto w1_at = [&](int col, int row) { return tile_bytes((uint32_t)row * w1_row4 + (nb * RM_COLS + (uint32_t)col) * 4u, skip); };
    // the same from the strip's first row of a lane (4 half) on: that row's parameter, rows behind it as scalars
    auto w1_from = [&](int col, int half, int strip) { return (uint32_t)(32 * strip + 4 * half) * w1_row4 + (nb * RM_COLS + (uint32_t)col) * 4u; };
    auto w1_next = [&](uint32_t from, int v) { return tile_bytes(from + (uint32_t)(8 * (v >> 2) + (v & 3)) * w1_row4, skip); };

    // ---- before the first iteration
    draw_group(0, 0);
    float vel[RM_STRIPS][16];                                 // momentum of this wave's strips: strip0, strip0 + 8, ...
#pragma unroll
    for (int n = 0; n < RM_STRIPS; ++n) {
        const int strip = min(strip0 + RM_WAVES * n, n_strips - 1);
#pragma unroll
        for (int v = 0; v < 16; ++v) vel[n][v] = *at_bytes(p.V + first, w1_at(col, min(w1_row(half, strip, v), p.din - 1)));
    }
    for (int e = t; e < p.din * (RM_COLS / 4); e += RM_THREADS) {
        const int row = e / (RM_COLS / 4), c4 = e % (RM_COLS / 4) * 4;
        *reinterpret_cast<f32x4 *>(wl + row * RM_COLS + c4) = load4(at_bytes(p.x_first + first, tile_bytes((uint32_t)row * w1_row4 + (nb * RM_COLS + (uint32_t)c4) * 4u, skip)));
    }
    // waves 0 and 1: rows 16 wave + 4 q + v of W2's block, class r, and (lanes 0 .. 15) the units' biases; the last wave's lanes 0 .. 15: the
    // output bias, which every workgroup keeps up to date
    const uint32_t b1_j = (uint32_t)(p.din * p.H) + nb * RM_COLS, w2_j = (uint32_t)(p.din * p.H + p.H) + nb * RM_COLS * (uint32_t)p.C;
    const uint32_t b2_at = tile_bytes(4u * ((uint32_t)(p.din * p.H + p.H + p.H * p.C) + (uint32_t)min(r, p.C - 1)), skip);
    const int kt = wave & 1;
    uint32_t w2_at[4];
    float x2[4], v2[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        w2_at[v] = tile_bytes(4u * (w2_j + (uint32_t)((16 * kt + 4 * q + v) * p.C + min(r, p.C - 1))), skip);
        x2[v] = *at_bytes(p.x_first + first, w2_at[v]);
        v2[v] = *at_bytes(p.V + first, w2_at[v]);
    }
    const bool bias1 = wave < 2 && lane < 16, bias2 = wave == RM_WAVES - 1 && lane < 16;
    const uint32_t bias_at = bias2 ? b2_at : tile_bytes(4u * (b1_j + (uint32_t)(16 * kt + r)), skip);
    float bias_x = *at_bytes(p.x_first + first, bias_at), bias_v = *at_bytes(p.V + first, bias_at);
    for (int e = t; e < RM_COLS * RM_P16; e += RM_THREADS) w2l[e] = 0.0f;
    for (int e = t; e < pad; e += RM_THREADS) {
        const size_t at = tiled_offset(p.M, i, p.D + e);
        px[e] = p.x_first[at];
        pv[e] = p.V[at];
    }
    if (t < 64) lr[t] = 0.0f;
    __syncthreads();
    if (wave < 2 && r < p.C) {
#pragma unroll
        for (int v = 0; v < 4; ++v) w2l[(16 * kt + 4 * q + v) * RM_P16 + r] = x2[v];
    }
    if (bias1) b1l[16 * kt + r] = bias_x;
    if (bias2) {
        b2l[r] = bias_x;
        // The peer's output bias of the first iteration.  All workgroups read the one that the peer's last workgroup replaces in the second, so it
        // is in LDS (behind a row of W2) before this workgroup sends its first partial logits: the peer's last workgroup writes behind the arrivals
        // of all last workgroups, and the one of this worker arrives behind the logits of all of its workgroups.  What else a workgroup reads
        // of a peer comes from the workgroup of the same units, whose arrival it has waited for.
        w2l[r * RM_P16 + RM_MAX_C] = *at_bytes(p.x_first + ((size_t)drawn_peer(0, 0) << TILE_SHIFT), b2_at);
    }
    if (t < B) yl[t] = p.labels[r0 + ib[t]];

    int at = 0, group = 0;                                    // the iteration's place in its group of draws, the group's parity
    for (int it = 0; it < p.n_iters; ++it) {
        // what comes from the lane's number is computed where it is used, not kept across the iteration
        const int t = opaque(t0), lane = t & 63, col = lane & 31, half = lane >> 5, r = lane & 15, q = lane >> 4;
        const int cur = it & 1, nxt = cur ^ 1;
        const bool more = it + 1 < p.n_iters;
        float *Xcur = (cur ? p.x_second : p.x_first) + first, *Xnext = (cur ? p.x_first : p.x_second) + first;
        if (t < B) ro[t] = (uint32_t)ib[at * B + t] * ((uint32_t)p.din * 4u);
        if (it > 0) stores_arrived();                         // this wave's new parameters
        __syncthreads();
        if (it > 0 && t == 0) __hip_atomic_fetch_add(p.rows_count + 32 * nb, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // ---- forward: wave w takes the contraction indices 64 s + 8 w .. + 7 (the two lane halves four consecutive ones each)
        rm_f32x16 acc[RT];
#pragma unroll
        for (int k = 0; k < RT; ++k)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[k][v] = 0.0f;
        {
            const int total = p.din / RM_KS, n_mine = wave < total ? (total - wave + RM_WAVES - 1) / RM_WAVES : 0, s_last = wave + RM_WAVES * (n_mine - 1);
            uint32_t arow[RT];
#pragma unroll
            for (int k = 0; k < RT; ++k) arow[k] = ro[32 * k + col] + 16u * (uint32_t)half;
            f32x4 fa[RM_DEPTH][RT];
            auto request = [&](int d, int s) {                // past the last step: that one again, never used
                const int sc = s < s_last ? s : s_last;
#pragma unroll
                for (int k = 0; k < RT; ++k) fa[d][k] = *reinterpret_cast<const f32x4 *>(at_bytes(shard, arow[k] + (uint32_t)sc * (RM_KS * 4)));
            };
            auto consume = [&](int d, int s) {
                const float *ws = wl + (RM_KS * s + 4 * half) * RM_COLS + col;
                float b[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) b[j] = ws[j * RM_COLS];
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int k = 0; k < RT; ++k) acc[k] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[d][k][j], b[j], acc[k], 0, 0, 0);
            };
            if (n_mine > 0) {
#pragma unroll
                for (int d = 0; d < RM_DEPTH; ++d) request(d, wave + RM_WAVES * d);
                int done = 0;
                for (; done + RM_DEPTH <= n_mine; done += RM_DEPTH) {
#pragma unroll
                    for (int d = 0; d < RM_DEPTH; ++d) {
                        consume(d, wave + RM_WAVES * (done + d));
                        request(d, wave + RM_WAVES * (done + d + RM_DEPTH));
                    }
                }
#pragma unroll
                for (int d = 0; d < RM_DEPTH - 1; ++d)
                    if (done + d < n_mine) consume(d, wave + RM_WAVES * (done + d));
            }
        }
        // the waves' tiles added in their order, bias, ReLU: one row tile after the other
#pragma unroll
        for (int k = 0; k < RT; ++k) {
#pragma unroll
            for (int v = 0; v < 16; ++v) part[(wave * 32 + 8 * (v >> 2) + 4 * half + (v & 3)) * RM_PP + col] = acc[k][v];
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int row = (t >> 5) + 16 * u, c = t & 31;
                float z = part[row * RM_PP + c];
#pragma unroll
                for (int w = 1; w < RM_WAVES; ++w) z += part[(w * 32 + row) * RM_PP + c];
                z += b1l[c];
                z = z > 0.0f ? z : 0.0f;
                hs[(32 * k + row) * RM_HP + c] = z;
                if (!more) p.hidden[((size_t)i * B + 32 * k + row) * p.H + nb * RM_COLS + c] = z;
            }
            __syncthreads();
        }
        // ---- partial logits: a wave per sixteen batch rows, two steps of sixteen units
        const unsigned ticket = p.ticket + (unsigned)it;
        const size_t words_of = (((size_t)cur * p.M + i) * p.NB) * T16 * 256 + lane;     // slice k at k T16 256, row tile at 256, element v at 64 v
        if (wave < T16) {
            __builtin_amdgcn_s_setprio(3);                    // everybody waits for these
            f32x4 z = {0.0f, 0.0f, 0.0f, 0.0f};
            f32x4 a[2];
            float b[2][4];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                a[s] = *reinterpret_cast<const f32x4 *>(hs + (16 * wave + r) * RM_HP + 16 * s + 4 * q);
#pragma unroll
                for (int j = 0; j < 4; ++j) b[s][j] = w2l[(16 * s + 4 * q + j) * RM_P16 + r];
            }
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int j = 0; j < 4; ++j) z = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s][j], b[s][j], z, 0, 0, 0);
            if (r < p.C) {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    __hip_atomic_store(p.words + words_of + ((size_t)nb * T16 + wave) * 256 + 64 * v, ((unsigned long long)ticket << 32) | __float_as_uint(z[v]),
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __builtin_amdgcn_s_setprio(0);
        }
        // the peer, the next group of draws, the next iteration's labels; its rows are brought into this XCD's L2, a share by each workgroup
        const int m = drawn_peer(group, at);
        const float wi = p.w[(size_t)i * p.M + m];
        const ptrdiff_t shift = ((ptrdiff_t)m - i) * TILE;    // from a worker's element to its peer's
        if (t == 0 && nb == 0 && !more) p.peers[i] = m;
        const bool fresh = more && at + 1 == ahead;
        const int next_at = fresh ? 0 : more ? at + 1 : at;
        if (fresh) {
            draw_group(it + 1, group ^ 1);
            __syncthreads();
        }
        int32_t label = 0;
        float touched = 0.0f;
        if (more) {
            if (t < B) label = p.labels[r0 + ib[next_at * B + t]];
            const int lines = (p.din + 31) / 32, share = (B * lines + p.NB - 1) / p.NB, line = (int)nb * share + t;
            if (t < share && line < B * lines) {
                const int b = line / lines;
                touched = shard[(size_t)ib[next_at * B + b] * p.din + min(32 * (line - b * lines), p.din - 1)];
            }
        }
        // ---- all partial logits of this wave's rows, added as head_logits_kernel does; softmax cross-entropy: sixteen lanes have a
        // batch row's classes
        unsigned seen = 0;
        {
            constexpr int VPW = T16 * 4 / RM_WAVES;           // of a lane's four rows
            const int tile = wave % T16, v0 = wave / T16 * VPW;
            const unsigned long long *from = p.words + words_of + (size_t)tile * 256 + 64 * v0;
            float z[VPW];
#pragma unroll
            for (int e = 0; e < VPW; ++e) z[e] = 0.0f;
            long long polls = 0;
            for (int k0 = 0; k0 < p.NB; k0 += 4 * p.run) {    // the parts of four waves of head_logits_kernel
                unsigned long long word[RM_WORDS][VPW];
                bool here;
                do {
                    here = true;
#pragma unroll
                    for (int k = 0; k < RM_WORDS; ++k)
#pragma unroll
                        for (int e = 0; e < VPW; ++e)
                            word[k][e] = __hip_atomic_load(from + (size_t)min(k0 + k, p.NB - 1) * T16 * 256 + 64 * e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                    for (int k = 0; k < RM_WORDS; ++k)
#pragma unroll
                        for (int e = 0; e < VPW; ++e) here &= (unsigned)(word[k][e] >> 32) == ticket;
                } while ((p.patience == 0 || __any(!here && r < p.C)) && !gives_up(++polls, p.fault, p.patience));
                auto part = [&](int k, int e) { return k0 + k < p.NB ? __uint_as_float((unsigned)word[k][e]) : 0.0f; };
                auto add = [&](auto run) {
                    constexpr int R = decltype(run)::value;
#pragma unroll
                    for (int e = 0; e < VPW; ++e) {
                        float of[4];
#pragma unroll
                        for (int w = 0; w < 4; ++w) {
                            of[w] = part(R * w, e);
                            if constexpr (R > 1) of[w] += part(R * w + 1, e);
                            if constexpr (R == 3) of[w] += part(R * w + 2, e);
                            if constexpr (R == 4) of[w] += part(R * w + 2, e) + part(R * w + 3, e);
                        }
                        z[e] += (of[0] + of[1]) + (of[2] + of[3]);
                    }
                };
                if (p.run == 1) add(std::integral_constant<int, 1>{});
                else if (p.run == 2) add(std::integral_constant<int, 2>{});
                else if (p.run == 3) add(std::integral_constant<int, 3>{});
                else add(std::integral_constant<int, 4>{});
            }
            if (wave == 0) seen = arrivals(p.rows_count + 32 * nb);
            const bool real = r < p.C;
#pragma unroll
            for (int e = 0; e < VPW; ++e) {
                const int b = 16 * tile + 4 * q + v0 + e;
                const float ze = real ? z[e] + b2l[r] : -INFINITY;
                float mx = ze;
                mx = fmaxf(mx, xor_lane<1>(mx));
                mx = fmaxf(mx, xor_lane<2>(mx));
                mx = fmaxf(mx, xor_lane<4>(mx));
                mx = fmaxf(mx, xor_lane<8>(mx));
                const float ex = real ? expf(ze - mx) : 0.0f;
                float sum = ex;
                sum += xor_lane<1>(sum);
                sum += xor_lane<2>(sum);
                sum += xor_lane<4>(sum);
                sum += xor_lane<8>(sum);
                const int y = yl[cur * B + b];
                const float d = (ex * (1.0f / sum) - (r == y ? 1.0f : 0.0f)) * (1.0f / (float)B);
                dzs[b * RM_P16 + r] = real ? d : 0.0f;
                if (!more && r == y) lr[b] = logf(sum) - (ze - mx);
            }
        }
        if (it > 0 && t == 0) await_arrivals(p.rows_count + 32 * nb, seen, p.rows_base + (unsigned)it * (unsigned)p.M, p.fault, p.patience);
        __syncthreads();
        // ---- the units' error dZ2 W2^T where h > 0: a wave per sixteen batch rows and sixteen units
        for (int e = wave; e < 2 * T16; e += RM_WAVES) {
            const int u = e & 1, k = e >> 1;
            f32x4 dh = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int s = 0; s < 4; ++s)
                dh = __builtin_amdgcn_mfma_f32_16x16x4f32(dzs[(16 * k + r) * RM_P16 + 4 * s + q], w2l[(16 * u + r) * RM_P16 + 4 * s + q], dh, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int b = 16 * k + 4 * q + v;
                dhs[b * RM_HP + 16 * u + r] = hs[b * RM_HP + 16 * u + r] > 0.0f ? dh[v] : 0.0f;
            }
        }
        float a[HB], xp[16];
        auto request_rows = [&](int strip) {
            const int lane = opaque(t0) & 63, col = lane & 31, half = lane >> 5;
            const uint32_t f4 = (uint32_t)min(32 * strip + col, p.din - 1) * 4u;
            const uint32_t *rows = ro + half;
#pragma unroll
            for (int j = 0; j < HB; ++j) a[j] = *at_bytes(shard, rows[2 * j] + f4);
        };
        auto request_peer = [&](int strip) {
            const int lane = opaque(t0) & 63, col = lane & 31, half = lane >> 5;
            const float *Xp = Xcur + shift;
            if (32 * strip + 32 <= p.din) {
                const uint32_t from = w1_from(col, half, strip);
#pragma unroll
                for (int v = 0; v < 16; ++v) xp[v] = __hip_atomic_load(at_bytes(Xp, w1_next(from, v)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    xp[v] = __hip_atomic_load(at_bytes(Xp, w1_at(col, min(w1_row(half, strip, v), p.din - 1))), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        };
        if (wave >= 2 && strip0 < n_strips) request_rows(strip0);
        __syncthreads();                                      // the units' error; W2 has been read
        // ---- waves 0 and 1, sixteen units each: dW2 = h^T dZ2 and the column sums of the error; their update (Eq. (c0), (c1)).  The last wave:
        // the output bias.
        if (wave < 2) {
            float x2p[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) x2p[v] = __hip_atomic_load(at_bytes(Xcur + shift, w2_at[v]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const float bias_p = __hip_atomic_load(at_bytes(Xcur + shift, bias_at), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (strip0 < n_strips) request_rows(strip0);
            f32x4 dw = {0.0f, 0.0f, 0.0f, 0.0f};
            float colsum = 0.0f;
#pragma unroll
            for (int k = 0; k < T16; ++k)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int b = 16 * k + 4 * q + v;
                    dw = __builtin_amdgcn_mfma_f32_16x16x4f32(hs[b * RM_HP + 16 * kt + r], dzs[b * RM_P16 + r], dw, 0, 0, 0);
                    colsum += dhs[b * RM_HP + 16 * kt + r];
                }
            colsum += __shfl_xor(colsum, 16);
            colsum += __shfl_xor(colsum, 32);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float xn, vn;
                momentum_mix1(x2[v], v2[v], dw[v], x2p[v], wi, p.alpha, p.mu, p.wd, xn, vn);
                x2[v] = xn;
                v2[v] = vn;
                if (r < p.C) {
                    w2l[(16 * kt + 4 * q + v) * RM_P16 + r] = xn;
                    store_row(at_bytes(Xnext, w2_at[v]), xn, more);
                    if (!more) { *at_bytes(p.V + first, w2_at[v]) = vn; *at_bytes(p.G + first, w2_at[v]) = dw[v]; }
                }
            }
            if (bias1) {
                float xn, vn;
                momentum_mix1(bias_x, bias_v, colsum, bias_p, wi, p.alpha, p.mu, p.wd, xn, vn);
                bias_x = xn;
                bias_v = vn;
                b1l[16 * kt + r] = xn;
                store_row(at_bytes(Xnext, bias_at), xn, more);
                if (!more) { *at_bytes(p.V + first, bias_at) = vn; *at_bytes(p.G + first, bias_at) = colsum; }
            }
        }
        if (wave == RM_WAVES - 1) {
            const float bias_p = __hip_atomic_load(p.biases + (((size_t)cur * p.M + m) * p.NB + nb) * 16 + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            f32x4 db = {0.0f, 0.0f, 0.0f, 0.0f};
            const float one = r == 0 ? 1.0f : 0.0f;
#pragma unroll
            for (int k = 0; k < 4 * T16; ++k) db = __builtin_amdgcn_mfma_f32_16x16x4f32(one, dzs[(4 * k + q) * RM_P16 + r], db, 0, 0, 0);
            if (bias2) {
                float xn, vn;
                momentum_mix1(bias_x, bias_v, db[0], it == 0 ? w2l[r * RM_P16 + RM_MAX_C] : bias_p, wi, p.alpha, p.mu, p.wd, xn, vn);
                bias_x = xn;
                bias_v = vn;
                b2l[r] = xn;
                __hip_atomic_store(p.biases + (((size_t)nxt * p.M + i) * p.NB + nb) * 16 + r, xn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (tail && r < p.C) {
                    store_row(at_bytes(Xnext, b2_at), xn, more);
                    if (!more) { *at_bytes(p.V + first, b2_at) = vn; *at_bytes(p.G + first, b2_at) = db[0]; }
                }
            }
        }
        for (int e = RM_THREADS - 1 - t; e < pad; e += RM_THREADS) {
            const size_t to = tiled_offset(p.M, i, p.D + e) - first;
            float xn, vn;
            momentum_mix1(px[e], pv[e], 0.0f, __hip_atomic_load(Xcur + shift + to, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), wi, p.alpha, p.mu, p.wd, xn, vn);
            px[e] = xn;
            pv[e] = vn;
            store_row(Xnext + to, xn, more);
            if (!more) { p.V[first + to] = vn; p.G[first + to] = 0.0f; }
        }
        if (wave == 2 && nb == 0 && !more) {
            float l = lane < B ? lr[lane] : 0.0f;
#pragma unroll
            for (int k = 32; k > 0; k >>= 1) l += __shfl_xor(l, k);
            if (lane == 0) p.loss[i] = l / (float)B;
        }
        // ---- dW1 = A^T dZ1 strip by strip (32 features x 32 units), the batch rows straight from memory; updated where the product leaves
        // it.  The next strip's batch rows are asked for before this one's results are stored, its peer's parameters ahead of its products: a
        // load waited for behind a store waits for the store.
#pragma unroll
        for (int n = 0; n < RM_STRIPS; ++n) {
            const int strip = strip0 + RM_WAVES * n;
            if (strip >= n_strips) break;
            const int lane = opaque(t0) & 63, col = lane & 31, half = lane >> 5;
            request_peer(strip);
            __builtin_amdgcn_sched_barrier(0);
            rm_f32x16 dw;
#pragma unroll
            for (int v = 0; v < 16; ++v) dw[v] = 0.0f;
            const float *zs = dhs + half * RM_HP + col;
#pragma unroll
            for (int j = 0; j < HB; ++j) dw = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j], zs[2 * j * RM_HP], dw, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (n + 1 < RM_STRIPS && strip + RM_WAVES < n_strips) request_rows(strip + RM_WAVES);
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t from = w1_from(col, half, strip);
            float *ws = wl + (32 * strip + 4 * half) * RM_COLS + col;
            auto update = [&](auto whole) {                   // whole: all 32 features exist
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    if (!decltype(whole)::value && w1_row(half, strip, v) >= p.din) continue;
                    float *wv = ws + (8 * (v >> 2) + (v & 3)) * RM_COLS;
                    float xn, vn;
                    momentum_mix1(*wv, vel[n][v], dw[v], xp[v], wi, p.alpha, p.mu, p.wd, xn, vn);
                    vel[n][v] = vn;
                    *wv = xn;
                    __hip_atomic_store(at_bytes(Xnext, w1_next(from, v)), xn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            };
            if (32 * strip + 32 <= p.din) update(std::true_type{});
            else update(std::false_type{});
            if (!more) {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (w1_row(half, strip, v) < p.din) {
                        const uint32_t to = w1_next(from, v);
                        *at_bytes(p.V + first, to) = vel[n][v];
                        *at_bytes(p.G + first, to) = dw[v];
                    }
            }
        }
        asm volatile("" ::"v"(touched));
        if (more && t < B) yl[nxt * B + t] = label;
        at = next_at;
        group ^= fresh;
        __syncthreads();                                      // the rows' offsets, the error and W1 have been read
    }
}

static int64_t rm_padding(const MlpPlan &p) { return p.ld - (p.dims[0] * p.dims[1] + p.dims[1] + p.dims[1] * p.dims[2] + p.dims[2]); }

// One hidden layer that fwd_f32_kernel and wgrad_f32_kernel take, classes and units in the parts that head_logits_kernel then adds, 32-bit byte
// offsets inside the parameters, columns that fit LDS (32 features x 4 bytes and the padding's x and v, which every workgroup has room for: features +
// padding / 16 up to 870 with a batch of 64, 925 with one of 32).  Of the data netmax_bind_data asks the rest.
bool resident_mlp_ok(const MlpPlan &p)
{
    return p.n_layers == 2 && !p.bf16 && (p.B == 32 || p.B == 64) && p.dims[0] % RM_KS == 0 && p.dims[1] % RM_COLS == 0 && head_parts_of_two(p) &&
           p.dims[2] <= RM_MAX_C && p.M <= RM_THREADS && p.ld * p.M < (int64_t)1 << 30 && p.dims[0] <= 32 * RM_STRIPS * RM_WAVES &&
           rm_padding(p) <= RM_MAX_PAD && rm_lds(p.B, p.dims[0], rm_padding(p)) <= (size_t)RM_LDS_LIMIT;
}
// Whether n iterations are faster here than by the separate kernels, from a model of both in us: work, features x batch of a workgroup; the separate
// kernels' time also grows with the workgroups and with the parameters once these leave the L2.  Fitted to the 450 shapes of profiles/whole_iterations.csv
// (16 to 864 features, 32 to 1024 hidden units, 2 to 128 workers, up to 256 workgroups, both batches; 1, 2, 3, 4 and 8 iterations): it takes the faster way
// in 92 % of them, and in all but 1 % a way at most 3 % slower or, where it stays with the separate kernels, in all but 3 % one at most 5 % slower.
// One iteration is never faster here: the cooperative launch costs 20 us.
bool resident_mlp_pays(const MlpPlan &p, int n_iters)
{
    const double work = 1e-3 * (double)p.dims[0] * p.B, groups = (double)p.M * (double)(p.dims[1] / RM_COLS);
    const double traffic = fmax(0.0, 1e-3 * groups * (double)p.dims[0] - 25.0), more = n_iters - 1;
    const double here = 33.5 + 0.6 * work + more * (8.5 + 0.41 * work);
    const double there = 22.2 + 0.17 * work + 0.094 * traffic + 0.022 * groups + more * (18.5 + 0.156 * work + 0.08 * traffic + 0.019 * groups);
    return n_iters > 1 && here < there;
}
int resident_mlp_grid(const MlpPlan &p) { return (int)grouped_grid(p.M, (unsigned)(p.dims[1] / RM_COLS)); }

void resident_mlp_scratch(const MlpPlan &p, size_t &words, size_t &biases, size_t &counters)
{
    const size_t groups = (size_t)p.M * (p.dims[1] / RM_COLS);
    words = 2 * groups * 4 * 256;
    biases = 2 * groups * 16;
    counters = (size_t)(p.dims[1] / RM_COLS) * 32;
}

typedef void (*ResidentKernel)(ResidentArgs);
static ResidentKernel resident_kernel(int B) { return B == 32 ? resident_mlp_kernel<1> : resident_mlp_kernel<2>; }

hipError_t prepare_resident_mlp(const MlpPlan &p, int *resident)
{
    int dev = 0, per_cu = 0, cus = 0, cooperative = 0;
    const void *kernel = reinterpret_cast<const void *>(resident_kernel(p.B));
    *resident = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cooperative, hipDeviceAttributeCooperativeLaunch, dev);
    if (e == hipSuccess) e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, RM_LDS_LIMIT);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, RM_THREADS, rm_lds(p.B, p.dims[0], rm_padding(p)));
    if (e == hipSuccess && cooperative) *resident = per_cu * cus;
    return e;
}

hipError_t launch_resident_mlp(hipStream_t s, const MlpPlan &p, const SlicedIterLaunch &a)
{
    ResidentArgs k{};
    k.M = p.M; k.B = p.B; k.din = (int)p.dims[0]; k.H = (int)p.dims[1]; k.C = (int)p.dims[2]; k.NB = k.H / RM_COLS; k.run = head_pairs_per_wave(p);
    k.D = p.ld - rm_padding(p); k.ld = p.ld;
    k.feats = (const float *)p.feats; k.labels = p.labels; k.row0 = p.row0; k.n_rows = a.n_rows;
    k.thr = a.thr; k.last = a.last; k.w = a.mix.w;
    k.x_first = const_cast<float *>(a.mix.Xcur); k.x_second = a.mix.Xnext; k.V = a.mix.V; k.G = a.G; k.loss = p.loss; k.hidden = p.act[1]; k.peers = a.peers;
    k.alpha = a.mix.alpha; k.mu = a.mix.mu; k.wd = a.mix.wd; k.seed = a.seed; k.iter = a.iter; k.n_iters = a.n_iters;
    k.words = a.parts; k.biases = a.biases; k.ticket = a.ticket; k.rows_count = a.counters; k.rows_base = a.rows_base;
    k.fault = a.fault; k.patience = a.patience;
    void *args[] = {&k};
    return hipLaunchCooperativeKernel(reinterpret_cast<const void *>(resident_kernel(p.B)), dim3((unsigned)resident_mlp_grid(p)), dim3(RM_THREADS), args,
                                      (unsigned)rm_lds(p.B, p.dims[0], rm_padding(p)), s);
}

}  // namespace netmax
