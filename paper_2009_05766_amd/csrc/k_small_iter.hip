// Whole NetMax iterations of a small softmax-regression model in ONE kernel (Algorithm 2, all of its steps): one
// workgroup per worker draws its peer and its batch, computes logits, loss and gradient with the worker's parameters
// and batch rows held in LDS, and applies the momentum step and the mix (Eq. (c0), (c1)) against the peer's copy of the
// previous iteration.  Models of this size are bound by launch latency (six dependent launches of a few microseconds
// each otherwise); here an iteration is one launch, or one step between two barriers inside a cooperative launch that runs many.
//
// Three modes share the code, so their results agree bit for bit:
//   GRAD      batch draw, loss, gradient -> G (netmax_local_step; the mix kernel then applies the same update function)
//   STEP      peer draw + GRAD + update  -> Xnext, V, G (one iteration per launch; also what a captured graph replays)
//   the same with n_iters > 1: cooperative launch, a split barrier per iteration; G, loss and peers are written by the last one only.
//
// Arithmetic: fp32, fixed order.  Forward: eight lanes share a batch row, lane s takes the features k = s, s + 8, ...
// in increasing order, the eight partial sums are added in halves.  Weight gradient: one thread per four features
// and four classes, batch rows in increasing order.  Shapes that tile (at most 16 classes, a batch of 16, 32 or 64
// rows, features a multiple of 128 or, batch 64, of 64) take both products on v_mfma_f32_16x16x4_f32 instead (exact fp32 products, fp32
// accumulation; lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16] and receives D[4 (l / 16) + v][l % 16]): the
// vector units are then left with the softmax and the update.
//
// The kernel lives on latency, so little is waited for that could have been asked for earlier: the peer's row and
// the own momentum are requested before the gradient is computed and used after it; draws depend on (seed, iteration, worker) only,
// so up to sixteen iterations' are made together, and the NEXT iteration's labels and batch rows are requested behind the forward pass;
// the new parameters stay in LDS, only the peer's row is read again.  A workgroup arrives at the barrier with its new row and looks for
// the others' arrival after the softmax of the next iteration, where it needs the peer's: half an iteration during which the last
// ones catch up.  256-10, batch 32, 8 workers, sixteen iterations in a call: 145 us with the barrier between iterations (release
// and acquire of the whole cache, about 2 us), a draw per iteration and stores between the loads of the update, 97 us now, 20 of them outside the
// kernel (a cooperative launch); an iteration takes 4.3 us (time stamps in a copy of the kernel): rows into LDS 0.2, forward 1.0, softmax 0.8, waiting 0.3, gradient 1.2, update 0.7.
#include "kernels.h"
#include "layout.h"
#include "philox.h"
#include "resident.h"

#include <type_traits>

namespace netmax {

constexpr int SI_THREADS = 512, SI_WAVES = SI_THREADS / 64;
constexpr int SI_SPLIT = 8;                 // lanes that share one batch row in the forward pass
constexpr int SI_MAX_OUT = 32;              // classes
constexpr int SI_LDS_LIMIT = 159 * 1024, SI_OPERANDS_LIMIT = 150 * 1024;
// What a thread has in flight: pieces of the batch rows while it fills LDS, vectors of x_peer and v per pass of the update.  The
// matrix-instruction form has a variant of half as many for models that they cover: requests that nobody needs cost their instructions.
constexpr int SI_BURST = 8, SI_UPD = 4;
static bool small_iter_few(int B, int64_t din, int64_t ld) { return B * din <= (int64_t)SI_BURST / 2 * SI_THREADS * 4 && ld <= (int64_t)SI_UPD / 2 * SI_THREADS * 4; }

struct SmallIterArgs {
    int M, B, din, dout;
    int64_t D, ld;
    const float *feats; const int32_t *labels; const int64_t *row0; const int32_t *n_rows;
    const uint32_t *thr; const int32_t *last; const float *w;
    float *x_first, *x_second;              // x_first holds x^t of the first iteration of the launch
    float *V, *G, *loss;
    int32_t *peers;
    float alpha, mu, wd;
    uint64_t seed;
    IterRef iter;                           // number of the first iteration
    int n_iters;
    unsigned *barrier; unsigned barrier_base; int *fault;
    long long patience;                     // polls of the barrier counter before a workgroup gives up
};
// grad_only for listed workers: workgroup s works for slot s.  (A struct of its own: the list in the arguments of the other launches
// would cost them 0.4 us each.)
struct SmallSlotArgs : SmallIterArgs { AsyncSlots slots; };

// The matrix-instruction form of the two products: classes padded to one 16-wide tile, 16-row tiles of the batch, up to two of them per
// wave; the waves split the features of the forward pass evenly in groups of 16 (no bounds test in any loop).
constexpr int si_row_tiles(int RT) { return RT < 2 ? 1 : 2; }                       // a wave's
constexpr int si_parts(int RT) { return SI_WAVES * si_row_tiles(RT) / RT; }         // of the features
static bool small_iter_mm(int B, int64_t din, int64_t dout)
{
    return dout <= 16 && (B == 16 || B == 32 || B == 64) && din % (16 * si_parts(B / 16)) == 0;
}
static int small_iter_cap(int B, int64_t din, int64_t dout)
{
    if (small_iter_mm(B, din, dout)) return 16;
    return dout <= 8 ? 8 : (dout <= 16 ? 16 : SI_MAX_OUT);
}
constexpr int SI_MM_PAD = 20;               // floats behind a batch row in that form: sixteen rows read together meet all banks, and four neighbouring
                                            // rows of sixteen features nearly so
constexpr int si_mm_part(int RT) { return si_parts(RT) * RT * 16 * 16; }            // floats of partial logits

// Iterations drawn together: a Philox block takes 0.45 us from its first multiplication to its last, whatever the number of lanes that
// work on one.  At most 4 KB of row numbers.
constexpr int SI_AHEAD = 16;
static __device__ __host__ __forceinline__ int si_ahead(int B) { return B >= 1024 ? 1 : (1024 / B < SI_AHEAD ? 1024 / B : SI_AHEAD); }

static size_t small_iter_lds(int B, int din, int dout, int64_t ld)
{
    const bool mm = small_iter_mm(B, din, dout);
    const size_t pitch = (size_t)din + (mm ? SI_MM_PAD : SI_SPLIT), cap = (size_t)small_iter_cap(B, din, dout);
    const size_t w = mm ? (size_t)si_mm_part(B / 16) : ((size_t)din + 1) * (cap + 4);
    return (2 * (size_t)ld + w + (size_t)B * pitch + (size_t)B * cap + (size_t)B) * sizeof(float) +
           ((size_t)si_ahead(B) * B + 2 * (size_t)B + 2 * SI_AHEAD * SI_WAVES) * sizeof(int32_t);
}

// The line up to which a worker's iterations are taken into one workgroup: parameters, gradient, padded weights and the batch.
static size_t small_iter_operands(int B, int din, int dout, int64_t ld)
{
    const size_t cap = (size_t)small_iter_cap(B, din, dout);
    return (2 * (size_t)ld + ((size_t)din + 1) * (cap + 4) + (size_t)B * (din + SI_SPLIT + cap + 5) + 2) * sizeof(float);
}

// CAP: classes the unrolled loops cover: dout <= CAP, CAP in {8, 16, 32}.  RT > 0: the two products on matrix
// instructions, RT = batch / 16 tiles of batch rows (CAP = 16, shapes accepted by small_iter_mm()).
// MODE: batch draw, loss and gradient of one iteration; the whole of one; several.  The last of several asks for its own batch rows
// again: a load under a branch is waited for where the branches join (4 us more for sixteen iterations of 256-10).
enum : int { SI_GRAD = 0, SI_ONE = 1, SI_RUN = 2 };
template <int CAP, int RT, int MODE, bool FEW, class Args = SmallIterArgs>
__global__ void __launch_bounds__(SI_THREADS) small_softmax_iteration_kernel(Args p)
{
    constexpr bool SLOTS = !std::is_same<Args, SmallIterArgs>::value;
    constexpr bool STEP = MODE != SI_GRAD, RUN = MODE == SI_RUN;
    static_assert(!SLOTS || !STEP, "listed workers: the gradient only");
    constexpr bool MM = RT > 0;
    constexpr int BURST = FEW ? SI_BURST / 2 : SI_BURST, UPD = FEW ? SI_UPD / 2 : SI_UPD;
    static_assert(!MM || CAP == 16, "the matrix-instruction form pads the classes to one 16-wide tile");
    extern __shared__ __attribute__((aligned(16))) unsigned char si_smem[];
    constexpr int SI_DEPTH = CAP <= 16 ? 4 : 2;               // steps of an inner product whose LDS reads are in flight together
    constexpr int OWN = CAP / SI_SPLIT;                       // classes a lane owns after the reduction of a row
    constexpr int WP = CAP + 4;                               // floats per padded row of W: the eight rows a wave reads
                                                              // together then lie in different LDS banks
    const int t0 = threadIdx.x;
    // the variant for few vectors has the registers for what it would compute anew in every iteration
    auto hidden = [](int v) { return FEW ? v : opaque(v); };
    int i = (int)blockIdx.x;
    if constexpr (SLOTS) i = p.slots.worker[blockIdx.x];
    const int pitch = p.din + (MM ? SI_MM_PAD : SI_SPLIT);
    float *xl = reinterpret_cast<float *>(si_smem);           // [ld]  the worker's parameters (W row-major [din][dout], b)
    float *gl = xl + p.ld;                                    // [ld]  its gradient
    float *wp = gl + p.ld;                                    // [din + 1][WP] W and then b with rows padded by zeros to
                                                              //       CAP classes: the inner loops run without a bounds test
    float *dz = MM ? wp : wp + ((size_t)p.din + 1) * WP;      // [B][CAP], zeros beyond dout (16-byte aligned rows); MM reads W where it lies
    float *xs = dz + (size_t)p.B * CAP;                       // [B][pitch] batch rows
    float *lb = xs + (size_t)p.B * pitch;                     // [B] per-row loss
    float *part = lb + p.B;                                   // MM: [parts of the features][B][16] partial logits
    const int ahead = si_ahead(p.B);
    int32_t *ib = reinterpret_cast<int32_t *>(part + (MM ? si_mm_part(RT) : 0));   // [ahead][B] batch rows (shard-local) of the iterations drawn together
    int32_t *yl = ib + ahead * p.B;                           // [2][B] labels of this and the next iteration
    int32_t *cnt = yl + 2 * p.B;                              // [2][SI_AHEAD][waves] thresholds of the peer draws that are <= u, two groups of draws
    uint64_t iter0;
    if constexpr (SLOTS) iter0 = p.slots.first + p.slots.step[blockIdx.x];
    else iter0 = iteration_of(p.iter);
    const int n_vec = (int)(p.ld >> 2);
    const float invB = 1.0f / (float)p.B;
    const uint32_t n_i = (uint32_t)p.n_rows[i];
    const int64_t r0 = p.row0[i];
    const int last_i = STEP ? p.last[i] : 0;
    const float *shard = p.feats + (size_t)r0 * p.din;
    const uint32_t *thr_row = p.thr + (size_t)i * p.M;
    const DivBy by_out(p.dout);
    const bool vec_rows = MM || (p.din & 3) == 0;             // batch rows as 128-bit pieces, else element by element
    const int row_units = vec_rows ? p.din >> 2 : p.din, feat_units = p.B * row_units;
    const DivBy by_row(row_units);

    // The draws of the iterations it0 .. of a group: batch row b is word b % 4 of block b / 4 of stream 1; the peer is the number of
    // thresholds of the worker's row that are <= u (they do not decrease), clamped to the last positive entry: every wave counts its
    // share for all iterations of the group.
    auto draw_group = [&](int t, int it0, int group, uint32_t first) {    // first: thr_row[t], read earlier
        const int n = p.n_iters - it0 < ahead ? p.n_iters - it0 : ahead, blocks = (p.B + 3) >> 2;
        for (int e = SI_THREADS - 1 - t; e < n * blocks; e += SI_THREADS) {      // from the last wave down: the first ones count
            const int k = e / blocks, q = e - k * blocks;
            const Words4 r = draw_block(p.seed, STREAM_BATCH, (uint32_t)q, (uint32_t)i, iter0 + (uint64_t)(it0 + k));
            const uint32_t word[4] = {r.a, r.b, r.c, r.d};
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (4 * q + c < p.B) ib[k * p.B + 4 * q + c] = (int32_t)__umulhi(word[c], n_i);
        }
        if (!STEP || (t & ~63) >= p.M) return;
        const int lane = t & 63;
        const uint32_t us = draw_block(p.seed, STREAM_PEER, 0u, (uint32_t)i, iter0 + (uint64_t)(it0 + (lane < n ? lane : 0))).a;
        int32_t *to = cnt + group * (SI_AHEAD * SI_WAVES) + (t >> 6);
        for (int k = 0; k < n; ++k) {
            const uint32_t u = (uint32_t)__builtin_amdgcn_readlane((int)us, k);
            int hits = (int)__popcll(__ballot(t < p.M && first <= u));
            for (int q0 = SI_THREADS; q0 < p.M; q0 += SI_THREADS) {
                const int q = q0 + t;
                hits += (int)__popcll(__ballot(q < p.M && thr_row[q < p.M ? q : 0] <= u));
            }
            if (lane == 0) to[k * SI_WAVES] = hits;
        }
    };
    // Requests the first BURST pieces per thread of the listed batch rows.
    auto request_rows = [&](int t, const int32_t *rows, f32x4 (&r)[BURST]) {
        const float *src[BURST];
#pragma unroll
        for (int e = 0; e < BURST; ++e) {
            const int q = e * SI_THREADS + t, qc = q < feat_units ? q : 0;     // unconditional, see the update's requests
            const int b = by_row(qc), c = qc - b * row_units;
            src[e] = shard + (size_t)rows[b] * p.din + (vec_rows ? 4 * c : c);
        }
        if (vec_rows) {                                       // one branch around all requests: one in each would make them wait for each other
#pragma unroll
            for (int e = 0; e < BURST; ++e) r[e] = load4(src[e]);
        } else {
#pragma unroll
            for (int e = 0; e < BURST; ++e) r[e] = f32x4{src[e][0], 0.0f, 0.0f, 0.0f};
        }
    };
    auto store_piece = [&](int q, const f32x4 &v) {
        const int b = by_row(q), c = q - b * row_units;
        float *dst = xs + (size_t)b * pitch;
        if (vec_rows) *reinterpret_cast<f32x4 *>(dst + 4 * c) = v;
        else dst[c] = v[0];
    };
    auto load4_peer = [](const float *at) { return RUN ? load4_device(at) : load4(at); };
    // Four neighbouring parameters into LDS: the flat copy and the padded rows.
    auto keep_params = [&](int q, const f32x4 &v) {
        *reinterpret_cast<f32x4 *>(xl + (size_t)q * 4) = v;
        if constexpr (MM) return;                             // reads W where it lies
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int j = q * 4 + c;
            if (j < (int)p.D) {
                const int k = by_out(j);        // row din holds the bias
                wp[(size_t)k * WP + (j - k * p.dout)] = v[c];
            }
        }
    };

    // ---- before the first iteration: parameters, draws and batch rows, all requested before any is waited for
    const int t = t0;
    f32x4 rf[BURST], rpar[BURST];
#pragma unroll
    for (int e = 0; e < BURST; ++e) {
        const int q = e * SI_THREADS + t;
        rpar[e] = load4(p.x_first + tiled_offset(p.M, i, (int64_t)(q < n_vec ? q : 0) * 4));
    }
    const uint32_t thr_own = STEP ? thr_row[t0 < p.M ? t0 : 0] : 0u;      // the row does not change during a launch
    draw_group(t, 0, 0, thr_own);
    __syncthreads();
    const int t_row = t0 < p.B ? t0 : p.B - 1;
    int32_t label = p.labels[r0 + ib[t_row]];
    request_rows(t, ib, rf);
#pragma unroll
    for (int e = 0; e < BURST; ++e) {
        const int q = e * SI_THREADS + t;
        if (q < n_vec) keep_params(q, rpar[e]);
    }
    for (int q = BURST * SI_THREADS + t; q < n_vec; q += SI_THREADS)
        keep_params(q, load4(p.x_first + tiled_offset(p.M, i, (int64_t)q * 4)));
    for (int q = t; !MM && q < (p.din + 1) * (CAP - p.dout); q += SI_THREADS) {       // the padding of every row
        const int k = q / (CAP - p.dout);
        wp[(size_t)k * WP + p.dout + (q - k * (CAP - p.dout))] = 0.0f;
    }
    if (t < p.B) yl[t] = label;
    for (int b = SI_THREADS + t; b < p.B; b += SI_THREADS) yl[b] = p.labels[r0 + ib[b]];       // batches beyond the threads
    for (int64_t j = p.D + t; j < p.ld; j += SI_THREADS) gl[j] = 0.0f;     // the padding behind the gradient: written here only

    uint32_t own_at[UPD];                                     // this thread's vectors of the first pass (beyond the end: the first vector, never used)
#pragma unroll
    for (int e = 0; e < UPD; ++e) {
        const int q = e * SI_THREADS + t0;
        own_at[e] = (uint32_t)tiled_offset(p.M, i, (int64_t)(q < n_vec ? q : 0) * 4);
    }
    const int n_iters = RUN ? p.n_iters : 1;
    int at = 0, group = 0;                                    // the iteration's place in its group of draws, the group's parity
    for (int it = 0; it < n_iters; ++it) {
        const int cur = it & 1, nxt = cur ^ 1;
        const bool more = RUN && it + 1 < n_iters;
        const int t = hidden(t0);
        float *Xcur = cur ? p.x_second : p.x_first;
        float *Xnext = cur ? p.x_first : p.x_second;
        // ---- this iteration's batch rows into LDS (the first pieces were requested an iteration ago)
#pragma unroll
        for (int e = 0; e < BURST; ++e) {
            const int q = e * SI_THREADS + t;
            if (q < feat_units) store_piece(q, rf[e]);
        }
        for (int q = BURST * SI_THREADS + t; q < feat_units; q += SI_THREADS) {
            const int b = by_row(q), c = q - b * row_units;
            const float *src = shard + (size_t)ib[at * p.B + b] * p.din;
            f32x4 v;
            if (vec_rows) v = load4(src + 4 * c); else v[0] = src[c];
            store_piece(q, v);
        }
        if (RUN && it > 0) stores_arrived();                  // this wave's new parameters, on their way since the update
        __syncthreads();
        if (RUN && it > 0 && t == 0) __hip_atomic_fetch_add(p.barrier, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // ---- the peer
        int m = i;
        if constexpr (STEP) {
            const int32_t *counts = cnt + group * (SI_AHEAD * SI_WAVES) + at * SI_WAVES;
            int c = counts[0];
            for (int w = 1; w < SI_WAVES && 64 * w < p.M; ++w) c += counts[w];
            m = __builtin_amdgcn_readfirstlane(c < last_i ? c : last_i);
            if (t == 0 && !more) p.peers[i] = m;
        }
        // the group of draws that the next iteration begins: the rows of this one are in LDS
        const bool fresh = more && at + 1 == ahead;
        const int next_at = fresh ? 0 : more ? at + 1 : at;
        const int32_t *next_rows = ib + next_at * p.B;
        if (fresh) draw_group(t, it + 1, group ^ 1, thr_own);
        unsigned seen = 0;
        // the count of arrivals and the next iteration's labels and batch rows, on their way while this iteration goes on (in this order:
        // a wave's loads are waited for in the order of their requests)
        auto request_ahead = [&]() {
            seen = arrivals(p.barrier);
            label = p.labels[r0 + next_rows[t_row]];
            request_rows(t, next_rows, rf);
        };
        if constexpr (MM) {
            // ---- forward on matrix instructions: wave = (up to two 16-row tiles of the batch, part of the features); two steps of sixteen
            // features are read from LDS together, then multiplied
            const int t = hidden(t0);
            const int lane = t & 63, wave = t >> 6, r = lane & 15, q = lane >> 4;
            constexpr int TILES = si_row_tiles(MM ? RT : 1), KP = si_parts(MM ? RT : 1), DEPTH = 2;
            const int KW = p.din / KP, kp = wave % KP, row0 = wave / KP * (16 * TILES);
            const float *xrow = xs + (size_t)(row0 + r) * pitch + kp * KW + 4 * q;
            // classes past the last one multiply what follows in the row (in LDS, finite or not): their columns are never looked at
            const float *wcol = xl + (size_t)(kp * KW + 4 * q) * p.dout + r;
            f32x4 acc[TILES];
#pragma unroll
            for (int rt = 0; rt < TILES; ++rt) acc[rt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            auto steps = [&](int k0, auto n) {                // n steps of sixteen features: all reads, then all products
                constexpr int N = decltype(n)::value;
                f32x4 a[N][TILES];
                float b[N][4];
#pragma unroll
                for (int u = 0; u < N; ++u) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) b[u][j] = wcol[(k0 + 16 * u + j) * p.dout];
#pragma unroll
                    for (int rt = 0; rt < TILES; ++rt) a[u][rt] = *reinterpret_cast<const f32x4 *>(xrow + 16 * rt * pitch + k0 + 16 * u);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < N; ++u)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int rt = 0; rt < TILES; ++rt) acc[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][rt][j], b[u][j], acc[rt], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            };
            int k0 = 0;
            for (; k0 + 16 * DEPTH <= KW; k0 += 16 * DEPTH) steps(k0, std::integral_constant<int, DEPTH>{});
            for (; k0 < KW; k0 += 16) steps(k0, std::integral_constant<int, 1>{});
#pragma unroll
            for (int rt = 0; rt < TILES; ++rt)
#pragma unroll
                for (int v = 0; v < 4; ++v) part[(size_t)(kp * p.B + row0 + 16 * rt + 4 * q + v) * 16 + r] = acc[rt][v];
            __syncthreads();
            if constexpr (RUN) request_ahead();
            // ---- the parts added in order, bias, softmax, loss, dZ: sixteen lanes per batch row, one class each
            const float *bias = xl + (size_t)p.din * p.dout;
            for (int e = t; e < p.B * 16; e += SI_THREADS) {
                const int b = e >> 4, c = e & 15;
                float z = part[(size_t)b * 16 + c];
#pragma unroll
                for (int kk = 1; kk < KP; ++kk) z += part[(size_t)(kk * p.B + b) * 16 + c];
                const bool real = c < p.dout;
                z = real ? z + bias[c] : -INFINITY;
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
                const int y = yl[cur * p.B + b];
                dz[(size_t)b * CAP + c] = real ? (ex * (1.0f / sum) - (c == y ? 1.0f : 0.0f)) * invB : 0.0f;
                if (c == y && !more) lb[b] = logf(sum) - (z - mx);
            }
        } else {
        // ---- forward, softmax, loss, dZ: eight lanes per batch row; lane s adds the features s, s + 8, ... in order,
        // the lanes then add their partial sums in halves, so that each ends up owning OWN classes of the row
        {
            const int t = hidden(t0);
            const int sub = t & (SI_SPLIT - 1);
            const int own0 = ((sub >> 2) & 1) * (CAP / 2) + ((sub >> 1) & 1) * (CAP / 4) + (sub & 1) * (CAP / 8);
            const float *bias = wp + (size_t)p.din * WP;
            for (int b0 = 0; b0 < p.B; b0 += SI_THREADS / SI_SPLIT) {
                const int b = b0 + t / SI_SPLIT;
                const bool row_ok = b < p.B;
                float acc[CAP];
#pragma unroll
                for (int o = 0; o < CAP; ++o) acc[o] = 0.0f;
                if (row_ok) {
                    // SI_DEPTH steps at a time: all their LDS reads are requested, then all their products are added
                    for (int k0 = sub; k0 < p.din; k0 += SI_SPLIT * SI_DEPTH) {
                        float x[SI_DEPTH];
                        f32x4 wv[SI_DEPTH][CAP / 4];
#pragma unroll
                        for (int u = 0; u < SI_DEPTH; ++u) {
                            const int k = k0 + u * SI_SPLIT;
                            const bool in = k < p.din;
                            x[u] = in ? xs[(size_t)b * pitch + k] : 0.0f;
                            const f32x4 *wk = reinterpret_cast<const f32x4 *>(wp + (size_t)(in ? k : 0) * WP);
#pragma unroll
                            for (int o4 = 0; o4 < CAP / 4; ++o4) wv[u][o4] = wk[o4];
                        }
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int u = 0; u < SI_DEPTH; ++u)
#pragma unroll
                            for (int o4 = 0; o4 < CAP / 4; ++o4)
#pragma unroll
                                for (int c = 0; c < 4; ++c) acc[4 * o4 + c] = fmaf(x[u], wv[u][o4][c], acc[4 * o4 + c]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                // halving exchange over the lane bits 4, 2, 1: a lane keeps the half its bit selects and adds the partner's
                {
                    const bool up4 = (sub & 4) != 0, up2 = (sub & 2) != 0, up1 = (sub & 1) != 0;
#pragma unroll
                    for (int j = 0; j < CAP / 2; ++j)
                        acc[j] = (up4 ? acc[j + CAP / 2] : acc[j]) + xor_lane<4>(up4 ? acc[j] : acc[j + CAP / 2]);
#pragma unroll
                    for (int j = 0; j < CAP / 4; ++j)
                        acc[j] = (up2 ? acc[j + CAP / 4] : acc[j]) + xor_lane<2>(up2 ? acc[j] : acc[j + CAP / 4]);
#pragma unroll
                    for (int j = 0; j < CAP / 8; ++j)
                        acc[j] = (up1 ? acc[j + CAP / 8] : acc[j]) + xor_lane<1>(up1 ? acc[j] : acc[j + CAP / 8]);
                }
                float z[OWN], mx = -INFINITY;
#pragma unroll
                for (int j = 0; j < OWN; ++j) {
                    z[j] = acc[j] + bias[own0 + j];
                    if (own0 + j < p.dout) mx = fmaxf(mx, z[j]);
                }
                mx = fmaxf(mx, xor_lane<1>(mx));
                mx = fmaxf(mx, xor_lane<2>(mx));
                mx = fmaxf(mx, xor_lane<4>(mx));
                const int y = row_ok ? yl[cur * p.B + b] : 0;
                float ex[OWN], sum = 0.0f, zy = 0.0f;
#pragma unroll
                for (int j = 0; j < OWN; ++j) {
                    ex[j] = own0 + j < p.dout ? expf(z[j] - mx) : 0.0f;
                    sum += ex[j];
                    zy += own0 + j == y ? z[j] : 0.0f;
                }
                sum += xor_lane<1>(sum);
                sum += xor_lane<2>(sum);
                sum += xor_lane<4>(sum);
                zy += xor_lane<1>(zy);
                zy += xor_lane<2>(zy);
                zy += xor_lane<4>(zy);
                if (row_ok) {
                    const float inv = 1.0f / sum;
#pragma unroll
                    for (int j = 0; j < OWN; ++j)
                        dz[(size_t)b * CAP + own0 + j] =
                            own0 + j < p.dout ? (ex[j] * inv - (own0 + j == y ? 1.0f : 0.0f)) * invB : 0.0f;
                    if (sub == 0) lb[b] = logf(sum) - (zy - mx);
                }
            }
        }
        }
        if constexpr (RUN && !MM) {
            if (fresh) __syncthreads();       // the group of draws is complete
            request_ahead();
        }
        if (RUN && it > 0 && t == 0) await_arrivals(p.barrier, seen, p.barrier_base + (unsigned)it * (unsigned)p.M, p.fault, p.patience);
        __syncthreads();
        // the peer's row and the own momentum are requested before the gradient is computed and used after it
        f32x4 rxp[UPD], rv[UPD];
        const float wi = STEP ? p.w[(size_t)i * p.M + m] : 0.0f;
        const float *Xpeer = Xcur + ((ptrdiff_t)m - i) * TILE;           // from a worker's element to its peer's
        if constexpr (STEP) {
#pragma unroll
            for (int e = 0; e < UPD; ++e) {
                // unconditional: a load under a branch is waited for where the branches join, one round trip per pair
                // instead of one for all
                rxp[e] = load4_peer(Xpeer + own_at[e]);
                rv[e] = load4(p.V + own_at[e]);
            }
        }
        // ---- gradient into LDS: dW[k][o] = sum_b x[b][k] dz[b][o], db[o] = sum_b dz[b][o] (batch rows in order), padding 0
        if constexpr (MM) {
            // a wave takes sixteen features at a time; the batch is the contraction (step s, lane group q: row 4 s + q)
            const int t = hidden(t0);
            const int lane = t & 63, wave = t >> 6, r = lane & 15, q = lane >> 4;
            constexpr int STEPS = MM ? 4 * RT : 1;           // batch / 4
            float bz[STEPS];
#pragma unroll
            for (int s4 = 0; s4 < STEPS; ++s4) bz[s4] = dz[(size_t)(4 * s4 + q) * CAP + r];
            for (int kt = wave; kt < (p.din >> 4); kt += SI_THREADS / 64) {
                float av[STEPS];
#pragma unroll
                for (int s4 = 0; s4 < STEPS; ++s4) av[s4] = xs[(size_t)(4 * s4 + q) * pitch + 16 * kt + r];
                __builtin_amdgcn_sched_barrier(0);
                f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int s4 = 0; s4 < STEPS; ++s4) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[s4], bz[s4], acc, 0, 0, 0);
                if (r < p.dout) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) gl[(size_t)(16 * kt + 4 * q + v) * p.dout + r] = acc[v];
                }
            }
            if (wave == SI_THREADS / 64 - 1) {
                // db = column sums of dZ: the same product with a row of ones in place of the features
                f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
                const float one = r == 0 ? 1.0f : 0.0f;
#pragma unroll
                for (int s4 = 0; s4 < STEPS; ++s4) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(one, bz[s4], acc, 0, 0, 0);
                if (q == 0 && r < p.dout) gl[(size_t)p.din * p.dout + r] = acc[0];
            }
            if (wave == 0 && !more) {
                // the loss: the rows' terms added by one wave in a fixed tree
                float l = lane < p.B ? lb[lane] : 0.0f;
#pragma unroll
                for (int m2 = 32; m2 > 0; m2 >>= 1) l += __shfl_xor(l, m2);
                if (lane == 0) p.loss[i] = l * invB;
            }
        } else {
            constexpr int OG = CAP / 4;                       // groups of four classes
            const int t = hidden(t0);
            const int og = t % OG, n_kg = (p.din + 3) >> 2;
            for (int kg = t / OG; kg < n_kg; kg += SI_THREADS / OG) {
                float acc[4][4];
#pragma unroll
                for (int a = 0; a < 4; ++a)
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[a][c] = 0.0f;
                for (int b0 = 0; b0 < p.B; b0 += SI_DEPTH) {
                    float xv[SI_DEPTH][4];
                    f32x4 dv[SI_DEPTH];
#pragma unroll
                    for (int u = 0; u < SI_DEPTH; ++u) {
                        const int b = b0 + u < p.B ? b0 + u : p.B - 1;
                        const float *xr = xs + (size_t)b * pitch + 4 * kg;    // the row's pad keeps 4 kg + 3 inside it
#pragma unroll
                        for (int a = 0; a < 4; ++a) xv[u][a] = xr[a];
                        dv[u] = *reinterpret_cast<const f32x4 *>(dz + (size_t)b * CAP + 4 * og);
                        if (b0 + u >= p.B) dv[u] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < SI_DEPTH; ++u)
#pragma unroll
                        for (int a = 0; a < 4; ++a)
#pragma unroll
                            for (int c = 0; c < 4; ++c) acc[a][c] = fmaf(xv[u][a], dv[u][c], acc[a][c]);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int a = 0; a < 4; ++a)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (4 * kg + a < p.din && 4 * og + c < p.dout) gl[(size_t)(4 * kg + a) * p.dout + 4 * og + c] = acc[a][c];
            }
        }
        if (!MM && t < CAP) {                                 // the bias gradient
            float s = 0.0f;
#pragma unroll 8
            for (int b = 0; b < p.B; ++b) s += dz[(size_t)b * CAP + t];
            if (t < p.dout) gl[(size_t)p.din * p.dout + t] = s;
        }
        if (!MM && !more && t == SI_THREADS - 1) {                     // batch rows in order
            float s = 0.0f;
#pragma unroll 8
            for (int b = 0; b < p.B; ++b) s += lb[b];
            p.loss[i] = s * invB;
        }
        __syncthreads();
        // ---- gradient to memory; momentum step and mix (Eq. (c0), (c1)) against the peer's previous copy; the new
        // parameters stay in LDS for the next iteration
        for (int q0 = 0; q0 < n_vec; q0 += SI_THREADS * UPD) {
            if (STEP && q0 > 0) {                     // beyond what was requested ahead
#pragma unroll
                for (int e = 0; e < UPD; ++e) {
                    const int q = q0 + e * SI_THREADS + t, qc = q < n_vec ? q : 0;
                    rxp[e] = load4_peer(Xpeer + tiled_offset(p.M, i, (int64_t)qc * 4));
                    rv[e] = load4(p.V + tiled_offset(p.M, i, (int64_t)qc * 4));
                }
            }
            // all new values, then all stores: a wave's stores are counted with its loads, and a load waited for behind a
            // store waits for the store
            f32x4 g[UPD], xn[UPD], vn[UPD];
#pragma unroll
            for (int e = 0; e < UPD; ++e) {
                const int q = q0 + e * SI_THREADS + t, j = (q < n_vec ? q : 0) * 4;
                g[e] = *reinterpret_cast<const f32x4 *>(gl + j);
                if constexpr (STEP) momentum_mix4(*reinterpret_cast<const f32x4 *>(xl + j), rv[e], g[e], rxp[e], wi, p.alpha, p.mu, p.wd, xn[e], vn[e]);
            }
#pragma unroll
            for (int e = 0; e < UPD; ++e) {
                const int q = q0 + e * SI_THREADS + t;
                if (q < n_vec) {
                    const size_t own = MM && q0 == 0 ? own_at[e] : tiled_offset(p.M, i, (int64_t)q * 4);
                    if constexpr (STEP) {
                        if (more) store4_device(Xnext + own, xn[e]);
                        else store4(Xnext + own, xn[e]);
                        store4(p.V + own, vn[e]);
                        if (more) keep_params(q, xn[e]);
                    }
                    if (!more) store4(p.G + own, g[e]);       // the next iteration's gradient replaces it otherwise
                }
            }
        }
        if (more) {
            if (t < p.B) yl[nxt * p.B + t] = label;
            for (int b = SI_THREADS + t; b < p.B; b += SI_THREADS) yl[nxt * p.B + b] = p.labels[r0 + next_rows[b]];
        }
        at = next_at;
        group ^= fresh;
    }
}

bool small_iter_ok(int model_is_mlp, int n_layers, int bf16, int B, int64_t din, int64_t dout, int64_t ld)
{
    return model_is_mlp && n_layers == 1 && !bf16 && dout <= SI_MAX_OUT && din <= 4096 && ld <= 32768 &&
           small_iter_operands(B, (int)din, (int)dout, ld) <= (size_t)SI_OPERANDS_LIMIT && small_iter_lds(B, (int)din, (int)dout, ld) <= (size_t)SI_LDS_LIMIT;
}

template <int MODE, bool FEW, class Args> static const void *small_iter_mm_kernel(int B)
{
    if (B == 16) return reinterpret_cast<const void *>(small_softmax_iteration_kernel<16, 1, MODE, FEW, Args>);
    if (B == 32) return reinterpret_cast<const void *>(small_softmax_iteration_kernel<16, 2, MODE, FEW, Args>);
    return reinterpret_cast<const void *>(small_softmax_iteration_kernel<16, 4, MODE, FEW, Args>);
}
template <int MODE, class Args = SmallIterArgs> static const void *small_iter_kernel(int B, int64_t din, int64_t dout, int64_t ld)
{
    if (small_iter_mm(B, din, dout)) return small_iter_few(B, din, ld) ? small_iter_mm_kernel<MODE, true, Args>(B) : small_iter_mm_kernel<MODE, false, Args>(B);
    if (dout <= 8) return reinterpret_cast<const void *>(small_softmax_iteration_kernel<8, 0, MODE, false, Args>);
    if (dout <= 16) return reinterpret_cast<const void *>(small_softmax_iteration_kernel<16, 0, MODE, false, Args>);
    return reinterpret_cast<const void *>(small_softmax_iteration_kernel<SI_MAX_OUT, 0, MODE, false, Args>);
}

// For the shape of a context: the four forms of its kernel.
hipError_t prepare_small_iter(int B, int64_t din, int64_t dout, int64_t ld)
{
    for (const void *kernel : {small_iter_kernel<SI_RUN>(B, din, dout, ld), small_iter_kernel<SI_ONE>(B, din, dout, ld), small_iter_kernel<SI_GRAD>(B, din, dout, ld),
                               small_iter_kernel<SI_GRAD, SmallSlotArgs>(B, din, dout, ld)}) {
        const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, SI_LDS_LIMIT);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Several iterations in one launch.  A cooperative launch costs about 20 us more than a plain one, an iteration in it 4.5 us instead of 7.2 in a launch of
// its own (256-10, batch 32, 8 workers).  One launch each and all in one, us: 256-10, 4 iterations 30.5 and 43.1, 8 59.6 and 61.4 (alone 83 and 62),
// 16 115 and 97; 64-10, batch 64, 8 iterations 54.6 and 54.5; 21-9, batch 65, 16 workers, 6 iterations 86.2 and 88.0, 8 114 and 109.
bool small_iter_pays(int n_iters) { return n_iters >= 8; }

// n_iters > 1: every workgroup must be resident (the caller has checked M against small_iter_max_resident()).
hipError_t launch_small_iter(hipStream_t s, const SmallIterLaunch &a)
{
    SmallSlotArgs p{};
    p.M = a.M; p.B = a.B; p.din = (int)a.din; p.dout = (int)a.dout; p.D = a.D; p.ld = a.ld;
    p.feats = a.feats; p.labels = a.labels; p.row0 = a.row0; p.n_rows = a.n_rows;
    p.thr = a.thr; p.last = a.last; p.w = a.w;
    p.x_first = a.x_first; p.x_second = a.x_second; p.V = a.V; p.G = a.G; p.loss = a.loss; p.peers = a.peers;
    p.alpha = a.alpha; p.mu = a.mu; p.wd = a.wd; p.seed = a.seed; p.iter = a.iter; p.n_iters = a.n_iters;
    p.barrier = a.barrier; p.barrier_base = a.barrier_base; p.fault = a.fault;
    p.patience = a.patience;
    const size_t lds = small_iter_lds(a.B, p.din, p.dout, a.ld);
    void *args[] = {&p};                    // the shorter struct is its beginning
    if (a.grad_only && a.slots) {
        p.slots = *a.slots;
        return hipLaunchKernel(small_iter_kernel<SI_GRAD, SmallSlotArgs>(a.B, a.din, a.dout, a.ld), dim3((unsigned)p.slots.n), dim3(SI_THREADS), args, lds, s);
    }
    const void *kernel = a.grad_only ? small_iter_kernel<SI_GRAD>(a.B, a.din, a.dout, a.ld)
                         : a.n_iters == 1 ? small_iter_kernel<SI_ONE>(a.B, a.din, a.dout, a.ld)
                                          : small_iter_kernel<SI_RUN>(a.B, a.din, a.dout, a.ld);
    if (!a.grad_only && a.n_iters > 1) return hipLaunchCooperativeKernel(kernel, dim3((unsigned)a.M), dim3(SI_THREADS), args, (unsigned)lds, s);
    return hipLaunchKernel(kernel, dim3((unsigned)a.M), dim3(SI_THREADS), args, lds, s);
}

// How many workgroups of the kernel fit on the device at once with this much LDS each (0 if unknown, or if the device has no cooperative launches).
int small_iter_max_resident(int B, int64_t din, int64_t dout, int64_t ld)
{
    int per_cu = 0, dev = 0, cus = 0, cooperative = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipDeviceGetAttribute(&cooperative, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !cooperative)
        return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, small_iter_kernel<SI_RUN>(B, din, dout, ld), SI_THREADS,
                                                     small_iter_lds(B, (int)din, (int)dout, ld)) != hipSuccess)
        return 0;
    return per_cu * cus;
}

}  // namespace netmax
