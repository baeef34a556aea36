// Internal launch interface between the C ABI (netmax_api.hip) and the gfx950 kernels.
// X, V, G are in the worker-interleaved tile layout of layout.h; ld is a multiple of TILE.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "grouped.h"
#include "philox.h"   // IterRef: iteration number by value or from a device cell

namespace netmax {


// Peer selection of Algorithm 2: one Philox draw per worker against fixed-point cumulative thresholds.
void launch_sample_peers(hipStream_t s, int M, const uint32_t *thr, const int32_t *last, uint64_t seed,
                         const IterRef &iter, int32_t *peer);

// Batch draws (with replacement) for every worker; n_rows[i] = shard size of worker i.
void launch_sample_batch(hipStream_t s, int M, int B, const int32_t *n_rows, uint64_t seed, const IterRef &iter,
                         int32_t *idx);
// Peers [n_iters][M] and batch rows [n_iters][M][B] (B = 0: none) of consecutive iterations in one launch; the last iteration's
// peers also go to last_peer [M].
void launch_sample_iterations(hipStream_t s, int n_iters, int M, const uint32_t *thr, const int32_t *last, int32_t *peer, int32_t *last_peer,
                              int B, const int32_t *n_rows, int32_t *idx, uint64_t seed, const IterRef &iter);

// g[i][j] = sigma * N(0,1) from Philox + Box-Muller; padding columns are zeroed.
void launch_synth_grad(hipStream_t s, int M, int64_t D, int64_t ld, float sigma, uint64_t seed, const IterRef &iter,
                       float *G);

// Asynchronous schedule: all (active worker, peer) draws of a run, and the in-place update of one worker's row.
void launch_async_draw(hipStream_t s, int M, const uint32_t *act_thr, int act_last, const uint32_t *thr, const int32_t *last,
                       uint64_t seed, uint64_t first, uint64_t n_steps, int32_t *active, int32_t *peers);
// A batch of global steps that do not see each other: slot s is step number first + step[s] of worker[s], which pulls from peer[s].
// Handed to kernels by value; batches of few steps as a shorter list (a launch copies its arguments).
constexpr int ASYNC_MAX_BATCH = 32, ASYNC_FEW = 4;
template <int N> struct AsyncSlotList {
    int n; uint64_t first; int32_t worker[N], peer[N]; uint32_t step[N];
    AsyncSlotList() = default;
    template <int K> explicit AsyncSlotList(const AsyncSlotList<K> &o) : n(o.n), first(o.first)      // o.n <= N
    {
        for (int s = 0; s < o.n; ++s) { worker[s] = o.worker[s]; peer[s] = o.peer[s]; step[s] = o.step[s]; }
    }
};
typedef AsyncSlotList<ASYNC_MAX_BATCH> AsyncSlots;
// The update of the active workers' rows.  source 0: flat model, gradient generated; 1: read from the active worker's row of G;
// 2: read from slot s of the compact matrix Gc and copied to the worker's row of G, as loss_c[s] is to loss.
void launch_async_rows(hipStream_t s, int source, int M, int64_t D, int64_t ld, float *X, float *V, float *G, const float *Gc,
                       const AsyncSlots &slots, const float *w, float alpha, float mu, float wd, float sigma, uint64_t seed,
                       const float *loss_c, float *loss);
// Subset runs of the perceptron gradient: the active workers' rows into a compact matrix, the first feature rows of their shards
// and their batch draws.
void launch_gather_slots(hipStream_t s, int M, int64_t ld, const AsyncSlots &slots, const float *X, float *Xc, int B, const int64_t *row0,
                         const int32_t *n_rows, uint64_t seed, int64_t *row0_c, int32_t *idx);

// The lists of a window of steps for the gradient kernels that take one: place q holds step order[q] (of the window), its worker and peer
// from the draws, its batch rows [B].
constexpr int ASYNC_WINDOW = 512;
struct AsyncOrder { uint16_t step[ASYNC_WINDOW]; };
void launch_async_lists(hipStream_t s, int n, const AsyncOrder &order, const int32_t *active, const int32_t *peers, uint64_t first, int B,
                        const int32_t *n_rows, uint64_t seed, int32_t *worker, int32_t *peer, int32_t *idx);

void launch_async_times(hipStream_t s, int M, int64_t n_steps, const int32_t *active, const int32_t *peers, const float *t,
                        float beta, float *ema, float *clock);

// Iteration-time bookkeeping of Algorithm 2 (UpdateTimeVector) against a given time matrix.
void launch_update_times(hipStream_t s, int M, const int32_t *peer, const float *t, float beta, float *ema, float *clock);

// The device cell of the iteration number used by graph replays: set it, advance it by one.
void launch_set_iteration(hipStream_t s, uint64_t *cell, uint64_t value);
void launch_bump_iteration(hipStream_t s, uint64_t *cell);

// One-time kernel attributes (LDS limits); call once per process before the first launch.
void prepare_kernels();

// Momentum apply + mix, Eq. (c0)/(c1), for all workers.
void launch_mix(hipStream_t s, int M, int64_t ld, const float *Xcur, const float *G, float *V, float *Xnext,
                const int32_t *peer, const float *w, float alpha, float mu, float wd);
// Once per device before the first launch_mix: lets the kernel be launched with its large (unused) LDS request.
hipError_t prepare_mix();
hipError_t prepare_mix_synth();      // the same for launch_mix_synth

// Flat models: the synthetic gradient generated inside the update (g is still written).
void launch_mix_synth(hipStream_t s, int M, int64_t D, int64_t ld, const float *Xcur, float *G, float *V, float *Xnext,
                      const int32_t *peer, const float *w, float alpha, float mu, float wd, float sigma, uint64_t seed,
                      const IterRef &iter);

// What the second-step update needs besides the gradient: passed to the gradient code when the weight-gradient
// kernels of the matrix-core layers apply the update themselves instead of writing the gradient.
// keep_g: a kernel that applies the update to a gradient it holds also writes it to g (not in an iteration of netmax_run that another
// follows: that one's replaces it).
struct MixArgs {
    const float *Xcur; float *V, *Xnext; const int32_t *peer; const float *w; float alpha, mu, wd; int keep_g;
};
// The same update for a list of column tiles only, leaving out up to MIX_MAX_SKIP column ranges (multiples of four
// columns) that another kernel updates.  tiles: device [n_listed].
constexpr int MIX_MAX_SKIP = 8;
struct MixSkip { int n; int64_t lo[MIX_MAX_SKIP], hi[MIX_MAX_SKIP]; };
void launch_mix_subset(hipStream_t s, int M, const int32_t *tiles, int n_listed, const MixSkip &skip, const float *G, const MixArgs &mix);

// Consensus distance: per-block partial sums (double), then a fixed-order final sum into out_dev[0].
// partial must hold consensus_partials(ld) doubles: one per CONSENSUS_COLS columns.
constexpr int CONSENSUS_COLS = 1024;
int consensus_partials(int64_t ld);
void launch_consensus(hipStream_t s, int M, int64_t D, int64_t ld, const float *X, double *partial,
                      double *out_dev);

// Layout conversion between row-major [M][row_ld] and the tile layout.  pack: columns from `cols` on become 0; unpack: so do the
// columns cols .. wide - 1.
void launch_pack(hipStream_t s, int M, int64_t cols, int64_t ld, const float *rows, int64_t row_ld, float *tiled);
void launch_unpack(hipStream_t s, int M, int64_t cols, const float *tiled, float *rows, int64_t row_ld, int64_t wide);

// out[k] = bfloat16 in[k] as float, k < n.
void launch_widen_bf16(hipStream_t s, int64_t n, const uint16_t *in, float *out);

// Whole iterations of a small softmax-regression model in one kernel, one workgroup per worker (k_small_iter.hip).
// grad_only: batch draw, loss and gradient only (G, loss); otherwise also the peer draw (peers) and the update
// (x_second, V).  n_iters > 1 is a cooperative launch, for which all workgroups have to fit the device together: x_first / x_second swap roles after every iteration and
// the workgroups meet at a barrier (counter `barrier`, which the launch advances by (n_iters - 1) * M from
// barrier_base); *fault is raised if a workgroup waited in vain.
struct SmallIterLaunch {
    int M, B; int64_t din, dout, D, ld;
    const float *feats; const int32_t *labels; const int64_t *row0; const int32_t *n_rows;
    const uint32_t *thr; const int32_t *last; const float *w;
    float *x_first, *x_second, *V, *G, *loss; int32_t *peers;
    float alpha, mu, wd; uint64_t seed; IterRef iter; int n_iters, grad_only;
    unsigned *barrier; unsigned barrier_base; int *fault;
    const AsyncSlots *slots;                 // grad_only: one workgroup per slot instead of per worker (NULL: all workers at `iter`)
    long long patience;                      // polls of the barrier counter before a workgroup gives up and raises *fault
};
bool small_iter_ok(int model_is_mlp, int n_layers, int bf16, int B, int64_t din, int64_t dout, int64_t ld);
hipError_t prepare_small_iter(int B, int64_t din, int64_t dout, int64_t ld);
int small_iter_max_resident(int B, int64_t din, int64_t dout, int64_t ld);
bool small_iter_pays(int n_iters);           // several iterations in one launch
hipError_t launch_small_iter(hipStream_t s, const SmallIterLaunch &a);

// Per-worker MLP / softmax-regression gradient (grouped GEMMs).
// The workers may be a list (layer_list_ok()): M of them then, X, G, V, loss, the shards and the mix weights those of all Mx workers; idx, the
// peers and the scratch go by place in the list.
struct MlpPlan {
    int M, n_layers, B;
    int Mx;                 // workers of X, G and V
    int M_rule;             // workers by which the error's kernel is chosen: M, but the same for all batches of asynchronous steps
    const int32_t *worker;  // device [M], NULL: all of them
    int64_t dims[8];
    int64_t woff[8];        // offset of layer l's W inside a parameter row; the bias follows the matrix
    int64_t ld;
    int bf16;               // operands rounded to bfloat16 (features are stored as bfloat16)
    int head_pairs;         // logits summed by pairs of steps, as resident_mlp_kernel does (contexts that can run it)
    const void *feats;      // [n_total][dims[0]]
    const int32_t *labels;  // [n_total]
    const int64_t *row0;    // device [M]: first feature row of each worker's shard
    const int32_t *idx;     // device [M][B] shard-local batch rows
    float *act[8];          // act[l], l = 1..n_layers: [M][B][dims[l]] post-activation (logits for the last)
    float *dz[2];           // two ping-pong buffers [M][B][max width]
    float *loss;            // [M]
    // bf16 operands only: bfloat16 copies of activations and back-propagated errors, in both orientations
    uint16_t *hb[8];        // hb[l], l = 1..n_layers-1: [M][B][dims[l]]
    uint16_t *ht[8];        // ht[l], l = 1..n_layers-1: [M][dims[l]][B] (the first layer's weight gradient gathers its A^T from the data rows)
    uint16_t *dzb[2];       // [M][B][max width]
    uint16_t *dzt[2];       // [M][max width][B]
};
// The second-step update inside netmax_run, for the columns that no weight gradient has updated: the columns of the listed tiles
// (device [n_tiles]) outside `skip`.
struct TailArgs { MixArgs mix; const int32_t *tiles; int n_tiles; MixSkip skip; };
// fuse != nullptr: layers accepted by mfma_layer_ok() do not write their weight gradient to G; they write
// x' and v' of their weight columns (Eq. (c0)/(c1)) straight from the product.
// tail != nullptr (not together with fuse): the weight gradients of the layers whose update_end() is not 0 write G (mix.keep_g) and apply the
// update to the columns woff .. update_end() - 1 (multiples of four) while they hold them.  The others are updated by the first
// layer's weight gradient where it can (it is the last launch then), else by the caller: false is returned in that case.
// With a list: X, G and the update in place (mix.Xnext = mix.Xcur); no listed worker is another's peer.
bool launch_mlp_grad(hipStream_t s, const MlpPlan &p, const float *X, float *G, const MixArgs *fuse = nullptr, const TailArgs *tail = nullptr);
int64_t update_end(const MlpPlan &p, int l);
bool update_beside_g(const MlpPlan &p);                  // in iterations that keep g, too
// All kernels of the plan take a list of workers and between them update all of their columns.
bool layer_list_ok(const MlpPlan &p);

// Matrix-core kernels (k_grad_mfma.hip) for layers that mfma_layer_ok() accepts.
bool mfma_layer_ok(const MlpPlan &p, int l);
void launch_fwd_mfma(hipStream_t s, const MlpPlan &p, int l, const float *X);
// also writes the bias gradient of layer l - 1 into G; want_f32: keep the fp32 copy of the error as well
void launch_dgrad_mfma(hipStream_t s, const MlpPlan &p, int l, const float *X, float *G, int cur, bool want_f32);
void launch_wgrad_mfma(hipStream_t s, const MlpPlan &p, int l, float *G, int cur);
double wgrad_mix_saves(const MlpPlan &p, bool keep_g);   // bytes a parameter, by count, that the update in all of them saves an iteration
void launch_wgrad_mix_mfma(hipStream_t s, const MlpPlan &p, int l, float *G, int cur, const MixArgs &mix);
// Last layer with at most 32 outputs.
bool mfma_small_last_ok(const MlpPlan &p);
// also: softmax cross-entropy on the logits (loss, dZ, the last layer's bias gradient, the gradient's padding)
void launch_fwd_small(hipStream_t s, const MlpPlan &p, const float *X, float *G);
void launch_wgrad_small(hipStream_t s, const MlpPlan &p, float *G, int cur);
void launch_dgrad_small(hipStream_t s, const MlpPlan &p, const float *X, float *G, int cur, bool want_f32);

// Layers on fp32 operands with a batch of 32 or 64 rows and a multiple of 32 outputs (k_grad_f32.hip): forward pass
// and weight gradient that read W / write dW exactly once with many loads in flight.
bool fwd_f32_ok(const MlpPlan &p, int l);
bool wgrad_f32_ok(const MlpPlan &p, int l);
hipError_t prepare_f32_layers();
void launch_fwd_f32(hipStream_t s, const MlpPlan &p, int l, const float *X);
// tail: see launch_mlp_grad(); others: this launch also updates the columns of tail->tiles (first layer only)
void launch_wgrad_f32(hipStream_t s, const MlpPlan &p, int l, float *G, const float *dz, const TailArgs *tail, bool others);

// Whole iterations of a softmax regression whose worker takes several workgroups (k_sliced_iter.hip), for netmax_run: mix, G, loss,
// peers as the separate kernels leave them after the last iteration.  All workgroups have to be resident together: M times
// sliced_iter_slices() of them.  Tickets: one per iteration, never 0, in turn.  The launch advances rows_base by (n_iters - 1) M.
struct SlicedIterLaunch {
    MixArgs mix; float *G; int32_t *peers; const int32_t *n_rows; const uint32_t *thr; const int32_t *last; uint64_t seed; IterRef iter; int n_iters;
    unsigned long long *parts; float *biases; unsigned *counters; unsigned ticket, rows_base;
    int *fault; long long patience;
};
bool sliced_iter_ok(const MlpPlan &p);
int sliced_iter_slices(const MlpPlan &p);
void sliced_iter_scratch(const MlpPlan &p, size_t &parts, size_t &biases, size_t &counters);
hipError_t prepare_sliced_iter(const MlpPlan &p, int *resident);
bool sliced_iter_pays(int n_iters);
hipError_t launch_sliced_iter(hipStream_t s, const MlpPlan &p, const SlicedIterLaunch &a);

// The same for a perceptron with one hidden layer whose first weight matrices fit the chip's LDS together (k_resident_mlp.hip): a grid of
// resident_mlp_grid() workgroups, all resident together.  Shards of fewer than 2^32 bytes, features where fwd_f32_ok() takes them.
bool resident_mlp_ok(const MlpPlan &p);
bool resident_mlp_pays(const MlpPlan &p, int n_iters);
int resident_mlp_grid(const MlpPlan &p);
void resident_mlp_scratch(const MlpPlan &p, size_t &parts, size_t &biases, size_t &counters);
hipError_t prepare_resident_mlp(const MlpPlan &p, int *resident);
hipError_t launch_resident_mlp(hipStream_t s, const MlpPlan &p, const SlicedIterLaunch &a);

// Tiled kernels for layers of any shape, fp32 or bfloat16 operands.  need_t: the transposed bfloat16 activation is wanted (by a
// matrix-core kernel above); below_fast: so are both bfloat16 copies of the error.  launch_tile_dgrad: true if it has also
// written the bias gradient of the layer below (its workgroups held the whole batch).
void launch_tile_fwd(hipStream_t s, const MlpPlan &p, int l, const float *X, bool need_t);
bool tile_fwd_one_chain(const MlpPlan &p, int l);        // its sums are one chain over the contraction, not four (blocks enough)
constexpr int TILE_DGRAD_BATCH = 128;                   // up to here they do
bool launch_tile_dgrad(hipStream_t s, const MlpPlan &p, int l, const float *X, float *G, int cur, bool below_fast);
bool tile_wgrad_update_ok(const MlpPlan &p, int l);      // its update: fp32 operands, aligned rows
void launch_tile_wgrad(hipStream_t s, const MlpPlan &p, int l, float *G, int cur, const TailArgs *tail, bool others);

// Layers on bfloat16 operands in few blocks (k_chain.hip), bit for bit as the tiled and the matrix-core kernels; the error's kernel also writes the
// bias gradient of the layer below.
bool chain_fwd_pays(const MlpPlan &p, int l);
void launch_chain_fwd(hipStream_t s, const MlpPlan &p, int l, const float *X, bool need_t);
bool chain_dgrad_pays(const MlpPlan &p, int l);
void launch_chain_dgrad(hipStream_t s, const MlpPlan &p, int l, const float *X, float *G, int cur, bool below_fast);

// Last layer with at most 32 classes, fp32 or bfloat16 operands (k_grad_head.hip): from its input to the error of the layer
// below in two kernels: logits, loss, dW, db, dH and the column sums of dH.
bool head_ok(const MlpPlan &p);
// Its logits are then sums of parts of 32 hidden units, added two by two: head_pairs_per_wave() of them at a time, then these.
bool head_parts_of_two(const MlpPlan &p);
int head_pairs_per_wave(const MlpPlan &p);
void launch_head(hipStream_t s, const MlpPlan &p, const float *X, float *G, const MixArgs *tail);

}  // namespace netmax
