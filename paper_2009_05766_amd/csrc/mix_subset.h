// The fused momentum apply + consensus mix (Eq. (c0), (c1)) of one worker's part of one column tile, column ranges left out: by
// the THREADS threads of a workgroup.  A function of its own because the stand-alone kernel and the weight gradients that finish
// an iteration share it: 784-512-10, 16 workers, batch 64, 2 % of the columns, 63 us an iteration with the launch of its own and
// 58 us without.
#pragma once
#include "kernels.h"
#include "layout.h"
#include "vec.h"

namespace netmax {

// i: the worker; g: its place in the list of peers.
template <int THREADS>
__device__ __forceinline__ void mix_subset_block(int M, int64_t tile, int i, int g, const MixSkip &skip, const float *G, const MixArgs &mix)
{
    static_assert(TILE % (4 * THREADS) == 0, "every thread has the same share of a tile");
    int m = mix.peer[g];
    if ((unsigned)m >= (unsigned)M) m = i;                   // an index outside [0, M) is treated as a self draw
    const float wi = mix.w[(size_t)i * M + m];
    const size_t own = ((size_t)tile * M + i) * TILE, other = ((size_t)tile * M + m) * TILE;
#pragma unroll
    for (int u = 0; u < TILE / 4 / THREADS; ++u) {
        const int q = (u * THREADS + (int)threadIdx.x) * 4;
        const int64_t col = tile * TILE + q;
        bool left_out = false;
        for (int r = 0; r < skip.n; ++r) left_out |= (col >= skip.lo[r] && col < skip.hi[r]);
        if (left_out) continue;
        const f32x4 x = load4(mix.Xcur + own + q), xp = load4(mix.Xcur + other + q);
        const f32x4 v = load4_stream(mix.V + own + q), g = load4_stream(G + own + q);
        f32x4 xn, vn;
        momentum_mix4(x, v, g, xp, wi, mix.alpha, mix.mu, mix.wd, xn, vn);
        store4_stream(mix.Xnext + own + q, xn);
        store4_stream(mix.V + own + q, vn);
    }
}

}  // namespace netmax
