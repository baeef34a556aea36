// The fused momentum apply + consensus mix (Eq. (c0), (c1)) restricted to a list of column tiles and with column
// ranges left out: the companion of the weight-gradient kernels that apply the update to their own columns.  It
// covers what those leave (biases, layers they do not handle, the padding, tiles that straddle a boundary).
#include "mix_subset.h"

namespace netmax {

__global__ void __launch_bounds__(256) mix_subset_kernel(int M, const int32_t *__restrict__ tiles, MixSkip skip, const float *G, MixArgs mix)
{
    mix_subset_block<256>(M, tiles[blockIdx.x / (unsigned)M], (int)(blockIdx.x % (unsigned)M), (int)(blockIdx.x % (unsigned)M), skip, G, mix);
}

void launch_mix_subset(hipStream_t s, int M, const int32_t *tiles, int n_listed, const MixSkip &skip, const float *G, const MixArgs &mix)
{
    if (n_listed <= 0) return;
    hipLaunchKernelGGL(mix_subset_kernel, dim3((unsigned)n_listed * (unsigned)M), dim3(256), 0, s, M, tiles, skip, G, mix);
}

}  // namespace netmax
