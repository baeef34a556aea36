// Conversion between a plain row-major matrix [M][row_ld] and the worker-interleaved tile layout.
#include "kernels.h"
#include "layout.h"
#include "vec.h"

namespace netmax {

// A workgroup moves one slot = (column tile, worker): 8 KB that are contiguous on both sides, so both conversions are plain
// copies bound by HBM.  Rows that start at multiples of 16 bytes go as 128-bit pieces (two per thread, both requested
// before the first is stored), others float by float (eight per thread, neighbouring lanes neighbouring floats); either
// way every element is touched once, hence non-temporal accesses.  Slots are walked in the order of the tile layout.
// Measured at 32 workers x 11.2 M columns (2.87 GB moved): unpack 502 us, pack 482 us (5.7 and 6.0 TB/s); with one thread per element, a
// 64-bit division each and 4-byte accesses 1000 and 1070 us.
constexpr int LAYOUT_THREADS = 256, LAYOUT_VECS = TILE / (4 * LAYOUT_THREADS), LAYOUT_FLOATS = TILE / LAYOUT_THREADS;

// tiled[tile][i][..] = rows[i][tile * TILE ..], 0 from column `cols` on.
template <bool VEC>
__global__ void __launch_bounds__(LAYOUT_THREADS) pack_kernel(int M, int64_t cols, const float *__restrict__ rows,
                                                              int64_t row_ld, float *__restrict__ tiled)
{
    const unsigned tile = blockIdx.x / (unsigned)M, i = blockIdx.x - tile * (unsigned)M;
    const int64_t j0 = (int64_t)tile << TILE_SHIFT;
    const float *src = rows + (size_t)i * row_ld + j0;
    float *dst = tiled + ((size_t)blockIdx.x << TILE_SHIFT);
    const int n = (int)(cols - j0 < TILE ? cols - j0 : TILE);        // at most 0 in a tile of padding
    const int t = (int)threadIdx.x;
    if (VEC && n == TILE) {
        f32x4 v[LAYOUT_VECS];
#pragma unroll
        for (int u = 0; u < LAYOUT_VECS; ++u) v[u] = load4_stream(src + (u * LAYOUT_THREADS + t) * 4);
#pragma unroll
        for (int u = 0; u < LAYOUT_VECS; ++u) store4_stream(dst + (u * LAYOUT_THREADS + t) * 4, v[u]);
    } else {
        float v[LAYOUT_FLOATS];
#pragma unroll
        for (int u = 0; u < LAYOUT_FLOATS; ++u) {
            const int q = u * LAYOUT_THREADS + t;
            v[u] = q < n ? __builtin_nontemporal_load(src + q) : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < LAYOUT_FLOATS; ++u) __builtin_nontemporal_store(v[u], dst + u * LAYOUT_THREADS + t);
    }
}

// rows[i][tile * TILE ..] = tiled[tile][i][..] for columns below `cols`, 0 for the columns cols .. wide - 1 (whoever wants them needs
// no fill of his own; the distance and two copies of 2 to 7 workers x 11 to 270 thousand columns: 47.6 us, with a fill of the padding
// of each copy 58 us, with one of all of it 53 us).  The tiles behind the last one with such a column need not exist in `tiled`.
template <bool VEC>
__global__ void __launch_bounds__(LAYOUT_THREADS) unpack_kernel(int M, int64_t cols, int64_t wide, const float *__restrict__ tiled,
                                                                float *__restrict__ rows, int64_t row_ld)
{
    const unsigned tile = blockIdx.x / (unsigned)M, i = blockIdx.x - tile * (unsigned)M;
    const int64_t j0 = (int64_t)tile << TILE_SHIFT;
    const float *src = tiled + ((size_t)blockIdx.x << TILE_SHIFT);
    float *dst = rows + (size_t)i * row_ld + j0;
    const int n = (int)(cols - j0 < TILE ? cols - j0 : TILE);
    const int t = (int)threadIdx.x;
    if (VEC && n == TILE) {
        f32x4 v[LAYOUT_VECS];
#pragma unroll
        for (int u = 0; u < LAYOUT_VECS; ++u) v[u] = load4_stream(src + (u * LAYOUT_THREADS + t) * 4);
#pragma unroll
        for (int u = 0; u < LAYOUT_VECS; ++u) store4_stream(dst + (u * LAYOUT_THREADS + t) * 4, v[u]);
    } else {
        const int end = (int)(wide - j0 < TILE ? wide - j0 : TILE);
        float v[LAYOUT_FLOATS];
#pragma unroll
        for (int u = 0; u < LAYOUT_FLOATS; ++u) {
            const int q = u * LAYOUT_THREADS + t;
            v[u] = q < n ? __builtin_nontemporal_load(src + q) : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < LAYOUT_FLOATS; ++u) {
            const int q = u * LAYOUT_THREADS + t;
            if (q < end) __builtin_nontemporal_store(v[u], dst + q);
        }
    }
}

// out[k] = the bfloat16 value in[k] widened to float.
__global__ void __launch_bounds__(256) widen_bf16_kernel(int64_t n, const uint16_t *__restrict__ in, float *__restrict__ out)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) out[k] = __uint_as_float((uint32_t)in[k] << 16);
}

void launch_widen_bf16(hipStream_t s, int64_t n, const uint16_t *in, float *out)
{
    hipLaunchKernelGGL(widen_bf16_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, in, out);
}

// 128-bit pieces need every row, and the tiled matrix, to start at a multiple of 16 bytes.
static bool rows_aligned(const float *rows, int64_t row_ld, const float *tiled)
{
    return row_ld % 4 == 0 && reinterpret_cast<uintptr_t>(rows) % 16 == 0 && reinterpret_cast<uintptr_t>(tiled) % 16 == 0;
}

void launch_pack(hipStream_t s, int M, int64_t cols, int64_t ld, const float *rows, int64_t row_ld, float *tiled)
{
    const dim3 grid((unsigned)(ld / TILE * M)), block(LAYOUT_THREADS);
    if (rows_aligned(rows, row_ld, tiled)) hipLaunchKernelGGL(pack_kernel<true>, grid, block, 0, s, M, cols, rows, row_ld, tiled);
    else hipLaunchKernelGGL(pack_kernel<false>, grid, block, 0, s, M, cols, rows, row_ld, tiled);
}

void launch_unpack(hipStream_t s, int M, int64_t cols, const float *tiled, float *rows, int64_t row_ld, int64_t wide)
{
    const dim3 grid((unsigned)((wide + TILE - 1) / TILE * M)), block(LAYOUT_THREADS);
    if (rows_aligned(rows, row_ld, tiled)) hipLaunchKernelGGL(unpack_kernel<true>, grid, block, 0, s, M, cols, wide, tiled, rows, row_ld);
    else hipLaunchKernelGGL(unpack_kernel<false>, grid, block, 0, s, M, cols, wide, tiled, rows, row_ld);
}

}  // namespace netmax
