// Grids of the kernels that work on one block of one worker per workgroup.
#pragma once

namespace netmax {

// Workgroup id -> (worker, block inside the worker's GEMM).  Workgroup ids are dealt round-robin to the 8
// XCDs; all blocks of one worker are placed on the same XCD, next to each other, so the operand every
// block of that worker re-reads (its activations / back-propagated errors) comes from HBM once and from
// that XCD's L2 afterwards.  The blocks of the workers beyond whole rounds of eight are dealt to all XCDs in eight equal runs: in
// a round of its own they leave XCDs idle.  Unless every block finds a compute unit of its own either way: then the
// operands should come into one L2 only.  Returns false for the padding ids.
// Per iteration, a round of its own and dealt: fp32 784-512-10, batch 64, 2 workers 39.8 and 31.5 us, 9 workers 50.2 and 41.2 us;
// 3072-1024-10, batch 64, 2 workers 119 and 74 us, batch 128, 9 workers 393 and 316 us; bfloat16 784-500-300-10, batch 100, 50
// workers 229 and 223 us; dealt also where they fit: bfloat16 784-500-300-10, 5 workers 75.5 and 77.4 us.
constexpr int MF_XCD = 8, XCD_CUS = 32;
__host__ __device__ inline unsigned dealt_workers(unsigned blocks_per_worker, int M)
{
    return ((unsigned)M / MF_XCD + 1) * blocks_per_worker <= XCD_CUS ? 0 : (unsigned)M % MF_XCD;
}
__device__ __forceinline__ bool decode_group(unsigned bid, unsigned blocks_per_worker, int M, int &g, unsigned &local)
{
    const unsigned xcd = bid % MF_XCD, slot = bid / MF_XCD, dealt = dealt_workers(blocks_per_worker, M), rounds = (unsigned)M / MF_XCD;
    if (dealt == 0 || slot < rounds * blocks_per_worker) {
        const unsigned round = slot / blocks_per_worker;
        local = slot - round * blocks_per_worker;
        g = (int)(round * MF_XCD + xcd);
        return g < M;
    }
    const unsigned run = (dealt * blocks_per_worker + MF_XCD - 1) / MF_XCD, nth = slot - rounds * blocks_per_worker;
    if (nth >= run) return false;                            // behind the grid
    const unsigned at = xcd * run + nth, w = at / blocks_per_worker;
    local = at - w * blocks_per_worker;
    g = (int)(rounds * MF_XCD + w);
    return w < dealt;
}
inline unsigned grouped_grid(int M, unsigned blocks_per_worker)
{
    const unsigned dealt = dealt_workers(blocks_per_worker, M);
    if (dealt == 0) return (unsigned)((M + MF_XCD - 1) / MF_XCD * MF_XCD) * blocks_per_worker;
    return ((unsigned)M / MF_XCD * blocks_per_worker + (dealt * blocks_per_worker + MF_XCD - 1) / MF_XCD) * MF_XCD;
}

// One direction of a launch holds fewer than 2^32 work-items (beyond, the count wraps and most of the launch is left out, without an
// error), which many workers with wide layers of few outputs can exceed.  Such a grid is cut into rows of whole rounds over the
// XCDs; a workgroup's id is then its row's start plus its place in the row, and ids behind the grid decode to nothing.
constexpr unsigned GRID_ROW = 1u << 21;                     // x 1024 threads at the most
struct GridRows { unsigned x, y; };
inline GridRows grid_rows(unsigned workgroups)
{
    if (workgroups <= GRID_ROW) return {workgroups, 1};
    return {GRID_ROW, (workgroups - 1) / GRID_ROW + 1};
}

// A number of workgroups rounded up to whole rounds over the XCDs: what follows them in a grid keeps its place in the deal.
inline unsigned grouped_blocks(unsigned n) { return (n + MF_XCD - 1) / MF_XCD * MF_XCD; }

}  // namespace netmax
