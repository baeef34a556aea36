// Every block of every worker once, nothing else, also from ids behind the grid; at most one block more on an XCD than on another
// where blocks are dealt.  Grids of any size are cut into rows that a launch can hold.
#include <cstdio>
#include <vector>
#define __host__
#define __device__
#define __forceinline__ inline
#include "../paper_2009_05766_amd/csrc/grouped.h"
using namespace netmax;

int main()
{
    for (int M = 1; M <= 140; ++M)
        for (unsigned b = 1; b <= 700; b += (b < 70 ? 1 : 37)) {
            std::vector<int> seen((size_t)M * b, 0);
            unsigned on_xcd[MF_XCD] = {};
            const unsigned grid = grouped_grid(M, b);
            for (unsigned i = 0; i < grid + 3 * MF_XCD * b + 5; ++i) {
                int g;
                unsigned local;
                if (!decode_group(i, b, M, g, local)) continue;
                if (g < 0 || g >= M || local >= b) { printf("M %d, %u blocks: id %u is (%d, %u)\n", M, b, i, g, local); return 1; }
                if (i >= grid) { printf("M %d, %u blocks: id %u behind the grid is (%d, %u)\n", M, b, i, g, local); return 1; }
                ++seen[(size_t)g * b + local];
                ++on_xcd[i % MF_XCD];
            }
            for (int n : seen)
                if (n != 1) { printf("M %d, %u blocks: a block %d times\n", M, b, n); return 1; }
            unsigned most = 0;
            for (unsigned n : on_xcd) most = n > most ? n : most;
            const unsigned even = ((unsigned)M * b + MF_XCD - 1) / MF_XCD;
            if (most > (even > XCD_CUS ? even : (unsigned)XCD_CUS)) { printf("M %d, %u blocks: %u on an XCD\n", M, b, most); return 1; }
        }
    for (unsigned n : {1u, 8u, GRID_ROW - 1, GRID_ROW, GRID_ROW + 1, 8519550u, 1u << 23, 0x7FFFFFFFu, 0xFFF00000u}) {
        const GridRows r = grid_rows(n);
        const unsigned long long all = (unsigned long long)r.x * r.y;
        if (all < n || all - n >= r.x || (unsigned long long)r.x * 1024 >= 1ull << 32 || r.y > 65535 || (r.y > 1 && r.x != GRID_ROW) || GRID_ROW % MF_XCD) {
            printf("%u workgroups: %u x %u\n", n, r.x, r.y);
            return 1;
        }
    }
    printf("ok\n");
    return 0;
}
