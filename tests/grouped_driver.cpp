// Every block of every worker once, nothing else; at most one block more on an XCD than on another where blocks are dealt.
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
            for (unsigned i = 0; i < grid; ++i) {
                int g;
                unsigned local;
                if (!decode_group(i, b, M, g, local)) continue;
                if (g < 0 || g >= M || local >= b) { printf("M %d, %u blocks: id %u is (%d, %u)\n", M, b, i, g, local); return 1; }
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
    printf("ok\n");
    return 0;
}
