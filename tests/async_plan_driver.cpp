// Runs random schedules step by step and batch by batch (all reads of a batch before its writes) and compares the states.
#include "../paper_2009_05766_amd/csrc/async_plan.h"
#include <cstdint>
#include <cstdio>
#include <random>

int main()
{
    std::mt19937_64 rng(7);
    long steps = 0, batches = 0;
    for (int trial = 0; trial < 3000; ++trial) {
        const int M = 2 + (int)(rng() % (trial % 3 == 0 ? 4 : 130)), n = 1 + (int)(rng() % 600), cap = 1 + (int)(rng() % 32);
        netmax::AsyncPlanner planner(M);
        std::vector<uint64_t> a(M), b;
        for (auto &x : a) x = rng();
        b = a;
        for (int window = 0; window < 3; ++window) {             // the planner is used again for the next steps
            std::vector<int> act(n), peer(n), seen(n, 0);
            for (int s = 0; s < n; ++s) {
                act[s] = (int)(rng() % M);
                peer[s] = rng() % 8 == 0 ? act[s] : (int)(rng() % M);
                a[act[s]] = a[act[s]] * 3 + a[peer[s]] * 5 + (uint64_t)s;
            }
            const bool in_order = (trial + window) % 2 != 0;
            planner.plan(act.data(), peer.data(), n, cap, in_order);
            for (int q = 0; in_order && q < n; ++q)
                if (planner.order()[q] != q) return std::puts("steps out of order"), 1;
            for (int k = 0; k < planner.batches(); ++k) {
                const int lo = planner.start(k), hi = planner.start(k + 1);
                if (hi - lo < 1 || hi - lo > cap) return std::printf("a batch of %d\n", hi - lo), 1;
                std::vector<uint64_t> next;
                for (int q = lo; q < hi; ++q) {
                    const int s = planner.order()[q];
                    ++seen[s];
                    next.push_back(b[act[s]] * 3 + b[peer[s]] * 5 + (uint64_t)s);
                }
                std::vector<int> written(M, 0), pulled(M, 0);
                for (int q = lo; q < hi; ++q) {
                    const int s = planner.order()[q];
                    if (written[act[s]]++) return std::puts("a worker active twice in a batch"), 1;
                    if (peer[s] != act[s]) pulled[peer[s]] = 1;
                    b[act[s]] = next[q - lo];
                }
                for (int q = lo; q < hi; ++q)
                    if (pulled[act[planner.order()[q]]]) return std::puts("a row written and pulled in a batch"), 1;
            }
            for (int s = 0; s < n; ++s)
                if (seen[s] != 1) return std::puts("a step left out or taken twice"), 1;
            if (a != b) return std::puts("another state"), 1;
            steps += n;
            batches += planner.batches();
        }
    }
    std::printf("ok %ld steps %ld batches\n", steps, batches);
    return 0;
}
