// Which global steps of the asynchronous schedule can run side by side (host code).
//
// Step s reads the rows of its active worker and of its peer and writes the row of its active worker.  Its level is one more
// than the highest level of an earlier step that wrote a row it reads or read a row it writes; steps of one level do not see
// each other, and running the levels one after the other gives every step the rows it would have found in step order.  Against
// cutting the run where the first step sees an earlier one of its group, a level also takes the steps behind that cut that wait
// for nobody: 64 steps of 16 workers are 18 batches instead of 23.  `in_order` cuts the run there all the same.
#pragma once
#include <algorithm>
#include <vector>

namespace netmax {

class AsyncPlanner {
public:
    explicit AsyncPlanner(int M) : wrote_(M, 0), read_(M, 0) {}

    // active, peer: n steps.  Afterwards order() lists the steps level by level (in step order inside a level), and batch b is
    // order()[start(b)] .. order()[start(b + 1) - 1]: steps of one level, at most cap of them.  in_order: consecutive steps, as many
    // as do not see each other.
    void plan(const int *active, const int *peer, int n, int cap, bool in_order = false)
    {
        level_.resize(n);
        order_.resize(n);
        count_.clear();
        int top = 0;
        for (int s = 0; s < n; ++s) {
            const int i = active[s], m = peer[s];
            const int after = std::max(std::max(wrote_[i], wrote_[m]), read_[i]);     // the step has to come behind this level
            const int l = in_order ? std::max(std::max(top, 1), after + 1) : after + 1;
            wrote_[i] = l;
            read_[m] = std::max(read_[m], l);
            level_[s] = l;
            if (l > top) { top = l; count_.resize(top + 1, 0); }
            ++count_[l];
        }
        start_.assign(1, 0);
        int at = 0;
        for (int l = 1; l <= top; ++l) {
            const int end = at + count_[l];
            count_[l] = at;                                  // where the level's next step goes
            for (; at < end; at = std::min(at + cap, end)) start_.push_back(std::min(at + cap, end));
        }
        for (int s = 0; s < n; ++s) order_[count_[level_[s]]++] = s;
        for (int s = 0; s < n; ++s) wrote_[active[s]] = read_[active[s]] = read_[peer[s]] = wrote_[peer[s]] = 0;
    }
    int batches() const { return (int)start_.size() - 1; }
    int start(int b) const { return start_[b]; }
    const std::vector<int> &order() const { return order_; }

private:
    std::vector<int> wrote_, read_;                          // per worker: highest level that wrote / pulled its row (0: none)
    std::vector<int> level_, order_, count_, start_;
};

}  // namespace netmax
