// Key splits of one attention launch (host only).
//
// A workgroup of the attention kernels occupies a whole CU and the dispatcher hands the next
// one to the first CU that frees up, so a launch takes about as long as its workgroups,
// dispatched in order over `slots` CUs, do.  For every budget of tiles per workgroup each
// stream gets the fewest splits that respect it, and the budget whose launch ends first wins.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <utility>
#include <vector>

namespace a2t {

// Most key splits of a stream.
constexpr int kMaxSplits = 128;

// Floats one stream's key-split partials take in the workspace (none without a
// split), rounded up to 64 floats (256 bytes) so that every stream's rows start
// 16-byte aligned for the kernels' 16-byte stores and loads.
#if defined(__HIPCC__)
__host__ __device__
#endif
inline int64_t stream_partials(int splits, int64_t floats_per_split) {
    return splits > 1 ? (splits * floats_per_split + 63) / 64 * 64 : 0;
}

// One stream of a launch.
struct SplitStream {
    int tiles;        // key tiles, at least 1
    int wgs;          // workgroups of each key split
    int64_t floats;   // partials of each key split
    bool operator==(const SplitStream& o) const { return tiles == o.tiles && wgs == o.wgs && floats == o.floats; }
};

// What a kernel's workgroups cost, in tiles.
struct SplitCosts {
    int fixed;       // of a workgroup besides its tiles (setup, first loads, its output)
    int merge;       // of the merge launch that splits need,
    int64_t merge_floats;   // one more for so many floats of partials
    int min_tiles;   // fewest tiles worth a workgroup
};

class SplitPlanner {
public:
    // no later call with at most n streams and as many slots allocates
    void reserve(int n, int slots) {
        last_.reserve(n);
        splits_.reserve(n);
        order_.reserve(n);
        try_.reserve(n);
        levels_.reserve(slots + 1);
    }

    // force > 0: that many splits (bounded by a stream's tiles) wherever they fit
    void plan(int n, const SplitStream* s, const SplitCosts& costs, int slots, int force, int64_t ws_limit, int* splits) {
        // every layer of a step plans the same launch
        if (force == force_ && ws_limit == limit_ && slots == slots_ && costs.fixed == costs_.fixed && costs.merge == costs_.merge && costs.merge_floats == costs_.merge_floats &&
            costs.min_tiles == costs_.min_tiles && (int)last_.size() == n &&
            std::equal(s, s + n, last_.begin())) {
            std::copy(splits_.begin(), splits_.end(), splits);
            return;
        }
        splits_.assign(n, 1);
        cost_ = 0;
        int max_tiles = 1;
        for (int i = 0; i < n; ++i) max_tiles = std::max(max_tiles, s[i].tiles);
        if (force > 0) {
            int64_t ws = 0;
            for (int i = 0; i < n; ++i) {
                splits_[i] = std::max(1, std::min({force, s[i].tiles, kMaxSplits}));
                ws += stream_partials(splits_[i], s[i].floats);
            }
            if (ws > ws_limit) splits_.assign(n, 1);
        } else {
            try_.resize(n);
            int64_t best = INT64_MAX, best_wgs = 0;
            // budgets a sixteenth apart; the last one splits nothing.  The longest stream's
            // workgroups only get longer with the budget: once they alone take more than the
            // best launch so far, no later budget is better.
            for (int budget = std::min(costs.min_tiles, max_tiles);; budget = std::min(max_tiles, budget + std::max(1, budget / 16))) {
                const int cut = std::min((max_tiles + budget - 1) / budget, kMaxSplits);
                if ((max_tiles + cut - 1) / cut + costs.fixed > best) break;
                int64_t wgs = 0, ws = 0;
                bool any = false;
                for (int i = 0; i < n; ++i) {
                    try_[i] = std::min((s[i].tiles + budget - 1) / budget, kMaxSplits);
                    any |= try_[i] > 1;
                    wgs += (int64_t)try_[i] * s[i].wgs;
                    ws += stream_partials(try_[i], s[i].floats);
                }
                if (ws <= ws_limit) {
                    const int64_t t = makespan(n, s, try_.data(), costs.fixed, slots) + (any ? costs.merge + ws / costs.merge_floats : 0);
                    if (t < best || (t == best && wgs < best_wgs)) {
                        best = cost_ = t;
                        best_wgs = wgs;
                        splits_.assign(try_.begin(), try_.end());
                    }
                }
                if (budget == max_tiles) break;
            }
        }
        last_.assign(s, s + n);
        force_ = force, limit_ = ws_limit, slots_ = slots, costs_ = costs;
        std::copy(splits_.begin(), splits_.end(), splits);
    }

    // what the last plan takes, in tiles, its merge included (0 where the splits were forced)
    int64_t cost() const { return cost_; }

    // when the last workgroup ends
    int64_t makespan(int n, const SplitStream* s, const int* splits, int fixed, int slots) {
        return dispatch(n, s, splits, slots, [&](int i) { return (int64_t)(s[i].tiles + splits[i] - 1) / splits[i] + fixed; });
    }

    // the same with a cost of its own for each stream's workgroups; the streams with the most
    // tiles a workgroup are dispatched first
    template <class Cost>
    int64_t dispatch(int n, const SplitStream* s, const int* splits, int slots, Cost&& cost) {
        auto per = [&](int i) { return (s[i].tiles + splits[i] - 1) / splits[i]; };
        int64_t wgs = 0, longest = 0;
        order_.resize(n);
        for (int i = 0; i < n; ++i) {
            order_[i] = i;
            wgs += (int64_t)splits[i] * s[i].wgs;
            longest = std::max(longest, cost(i));
        }
        if (wgs <= slots) return longest;
        std::sort(order_.begin(), order_.end(), [&](int a, int b) { return per(a) != per(b) ? per(a) > per(b) : a < b; });
        // (time, CUs that are free from then on), by falling time
        levels_.clear();
        levels_.push_back({0, slots});
        for (int i : order_) {
            for (int64_t left = (int64_t)splits[i] * s[i].wgs; left > 0;) {
                const int64_t use = std::min(left, levels_.back().second), end = levels_.back().first + cost(i);
                left -= use;
                if ((levels_.back().second -= use) == 0) levels_.pop_back();
                auto at = std::lower_bound(levels_.begin(), levels_.end(), end,
                                           [](const std::pair<int64_t, int64_t>& l, int64_t t) { return l.first > t; });
                if (at != levels_.end() && at->first == end)
                    at->second += use;
                else
                    levels_.insert(at, {end, use});
            }
        }
        return levels_.front().first;
    }

private:
    std::vector<SplitStream> last_;
    std::vector<int> splits_, order_, try_;
    std::vector<std::pair<int64_t, int64_t>> levels_;
    SplitCosts costs_{};
    int force_ = -1, slots_ = -1;
    int64_t limit_ = -1, cost_ = 0;
};

}  // namespace a2t
