// How the rows of a projection are dealt to 256- and 128-token tiles (host code, no GPU): list scheduling of the two-size launch.
#pragma once
#include <algorithm>
#include <functional>
#include <utility>
#include <vector>

namespace slim {

// The CUs of a launch, each with a speed (time per unit of work) and the time at which it becomes free.  Workgroups go in id order to the
// CU that is free first, the lowest one of several.
class CuSchedule {
public:
    explicit CuSchedule(int n_cu) : free_(n_cu, 0.0), speed_(n_cu) {
        // spread over +-8 %: tiles do not run equally fast on all CUs, which is what makes a fine-grained tail pay even
        // when the large tiles fill whole rounds
        for (int c = 0; c < n_cu; ++c) {
            speed_[c] = 1.0 + 0.08 * (n_cu > 1 ? (double)((c * 97) % n_cu) / (n_cu - 1) * 2.0 - 1.0 : 0.0);
            per_time_ += 1.0 / speed_[c];
        }
    }
    // Deals out `jobs` workgroups of `cost` each.  Whatever starts before the time `sure` (by which no more than `jobs` can have started) is
    // dealt CU by CU; only the last one or two per CU go through a heap.  Job by job the plans of one layer took 10 to 20 ms of host
    // time for a new number of rows, more than the layer on the GPU; the result is the same to the last bit.
    void deal(long jobs, double cost) {
        const long n_cu = (long)free_.size();
        if (jobs <= 0) return;
        const double sure = *std::min_element(free_.begin(), free_.end()) + (double)(jobs - n_cu - 1) * cost / per_time_;
        for (int c = 0; c < n_cu; ++c)
            while (free_[c] < sure) { start(c, cost); --jobs; }
        typedef std::pair<double, int> Slot;             // (time the CU becomes free, CU): the heap's top is the smallest
        std::vector<Slot> heap(n_cu);
        for (int c = 0; c < n_cu; ++c) heap[c] = Slot(free_[c], c);
        std::make_heap(heap.begin(), heap.end(), std::greater<Slot>());
        for (; jobs > 0; --jobs) {
            const int c = heap[0].second;
            start(c, cost);
            long i = 0;                                  // the top grows to its new time and sinks
            const Slot s(free_[c], c);
            for (long k; (k = 2 * i + 1) < n_cu; i = k) {
                if (k + 1 < n_cu && heap[k + 1] < heap[k]) ++k;
                if (!(heap[k] < s)) break;
                heap[i] = heap[k];
            }
            heap[i] = s;
        }
    }
    double makespan() const { return makespan_; }

private:
    void start(int c, double cost) {
        free_[c] += speed_[c] * cost;
        makespan_ = std::max(makespan_, free_[c]);
    }
    std::vector<double> free_, speed_;
    double per_time_ = 0.0, makespan_ = 0.0;
};

// How many 256-token tiles to run before the 128-token tiles: first = tiles, second = makespan of the plan in times of a 256-token tile.  Each
// candidate is simulated and the shortest makespan wins.  The model, fitted to sweeps of the split on the layer's shapes:
//   a 128-token tile costs small_cost of a 256-token one;
//   CU speeds are spread (CuSchedule);
//   for the 8-wave tiles only (the sweeps of the 4-wave tiles show neither effect):
//     +1 % / +3 % when the per-XCD run of large tiles is not a multiple of 8 / of 4 tiles (the run then
//     straddles columns of the band walk and shares fewer operand panels in that XCD's L2);
//     +5 % for fewer than 4 token-tiles of small tiles (too few rows to share a weight panel between the
//     workgroups that run together);
//   a ragged last tile of 256 is taken only for a gain of 3 % or more: it saves a round (SwiGLU, 14336 features: 400 rows 138 -> 102 us,
//     1000 rows 224 -> 200, 1511 rows 330 -> 296; Query + Value of 2983 rows 127 -> 97), but where the model sees a tie the launch with
//     128-token tiles is the faster one (SwiGLU 300 rows 88 against 102, down projection of 2983 rows 293 against 316).
inline std::pair<int, double> plan_tiles(int M, int tiles_n, int n_cu, double small_cost, bool eight_waves) {
    const int mb_floor = M / 256, mb_max = (M + 255) / 256, mb_min = std::max(0, mb_max - 24);
    int best_mb = mb_floor;
    double best = 1e300, ragged = 1e300;
    CuSchedule large(n_cu);                              // grows by a row of large tiles from candidate to candidate
    large.deal((long)mb_min * tiles_n, 1.0);
    for (int mb = mb_min; mb <= mb_max; ++mb) {
        if (mb > mb_min) large.deal(tiles_n, 1.0);
        const int small_tiles_m = std::max(0, M - mb * 256 + 127) / 128;
        CuSchedule all = large;
        all.deal((long)small_tiles_m * tiles_n, small_cost);
        double makespan = all.makespan();
        const long nb = (long)mb * tiles_n;
        if (eight_waves && nb > 0 && nb % 8 == 0) {
            const long run = nb / 8;
            if (run % 8 != 0) makespan *= 1.01;
            if (run % 4 != 0) makespan *= 1.03;
        }
        if (eight_waves && small_tiles_m > 0 && small_tiles_m < 4 && mb > 0) makespan *= 1.05;
        if (mb > mb_floor) ragged = makespan * 1.03;
        else if (makespan <= best) { best = makespan; best_mb = mb; }   // (of equal ones the most large tiles)
    }
    if (ragged < best) { best = ragged; best_mb = mb_max; }
    return std::make_pair(best_mb, best);
}

}  // namespace slim
