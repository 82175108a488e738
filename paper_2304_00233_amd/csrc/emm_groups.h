// Which sources of a forward, and which jobs of a batch, run side by side.
// Plain C++: its tests use it without HIP.
#pragma once

#include <algorithm>
#include <vector>

namespace emm {

// Bytes a step may touch for several sources of one model to share the 256 MB
// Infinity Cache.  ms a forward of 100 steps, in groups of the size named:
//   48^3 nodes, 9 sources (23 MB each)     8.6 in 9 (207 MB), 9.1 in 8, 9.5 in 5
//   48^3, 16 sources                       15.6 in 8 (184 MB), 16.7 in 10 (229), 18.4 in 16 (365)
//   37 x 29 x 23, 16 (13 MB)               9.1 in 16 (211 MB), 10.0 in 8
//   80 x 64 x 50, 12 (35 MB)               17.0 in 6 (214 MB), 18.7 in 4, 20.1 in 8 (285)
//   64^3, 8 (41 MB)                        11.8 in 4 (167 MB), 13.3 in 8 (332)
//   90^3, smooth, 6 (62 + 24 MB)           18.4 in 3 (211 MB), 20.2 in 2, 22.3 in 5 (335)
//   140 x 130 x 130, smooth, 4 (153 + 62)  36.9 in 1 (215 MB), 39.4 in 4
constexpr double kSourceBudget = 240e6;

// Sources per time loop: as few loops of even size as keep the bytes of a step
// (per a source and shared by all) within the budget, or all of them in one
// when one source alone does not fit.
inline int source_group(double per, double shared, int nsrc) {
    if (per + shared > kSourceBudget) return nsrc;
    const int most = std::max(1, (int)((kSourceBudget - shared) / per)), groups = (nsrc + most - 1) / most;
    return (nsrc + groups - 1) / groups;
}

// Bytes a step may touch for jobs to share the 256 MB Infinity Cache, and cells
// that fill the chip (below them more jobs are never worse).  ms for 6 equal
// jobs of 60 steps (12 of 56 to 78 MB), by jobs side by side:
//   need each         1      2      3      4      6
//   56 MB            27.1   20.6   19.5   19.8   19.7    (169 MB in threes, 225 in fours)
//   64 MB            29.2   21.5   20.4   21.7   21.5    (192, 256)
//   76 MB            17.3   13.1   12.5   14.3   14.7    (227, 302)
//   78 MB            30.8   22.9   22.1   25.6   24.4    (235, 313)
//   97 MB            19.5   15.6   18.7   18.2   18.3    (194 in pairs, 291)
//   119 MB           22.7   20.9   21.9   22.5   23.0    (238, 356)
//   131 MB           24.7   24.8   25.0   26.0   26.3
//   240 MB           39.6   36.3   38.0
// A job of one or two sources leaves the chip idle between its launches, so
// two of them also go together beyond the cache (262 MB each 17.0 -> 16.5 ms,
// 277 MB at r = 4 12.4 -> 10.7; 375 MB each 22.1 -> 23.3).  Jobs of more
// sources do not (178 MB, three sources, 16.4 -> 17.6 in a pair; 184 MB, eight
// sources, 16.1 -> 18.1).
constexpr double kBatchBudget = 240e6;
constexpr double kPairBudget = 560e6;
constexpr int kPairSources = 2;
constexpr double kFillCells = 2.5e6;

// Sizes of consecutive groups of jobs that touch need[j] bytes a step, have
// cells[j] cells (of all sources) and nsrc[j] sources: as few groups as the budget allows, of even size where that
// keeps to it (four jobs of 76 MB 8.8 ms in twos, 9.2 in three and one).
inline std::vector<int> batch_groups(const std::vector<double> &need, const std::vector<double> &cells,
                                     const std::vector<int> &nsrc) {
    const size_t n = need.size();
    double total = 0.0;
    for (double b : need) total += b;
    bool over = false;                                   // a group of the last split exceeds the budget
    // parts = 0: packed, else by parts of all bytes
    auto split = [&](int parts) {
        std::vector<int> sizes;
        double before = 0.0, held = 0.0, filled = 0.0;   // bytes of the jobs before j; bytes and cells of the group
        int at = 0;                                      // part that the group's first job lies in
        over = false;
        for (size_t j = 0; j < n; ++j) {
            // (a job goes with the part that its middle lies in)
            const int next = parts > 0 ? (int)((before + 0.5 * need[j]) / (total / parts)) : 0;
            const bool pair = j > 0 && sizes.back() == 1 && nsrc[j - 1] <= kPairSources && nsrc[j] <= kPairSources;
            const bool some = j > 0 && filled >= kFillCells && !(pair && held + need[j] <= kPairBudget);
            const bool beyond = held + need[j] > kBatchBudget;
            if (j == 0 || (some && (parts > 0 ? next > at : beyond))) {
                sizes.push_back(0);
                held = filled = 0.0;
                at = next;
            } else if (some && beyond) {
                over = true;
            }
            ++sizes.back();
            before += need[j];
            held += need[j];
            filled += cells[j];
        }
        return sizes;
    };
    const std::vector<int> packed = split(0), even = split((int)packed.size());
    return over || even.size() > packed.size() ? packed : even;
}

}  // namespace emm
