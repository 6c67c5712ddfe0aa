// asd_tune.h -- the autotuner's choice among timed candidates (host only).
#pragma once

#include <stddef.h>

#include <algorithm>
#include <vector>

namespace asd {

// Candidate of least median over the rounds.  Where that is not the incumbent
// (the variant a handle starts with), it has to be ahead of it by more than the
// larger spread of the two, slowest and fastest round left out: near-ties stay
// with the incumbent instead of falling to whichever round was disturbed.
inline size_t tune_pick(std::vector<std::vector<double>> rounds, size_t incumbent)
{
    if (rounds.empty()) return 0;
    for (auto &v : rounds) std::sort(v.begin(), v.end());
    auto median = [&](size_t j) { return rounds[j][rounds[j].size() / 2]; };
    auto spread = [&](size_t j) {
        const size_t cut = rounds[j].size() > 2 ? 1 : 0;
        return rounds[j][rounds[j].size() - 1 - cut] - rounds[j][cut];
    };
    size_t pick = 0;
    for (size_t j = 1; j < rounds.size(); ++j)
        if (median(j) < median(pick)) pick = j;
    if (incumbent < rounds.size() &&
        median(incumbent) - median(pick) <= std::max(spread(incumbent), spread(pick)))
        return incumbent;
    return pick;
}

}  // namespace asd
