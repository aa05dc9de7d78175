// How a memoised schedule is corrected from the times of its own launches (host code only).
#pragma once
#include <stdint.h>
#include <string.h>

#include <algorithm>

namespace difa {

constexpr int kMaxDies = 16;
constexpr int kTrials = 4;     // versions of a memoised schedule that are timed, and for how many launches each
constexpr int kTrialLaunches[kTrials] = {3, 3, 16, 32};

// A schedule is made for die speeds: at first those the plan object has learnt so far, then the rates at which the dies
// have gone through this very schedule (how fast a die goes depends on what it is given: dies with short band records
// clock higher than dies with full heads).  A version runs until a few launches of it have been timed (kTrialLaunches);
// the dies not finishing together, the next one is made from what they took, and one that turned out slower gives
// way to the best so far for good.
struct Trial {
    double speed[kMaxDies] = {};        // what the schedule in use was made for
    double best_speed[kMaxDies] = {};   // ... the fastest one before it
    double best_ticks = 0.0;            // mean launch time of that one
    int trial = 0;                      // versions timed so far; kTrials: settled
    double ticks = 0.0, die_ticks[kMaxDies] = {};   // measured times of this version's launches and of their dies, summed
    int timed = 0;
    bool held = false;                  // a captured graph launches this schedule: its buffer is to stay as it is

    void start_version() {
        ticks = 0.0;
        memset(die_ticks, 0, sizeof die_ticks);
        timed = 0;
    }
    // One launch of this version has been timed: what each die took.
    void add(const unsigned long long* die, int n_dies) {
        unsigned long long longest = 0;
        for (int x = 0; x < n_dies; ++x) longest = std::max(longest, die[x]);
        if (trial >= kTrials || longest == 0) return;
        ticks += (double)longest;
        for (int x = 0; x < n_dies; ++x) die_ticks[x] += (double)die[x];
        ++timed;
    }
    // What the timed launches say: false if the schedule stays (for now, or for good), true if it is to be made again for
    // the speeds in `want`.  die_span: predicted finishing time of each die, in the scheduler's cost units.
    // capturing: the launch that is about to be made is recorded into a graph.  A remake would put its upload into the graph,
    // from a staging buffer that later uploads overwrite, and a later one would change under the graph what it launches: a
    // schedule that has been captured is not made again.
    bool remake_wanted(const int64_t* die_span, int n_dies, double* want, bool capturing) {
        held |= capturing;
        if (held || trial >= kTrials || timed < kTrialLaunches[trial]) return false;
        const double mine = ticks / timed;
        double mean = 0.0, rate_mean = 0.0, longest = 0.0;
        for (int x = 0; x < n_dies; ++x) {
            mean += die_ticks[x] / timed / n_dies;
            longest = std::max(longest, die_ticks[x] / timed);
        }
        bool rates = true;                                            // every die was busy long enough to have a rate
        for (int x = 0; x < n_dies; ++x) {
            rates &= die_span[x] >= 256 && die_ticks[x] >= 1000.0 * timed;
            want[x] = rates ? (double)die_span[x] * timed / die_ticks[x] : 1.0;
            rate_mean += want[x] / n_dies;
        }
        for (int x = 0; x < kMaxDies; ++x)
            want[x] = x < n_dies ? std::min(1.3, std::max(0.7, want[x] / rate_mean)) : 1.0;
        if (trial > 0 && mine > best_ticks * 0.997) {                 // the earlier version was faster after all
            memcpy(want, best_speed, sizeof best_speed);
            trial = kTrials;
            return true;
        }
        ++trial;
        if (!rates || longest < mean * 1.015 || trial == kTrials) {   // the dies finish together, as far as that goes
            trial = kTrials;
            return false;
        }
        memcpy(best_speed, speed, sizeof speed);
        best_ticks = mine;
        return true;
    }
};

}  // namespace difa
