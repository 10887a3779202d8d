// tune_times.h -- the tuner's measure of a candidate (host code, plain C++).
#pragma once

namespace hqa {

// Runs of `steps` and of 2 `steps` steps, milliseconds: their difference is the cost of `steps` steps
// without the plan's fixed cost per run (state staging of the one-launch plans).  A run held up by
// something else counts by its repetition, so one that shortens the difference cannot make a slow
// plan the choice: 2 of 60 first tunings of N = 64, R = 8 took the per-step plan, four times slower.
struct TuneTimes {
    float one = 1e30f, two = 1e30f;
    void add(bool twice, float ms) {
        float &t = twice ? two : one;
        if (ms < t) t = ms;
    }
    float slope() const { return one >= 1e30f || two >= 1e30f ? 1e30f : two > one ? two - one : 0.0f; }
};

// Passes over a candidate: a warm-up, one pair of runs, and a second pair if the first would make
// it the choice.
constexpr int TUNE_PASSES = 5;
inline bool tune_pass_twice(int pass) { return pass > 0 && pass % 2 == 0; }
inline bool tune_done(int pass, const TuneTimes &t, float best) { return pass == 3 && t.slope() >= best; }

}  // namespace hqa
