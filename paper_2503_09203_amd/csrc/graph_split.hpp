// Split of a captured chunk into launches (host code without HIP).
#pragma once
#include <cstdint>

namespace mgx {

// Launches are bounded, so that no kernel holds the device for long.
constexpr int32_t kMaxLaunchSteps = 4096;

struct ChunkSplit {
    int32_t n_steps, K;
    bool single;       // one step per launch
    bool join;         // stretches of K steps share launches (K < kMaxLaunchSteps)
    bool stats;        // the last stretch's end takes statistics: a launch of its own
    int32_t min_join;  // the fewest steps a joined launch takes; fewer go stretch by stretch

    // Steps of the launch that starts after `done` steps.
    int32_t next(int32_t done) const {
        const int32_t per = single ? 1 : join ? kMaxLaunchSteps / K * K : K;
        int32_t k = n_steps - done < per ? n_steps - done : per;
        if (join && stats && done + k == n_steps && k > K) k = (k - 1) / K * K;
        if (join && k < min_join && k > K) k = K;
        return k;
    }
    // Whether some launch is of one step (such launches use the step hints).
    bool any_single() const {
        for (int32_t done = 0; done < n_steps;) {
            const int32_t k = next(done);
            if (k == 1) return true;
            done += k;
        }
        return false;
    }
};

}  // namespace mgx
