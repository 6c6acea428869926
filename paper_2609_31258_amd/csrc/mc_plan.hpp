// mc_plan.hpp -- rules by which the host plans its launches: plain C++.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>

namespace mc {

// Time at which a run of adaptive steps from t0 hands over to the space-charge
// update due at t_pic (later than t0; updates within tol count as due).  Later
// than t0 also where tol vanishes beside the times, so that every run takes a
// step.
inline double pause_time(double t0, double t_pic, double tol) {
    return std::max(t_pic - tol, std::nextafter(t0, HUGE_VAL));
}

// How many adaptive steps to enqueue before the next space-charge update: as
// many as fit at the mean length of the run's last steps, and one more.  Steps
// enqueued beyond the update are not taken, but each is a launch (4 us); too few
// cost another round with the host (25 us).  A step that an update cut short
// tells nothing of the others: 1000 FP32 packs on the Langevin branch with
// updates every 50 ns took 23.6 us a step of 3.3 ns where the last step's length
// was the guess (most launches beyond the update, each time for the 0.5 ns left
// to it), 13.9 us so.
class StepPace {
public:
    int64_t steps_for(double room, double dt_max) const {
        const bool known = mean_ > 0.0 && mean_ < dt_max;
        const double n = std::ceil(room / (known ? mean_ : dt_max)) + (known ? 1.0 : 0.0);
        return (int64_t)std::max(1.0, std::min(n, 1024.0));
    }
    // A run took `steps` steps in `time`, the last one of length `last` up to
    // an update if `cut`.
    void took(int64_t steps, double time, double last, bool cut) {
        const int64_t whole = cut ? steps - 1 : steps;
        if (whole > 0) mean_ = (cut ? time - last : time) / (double)whole;
    }

private:
    double mean_ = 0.0;
};

}  // namespace mc
