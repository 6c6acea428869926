// mc_plan.hpp -- rules by which the host plans its launches: plain C++.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <vector>

namespace mc {

// Largest number density (in p/T) of every axial row of a gas table, and its
// largest pressure and temperature (none is negative).  Ratios are compared by
// products: a division a node took 65,536 nodes 90 us of a field load of 0.53 ms.
struct GasRows {
    std::vector<double> densest;
    double p_max = 0.0, t_max = 0.0;

    void scan(const double *p, const double *t, int32_t nr, int32_t nz) {
        densest.assign((size_t)nz, 0.0);
        p_max = t_max = 0.0;
        for (int32_t j = 0; j < nz; ++j, p += nr, t += nr) {
            double pd = 0.0, td = 1.0;
            for (int32_t i = 0; i < nr; ++i) {
                p_max = std::max(p_max, p[i]);
                t_max = std::max(t_max, t[i]);
                if (t[i] > 0.0 && p[i] * td > pd * t[i]) {
                    pd = p[i];
                    td = t[i];
                }
            }
            densest[(size_t)j] = pd / td;
        }
    }
};

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
