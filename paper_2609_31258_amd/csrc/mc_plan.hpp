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

}  // namespace mc
