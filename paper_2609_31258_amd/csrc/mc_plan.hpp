// mc_plan.hpp -- rules by which the host plans its launches: plain C++.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <vector>

#include "../../include/mucite.h"

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

// Largest number of candidates that a step may hold for a pack on the explicit
// branch, moving slowly in the gas: that of the densest gas, but where the pack
// would take the Langevin branch no more than its switch (at the ends of the
// window the cells with a node on either side count as outside it).
inline double densest_explicit(const GasRows &gas, double dz, const mc_operating &op, double ccs, double gas_mass_da) {
    constexpr double kBoltzmann = 1.380649e-23, kDalton = 1.66053906660e-27, pi = 3.14159265358979323846;
    if (!op.collisions_on) return 0.0;
    const double per = ccs * op.dt * std::sqrt(8.0 * gas.t_max / (pi * gas_mass_da * kDalton * kBoltzmann));
    const bool window = op.lv_z_hi > op.lv_z_lo;
    const int32_t nz = (int32_t)gas.densest.size();
    double most = 0.0;
    for (int32_t j = 0; j < nz; ++j) {
        const double c = per * gas.densest[(size_t)j];
        const bool inside = !window || (std::max(j - 1, 0) * dz >= op.lv_z_lo && std::min(j + 1, nz - 1) * dz < op.lv_z_hi);
        most = std::max(most, op.langevin_on && inside ? std::min(c, op.lv_switch) : c);
    }
    return most;
}

// Fewer candidates a step than these count as thin gas: one lane per pack is
// then the better one for any population.  1e6 packs, us a step, against one
// launch of the step kernel per step: FP32 form 41 / 53 / 77 / 106 / 181 at 0.3
// / 0.9 / 2.7 / 5.4 / 13 candidates, 52 / 61 / 84 / 112 / 184 by the step
// kernel; FP64 74 / 101 / 157 / 226 / 395 against 136 / 146 / 183 / 244 / 408.
constexpr double kThinGas = 16.0;

// Share of the pack-steps on the Langevin branch from which a large population
// that has both kinds is the stretch kernel's: one explicit pack keeps its whole
// wavefront, so it takes nearly all of them, or the slots sorted by cell.  1e6
// packs at 1e5 Pa, step kernel against stretch kernel, us a step at a share of
// 0.8 / 0.95 / 0.98 / 0.995 / 1: FP64 779 / 656 / 517 / 327 / 121 against 849 /
// 687 / 518 / 274 / 45, sorted (0.5 / 0.8 / 0.9 / 0.98 / 1) 551 / 328 / 273 / 216 /
// 98 against 561 / 312 / 198 / 182 / 44; FP32 360 / 302 / 239 / 154 / 37 against 376
// / 309 / 238 / 134 / 28, sorted 291 / 199 / 168 / 147 / 37 against 296 / 187 / 160 /
// 131 / 28.
inline bool mostly_langevin(double share, bool sorted) { return share >= (sorted ? 0.9 : 0.99); }

// That share as the program's own reads of the counters show it, for the next
// thousand steps (packs drift through a window in some thousands); -1 while
// nothing is known.
class LangevinShare {
public:
    void read(int64_t step, int64_t langevin, int64_t pack_steps) {
        if (known_ && pack_steps > steps_) {
            share_ = (double)(langevin - langevin_) / (double)(pack_steps - steps_);
            at_ = step;
        }
        known_ = true;
        langevin_ = langevin;
        steps_ = pack_steps;
    }
    void forget(bool counters) {  // (counters: they go on from another state too)
        share_ = -1.0;
        if (counters) known_ = false;
    }
    double at(int64_t step) const { return step - at_ <= 1000 ? share_ : -1.0; }

private:
    double share_ = -1.0;
    int64_t at_ = 0, langevin_ = 0, steps_ = 0;
    bool known_ = true;  // a context's counters begin at zero
};

// Lanes per pack for a launch of several steps over n slots, or 0 where the
// step kernels, one step a launch, are the faster ones.  light: no pack, or
// nearly none, runs the collision loop for more than thin gas; langevin: most
// take the Langevin branch.
//
// Lanes: the most, up to 16, that leave one wavefront per SIMD (65536 lanes);
// the FP32 form's candidates cost less of what the lanes share out than of
// what each repeats, and two wavefronts per SIMD still gain (FP64 form at
// 1.2e4 packs: 4 lanes 31 us, 8 lanes 34 us; FP32 form at 3.2e4 packs: 4 lanes
// 25 us, 2 lanes 27 us).  On the Langevin branch there is nothing to share.
//
// One lane per pack: for light populations, and up to the sizes where the step
// kernel's larger occupancy (three wavefronts per SIMD in the FP64 form, five
// in the FP32 form) outweighs the end of its launches: FP64 3e5 packs 380
// against 380 us and 6e5 packs 716 against 669, FP32 6e5 packs 301 against 305
// us and 1e6 479 against 468.
constexpr int64_t kStretchLanes = 65536;
constexpr int64_t kStretchPacks64 = 300000, kStretchPacks32 = 700000;
inline int lanes_for(bool fp32, bool langevin, bool light, int64_t n) {
    if (n <= 0) return 0;
    const int64_t lanes = fp32 && !langevin ? 2 * kStretchLanes : kStretchLanes;
    int g = 16;
    while (g > 1 && n * g > lanes) g >>= 1;
    return g > 1 || light || n <= (fp32 ? kStretchPacks32 : kStretchPacks64) ? g : 0;
}

// Whether a launch of a single step, too, is better off with several lanes per
// pack.  They must have candidates to share: with none, their loads and draws
// make the step slower than the step kernel's.  Us a step, step kernel against
// lanes, at 0 / 0.05 / 1 / 4 / 15 candidates: FP32 form 4000 packs 4.8 / 6.7 / 9.9 /
// 15 / 30 against 6.9 / 8.1 / 9.4 / 11 / 18, 3e4 packs 5.0 / 7.4 / 11 / 17 / 33
// against 6.8 / 9.5 / 11 / 15 / 25, 6e4 (two lanes) 5.3 / 7.8 / 11 / 17 / 32 against
// 5.4 / 9.9 / 13 / 18 / 31; FP64 4000 packs 7.7 / 11 / 16 / 25 / 50 against 9.4 / 12 /
// 13 / 16 / 26, 3e4 packs 9.3 / 12 / 19 / 29 / 57 against 9.4 / 13 / 17 / 24 / 44.
// (Of two steps or more all of these are faster in one launch.)
inline bool lanes_pay_in_one_step(bool fp32, int lanes, double candidates) {
    return lanes > 1 && candidates >= (!fp32 ? 1.0 : lanes > 2 ? 4.0 : 10.0);
}

// Whether no pack of a run meets more than thin gas but on the Langevin branch.
inline bool takes_only_langevin(const mc_operating &op, double most_cand) {
    return op.langevin_on && most_cand < kThinGas;
}

// What a step of a query's packs costs at most, to order the queries of a
// launch by: the long ones go first, or the launch ends with their wavefronts
// alone on the chip.
inline double step_cost(const mc_operating &op, double most_cand, double dt_now) {
    return op.adaptive ? most_cand * (dt_now / op.dt) : most_cand;
}

}  // namespace mc
