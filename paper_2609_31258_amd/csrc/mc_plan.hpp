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
        const bool inside = !window || (std::max(j - 1, 0) * dz >= op.lv_z_lo &&
                                        std::min(j + 1, nz - 1) * dz < op.lv_z_hi);
        most = std::max(most, op.langevin_on && inside ? std::min(c, op.lv_switch) : c);
    }
    return most;
}

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

// Lanes per pack for a launch over n slots: the most, up to 16, that leave one
// wavefront per SIMD (65536 lanes); the FP32 form's candidates cost less of what
// the lanes share out than of what each repeats, and two wavefronts per SIMD
// still gain (FP64 form at 1.2e4 packs: 4 lanes 31 us, 8 lanes 34 us; FP32 form
// at 3.2e4 packs: 4 lanes 25 us, 2 lanes 27 us).  On the Langevin branch there is
// nothing to share.
constexpr int64_t kStretchLanes = 65536;
inline int lanes_for(bool fp32, bool langevin, int64_t n) {
    const int64_t lanes = fp32 && !langevin ? 2 * kStretchLanes : kStretchLanes;
    int g = 16;
    while (g > 1 && n * g > lanes) g >>= 1;
    return g;
}

// Whether a launch of `steps` steps with one lane per pack is the better one for
// n packs of up to `candidates` a step, against a launch of the step kernel per
// step.  What it saves -- the ends of the launches and the state's way to memory
// and back -- it saves per step beyond the first; what it loses, by a lower
// occupancy (two wavefronts per SIMD against three in the FP64 form, three
// against five in the FP32 form), goes with packs and candidates, and begins
// where the packs no longer fit on the chip at once (131072 in the FP64 form).
// The rows are the candidates measured and a tenth more, the columns 2, 3 to 4, 5
// to 9 and more steps, and what they hold the largest of 1.4e5, 2e5, 3e5, 5e5,
// 7e5, 1e6, 2e6 and 4e6 packs that gained (or lost less than a hundredth).  Step
// kernel against stretch kernel, us a step of ten: FP64 1 candidate 1e6 packs 128
// / 90, 4 candidates 1e6 181 / 171, 4e6 657 / 644, 10 candidates 7e5 216 / 214, 1e6
// 295 / 303, 25 candidates 3e5 206 / 204, 5e5 304 / 313, 49 candidates 1.2e5 172 /
// 152, 1.4e5 224 / 226, 1e6 957 / 1059; FP32 0.05 candidates 4e6 108 / 95, 1
// candidate 2e6 87 / 84, 4e6 158 / 162, 4 candidates 1e6 81 / 79, 2e6 144 / 148, 10
// candidates 7e5 99 / 95, 1e6 133 / 134, 49 candidates 5e5 238 / 234, 7e5 312 / 316,
// 1e6 430 / 445.
struct OneLaneLimit {
    double candidates;
    int64_t packs[4];
};
inline bool one_lane_pays(bool fp32, bool langevin, double candidates, int64_t n, int64_t steps) {
    constexpr int64_t any = INT64_MAX;
    constexpr OneLaneLimit limits64[] = {{1.1, {any, any, any, any}},
                                         {4.4, {500'000, 1'000'000, 2'000'000, any}},
                                         {11.0, {300'000, 500'000, 500'000, 700'000}},
                                         {27.0, {131'072, 200'000, 300'000, 300'000}},
                                         {HUGE_VAL, {131'072, 131'072, 131'072, 131'072}}};
    constexpr OneLaneLimit limits32[] = {{0.1, {1'000'000, any, any, any}},
                                         {1.1, {700'000, 2'000'000, 2'000'000, 2'000'000}},
                                         {4.4, {500'000, 1'000'000, 1'000'000, 1'000'000}},
                                         {11.0, {300'000, 700'000, 700'000, 700'000}},
                                         {27.0, {300'000, 500'000, 500'000, 700'000}},
                                         {HUGE_VAL, {300'000, 300'000, 500'000, 500'000}}};
    if (steps < 2) return false;
    const int column = steps < 3 ? 0 : steps < 5 ? 1 : steps < 10 ? 2 : 3;
    const OneLaneLimit *row = fp32 ? limits32 : limits64;
    while (!langevin && candidates > row->candidates) ++row;  // (on the Langevin branch: as without candidates)
    return n <= row->packs[column];
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

// Whether no pack of a run meets a candidate to speak of but on the Langevin
// branch.
inline bool takes_only_langevin(const mc_operating &op, double most_cand) {
    return op.langevin_on && most_cand <= 0.1;
}

// What a step of a query's packs costs at most, to order the queries of a
// launch by: the long ones go first, or the launch ends with their wavefronts
// alone on the chip.
inline double step_cost(const mc_operating &op, double most_cand, double dt_now) {
    return op.adaptive ? most_cand * (dt_now / op.dt) : most_cand;
}

// Lanes per pack for the queries of a server, over the packs of all of them; 0:
// the step kernel, one step a launch.  (Queries of unlike ions leave more of
// every launch's end idle than one population does, so that many steps a launch
// still pay where one_lane_pays has long said no.)
constexpr int64_t kQueryPacks64 = 300'000, kQueryPacks32 = 700'000;
inline int query_lanes(bool fp32, bool langevin, int64_t n) {
    if (n <= 0) return 0;
    const int g = lanes_for(fp32, langevin, n);
    return g > 1 || langevin || n <= (fp32 ? kQueryPacks32 : kQueryPacks64) ? g : 0;
}

}  // namespace mc
