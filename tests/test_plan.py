"""The rules by which the host plans its launches (mc_plan.hpp), compiled with
g++ and called over ranges of their arguments."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _check(tmp_path, name, body):
    """Compile and run `body`, the inside of a main that returns 0 where all is well."""
    src = tmp_path / (name + ".cpp")
    src.write_text('#include "mc_plan.hpp"\n#include <cstdio>\n#include <random>\n'
                   "#define CHECK(x) do { if (!(x)) { std::printf(\"%d: %s\\n\", __LINE__, #x); return 1; } } while (0)\n"
                   "using namespace mc;\nint main() {\n" + body + "\nreturn 0; }\n")
    exe = tmp_path / name
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-Xlinker", "--no-as-needed",
                    "-fsanitize=address,undefined", "-I" + os.path.join(ROOT, "paper_2609_31258_amd", "csrc"), str(src),
                    "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout + run.stderr


def test_a_run_of_adaptive_steps_always_takes_one(tmp_path):
    """The pause lies after the run's start for every next update that is not yet due, from times of a few steps
    to times beside which the tolerance is half their last bit."""
    _check(tmp_path, "pause", r'''
    std::mt19937_64 rng(3);
    for (int k = 0; k < 200000; ++k) {
        const double dt = std::ldexp(1.0, -31 - (int)(rng() % 4)), tol = k % 2 ? 1e-6 * dt : std::ldexp(dt, -20);
        const double t0 = std::ldexp(1.0 + (double)(rng() % 1024) / 1024, (int)(rng() % 36) - 31);
        double t_pic = t0 + (double)(rng() % 4) * tol;
        for (int j = 0; j < 3; ++j, t_pic = std::nextafter(t_pic, HUGE_VAL)) {
            if (t_pic <= t0 + tol) continue;  // due: the update comes first
            CHECK(pause_time(t0, t_pic, tol) > t0);
            CHECK(pause_time(t0, t_pic, tol) <= t_pic);
        }
    }
    CHECK(pause_time(0.0, 5e-9, 5e-16) == 5e-9 - 5e-16);''')


def test_adaptive_steps_enqueued_beyond_an_update_stay_few(tmp_path):
    """Runs of steps at a limit, updates every ten largest steps: a step more than are taken in each run, and the
    runs no more than two an update, whatever is left for the step that an update cuts short."""
    _check(tmp_path, "pace", r'''
    std::mt19937_64 rng(5);
    for (int trial = 0; trial < 400; ++trial) {
        const double dt = 5e-9, period = 10 * dt, tol = 1e-6 * dt;
        // limits from dt/60 up to dt; every other one with a tiny remainder
        double limit = dt / (1.0 + (double)(rng() % 59000) / 1000);
        if (trial % 2) limit = period / (std::floor(period / limit) + std::ldexp(1.0, -4 - (int)(rng() % 12)));
        StepPace pace;
        double t = 0.0, next = period;
        long enqueued = 0, taken = 0, runs = 0;
        const int updates = 100;
        for (int u = 0; u < updates; ) {
            while (next <= t + tol) { next += period; ++u; }
            const double t0 = t, pause = pause_time(t0, next, tol);
            const long k = pace.steps_for(next - tol - t0, dt);
            CHECK(k >= 1 && k <= 1024);
            long j = 0;
            double d = 0.0;
            for (; j < k && t < pause; ++j) {
                d = std::min(std::min(dt, limit * (0.98 + (double)(rng() % 400) / 10000)), next - t);
                t += d;
            }
            pace.took(j, t - t0, d, t >= pause);
            enqueued += k;
            taken += j;
            ++runs;
        }
        CHECK(taken <= enqueued);
        CHECK(runs <= 2 * updates + 10);
        CHECK(enqueued <= taken + taken / 20 + 2 * runs);
    }
    StepPace fresh;
    CHECK(fresh.steps_for(5e-9, 5e-9) == 1 && fresh.steps_for(51e-9, 5e-9) == 11 && fresh.steps_for(-1e-12, 5e-9) == 1);
    fresh.took(1, 1e-15, 1e-15, true);  // nothing but a step cut short
    CHECK(fresh.steps_for(50e-9, 5e-9) == 10);''')


def test_densest_gas_of_each_row(tmp_path):
    """Largest p/T of a row over its nodes with gas, from division; rows of vacuum and of zero temperature."""
    _check(tmp_path, "gas", r'''
    std::mt19937_64 rng(9);
    std::uniform_real_distribution<double> u(0.0, 1.0);
    const int nr = 37, nz = 50;
    std::vector<double> p(nr * nz), t(nr * nz);
    for (int k = 0; k < nr * nz; ++k) {
        p[k] = k / nr == 3 ? 0.0 : std::exp(12 * u(rng));
        t[k] = k / nr == 5 || u(rng) < 0.1 ? 0.0 : 20 + 400 * u(rng);
    }
    GasRows g;
    g.scan(p.data(), t.data(), nr, nz);
    double t_max = 0;
    for (int j = 0; j < nz; ++j) {
        double most = 0;
        for (int k = j * nr; k < (j + 1) * nr; ++k) {
            if (t[k] > 0) most = std::max(most, p[k] / t[k]);
            t_max = std::max(t_max, t[k]);
        }
        CHECK(std::fabs(g.densest[j] - most) <= 1e-14 * most);
    }
    CHECK(g.t_max == t_max && g.p_max == *std::max_element(p.begin(), p.end()));
    CHECK( g.densest[3] == 0.0 && g.densest[5] == 0.0);''')


def test_which_populations_take_the_stretch_kernel(tmp_path):
    """Large populations take it only where no pack, or next to none, runs the collision loop in dense gas: not for
    the Langevin branch being on, with a window or a switch that leaves dense gas to the explicit branch."""
    _check(tmp_path, "lanes", r'''
    // 100 rows 50 um apart, 1e5 Pa in the first 40, 100 Pa from there on; about 49 candidates a step in the dense gas
    const int nr = 4, nz = 100;
    const double dz = 5e-5;
    std::vector<double> p(nr * nz), t(nr * nz, 300.0);
    for (int k = 0; k < nr * nz; ++k) p[k] = k / nr < 40 ? 1e5 : 100.0;
    GasRows g;
    g.scan(p.data(), t.data(), nr, nz);
    mc_operating op{};
    op.dt = 0.5e-9;
    op.collisions_on = 1;
    op.lv_switch = 0.05;
    const double ccs = 9.28e-18;
    const auto most = [&] { return densest_explicit(g, dz, op, ccs, 28.0134); };
    const double dense = most();
    CHECK(dense > 40.0 && dense < 70.0);
    op.langevin_on = 1;                                   // no window: explicit only below the switch
    CHECK(most() == 0.05);
    op.lv_switch = 20.0;
    CHECK(most() == 20.0);
    op.lv_switch = 1e9;
    CHECK(most() == dense);
    op.lv_switch = 0.05;
    op.lv_z_hi = 1e-3;                                    // dense gas beyond the window
    CHECK(most() == dense);
    op.lv_z_hi = 39 * dz + 1e-9;                          // rows of dense gas share cells with the end of the window
    CHECK(most() == dense);
    op.lv_z_hi = 42 * dz;                                 // the window holds the dense gas
    CHECK(std::fabs(most() - dense * 1e-3) < 1e-12);
    op.lv_z_lo = 10 * dz;                                 // dense gas before the window
    CHECK(most() == dense);
    op.lv_z_lo = 0.0, op.lv_z_hi = 1.0;                   // over the whole grid
    CHECK(most() == 0.05);
    op.collisions_on = 0;
    CHECK(most() == 0.0);
    CHECK(densest_explicit(GasRows{}, dz, op, ccs, 28.0134) == 0.0);

    for (int fp32 = 0; fp32 < 2; ++fp32)
        for (int langevin = 0; langevin < 2; ++langevin) {
            const int64_t lanes = fp32 && !langevin ? 131072 : 65536;
            for (int g = 16; g > 1; g /= 2) {
                CHECK(lanes_for(fp32, langevin, lanes / g) == g);
                CHECK(lanes_for(fp32, langevin, lanes / g + 1) == g / 2);
            }
            CHECK(lanes_for(fp32, langevin, 1) == 16 && lanes_for(fp32, langevin, INT64_C(1) << 40) == 1);
            CHECK(query_lanes(fp32, langevin, 0) == 0);
            const int64_t edge = fp32 ? kQueryPacks32 : kQueryPacks64;
            CHECK(query_lanes(fp32, langevin, edge) == 1 && query_lanes(fp32, langevin, edge + 1) == langevin);
        }

    LangevinShare s;
    CHECK(!mostly_langevin(s.at(0), true));
    s.read(10, 995, 1000);
    CHECK(mostly_langevin(s.at(10), false) && mostly_langevin(s.at(1010), false) && !mostly_langevin(s.at(1011), true));
    s.read(20, 1095, 2000);                               // 100 of the next 1000
    CHECK(s.at(20) == 0.1 && !mostly_langevin(s.at(20), true));
    s.read(30, 1095, 2000);                               // no steps since: what is known stays
    CHECK(s.at(1020) == 0.1 && s.at(1021) == -1.0);
    s.forget(false);
    CHECK(s.at(20) == -1.0);
    s.read(40, 2095, 3000);
    CHECK(s.at(40) == 1.0);
    s.forget(true);                                       // a state from elsewhere: its counters say nothing
    s.read(5, 7000, 7000);
    CHECK(s.at(5) == -1.0);
    s.read(15, 7950, 8000);
    CHECK(s.at(15) == 0.95 && mostly_langevin(s.at(15), true) && !mostly_langevin(s.at(15), false));''')


def test_queries_are_ordered_by_the_collisions_of_their_packs(tmp_path):
    """The branch being on does not make a query cheap: where its window leaves dense gas to the explicit branch it
    costs what an explicit one does."""
    _check(tmp_path, "cost", r'''
    const int nr = 3, nz = 60;
    std::vector<double> p(nr * nz, 1e5), t(nr * nz, 300.0);
    GasRows g;
    g.scan(p.data(), t.data(), nr, nz);
    mc_operating op{};
    op.dt = 0.5e-9;
    op.collisions_on = 1;
    op.lv_switch = 0.05;
    const auto cost = [&](double ccs, double dt_now = 0.0) {
        return step_cost(op, densest_explicit(g, 5e-5, op, ccs, 28.0134), dt_now);
    };
    const double small = cost(1e-18), large = cost(5e-18);
    CHECK(small > 0.0 && std::fabs(large - 5 * small) < 1e-9 * large);
    op.langevin_on = 1;
    CHECK(cost(5e-18) < small && takes_only_langevin(op, densest_explicit(g, 5e-5, op, 5e-18, 28.0134)));
    op.lv_z_hi = 1e-3;
    CHECK(cost(5e-18) == large && !takes_only_langevin(op, densest_explicit(g, 5e-5, op, 5e-18, 28.0134)));
    op.langevin_on = 0;
    op.adaptive = 1;
    CHECK(std::fabs(cost(5e-18, 0.1 * op.dt) - 0.1 * large) < 1e-9 * large);
    op.collisions_on = 0;
    CHECK(cost(5e-18, op.dt) == 0.0);''')


def test_single_steps_take_lanes_only_with_candidates_to_share(tmp_path):
    _check(tmp_path, "single", r'''
    for (int fp32 = 0; fp32 < 2; ++fp32)
        for (int lanes = 1; lanes <= 16; lanes *= 2) {
            CHECK(!lanes_pay_in_one_step(fp32, lanes, 0.0) && !lanes_pay_in_one_step(fp32, lanes, 0.05));
            CHECK(lanes_pay_in_one_step(fp32, lanes, 50.0) == (lanes > 1));
        }
    CHECK(lanes_pay_in_one_step(false, 2, 1.0) && !lanes_pay_in_one_step(true, 16, 1.0));
    CHECK(lanes_pay_in_one_step(true, 4, 4.0) && !lanes_pay_in_one_step(true, 2, 4.0));''')


def test_one_lane_per_pack_by_candidates_and_steps(tmp_path):
    """More packs, more candidates or fewer steps never bring the stretch kernel back; a million packs in dense gas
    are the step kernel's, a million in next to none are not."""
    _check(tmp_path, "one_lane", r'''
    const double cand[] = {0.0, 0.05, 0.06, 0.9, 1.0, 1.1, 4.0, 5.0, 10.0, 11.0, 25.0, 26.0, 1e4, HUGE_VAL};
    const int64_t packs[] = {70'000, 131'072, 131'073, 200'000, 300'001, 500'000, 700'001, 1'000'000, 2'000'001, 1 << 28};
    const int64_t steps[] = {2, 3, 4, 5, 9, 10, 32};
    for (int fp32 = 0; fp32 < 2; ++fp32) {
        for (double c : cand)
            for (int64_t n : packs) {
                CHECK(!one_lane_pays(fp32, false, c, n, 1) && !one_lane_pays(fp32, true, c, n, 1));
                bool before = false;
                for (int64_t k : steps) {
                    const bool pays = one_lane_pays(fp32, false, c, n, k);
                    CHECK(pays || !before);
                    before = pays;
                    if (pays)
                        for (double c2 : cand)
                            for (int64_t n2 : packs)
                                if (c2 <= c && n2 <= n) CHECK(one_lane_pays(fp32, false, c2, n2, k));
                    CHECK(one_lane_pays(fp32, true, c, n, k) == one_lane_pays(fp32, false, 0.0, n, k));
                }
            }
        CHECK(one_lane_pays(fp32, false, 0.05, 1'000'000, 10) && !one_lane_pays(fp32, false, 49.0, 1'000'000, 10));
        CHECK(!one_lane_pays(fp32, false, 10.0, 1'000'000, 32) && one_lane_pays(fp32, false, 120.0, 100'000, 2));
    }''')
