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
