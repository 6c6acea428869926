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
