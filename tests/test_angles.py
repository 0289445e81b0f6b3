"""The angle classes that decide which faces a run of velocities leaves or enters
(csrc/angles.h), compiled alone: as constant expressions, where an overflow of a
signed difference does not compile, at both ends of the range (a run that crosses
the wrap, the whole turn that stands for the point at rest), and against the
angles themselves in double over seeded runs and normals."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "angles.h"
#include <climits>
#include <cmath>
#include <cstdio>
#include <random>
using namespace mlvs;
constexpr bool within(unsigned span, unsigned t) { return span <= ANG_HALF && t <= ANG_HALF - span; }
constexpr bool out(int a0, int a1, int n) { return within(ang_span(a0, a1), ang_turn(a0, n)); }
constexpr bool in(int a0, int a1, int n) { return within(ang_span(a0, a1), ang_turn(a0, n) + 0x80000000u); }
// the point at rest: the whole turn is within no quarter of any normal
static_assert(!out(INT_MIN, INT_MAX, 0) && !in(INT_MIN, INT_MAX, 0), "");
static_assert(!out(INT_MIN, INT_MAX, INT_MIN) && !in(INT_MIN, INT_MAX, INT_MAX), "");
// normals and runs at the two ends of the range
static_assert(out(INT_MIN, INT_MIN + 9, INT_MAX) && !in(INT_MIN, INT_MIN + 9, INT_MAX), "");
static_assert(out(INT_MAX - 9, INT_MAX, INT_MIN) && in(INT_MAX - 9, INT_MAX, 0), "");
static_assert(in(INT_MIN, INT_MIN, 0) && out(-5, 5, 0) && in(-5, 5, INT_MIN), "");
// a right angle is neither, and the margin counts on both sides
static_assert(!out(ANG_QUARTER, ANG_QUARTER, 0) && !in(ANG_QUARTER, ANG_QUARTER, 0), "");
static_assert(!out(0, ANG_QUARTER - ANG_MARGIN + 1, 0) && out(0, ANG_QUARTER - ANG_MARGIN - 1, 0), "");

int main() {
    std::mt19937_64 rng(7);
    const double unit = 3.14159265358979323846 / 2147483648.0;
    long bad = 0, n_out = 0, n_in = 0;
    for (int k = 0; k < 200000; ++k) {
        const int n = (int)(unsigned)rng(), a = (int)(unsigned)rng();
        const long long room = (long long)INT_MAX - a;
        const int b = a + (int)std::llround(room * std::pow(std::uniform_real_distribution<>()(rng), 8));
        const bool o = out(a, b, n), i = in(a, b, n);
        n_out += o; n_in += i;
        if (o && i) ++bad;
        for (int t = 0; t <= 16; ++t) {       // xi . n over the run, ends included
            const double ang = unit * (a + (double)((long long)b - a) * t / 16);
            const double dn = std::cos(ang - unit * n);
            if ((o && !(dn > 0)) || (i && !(dn < 0))) ++bad;
        }
    }
    std::printf("%ld wrong, %ld out, %ld in\n", bad, n_out, n_in);
    return bad != 0 || n_out < 10000 || n_in < 10000;
}
"""


def test_angle_classes(tmp_path):
    src, exe = tmp_path / "angles.cpp", tmp_path / "angles"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2609_35258_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
