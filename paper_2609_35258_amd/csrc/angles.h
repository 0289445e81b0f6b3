// Angles of velocities and face normals as 32-bit integers, a whole turn 2^32
// (plain C++: the tests compile it alone).
#pragma once

namespace mlvs {

// A quarter turn, and the margin (2.4e-5 rad) by which a decision from angles
// must be clear of it: far above the rounding of an angle or of a float velocity
// (about 1e-7).
constexpr int ANG_QUARTER = 1 << 30, ANG_MARGIN = 1 << 14;

// Whether every angle of the run from a0 on to a1 (counted upwards, across the
// wrap as well) is within a quarter turn, less the margin, of the direction n
// (of the opposite one for `in`).  Unsigned throughout: the differences wrap.
constexpr bool ang_within(unsigned a0, unsigned a1, unsigned n) {
    constexpr unsigned W = 2u * (unsigned)(ANG_QUARTER - ANG_MARGIN);
    const unsigned span = a1 - a0;
    return span <= W && a0 - n + W / 2 <= W - span;
}
// ... velocities that all leave through a face of outward normal n, or all enter.
constexpr bool ang_out(int a0, int a1, int n) { return ang_within((unsigned)a0, (unsigned)a1, (unsigned)n); }
constexpr bool ang_in(int a0, int a1, int n) {
    return ang_within((unsigned)a0, (unsigned)a1, (unsigned)n + 0x80000000u);
}

}  // namespace mlvs
