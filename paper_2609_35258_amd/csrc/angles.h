// Angles of velocities and face normals as 32-bit integers, a whole turn 2^32
// (plain C++: the tests compile it alone).
#pragma once

namespace mlvs {

// A quarter turn, and the margin (2.4e-5 rad) by which a decision from angles
// must be clear of it: far above the rounding of an angle or of a float velocity
// (about 1e-7).
constexpr int ANG_QUARTER = 1 << 30, ANG_MARGIN = 1 << 14;

// A run of angles from a0 on to a1 and a face of outward normal n.  With span =
// ang_span(a0, a1) and t = ang_turn(a0, n), all of the run is within a quarter
// turn, less the margin, of n (velocities that all leave) where span <= ANG_HALF
// and t <= ANG_HALF - span, and of the opposite direction (all enter) where this
// holds with t + 2^31.  Unsigned: the differences wrap.
constexpr unsigned ANG_HALF = 2u * (ANG_QUARTER - ANG_MARGIN);
__attribute__((always_inline)) constexpr unsigned ang_span(int a0, int a1) { return (unsigned)a1 - (unsigned)a0; }
__attribute__((always_inline)) constexpr unsigned ang_turn(int a0, int n) {
    return (unsigned)a0 - (unsigned)n + ANG_HALF / 2;
}

}  // namespace mlvs
