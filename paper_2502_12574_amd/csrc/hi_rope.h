// The rotary angles of consecutive positions.  The kernels that need a run of them (the table of the 256-row projection tile, the
// 128-row tile) take them from here, so that every form rotates by the same bits; the host replays it in a test.
#pragma once
#include <math.h>
#include <stdint.h>
#if defined(__HIPCC__)
#define HI_ROPE_HD __host__ __device__ __forceinline__
#else
#define HI_ROPE_HD inline
#endif

namespace hi {

constexpr int kRopeRun = 32;     // positions of a run: the first one, then 31 steps

// (cos, sin) of position p times w, p = first .. first + 31, in double precision: at a million tokens the angle of the fastest pair is
// a million radians, beyond what fp32 can reduce.  Two sincos, then rotations by w.  What is wanted is the angle p * w as rounded, which
// is half an ulp of the angle off (6e-11 at a million): the rotations go by the product itself, and each result turns back by what its
// rounding left out, to first order.  That leaves some 1e-15 (angles up to 2^33): of 1.6 million fp32 values at positions from 0 to
// 2^31 none or one differ from those of a sincos per position; steps between rounded angles miss 5e-5 of them at 131 thousand
// positions, 3e-4 at a million, 1e-3 at four.  Every rounding is written out, so that no compiler fuses here what it does not there.
struct RopeRun {
  double w, p, c, s, c1, s1;
  HI_ROPE_HD RopeRun(int64_t first, double frequency) : w(frequency), p((double)first) {
#if defined(__clang__)
#pragma clang fp contract(off)
#endif
    const double angle = p * w, rest = __builtin_fma(p, w, -angle);
    double s0, c0;
    sincos(angle, &s0, &c0);
    sincos(w, &s1, &c1);
    c = __builtin_fma(-s0, rest, c0);
    s = __builtin_fma(c0, rest, s0);
  }
  // the next position's
  HI_ROPE_HD void next(float& cos_out, float& sin_out) {
#if defined(__clang__)
#pragma clang fp contract(off)
#endif
    const double angle = p * w, rest = __builtin_fma(p, w, -angle);
    cos_out = (float)__builtin_fma(s, rest, c);
    sin_out = (float)__builtin_fma(-c, rest, s);
    const double cn = __builtin_fma(c, c1, -(s * s1));
    s = __builtin_fma(s, c1, c * s1);
    c = cn;
    p += 1.0;
  }
};

}  // namespace hi
