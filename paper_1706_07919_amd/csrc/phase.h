// Sine and cosine of the float64 phases of the operator.  For |x| < 2^20
// (k r and k n.d of any surface here) x = n pi/2 + y with a three-part
// Cody-Waite reduction (pi/2 split into two 33-bit parts, exact in n * part,
// and a remainder) and |y| <= pi/4; sin y and cos y by their Taylor series to
// y^15 and y^16 (the first omitted terms are below 7e-17 and 3e-18 on
// [-pi/4, pi/4]); the quadrant n mod 4 permutes and signs them.  Larger
// arguments take the library sincos (phase_sincos), or are the caller's to
// route elsewhere (phase_sincos_near, branch-free, for loops whose callers
// check the range of their arguments up front).
#pragma once

#include <hip/hip_runtime.h>

namespace bem {

constexpr double kPhaseNear = 1048576.0;   // 2^20

// Valid for |x| < kPhaseNear only.
__device__ inline void phase_sincos_near(double x, double* s, double* c) {
  const double n = rint(x * 0.6366197723675814);   // 2/pi
  double y = fma(-n, 1.5707963267341256, x);
  y = fma(-n, 6.077100506303966e-11, y);
  y = fma(-n, 2.0222662487959506e-21, y);
  const double y2 = y * y;
  double ps = -7.647163731819816e-13;   // -1/15!
  ps = fma(ps, y2, 1.6059043836821613e-10);   // +1/13!
  ps = fma(ps, y2, -2.505210838544172e-08);   // -1/11!
  ps = fma(ps, y2, 2.7557319223985893e-06);   // +1/9!
  ps = fma(ps, y2, -0.0001984126984126984);   // -1/7!
  ps = fma(ps, y2, 0.008333333333333333);   // +1/5!
  ps = fma(ps, y2, -0.16666666666666666);   // -1/3!
  const double sy = fma(ps * y2, y, y);
  double pc = 4.779477332387385e-14;   // 1/16!
  pc = fma(pc, y2, -1.1470745597729725e-11);   // -1/14!
  pc = fma(pc, y2, 2.08767569878681e-09);   // +1/12!
  pc = fma(pc, y2, -2.755731922398589e-07);   // -1/10!
  pc = fma(pc, y2, 2.48015873015873e-05);   // +1/8!
  pc = fma(pc, y2, -0.001388888888888889);   // -1/6!
  pc = fma(pc, y2, 0.041666666666666664);   // +1/4!
  pc = fma(pc, y2, -0.5);
  const double cy = fma(pc, y2, 1.0);
  const int q = (int)n & 3;
  const double sa = (q & 1) ? cy : sy, ca = (q & 1) ? sy : cy;
  *s = (q & 2) ? -sa : sa;
  *c = ((q + 1) & 2) ? -ca : ca;
}

// e^{i k t} of the exact product k t (|k t| < kPhaseNear): the rounded product's,
// turned by what the rounding took off.
__device__ inline double2 unit_phase(double k, double t) {
  const double p = k * t, lo = fma(k, t, -p);
  double s, c;
  phase_sincos_near(p, &s, &c);
  return make_double2(fma(-lo, s, c), fma(lo, c, s));
}
__device__ inline double2 rotate(double2 a, double2 b) {   // a b
  return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}
__device__ inline double2 rotate_back(double2 a, double2 b) {   // a conj(b)
  return make_double2(fma(a.x, b.x, a.y * b.y), fma(a.y, b.x, -a.x * b.y));
}
__device__ inline double2 turn(double2 a, double e) {   // a e^{i e}, e tiny
  return make_double2(fma(-e, a.y, a.x), fma(e, a.x, a.y));
}

// A workgroup's chunk of KC wavenumbers on an even grid, k[q] = k0 + q dk up to their
// roundings, along which phases advance by rotation: step[q] = (k[q] - k[q - 1]) - dk,
// which a phase k t takes as a further turn by step[q] t.  (Without it the wavenumbers'
// own roundings, times t, are an error of every rotated phase: float64 fields at
// 32 wavenumbers were 1.2 to 1.5 times further off than with a sincos each.)
template <int KC>
struct EvenChunk {
  double k[KC], step[KC], dk, kmax;
  bool even;
  // Phases start from the middle wavenumber: a rotation's rounding counts once per step
  // taken, so the ends are up to KC / 2 steps off instead of KC - 1.  The i-th value
  // is wavenumber order(i): up from the middle, then, from it again, down.
  static constexpr int kMid = (KC - 1) / 2, kUp = KC - kMid;
  static constexpr int order(int i) { return i < kUp ? kMid + i : KC - 1 - i; }
  // phase of wavenumber order(i), i > 0, from that of the one before it (from the
  // middle one's for i == kUp), d = e^{i dk t}
  __device__ inline double2 advance(int i, double2 e, double2 d, double t) const {
    const int q = order(i);
    return i < kUp ? turn(rotate(e, d), step[q] * t) : turn(rotate_back(e, d), -step[q + 1] * t);
  }
  // wavenumbers kv[0 .. n - 1], 1 <= n <= KC, continued evenly past n
  __device__ inline void load(const double* kv, int n) {
    const double k0 = kv[0];
    dk = n > 1 ? (kv[n - 1] - k0) / (n - 1) : 0.0;
    even = true;
    kmax = 0.0;
    double last = 0.0;   // k[q] - (k0 + q dk)
#pragma unroll
    for (int q = 0; q < KC; ++q) {
      const double v = q < n ? kv[q] : fma((double)q, dk, k0);
      // v - k0 = d + e exactly
      const double d = v - k0, bv = d - v, e = (v - (d - bv)) + (-k0 - bv);
      const double off = fma(-(double)q, dk, d) + e;
      k[q] = v;
      step[q] = q < n ? off - last : 0.0;
      last = off;
      kmax = fmax(kmax, fabs(v));
      if (!(fabs(off) <= 1e-15 * fabs(v))) even = false;
    }
  }
};

// r and 1/r from r^2 > 0 without the library's square root and division: the
// float64 reciprocal square root estimate (any float64 r^2, where the float32 one
// ends at distances of 1e-19 and 1e19), two Newton steps, and a correction step for
// each, which keep them to the rounding of a square root and a division.
__device__ inline void dist_and_inverse64(double r2, double& r, double& rinv) {
  double y = __builtin_amdgcn_rsq(r2);
  y *= fma(-0.5 * r2, y * y, 1.5);
  y *= fma(-0.5 * r2, y * y, 1.5);
  const double r1 = r2 * y;
  r = fma(fma(-r1, r1, r2), 0.5 * y, r1);
  rinv = fma(y, fma(-r, y, 1.0), y);
}

__device__ inline void phase_sincos(double x, double* s, double* c) {
  if (!(fabs(x) < kPhaseNear)) {
    sincos(x, s, c);
    return;
  }
  phase_sincos_near(x, s, c);
}

}  // namespace bem
