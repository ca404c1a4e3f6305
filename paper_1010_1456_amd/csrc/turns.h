// Sine and cosine of an angle in turns, for the set-up and far-field kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "fft_core.h"

namespace aim {

constexpr double signed_inv_factorial(int n) {
  double f = 1.0;
  for (int m = 2; m <= n; ++m) f /= m;
  return n / 2 % 2 ? -f : f;
}
// Taylor coefficients of sine (x^21 .. x) and cosine (x^20 .. 1), highest power
// first. Kernels keep them in constant memory and read them with scalar loads.
struct TurnsConst {
  double s[11], c[11];
  constexpr TurnsConst() : s{}, c{} {
    for (int i = 0; i < 11; ++i) {
      s[i] = signed_inv_factorial(21 - 2 * i);
      c[i] = signed_inv_factorial(20 - 2 * i);
    }
  }
};
using TurnsPtr = const __attribute__((address_space(4))) TurnsConst *;

// sin and cos of 2 pi t (|t| < 2^50): t is reduced by half turns (exactly), the
// sign taken from the parity of their number; on |x| <= pi / 2 the first terms
// left out are below 2e-17. 26 FP64 instructions and no branch, where the
// library's sincos carries a path for huge arguments.
__device__ __forceinline__ void sincos_turns(TurnsPtr k, double t, double &sn, double &cs) {
  constexpr double kRound = 6755399441055744.0;  // 1.5 * 2^52: rounds to an integer
  const double z = fma(2.0, t, kRound);
  const double x = (2.0 * 3.14159265358979323846) * fma(-0.5, z - kRound, t);
  const double x2 = x * x;
  double s = k->s[0], c = k->c[0];
  fftc::static_for<10>([&](auto i_) AIM_AI {
    constexpr int i = decltype(i_)::value + 1;
    s = fma(s, x2, k->s[i]);
    c = fma(c, x2, k->c[i]);
  });
  s *= x;
  const int flip = (int)((unsigned)__double2loint(z) << 31);
  sn = __hiloint2double(__double2hiint(s) ^ flip, __double2loint(s));
  cs = __hiloint2double(__double2hiint(c) ^ flip, __double2loint(c));
}

}  // namespace aim
