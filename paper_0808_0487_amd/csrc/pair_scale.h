// Scales of the paired variance columns (p odd).  Host code, no device
// dependence.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <vector>

namespace fdwt {

// The variance columns U_1..U_s, Q_1..Q_{s-1} (Section 4) are transformed two
// to a complex column; ix[i], i < s, is the exponent of the power of two that
// multiplies the second column of pair i before the transform (and divides its
// spectrum after it), so that both columns have about the same norm.
// The rounding errors of a transform follow the norm of what it transforms,
// half of them in the real part: with equal norms each column's spectrum is
// about as far off as when it is transformed alone, and the sums over h, which
// weigh h and (-)h alike, exactly as far in the mean (alone, the errors at h
// and (-)h are the same; in a pair they are independent).  Against extended
// precision, 12 kernels of p = 3, 5, 7, alone / paired: spectra, relative to
// their norm, rms 2.2e-16 / 2.3e-16, largest 3.7e-16 / 4.1e-16; sums rms
// 2.10e-15 / 2.10e-15.  (With the values at x = 0 made equal in place of the
// norms, the largest spectrum error was 1.3e-15: Q_j is far more peaked than
// Q_{j-1} and U_s.)
// The norms: the mean square over [0, 1)^s, from that of a_j = gamma_j^2 R'(x_j)
// (the a_j are independent with mean 0, up to p^-m), times p^m points, plus the
// square at x = 0, the maximum, which counts for much of the norm on few points.
// rp: R' by the index of the first non-zero digit, rp[m] that of x = 0.
// In long double: products of up to 64 squares leave the range of double where
// the columns themselves do not.
inline void pair_exponents(int p, int m, int s, const double* gamma, const double* rp, int32_t* ix) {
  using ld = long double;
  ld q = 0.0L, pt = 1.0L;  // mean of R'^2: index t has share (p - 1) p^-(t + 1), x = 0 has p^-m
  for (int t = 0; t < m; ++t) {
    pt /= p;
    q += (p - 1) * pt * (ld)rp[t] * rp[t];
  }
  q += pt * (ld)rp[m] * rp[m];
  const ld N = 1.0L / pt;
  std::vector<ld> sq(2 * s), e(s + 1, 0.0L), f(s + 1, 0.0L);  // squared norms; e_j of the values at 0 and of the mean squares
  e[0] = f[0] = 1.0L;
  ld u = 0.0L, v = 0.0L;
  for (int j = 0; j < s; ++j) {
    const ld g2 = (ld)gamma[j] * gamma[j], r = g2 * rp[m], w = g2 * g2 * q;
    u += r + u * r;
    v += w + v * w;
    sq[j] = N * v + u * u;
    for (int i = j + 1; i >= 1; --i) {
      e[i] += r * e[i - 1];
      f[i] += w * f[i - 1];
    }
  }
  for (int j = 1; j <= s; ++j) sq[s + j - 1] = N * f[j] + e[j] * e[j];
  for (int i = 0; i < s; ++i) {
    const ld a = sq[2 * i], b = sq[2 * i + 1];
    const bool ok = a > 0.0L && b > 0.0L && std::isfinite(a) && std::isfinite(b);
    const long x = ok ? std::lround(0.5L * (std::log2(a) - std::log2(b))) : 0;
    ix[i] = (int32_t)std::max(-1000L, std::min(1000L, x));
  }
}

}  // namespace fdwt
