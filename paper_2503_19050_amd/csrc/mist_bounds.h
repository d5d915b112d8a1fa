// The search's bound on how Algorithm 1's time grows with the host streams: the slopes, formed on the host
// per hardware sample, and what the kernel makes of them.
#pragma once

#include <algorithm>
#include <cmath>
#include <limits>

namespace mist {

// Least directional derivative of Algorithm 1's time along (0, 0, 1, 1), both host streams growing
// alike.  For a given order in which the streams finish, the time is linear in the stream times:
// each phase lasts the scaled time of the stream that finishes, and every other member's standalone
// time falls by that length over its factor.  The time is continuous where orders change (a phase of
// length 0), so along a segment it never grows by less than the least slope over the orders it meets:
// all (first = 0), those that start with GPU-GPU (1), or with GPU-GPU and then compute (2).
inline double host_slope(const double phi[16][4], int first) {
  int ord[4] = {0, 1, 2, 3};
  double least = std::numeric_limits<double>::infinity();
  do {
    if ((first >= 1 && ord[0] != 1) || (first >= 2 && ord[1] != 0)) continue;
    double x[4] = {0.0, 0.0, 1.0, 1.0}, T = 0.0;
    int mask = 15;
    for (int i = 0; i < 3; ++i) {
      const double ov = x[ord[i]] * phi[mask][ord[i]];
      T += ov;
      for (int j = 0; j < 4; ++j)
        if (mask >> j & 1) x[j] -= ov / phi[mask][j];
      mask &= ~(1 << ord[i]);
    }
    least = std::min(least, T + x[ord[3]]);
  } while (std::next_permutation(ord, ord + 4));
  return least - 1e-9 * (1.0 + std::fabs(least));
}

// Factors up to which the slopes bound the rounded time as well.  A round leaves a relative 2^-53 of a
// stream's time as noise, and each of the two rounds after it may scale that by a factor: with factors up
// to 2^6 the noise stays below 2^-38 of the time, far below the 2^-30 by which every bound is lowered; at
// 2^16 it reaches 2^-21, above it.
constexpr double kSlopeFactors = 0x1p6;

// The slopes of one hardware sample; -inf (no bound: the kernel's maxima drop what it makes of them) with
// larger factors.
inline void host_slopes(const double phi[16][4], double slope[3]) {
  double most = 1.0;
  for (int mask = 3; mask < 16; ++mask)
    for (int j = 0; j < 4; ++j)
      if ((mask & (mask - 1)) && (mask >> j & 1)) most = std::max(most, phi[mask][j]);
  for (int f = 0; f < 3; ++f)
    slope[f] = most <= kSlopeFactors ? host_slope(phi, f) : -std::numeric_limits<double>::infinity();
}

// A lower bound of the time with both host streams longer by any length x >= 0, from the time T at x = 0,
// the slope sl and the longer host stream h: max(T + sl x, h + x), whose least value lies at x = 0 or, with a
// falling slope, where the two meet.
constexpr double any_length(double T, double sl, double h) {
  const double neg = sl < 0.0 ? sl : 0.0;
  return T + neg * (1.0 / (1.0 - neg)) * (T - h);
}

}  // namespace mist
