// Bounds of the distance screens, from the cutoff and the cell side (host code).
// A screen may accept a pair beyond the cutoff, which the exact test of the walk
// then rejects; it must never drop one within it.
#pragma once

#include <cmath>

namespace mdlj {

// Bound on r^2 of the 32-bit screen, in the frame's units: frame coordinates lie
// within [-s, 2s) per axis, so |x|^2 <= 12 s^2; the FP32 dot-product form of r^2
// errs by a few ulp of that. 2^-17 * 12 s^2 leaves a wide margin, so the screen
// never drops a pair that the exact test accepts.
inline float screen_bound(double rc, double s) { return static_cast<float>(rc * rc + std::ldexp(12.0 * s * s, -17)); }

// Bound of the 16-bit screen, in units of the cell side s: (r / s)^2 plus a
// margin above what rounding to 16 bits can add to a pair with r_ij <= r. Home
// coordinates v lie in [-d, 1 + d] with d = (s - r_c) / 2s (atoms may leave their
// cell by half the side's margin between rebuilds), so that r_c / s = 1 - 2 d and a
// partner within r_c has |u| = |x_j - 1/2| <= 3/2 - d per axis and |x_j| <= sqrt(3)
// (1 + d) + 1 - 2 d < sqrt(8). What is rounded is 2 v (below 4: by 2^-10 at most),
// u (below 2: 2^-11) and |x_j|^2 (below 8: 2^-9):
//   sum |u| err(2 v) + sum |2 v| err(u) + err(|x_j|^2)
//   <= 3 (3/2 - d) 2^-10 + 3 (2 + 2 d) 2^-11 + 2^-9 = 9.5 x 2^-10 = 0.00928
// at any d. The same holds for a list radius r up to s right after a rebuild
// (d = 0). The rest of the margin covers the products of two roundings (1.5e-6)
// and what 32 bits add (scaling, |x|^2, C, accumulation: within 2e-5). The worst
// pairs that a search finds need 0.0069.
inline float screen16_bound(double r, double s) { return static_cast<float>(r * r / (s * s) + 0.0100); }

}  // namespace mdlj
