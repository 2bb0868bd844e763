// shp_nodes.h -- how many frequencies determine a shapelet's envelope over a
// band, free of any device code.
//
// Along a baseline the envelope is a function of frequency alone: the line
// (a, b) = nu (a_m, b_m) / c through the origin of the Hermite plane.  Rotated
// onto that line, a sum over n1 + n2 <= N is a combination of the Hermite
// functions phi_n(x), n <= N, of x = nu |(a_m, b_m)| / c (the functions of one
// order n1 + n2 are rotated among themselves).  phi_n oscillates at
// sqrt(2 n + 1 - x^2) where it is not small, so over a band of relative width
// its phase advances by at most x sqrt(2 n + 1 - x^2) <= n + 1/2 per unit of
// ln nu, whatever the baseline's length: the envelope is entire, of bounded
// bandwidth over the band, and a Chebyshev interpolation in nu converges as
// (w/2)^M / M! with w = (N + 1/2) x the band's half-width over its lower end.
#pragma once

#include <algorithm>
#include <cmath>

namespace vp {

constexpr int kNodesMax = 64;  // nodes a plan may have
// Absolute errors of phi_n allowed to the interpolation: a hundredth of the
// mixed path's own (its products carry FP32 sums), and below the rounding of
// the FP64 recurrence.
constexpr double kNodesTolMixed = 1e-10, kNodesTolFp64 = 2e-15;

// The least number of Chebyshev nodes on [f_lo, f_hi] for order nmax, or 0
// when kNodesMax do not suffice.  The series' leading term (damped as the
// Bessel function J_M(w) it stands for) against the tolerance; the order is
// raised by 6.5 for the functions' tails beyond their turning points, which
// matter at low orders.  Against the largest Chebyshev coefficients of phi_n
// over all n <= N and lines, N = 0 .. 96 and bands up to a factor of 2, it is
// never less than enough, and 1.6 more on average.
inline int shp_nodes(int nmax, double f_lo, double f_hi, double tol) {
  if (!(f_lo > 0.0) || !(f_hi >= f_lo)) return 0;
  const double w = (nmax + 7.0) * 0.5 * (f_hi - f_lo) / f_lo;
  if (!(w <= kNodesMax)) return 0;
  double t = 2.0;
  for (int m = 1; m <= kNodesMax; ++m) {
    t *= 0.5 * w / m;
    if (m >= w && t * std::exp(-0.25 * w * w / (m + 1)) <= tol) return m;
  }
  return 0;
}

// Points and Gaussians.  Along a baseline a component is S(nu) 2^(-Q nu^2)
// e^(2 pi i t0 nu / c), S(nu) = S0 nu^alpha e^(-A nu^2) with the power law and the
// beam, so that a row's sum over components in a narrow field, where every t0 is
// short, is determined by its values at a few frequencies too.
// w: the largest phase, in radians, from the band's middle to its end; delta:
// the band's half-width over its middle; amax: the largest |spectral index|;
// beam: A at the middle for the component furthest from the beam's centre.
// On the ellipse with foci -1, 1 and semi-axes a, b = (rho +- 1 / rho) / 2 (the
// band's variable being z in [-1, 1]) |nu|^alpha, over its least value in the
// band, is at most the larger of (1 + delta a) / (1 - delta) and (1 + delta) / (1 -
// delta a) to the amax, and the beam's Gaussian e^(beam ((1 + delta)^2 - m)), m the
// least real part of (1 + delta z)^2 there, which is >= 0 (so that the Gaussian
// envelopes stay below 1) while delta^2 (a^2 + b^2) <= 1.  With the phase's e^(w b),
// Chebyshev interpolation at M nodes errs by at most 4 rho^(1 - M) / (rho - 1) of
// that: an error over the flux that S leaves of the component at any channel.  The
// least M over the ellipses tried that brings it to tol, or 0 when kPgNodesMax do not.
constexpr int kPgNodesMax = 48;
inline int pg_nodes(double w, double delta, double amax, double tol, double beam = 0.0) {
  if (!(w >= 0.0) || !(w <= kPgNodesMax) || !(delta >= 0.0) || !(delta < 1.0) || !(amax >= 0.0) || !(beam >= 0.0)) return 0;
  int best = 0;
  for (double rho = 1.2; rho < 1e4; rho *= 1.15) {
    const double a = 0.5 * (rho + 1.0 / rho), b = 0.5 * (rho - 1.0 / rho);
    if (delta * delta * (a * a + b * b) > 0.9) break;
    const double ab = a * a + b * b;
    const double m = a >= delta * ab ? (1.0 - delta * a) * (1.0 - delta * a) : b * b * (1.0 / ab - delta * delta);
    const double lg = std::log(4.0 / ((rho - 1.0) * tol)) + w * b +
                      amax * std::log(std::max((1.0 + delta * a) / (1.0 - delta), (1.0 + delta) / (1.0 - delta * a))) +
                      beam * ((1.0 + delta) * (1.0 + delta) - m);
    if (!(lg <= kPgNodesMax * std::log(rho))) continue;
    const int M = 1 + (int)std::ceil(std::max(0.0, lg) / std::log(rho));
    if (M <= kPgNodesMax && (best == 0 || M < best)) best = M;
  }
  return best;
}

// The logarithm of a component's largest flux in the band over its least, at most.
// The sums at the nodes carry their rounding at the flux of the node, the channels
// between them at the least: the mixed path (FP32 terms) takes nodes only while
// that is a factor of 4, the FP64 path, whose sums are some 1e-16 off where
// phases cost it 1e-14 to 1e-13, up to 50.
constexpr double kPgSpreadMixed = 1.386, kPgSpreadFp64 = 3.912;
inline double pg_spread(double delta, double amax, double beam) {
  return amax * std::log((1.0 + delta) / (1.0 - delta)) + 4.0 * beam * delta;
}

}  // namespace vp
