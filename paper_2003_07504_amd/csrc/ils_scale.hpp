// The scale of the iterate and the penalty's constants of a frame descriptor
// (host only).
#pragma once

#include <algorithm>
#include <cmath>

#include "ils_desc.hpp"

namespace ilsk {

// Sets kappa and the scale s that the iterate is held times: `ideal` (eps^(-1/2),
// or sqrt(log2(e) / 2) / gamma for Welsch), kept within 1 / limit .. limit.  A
// rounding error of s / (2 H W) times 1 / s would scale the whole result, so
// 1 / s is taken among the floats within three units in the last place of it,
// where the larger of that error and width(s), the relative error of the
// penalty's width, is least.  d.H and d.W are set.  Returns s.
template <class Width>
inline double set_scale(FrameDesc& d, double kappa, double ideal, double limit, Width&& width) {
  const double hw2 = 2.0 * (double)d.H * (double)d.W;
  float c = (float)(1.0 / std::min(std::max(ideal, 1.0 / limit), limit));
  for (int i = 0; i < 3; ++i) c = std::nextafter(c, 0.0f);
  double best = HUGE_VAL;
  for (int i = -3; i <= 3; ++i, c = std::nextafter(c, HUGE_VALF)) {
    const float col = (float)(1.0 / (hw2 * (double)c));
    const double off = std::max(std::fabs((double)col * (double)c * hw2 - 1.0), width(1.0 / (double)c));
    if (off < best) {
      best = off;
      d.u_unscale = c;
      d.col_scale = col;
    }
  }
  const double s = 1.0 / (double)d.u_unscale;
  d.kappa = (float)kappa;
  d.u_scale = (float)s;
  d.kappa_mu = (float)(kappa / s);
  return s;
}

// Generalised Charbonnier penalty, c >= c0 = p eps^(p/2 - 1) (Eq. (7)): with
// h = s g, (c0 / c) (1 + g^2 / eps)^a = 2^(a log2(h^2 + pen_k) + log2_r), a = p/2 - 1.
// s stays within 2^-40 .. 2^40, so that s u stays in float32's range for images
// far larger or smaller than the penalty is wide.  Within, pen_k is 1: the
// choice of s moves eps by up to 7e-7 relative, which the results do not show
// (error against 64 bits over 45 cases, geometric mean: 4.2e-7 with an exact
// eps^(-1) and the iterate unscaled, 4.0e-7 so); at the limits pen_k makes up
// for it.  p = 2 (a = 0) stays the quadratic penalty exactly.
inline void set_charbonnier(FrameDesc& d, double lambda, double p, double eps, double c0_over_c, double c) {
  const double ideal = 1.0 / std::sqrt(eps), limit = std::ldexp(1.0, 40);
  const double s = set_scale(d, lambda * c / 2.0, ideal, limit, [](double) { return 0.0; });
  const double a = p / 2.0 - 1.0;
  const bool within = ideal <= limit && ideal >= 1.0 / limit;
  d.a_exp = (float)a;
  d.pen_k = within ? 1.0f : (float)(eps * s * s);
  d.log2_r = (float)(std::log2(c0_over_c) - a * std::log2((double)d.pen_k));
}

// Welsch penalty (Sec. 5): c = c0 = 2 (Eq. (20)), so kappa = lambda;
// exp(-g^2 / (2 gamma^2)) = 2^(-h^2).  No constant makes up for the choice of s
// here (one more multiply per difference: 450 x 600, N = 15 228 -> 230 us), so
// its error counts, and the limit of s lies beyond images of 2^-70 and 2^70.
inline void set_welsch(FrameDesc& d, double lambda, double gamma) {
  const double w = std::sqrt(1.4426950408889634 / 2.0) / gamma;
  set_scale(d, lambda, w, std::ldexp(1.0, 80), [&](double s) { return std::min(1.0, 2.0 * std::fabs(s / w - 1.0)); });
  d.a_exp = d.log2_r = 0.0f;
  d.pen_k = 1.0f;
}

}  // namespace ilsk
