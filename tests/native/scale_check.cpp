// Host check of csrc/ils_scale.hpp: for penalties of every width prints
// "bad <what> at <value>" for what does not hold, then "passed" or "failed".
#include <hip/hip_runtime.h>

#include <cstdio>
#include <random>

#include "../../paper_2003_07504_amd/csrc/ils_scale.hpp"

using ilsk::FrameDesc;

static const double kUlp = std::ldexp(1.0, -23);  // of a float32 between 1 and 2
static int bad = 0;
static void check(bool ok, const char* what, double at) {
  if (!ok) {
    std::printf("bad %s at %.9g\n", what, at);
    ++bad;
  }
}
static void common(const FrameDesc& d, double kappa, double limit, double at) {
  check(std::fabs((double)d.u_scale * d.u_unscale - 1.0) <= kUlp, "1 / s", at);
  check(d.u_scale >= 0.99999 / limit && d.u_scale <= 1.00001 * limit, "range of s", at);
  check(std::isfinite(d.pen_k) && std::isfinite(d.log2_r) && std::isfinite(d.col_scale), "finite", at);
  const double hw2 = 2.0 * d.H * d.W;
  check(std::fabs((double)d.col_scale * d.u_unscale * hw2 - 1.0) <= kUlp / 2, "col_scale", at);
  if (kappa > 1e-37 && kappa < 3e38 && kappa * d.u_unscale > 1e-37 && kappa * d.u_unscale < 3e38)
    check(std::fabs((double)d.kappa_mu / d.u_unscale / d.kappa - 1.0) <= kUlp, "kappa / s", at);
}

int main() {
  std::mt19937_64 rng(7);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  for (int i = 0; i < 200000; ++i) {
    FrameDesc d{};
    d.H = 2 + (int)(u(rng) * 4000);
    d.W = 2 * (1 + (int)(u(rng) * 4000));
    const bool wide = i % 4 == 0;
    const float p = (float)(0.05 + 1.95 * u(rng)), lam = (float)std::exp(8.0 * u(rng) - 4.0);
    const float eps = (float)std::exp(wide ? 176.0 * u(rng) - 88.0 : 23.0 * u(rng) - 18.0);
    if (!(eps > 0.0f) || !std::isfinite(eps)) continue;
    const double c0 = (double)p * std::pow((double)eps, (double)p / 2.0 - 1.0), c = i % 3 ? c0 : 1.5 * c0;
    ilsk::set_charbonnier(d, lam, p, eps, c0 / c, c);
    common(d, lam * c / 2.0, std::ldexp(1.0, 40), eps);
    // (h^2 + pen_k) / pen_k is 1 + g^2 / eps
    const double s = 1.0 / (double)d.u_unscale;
    check(std::fabs((double)d.pen_k / (s * s) / (double)eps - 1.0) <= 7.0 * kUlp, "eps in force", eps);
    const double r = std::exp2(d.a_exp * std::log2((double)d.pen_k) + d.log2_r) * c / c0;
    check(std::fabs(r - 1.0) <= kUlp * (1.0 + std::fabs(std::log2((double)d.pen_k))), "c0 / c", eps);
    if (!wide) check(d.pen_k == 1.0f, "pen_k 1", eps);

    const float gamma = (float)std::exp(wide ? 110.0 * u(rng) - 55.0 : 20.0 * u(rng) - 10.0);
    ilsk::set_welsch(d, lam, gamma);
    common(d, lam, std::ldexp(1.0, 80), gamma);
    const double w = std::sqrt(1.4426950408889634 / 2.0) / (double)gamma;
    if (w > std::ldexp(1.0, -80) && w < std::ldexp(1.0, 80))
      check(std::fabs(w * d.u_unscale - 1.0) <= kUlp, "gamma in force", gamma);
  }
  std::printf("%s\n", bad ? "failed" : "passed");
  return bad ? 1 : 0;
}
