// The kernels' logarithm, exponential and exp - 1 (integrands.hpp: log_pos, exp_fin,
// expm1_fin) compiled for the host in binary64 and compared with the C library's long double
// functions: the largest errors in units in the last place, as JSON.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "integrands.hpp"

static double ulp_of(long double r) {
  int e;
  frexpl(r, &e);
  return std::ldexp(1.0, e - 53);
}

int main(int argc, char** argv) {
  const long n = argc > 1 ? std::atol(argv[1]) : 1000000;
  std::mt19937_64 g(5);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  double e_log = 0, e_exp = 0, e_expm1 = 0;
  auto log_at = [&](double x) {
    const long double r = logl(static_cast<long double>(x));
    if (r != 0.0L) e_log = std::max(e_log, static_cast<double>(fabsl(vg::log_pos(x) - r)) / ulp_of(r));
    else if (vg::log_pos(x) != 0.0) e_log = 1e9;
  };
  auto exp_at = [&](double t) {
    const long double r = expl(static_cast<long double>(t)), m = expm1l(static_cast<long double>(t));
    e_exp = std::max(e_exp, static_cast<double>(fabsl(vg::exp_fin(t) - r)) / ulp_of(r));
    if (m != 0.0L) e_expm1 = std::max(e_expm1, static_cast<double>(fabsl(vg::expm1_fin(t) - m)) / ulp_of(m));
    else if (vg::expm1_fin(t) != 0.0) e_expm1 = 1e9;
  };
  for (long i = 0; i < n; ++i) {
    log_at(u(g));
    log_at(std::pow(10.0, -300.0 * u(g)));               // down to 1e-300
    log_at(1.0 + (u(g) - 0.5) * std::pow(2.0, -50.0 * u(g)));  // around 1
    exp_at(-40.0 * u(g));                                // logarithms of parton fractions
    exp_at(700.0 * (2.0 * u(g) - 1.0));
    exp_at(-std::pow(10.0, -15.0 * u(g)));               // fractions near 1
  }
  for (int k = -1000; k <= 1000; ++k)
    for (double f : {1.0, 0.70710678118654746, 0.70710678118654757, 0.70710678118654768})
      log_at(std::ldexp(f, k));
  for (int k = -200; k <= 200; ++k) exp_at(0.34657359027997264 * k);  // the folds' ends
  exp_at(0.0);
  // out of range: the limits
  const bool lim = vg::exp_fin(-1e5) == 0.0 && vg::expm1_fin(-1e5) == -1.0 && vg::exp_fin(1e5) > 1e308;
  std::printf("{\"log\": %.4f, \"exp\": %.4f, \"expm1\": %.4f, \"limits\": %s}\n", e_log, e_exp, e_expm1,
              lim ? "true" : "false");
  return 0;
}
