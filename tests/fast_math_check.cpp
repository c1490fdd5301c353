// Host check of ems_math.hpp against long double: largest error of the
// logarithm and the exponential in units in the last place, and of sine and
// cosine of a turn, over the ranges the transport uses (energies over 17
// decades, draws in (0, 1), arguments next to 1, quarter turns).  Prints the
// three figures; exits with 1 where one exceeds its bound: half a unit for
// the last rounding and a third for the terms before it (log), the same and
// the rounding of 1 + r over half a binade (exp), one rounding each of the
// angle and the polynomial below an eighth of a turn (sine, cosine).
#include <cmath>
#include <cstdio>
#include <random>

#include "../paper_2209_15445_amd/csrc/ems_core.hpp"

static double ulp(double v) { return std::nextafter(std::fabs(v), INFINITY) - std::fabs(v); }

int main() {
  std::mt19937_64 g(7);
  std::uniform_real_distribution<double> U(0.0, 1.0);
  double wl = 0.0, we = 0.0, ws = 0.0;
  const double edge[] = {1.0, 1.0 - 0x1p-53, 1.0 + 0x1p-52, 0x1p-53, 0.5, 2.0, 0x1.6a09ep-1, 0x1.6a09fp-1, 1e-300, 1e300};
  for (long i = 0; i < 2000000; ++i) {
    const int k = (int)(i % 4);
    double x = k == 0 ? std::exp(U(g) * 40.0 - 14.0) : k == 1 ? U(g) : k == 2 ? 1.0 + (U(g) - 0.5) * std::pow(2.0, -U(g) * 40.0) : 2.0 * U(g);
    if (i < (long)(sizeof edge / sizeof edge[0])) x = edge[i];
    if (!(x > 0.0)) continue;
    const long double l = logl((long double)x);
    if (l != 0.0L) wl = std::fmax(wl, std::fabs((double)(ems::pos_log(x) - l)) / ulp((double)l));
    else if (ems::pos_log(x) != 0.0) wl = INFINITY;
    const double y = (i % 3) ? (U(g) - 0.5) * 60.0 : -8.0 * U(g);
    const long double e = expl((long double)y);
    we = std::fmax(we, std::fabs((double)(ems::ranged_exp(y) - e)) / ulp((double)e));
    const double u = i < 9 ? 0.125 * (double)i : U(g);
    double s, c;
    ems::sincos_turn(u, &s, &c);
    const long double t = 2.0L * acosl(-1.0L) * (long double)u;
    ws = std::fmax(ws, std::fmax(std::fabs((double)(s - sinl(t))), std::fabs((double)(c - cosl(t)))));
  }
  std::printf("log %.3f ulp, exp %.3f ulp, sincos %.3g\n", wl, we, ws);
  return wl < 0.84 && we < 0.9 && ws < 2.3e-16 ? 0 : 1;
}
