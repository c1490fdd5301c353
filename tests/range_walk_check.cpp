// Host check of the range-table search at table sizes around the one from
// which it reads groups of nodes (below: node by node): the node found must
// be that of a one-by-one walk down, for every start and for r on a node,
// below the table and inside it, with runs of equal values, FP64 and FP32.
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "../paper_2209_15445_amd/csrc/ems_step.hpp"

template <class R>
static long check(int nodes) {
  std::mt19937_64 g(nodes);
  std::uniform_real_distribution<double> u01(0.0, 1.0);
  long bad = 0;
  for (int trial = 0; trial < 12; ++trial) {
    std::vector<R> Rt(nodes);
    double acc = std::exp(-15.0 * u01(g));
    for (int j = 0; j < nodes; ++j) {
      if (!(trial % 3 == 0 && j % 7 == 3)) acc += acc * (0.01 + 0.39 * u01(g));
      Rt[j] = (R)acc;
    }
    ems::StepEnv<R> e{};
    e.nodes = nodes;
    e.lnemin = R(-6.9);
    e.dlog = R(0.127);
    for (int jhi = 0; jhi <= nodes; ++jhi)
      for (int q = 0; q < 40; ++q) {
        const R r = q % 4 == 0 ? Rt[(size_t)(u01(g) * nodes) % nodes]
                               : (R)((double)Rt[0] * std::pow((double)Rt[nodes - 1] / Rt[0], 1.2 * u01(g) - 0.1));
        int j = jhi > nodes - 1 ? nodes - 1 : jhi;
        while (j > 0 && Rt[j] > r) --j;
        j = j > nodes - 2 ? nodes - 2 : j;
        const R want = e.lnemin + (R)j * e.dlog + e.dlog * (r - Rt[j]) / (Rt[j + 1] - Rt[j]);
        const R got = ems::inverse_range_ln<R>(e, Rt.data(), r, jhi);
        if (!(got == want) && !(std::isnan((double)got) && std::isnan((double)want))) ++bad;
      }
  }
  return bad;
}

int main() {
  long bad = 0;
  for (int nodes : {3, 8, 9, 63, 64, 65, 72, 73, 201}) {
    const long b = check<double>(nodes) + check<float>(nodes);
    std::printf("%d nodes: %ld mismatches\n", nodes, b);
    bad += b;
  }
  return bad != 0;
}
