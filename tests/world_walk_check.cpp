// The walk of the box hierarchy from the world volume, whose node tests are
// in single precision, against a test of every box: the distance has to be
// the same to the bit, at scales and offsets at which a position or a bound
// rounds, for rays along an axis, almost along one, and from points on faces.
#include <cstdio>
#include <random>

#include "../paper_2209_15445_amd/csrc/ems_geometry.cpp"

using namespace ems;

int main() {
  std::mt19937_64 rng(20);
  auto uni = [&] { return (double)(rng() >> 11) * 0x1p-53; };
  long rays = 0, hits = 0, bad = 0;
  for (double scale : {1e-3, 1.0, 37.3, 1e7})
    for (double off : {0.0, -1.7, 1e5, 1e9})
      for (int n : {1, 3, 7, 16}) {
        // an n^3 (at most 7 x 7 x 16) grid of boxes, each cell's box smaller
        // than the cell, or filling it so that boxes touch
        const int m = n > 7 ? 7 : n;
        std::vector<double> lo, hi;
        for (int i = 0; i < m; ++i)
          for (int j = 0; j < m; ++j)
            for (int k = 0; k < n; ++k) {
              if (n > 1 && uni() < 0.3) continue;
              const bool full = uni() < 0.5;
              const int c[3] = {i, j, k};
              for (int q = 0; q < 3; ++q) {
                lo.push_back(scale * (off + c[q] + (full ? 0.0 : 0.4 * uni())));
                hi.push_back(scale * (off + c[q] + (full ? 1.0 : 0.5 + 0.4 * uni())));
              }
            }
        const uint32_t nb = (uint32_t)(lo.size() / 3);
        if (nb == 0) continue;
        BvhHost h;
        std::string err;
        if (!build_bvh(lo.data(), hi.data(), nb, h, err)) return std::printf("build failed\n"), 1;
        BoxNav g{};
        g.node = h.node.data();
        g.leaf = h.leaf.data();
        g.box = h.box.data();
        g.rec = h.rec.data();
        g.nbr_off = h.nbr_off.data();
        g.nbr = h.nbr.data();
        g.n_boxes = nb;
        const int len[3] = {m, m, n};
        for (int q = 0; q < 3; ++q) {
          g.wlo[q] = scale * (off - 3.0);
          g.whi[q] = scale * (off + len[q] + 2.0);
        }
        for (int it = 0; it < 4000; ++it, ++rays) {
          double p[3], u[3];
          for (int q = 0; q < 3; ++q) p[q] = g.wlo[q] + (g.whi[q] - g.wlo[q]) * uni();
          const uint32_t b = (uint32_t)(rng() % nb);
          if (it % 3 == 1)  // on a face of a box, within it or beside it
            for (int q = 0; q < 3; ++q) p[q] = it % 9 == 1 + 3 * q ? (it & 1 ? lo : hi)[3 * b + q] : p[q];
          if (it % 5 == 2) {  // towards a box's edge
            for (int q = 0; q < 3; ++q) u[q] = (rng() & 1 ? lo : hi)[3 * b + q] - p[q];
          } else {
            for (int q = 0; q < 3; ++q) u[q] = uni() - 0.5;
          }
          const double tiny[5] = {0.0, 1e-8, -1e-20, 3e-31, -1e-300};
          for (int q = 0; q < 3; ++q)
            if (rng() % 4 == 0) u[q] = tiny[rng() % 5];
          const double len2 = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
          if (!(len2 > 0.0)) continue;
          for (int q = 0; q < 3; ++q) u[q] /= std::sqrt(len2);
          Face fw, fb, f;
          double best = ray_exit(g.wlo, g.whi, p, u, fb);
          fb.box = -1;
          for (uint32_t i = 0; i < nb; ++i) {
            const double d = ray_entry(&h.box[6 * (size_t)i], &h.box[6 * (size_t)i + 3], p, u, f);
            if (d <= best) {
              best = d;
              fb = f;
              fb.box = (int)i;
            }
          }
          const double got = world_distance(g, p, u, fw);
          hits += fb.box >= 0;
          if (got != best || (fw.box < 0) != (fb.box < 0)) {
            if (bad++ < 5)
              std::printf("scale %g offset %g n %d ray %d: %.17g box %d, every box %.17g box %d\n", scale, off, n, it,
                          got, fw.box, best, fb.box);
          }
        }
      }
  std::printf("%ld rays, %ld enter a box, %ld differ\n", rays, hits, bad);
  return bad != 0 || hits == 0;
}
