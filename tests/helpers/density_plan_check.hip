// Host-side check of the rules that send a setting of the density propagation to its
// coarse form: for every number of cells, step widths over the whole range and drifts up
// to the rule's limit, each table, buffer and thread of the coarse kernel reaches every
// index that the kernel forms.  Prints the first violation and exits nonzero.
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "../../paper_2110_15425_amd/csrc/density.hip"

namespace {

unsigned long long plans = 0;

void need(bool ok, const char* what, uint32_t cells, double b, double as) {
  if (ok) return;
  printf("%s: %u cells, b %.17g, as %.17g\n", what, cells, b, as);
  exit(1);
}

void check(uint32_t cells, double b, double as) {
  using namespace cm;
  const CoarsePlan p = coarse_plan(cells, 1.0, b, as, 0.0, INFINITY);
  if (!p.ok) return;
  ++plans;
  const DensityGeo g = density_geo(cells);
  const CoarseGeo c = coarse_geo(g, p);
  const int M = (int)cells, NB = (int)g.NB, NT = (int)g.NT, s = p.s;
  auto ft = [&](int d) { need(d >= -c.FO && d <= c.FO, "displacement", cells, b, as); };
  auto sc = [&](int d) { need(abs(d) <= c.SM, "sinc", cells, b, as); };
  need(p.r >= 1 && p.r <= kCoarse, "samples", cells, b, as);
  need(p.direct >= 1 && p.direct <= 31, "full-grid steps", cells, b, as);
  need(c.prep <= kCoarseLds, "LDS", cells, b, as);
  need(256 * NT <= kCoarseSlots * kCoarseThreads, "cells of the threads", cells, b, as);
  need(2 * M <= (int)g.CB * kBS, "absorption table", cells, b, as);
  ft(p.E);
  const double h = 2.0 / cells;
  ft((int)(b / h + 0.5));
  ft(s * (int)(b / (h * s) + 0.5));
  const int X0 = -s * p.mg, X1 = s * (p.r - 1 - p.mg);
  sc(M - 1 - X0);  // the sums over cells
  sc(X1);
  const int dlo = -((p.E + 15) / 16) - 1, dhi = (p.E + 15) / 16 + 1;
  for (int tile = 0; tile < NT; ++tile) {  // the full-grid steps
    const int c0 = 16 * tile, dA = std::max(dlo, c0 - NB + 1), dB = std::min(dhi, std::min(c0 + 15, NB - 1));
    if (dB < dA) continue;
    ft(16 * dA - 3 - 12);
    ft(16 * dB + 15);
    need(c0 + NB - dB >= 0 && c0 + 15 + NB - dA < (int)g.CB, "mass blocks", cells, b, as);
  }
  if (!p.mg) return;
  for (int w = 0; 16 * w < p.r; ++w) {  // the cells beyond the bounds
    const int Xlo = s * (16 * w - p.mg), Xhi = Xlo + 15 * s;
    const int left = (std::min(p.E, p.E - Xlo) + 3) / 4, right = (std::min(p.E, Xhi + p.E + 1 - M) + 3) / 4;
    for (int side = 0; side < 2; ++side) {
      const int n = side ? right : left;
      if (n <= 0) continue;
      const int i0 = side ? M : -4 * n, i1 = i0 + 4 * (n - 1);
      ft(Xlo - 3 - i1);
      ft(Xhi - i0);
      sc(i0 - X1);
      sc(i1 + 3 - X0);
    }
  }
}

// A propagation that ends early: the steps to the tolerance, from the discrete walk's
// leading eigenvalue, against those that the preparation is worth.
void check_tol(uint32_t cells, double b, double as, double tol, bool want) {
  const cm::CoarsePlan p = cm::coarse_plan(cells, 1.0, b, as, 0.0, log(4.0 / (M_PI * tol)));
  need(p.ok == want, want ? "left to the full grid" : "not left to the full grid", cells, b, as);
}

}  // namespace

int main() {
  check_tol(128, 0.24, 0.0, 0.5, false);   // ends after some 20 steps
  check_tol(128, 0.24, 0.0, 1e-5, true);   // 215
  check_tol(128, 0.1, 0.0, 0.5, false);    // 100
  check_tol(333, 0.1, 0.0, 0.5, false);    // 100
  check_tol(333, 0.1, 0.0, 0.1, true);     // 235
  check_tol(333, 0.2, 0.0, 0.5, false);    // 36
  check_tol(333, 0.2, 0.0, 1e-3, true);    // 195
  check_tol(1000, 0.1, 0.0, 0.5, true);    // 100
  check_tol(1000, 0.1, 0.0, 0.9, false);   // 45
  check_tol(48, 0.2, 0.0, 1e-3, true);     // 190
  check_tol(333, 0.1, 0.019, 1e-3, true);  // 250, with the drift
  check_tol(333, 0.1, 0.019, 0.1, false);  // 100
  for (uint32_t cells = 16; cells <= 2000; ++cells) {
    const double lo = 4.0, hi = cells / 8.0;  // step width in cells: the rule's ends
    for (int k = 0; k <= 48 && lo <= hi; ++k) {
      const double bc = lo * pow(hi / lo, k / 48.0), b = bc * 2.0 / cells, a = 2.0 * b * b;
      for (double as : {0.0, 0.5 * a, a, -a}) check(cells, b, as);
    }
    for (int s = 1; s < 90; ++s)  // either side of each change of the sample spacing
      for (double e : {-1e-9, 0.0, 1e-9}) {
        const double b = s * 8.9 / 3.14159265358979 * (1.0 + e) * 2.0 / cells;
        check(cells, b, 0.0);
        check(cells, b, 2.0 * b * b * (1.0 - 1e-12));
      }
  }
  printf("plans %llu\n", plans);
  return plans > 100000 ? 0 : 1;
}
