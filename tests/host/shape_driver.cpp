// The shape search of the operator's local part against every (rows, segments) pair.
// Input (stdin): lines "nx ny nz p nv elem".
// Output per line: rows, segments and cost of the search; rows, segments and cost of the best of all
// pairs; pairs looked at, all pairs; whether the rows are a shape.
#include <cstdio>

#include "apply_shape.hpp"

int main() {
  int nx, ny, nz, p, nv, elem;
  while (scanf("%d %d %d %d %d %d", &nx, &ny, &nz, &p, &nv, &elem) == 6) {
    int64_t evals = 0;
    const cbs::ApplyShape s = cbs::apply_shape(nx, ny, nz, p, nv, elem, &evals);
    int ty = 1, nseg = 1;
    double best = 0;
    long long pairs = 0;
    for (int t = 1; t <= ny && (t == 1 || nx * t <= 1024); ++t) {
      if (t > 1 && (size_t)(t + 2 * p) * nx * elem > 64 * 1024) break;
      const cbs::ApplyRows r(nx, ny, p, nv, t);
      for (int ns = 1; ns <= (nz / p > 1 ? nz / p : 1); ++ns) {
        const int zlen = (nz + ns - 1) / ns;
        const double c = r.cost(p, zlen, (nz + zlen - 1) / zlen);
        ++pairs;
        if (best == 0 || c < best) {
          best = c;
          ty = t;
          nseg = ns;
        }
      }
    }
    printf("%d %d %.17g %d %d %.17g %lld %lld %d\n", s.ty, s.nseg, s.cost, ty, nseg, best, (long long)evals, pairs,
           cbs::apply_rows_fit(nx, ny, p, elem, s.ty) && s.ty >= 1 && s.nseg >= 1 && s.nseg <= nz ? 1 : 0);
  }
  return 0;
}
