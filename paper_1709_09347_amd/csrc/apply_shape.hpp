// Rows per workgroup and z segments of the operator's local part (plain C++, used by the launch and
// compiled on its own by a CPU test).
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace cbs {

struct ApplyShape {
  int32_t ty, nseg;
  double cost;
};

// Modelled time of t rows in segments of zlen planes.  A workgroup's march costs its owned planes
// (staged rows with their halo, plus the points worked on) and 2p halo columns, or, when few points
// are in flight, one latency a plane (as long as 1500 points take); a CU holds 16 waves, and a launch
// runs in whole rounds of the chip.
struct ApplyRows {
  int32_t percu;   // workgroups a CU holds
  int64_t wgs;     // workgroups per segment
  double plane, halo, inv, latency;

  ApplyRows(int32_t nx, int32_t ny, int32_t p, int32_t nv, int32_t t) {
    const int32_t waves = (nx * t + 63) / 64;
    percu = std::max(1, 16 / waves);
    wgs = (int64_t)nv * ((ny + t - 1) / t);
    plane = (t + 2 * p) * nx + 2.0 * nx * t;
    halo = 0.5 * 2 * p * ((double)nx * t);
    inv = 1.0 / percu;
    latency = (t + 2 * p) * nx <= 128 * waves ? 1.0 : 2.0;   // a plane's staging ahead of its use, or not
  }
  double cost(int32_t p, int32_t zlen, int32_t nseg) const {
    const int32_t share = (int32_t)((wgs * nseg + 255) >> 8);   // per CU: below 64 N / 256 with N < 2^31
    const int32_t rounds = (int32_t)((share + percu - 0.5) * inv);   // share / percu rounded up
    const double work = std::min(percu, share) * (zlen * plane + halo);
    return (double)rounds * std::max(work, 1500.0 * (zlen * latency + 2 * p * 0.25));
  }
};

// Whether t rows are a shape: 1024 threads, a plane of them within 64 KB of LDS (one row always).
inline bool apply_rows_fit(int32_t nx, int32_t ny, int32_t p, size_t elem, int32_t t) {
  return t == 1 || (t <= ny && nx * t <= 1024 && (size_t)(t + 2 * p) * nx * elem <= 64 * 1024);
}

// The pair with the least modelled time.  Against every (rows, segments) pair on thirteen cells and
// block sizes from 8x8x12 to 160x160x48 the choice is within 6 % of the fastest call (19 % on
// 21x70x16), where the worst pairs take twice as long: 96x96x32, 24 vectors: 76 us with 10 rows in one
// segment, 127 us with 8.
// The search runs at every call, so it skips what cannot win: segment counts that leave a segment's
// planes as they are (and past 32 segments those within a sixteenth of the last), rows whose work alone
// takes longer than the best pair, and beyond 32 rows (nx below 32) those that leave the number of
// tiles as it is.  On a CPU, 48x48x32 order 8, 32 vectors: 0.4 us (every pair: 1.5); order 2, one vector:
// 5x96x48 2.2 us (46), 4x256x512 5 us (1300).
// evals: counts the pairs looked at, if given.
inline ApplyShape apply_shape(int32_t nx, int32_t ny, int32_t nz, int32_t p, int32_t nv, size_t elem,
                              int64_t* evals = nullptr) {
  int32_t tmax = 1;
  if (apply_rows_fit(nx, ny, p, elem, 2))
    tmax = (int32_t)std::min<int64_t>({ny, 1024 / nx, (int64_t)(64 * 1024 / ((size_t)nx * elem)) - 2 * p});
  // the counts of segments that differ in their planes, fewest first
  constexpr int32_t MAXS = 384;   // 32, a sixteenth each up to 2^31, and the last sixteen
  int32_t nseg[MAXS], zlen[MAXS], n = 0;
  for (int64_t ns = 1; n < MAXS && ns <= std::max(1, nz / p);) {
    const int64_t len = (nz + ns - 1) / ns;
    nseg[n] = (int32_t)((nz + len - 1) / len);
    zlen[n++] = (int32_t)len;
    if (len == 1) break;
    ns = std::max<int64_t>((nz + len - 2) / (len - 1), ns > 32 ? ns + ns / 16 : 0);
  }
  ApplyShape best{1, 1, 0};
  bool any = false;
  for (int32_t t = tmax; t >= 1; --t) {
    if (t > 32 && (ny + t - 2) / (t - 1) == (ny + t - 1) / t) continue;
    const ApplyRows r(nx, ny, p, nv, t);
    if (any && (double)r.wgs * nz * r.plane / 256 > best.cost) continue;   // rounds x sharing >= workgroups / 256
    int32_t at = 0;
    double here = r.cost(p, zlen[0], nseg[0]);
    for (int32_t i = 1; i < n; ++i) {
      const double c = r.cost(p, zlen[i], nseg[i]);
      if (c < here) {
        here = c;
        at = i;
      }
    }
    if (evals != nullptr) *evals += n;
    if (!any || here <= best.cost) best = ApplyShape{t, nseg[at], here};   // of equals the fewest rows
    any = true;
  }
  return best;
}

}  // namespace cbs
