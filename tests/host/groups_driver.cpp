// Energies per group of Hankel SVDs.
// Input (stdin): lines "ne moment_bytes n budget"; output per line: energies, bytes they hold.
#include <cstdio>

#include "groups.hpp"

int main() {
  int ne, n;
  double mom, budget;
  while (scanf("%d %lf %d %lf", &ne, &mom, &n, &budget) == 4) {
    const int g = cbs::svd_group_size(ne, mom, n, budget);
    printf("%d %.17g\n", g, g * cbs::svd_energy_bytes(mom, n));
  }
  return 0;
}
