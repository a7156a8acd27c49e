// The chunk rules of the residual update over a range of cells.
// Input (arguments): the first and the last N, and the runs of a batch.
// Output: "N trial_doubles buffer_doubles" for every N whose tuner trials would write past their
// buffer, "chunks N ..." for every N whose chunks do not cover it, then "checked <count>".
#include <cstdio>
#include <cstdlib>

#include "chunks.hpp"

int main(int argc, char** argv) {
  if (argc != 4) return 1;
  const long long n0 = atoll(argv[1]), n1 = atoll(argv[2]);
  const int nr = atoi(argv[3]);
  long long checked = 0;
  for (long long N = n0; N <= n1; ++N) {
    const size_t len = cbs::tune_part_len(N, nr);
    for (int pts : cbs::UPD_PTS_TUNE) {
      const int nch = cbs::tune_chunks(N, pts);
      // the last partial sum that run nr - 1 writes in chunk nch - 1
      const size_t last = ((size_t)(nr - 1) * nch + (nch - 1)) * 4 + 3;
      if (last >= len) printf("%lld %zu %zu\n", N, last + 1, len);
      if (nch < 1 || (long long)nch * pts < N) printf("chunks %lld %d x %d\n", N, nch, pts);
      // a solve with the tuned length: whole groups of 256 points or the tuned chunk
      const int ns = cbs::update_chunks_of(N, nr, pts);
      if (ns < nch || ns > (N + 255) / 256) printf("chunks %lld solve %d\n", N, ns);
      if (cbs::update_part_len(nr, ns) != (size_t)nr * ns * 4) printf("chunks %lld part\n", N);
      ++checked;
    }
  }
  printf("checked %lld\n", checked);
  return 0;
}
