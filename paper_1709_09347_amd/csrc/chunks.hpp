// Chunks of the residual update and the size of their partial sums (plain C++, shared by the
// launches and the tuner, and compiled on its own by a CPU test).
//
// The update leaves four partial sums per run and chunk of points, at ((run * nchunks) + chunk) * 4:
// whoever launches it owns UPD_PART * nruns * nchunks doubles for the nchunks that it launches with.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace cbs {

constexpr int UPD_RUNS = 4;                          // runs per workgroup of the update
constexpr int UPD_PART = 4;                          // partial sums per run and chunk
constexpr int UPD_PTS_MIN = 256;                     // points of the shortest chunk
constexpr int UPD_PTS_TUNE[3] = {1024, 2048, 4096};  // chunk lengths the tuner times, shortest first

// chunks of `pts` points that cover N
inline int32_t update_chunk_count(int64_t N, int32_t pts) {
  const int64_t per = std::max<int64_t>(pts, UPD_PTS_MIN);
  return (int32_t)((N + per - 1) / per);
}

// Chunks of a solve of nruns runs: the tuned length, halved down to a group of points per wave until
// there are two workgroups per CU: 23 x 19 x 17 points, 30 runs: 21.6 us in chunks of 1024 points,
// 12.6 us in chunks of 256.
inline int32_t update_chunks_of(int64_t N, int32_t nruns, int32_t tuned_pts) {
  int32_t per = std::max<int32_t>(tuned_pts, UPD_PTS_MIN);
  const int64_t groups = (nruns + UPD_RUNS - 1) / UPD_RUNS;
  while (per > UPD_PTS_MIN && groups * update_chunk_count(N, per) < 512) per = std::max<int32_t>(per / 2, UPD_PTS_MIN);
  return update_chunk_count(N, per);
}

// doubles that a launch of the update writes partial sums to
inline size_t update_part_len(int32_t nruns, int32_t nchunks) { return (size_t)nruns * nchunks * UPD_PART; }

// The tuner's trial of a chunk length (as it is: a solve's own shortening depends on its runs), and the
// buffer that holds every trial's partial sums.
inline int32_t tune_chunks(int64_t N, int32_t pts) { return update_chunk_count(N, pts); }
inline size_t tune_part_len(int64_t N, int32_t nruns) {
  size_t len = 0;
  for (int32_t pts : UPD_PTS_TUNE) len = std::max(len, update_part_len(nruns, tune_chunks(N, pts)));
  return len;
}

}  // namespace cbs
