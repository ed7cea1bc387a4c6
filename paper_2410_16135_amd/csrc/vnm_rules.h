// Rules that choose between kernels or launch shapes by sizes alone.  Plain C++ without HIP, so that they can be
// compiled and checked on any host.
#pragma once
#include <stdint.h>

namespace vnm {

// ---- RIA scores (vnm_score.hip)
// Column sums: waves per workgroup and rows in flight per thread.  One pass of a workgroup covers
// 8 * waves * flight rows; on short matrices the rows that a wide pass would repeat at the end cost more than the
// bandwidth it gains on tall ones.  Device time of the whole vnm_ria_scores with (waves, flight) =
// (4, 4) / (4, 8) / (8, 8) / (16, 8), us: 96 x 1000 9.6 / 10.1 / 11.4 / 12.8, 500 x 1000 12.0 / 11.8 / 11.6 / 14.4,
// 768 x 1000 13.8 / 13.3 / 14.7 / 14.7, 2048 x 1000 24.1 / 22.4 / 21.7 / 21.8, 4096 x 4096 64.0 / 58.3 / 55.2 / 54.2,
// 11008 x 4096 151 / 136 / 130 / 126.
// Rows without 16-byte alignment are read element by element, and only waves hide that: 1000 x 1031
// 42.6 / 42.5 / 31.5 / 25.5, 16 x 1031 12.5 / 12.6 / 12.5 / 12.5.
struct ColsumShape { int waves, flight; };
inline ColsumShape colsum_shape(int64_t out, bool aligned) {
  if (!aligned || out >= 3072) return {16, 8};
  if (out >= 1536) return {8, 8};
  if (out > 384) return {4, 8};
  return {4, out > 32 ? 4 : 1};                       // 16 x 1000: 7.8 us with one row in flight, 8.6 with four
}
// Scores: rows per workgroup, from the number of (1024 columns, row) units.  More rows share the column reciprocals;
// fewer give a small matrix workgroups for every compute unit.  Whole call with 1 / 4 / 8 / 16 rows, us:
// 96 x 1000 8.8 / 9.6 / 10.3 / 11.6, 1000 x 1000 16.5 / 15.7 / 16.3 / 17.7, 1000 x 4096 28.2 / 23.8 / 23.8 / 24.4,
// 2048 x 4096 47.1 / 38.4 / 36.8 / 36.9, 4096 x 4096 80.7 / 64.1 / 62.9 / 61.0, 11008 x 64 85.6 / 78.4 / 77.4 / 76.9.
inline int score_rows(int64_t out, int64_t in) {
  const int64_t units = (in + 1023) / 1024 * out;
  return units <= 1024 ? 1 : units <= 4096 ? 4 : units <= 12288 ? 8 : 16;
}

}  // namespace vnm
