// Choice among timed tile shapes (host only).  Candidates often lie closer
// together than two timings of one of them, which differ by 1 to 2 %; then the
// faster one is a matter of chance, while in a batch, whose large frames take
// the shape of a lone one, it matters: 4K grey takes 311 us a frame with bands
// of 7 rows and 314 with 5, but 235 and 273 in a batch of four; 720 x 2560 RGB
// 167 with 17 rows and 169 with 13, and 156 and 147 in the batch.  So within a
// margin a fixed preference decides.
#pragma once

#include <algorithm>
#include <cmath>

namespace ilsk {

// Index of a row shape: of those within 1.5 % of the fastest the one nearest to
// three quarters of the tallest band (whose blocks leave fewer compute units
// without work at the end of a pass) if that is eight rows or more, else the
// tallest (fewest halo rows).  Negative times are failures; 0 if nothing was
// timed.
inline int pick_row(const float* ms, const int* rows, int n) {
  float best = HUGE_VALF;
  int tallest = 0;
  for (int i = 0; i < n; ++i) {
    if (ms[i] >= 0.0f) best = std::min(best, ms[i]);
    tallest = std::max(tallest, rows[i]);
  }
  const float want = 0.75f * tallest >= 8.0f ? 0.75f * tallest : tallest;
  int pick = 0;
  float off = HUGE_VALF;
  for (int i = 0; i < n; ++i) {
    const float o = std::fabs(rows[i] - want);
    if (ms[i] >= 0.0f && ms[i] <= 1.015f * best && o < off) off = o, pick = i;
  }
  return pick;
}

// Index of a column tile: the first (shapes are in order of preference) within
// 1 % of the fastest.
inline int pick_col(const float* ms, int n) {
  float best = HUGE_VALF;
  for (int i = 0; i < n; ++i)
    if (ms[i] >= 0.0f) best = std::min(best, ms[i]);
  for (int i = 0; i < n; ++i)
    if (ms[i] >= 0.0f && ms[i] <= 1.01f * best) return i;
  return 0;
}

}  // namespace ilsk
