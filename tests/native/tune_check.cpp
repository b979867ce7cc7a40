// Host check of csrc/ils_tune.hpp: prints "passed" or what went wrong.
#include <cstdio>

#include "../../paper_2003_07504_amd/csrc/ils_tune.hpp"

static int bad = 0;
static void expect(int got, int want, const char* what) {
  if (got != want) std::printf("%s: %d, expected %d\n", what, got, want), ++bad;
}

int main() {
  const int r960[6] = {7, 17, 13, 11, 5, 4}, r1920[3] = {7, 5, 4}, r512[6] = {14, 30, 23, 19, 5, 4};
  const float clear[6] = {32.0f, 22.0f, 23.0f, 31.0f, 37.0f, 38.0f};
  expect(ilsk::pick_row(clear, r960, 6), 1, "a clearly faster shape");
  // two shapes that swap places from timing to timing
  for (float e : {-0.012f, -0.004f, 0.0f, 0.004f, 0.012f}) {
    const float tie[6] = {32.0f, 22.0f, 22.0f * (1.0f + e), 31.0f, 37.0f, 38.0f};
    expect(ilsk::pick_row(tie, r960, 6), 2, "three quarters of the tallest");
    const float tie4k[3] = {50.8f * (1.0f + e), 50.8f, 64.0f};
    expect(ilsk::pick_row(tie4k, r1920, 3), 0, "the tallest of short bands");
    const float near512[6] = {12.0f * (1.012f + e), 12.5f, 12.4f, 12.0f, 14.6f, 14.7f};
    expect(ilsk::pick_row(near512, r512, 6), 3, "a shape at the margin that is not preferred");
  }
  const float failed[6] = {-1.0f, -1.0f, -1.0f, -1.0f, -1.0f, -1.0f};
  expect(ilsk::pick_row(failed, r960, 6), 0, "nothing timed");
  expect(ilsk::pick_col(failed, 4), 0, "nothing timed");
  const float some[6] = {-1.0f, 9.0f, -1.0f, 8.0f, -1.0f, -1.0f};
  expect(ilsk::pick_row(some, r960, 6), 3, "failures are no times");
  const float c1[4] = {15.2f, 15.4f, 12.9f, 11.9f}, c2[4] = {16.9f, 18.2f, 24.4f, 16.8f}, c3[3] = {-1.0f, 5.0f, 5.02f};
  expect(ilsk::pick_col(c1, 4), 3, "the fastest tile");
  expect(ilsk::pick_col(c2, 4), 0, "the widest of two as fast");
  expect(ilsk::pick_col(c3, 3), 1, "the first that was timed");
  if (!bad) std::printf("passed\n");
  return bad ? 1 : 0;
}
