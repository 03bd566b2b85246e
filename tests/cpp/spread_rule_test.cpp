// Host test of the choice between full and spread workgroups (split_plan.hpp).
#include <stdio.h>
#include "split_plan.hpp"

static int failures = 0;
#define CHECK(c)                                          \
  do {                                                    \
    if (!(c)) {                                           \
      printf("FAIL %s:%d: %s\n", __FILE__, __LINE__, #c); \
      ++failures;                                         \
    }                                                     \
  } while (0)

int main() {
  using cfog::plan_split_choice;
  using cfog::takes_spread;
  const int cus = 256;
  // one spread workgroup to a CU, unsplit: up to a CU each
  for (int n = 1; n <= 2000; ++n) CHECK(takes_spread(n, n, n, cus, 1, true) == (n <= 256));
  // two to a CU: up to two each
  for (int n = 1; n <= 2000; ++n) CHECK(takes_spread(n, n, n, cus, 2, true) == (n <= 512));
  // P = 64, N = 44, r = 9, 9 channels, split: full workgroups share a CU by fours
  auto lane64 = [&](int n, bool rest) {
    const auto s = plan_split_choice(64, n, 2 * cus, 9, 44, 62, 19);
    const int items = s.G > 1 ? s.n_whole + (n - s.n_whole) * s.G : n;
    return takes_spread(n, s.n_whole, items < 4 * cus ? items : 4 * cus, cus, 2, rest);
  };
  CHECK(lane64(512, true));
  CHECK(lane64(520, true) && lane64(600, true) && lane64(700, true));  // a round and a small rest
  CHECK(!lane64(768, true) && !lane64(1024, true) && !lane64(1100, true));
  CHECK(!lane64(520, false));  // full workgroups of few waves
  CHECK(!lane64(200, true));   // no whole round: the split items fill the full workgroups
  // with one to a CU a round and a rest are full workgroups
  CHECK(!takes_spread(272, 256, 256 + 16 * 9, cus, 1, true));
  if (failures) return 1;
  printf("ALL OK\n");
  return 0;
}
