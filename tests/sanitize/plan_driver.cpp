// Checks of what a plan holds on the host, for the same build as abi_driver.cpp. Exit status 0 when all hold.
#include <cstdio>
#include <map>
#include <random>
#include <utility>
#include <vector>

#include "morlet.h"
#include "plan_internal.h"

static int g_fail = 0;
#define EXPECT(cond)                                                               \
  do {                                                                             \
    if (!(cond)) {                                                                 \
      std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #cond);      \
      ++g_fail;                                                                    \
    }                                                                              \
  } while (0)

// The split of a batch is found over its row shapes, each once: the counts add up to the rows, and the split
// is that of the rows themselves.
static void row_shapes() {
  std::mt19937_64 rng(7);
  std::vector<int64_t> lengths, windows{3, 3, 40, 700};
  for (int b = 0; b < 3000; ++b) lengths.push_back((int64_t)(rng() % 5000));
  lengths[5] = 0;
  std::map<std::pair<int64_t, int64_t>, int64_t> count;
  std::vector<mk::GranRow> rows;
  for (int64_t n : lengths)
    for (int64_t w : windows)
      if (n > 0) {
        ++count[{mk::granules_for(n), w}];
        rows.push_back({mk::granules_for(n), w, 1});
      }
  const std::vector<mk::GranRow> shapes = mk::gran_shapes(lengths, windows);
  EXPECT(shapes.size() == count.size());
  for (const mk::GranRow& s : shapes) EXPECT((count[{s.ng, s.nw}] == s.count));
  const mk::GranSplit a = mk::split_granules(shapes, 256), b = mk::split_granules(rows, 256);
  EXPECT(a.base == b.base && a.per_warm == b.per_warm);
}

int main() {
  row_shapes();
  if (g_fail == 0) std::printf("all checks passed\n");
  return g_fail ? 1 : 0;
}
