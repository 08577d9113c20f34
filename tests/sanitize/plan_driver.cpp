// Checks of what a plan holds on the host, for the same build as abi_driver.cpp. Exit status 0 when all hold.
#include <cstdio>
#include <map>
#include <memory>
#include <random>
#include <utility>
#include <vector>

#include "api.cpp"   // its internal functions too

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

// Whether a batch's rows are all alike is found when the plan is built, not by a pass over the lengths in
// every launch.
static void equal_rows() {
  const double sig[2] = {16.0, 32.0}, xi[2] = {0.4, 0.2};
  const int64_t same[3] = {500, 500, 500}, other[3] = {500, 501, 500}, none[2] = {0, 0};
  struct { const int64_t* len; int B, S; bool equal; } cases[] = {{same, 3, 1, true}, {same, 3, 2, false}, {other, 3, 1, false}, {same, 1, 1, true}, {none, 2, 1, true}};
  for (const auto& c : cases) {
    morlet_plan_t p = nullptr;
    EXPECT(morlet_scalogram_plan(&p, c.B, c.len, c.S, sig, xi, 4, 3.0) == MORLET_OK);
    EXPECT(p && p->equal_rows == c.equal);
    EXPECT(morlet_plan_set_tile(p, 8) == MORLET_OK && p->equal_rows == c.equal);
    EXPECT(c.equal == p->gran_segs.empty());
    morlet_destroy(p);
  }
}

// The backward workspace holds per-scale adjoints only where several are added up: with one scale a batch of one
// signal needs what the signal's own plan needs (up to its padding), not N floats more.
static void backward_scratch() {
  const int64_t N = 1 << 20;
  const double sig[2] = {16.0, 32.0}, xi[2] = {0.4, 0.2};
  morlet_plan_t one = nullptr, row = nullptr, two = nullptr;
  EXPECT(morlet_plan(&one, N, 16.0, 0.4, 5, 48) == MORLET_OK);
  EXPECT(morlet_scalogram_plan(&row, 1, &N, 1, sig, xi, 5, 3.0) == MORLET_OK);
  EXPECT(morlet_scalogram_plan(&two, 1, &N, 2, sig, xi, 5, 3.0) == MORLET_OK);
  size_t a = 0, b = 0, c = 0;
  EXPECT(morlet_backward_workspace_size(one, &a) == MORLET_OK && morlet_backward_workspace_size(row, &b) == MORLET_OK &&
         morlet_backward_workspace_size(two, &c) == MORLET_OK);
  EXPECT(b <= a + 4096 && a <= b + 4096);
  EXPECT(c >= 2 * a - 4096 + 2 * (size_t)N * sizeof(float));
  for (morlet_plan_t p : {one, row, two}) morlet_destroy(p);
}

// A batch of more pieces than a launch has room for (64 threads each, fewer than 2^32 in all) is left to the tile
// scan, whose grid is bounded.
static void launch_limit() {
  EXPECT(mk::launchable(((int64_t)1 << 26) - 1, 64) && !mk::launchable((int64_t)1 << 26, 64));
  EXPECT(mk::launchable(((int64_t)1 << 23) - 1, 512) && !mk::launchable((int64_t)1 << 23, 512));
  auto p = std::make_unique<morlet_plan_s>();
  p->batched = true;
  p->K = 5;
  p->rows.resize(4);
  mk::ScanLaunch a{};
  a.acc = mk::kAccF32;
  a.ntiles = (int64_t)1 << 30;
  p->gran_segs.resize(((size_t)1 << 26) - 1);
  EXPECT(gran_launch(p.get(), a, mk::kVarForward) && a.gran_nseg == ((int64_t)1 << 26) - 1);
  p->gran_segs.push_back({});
  EXPECT(!gran_launch(p.get(), a, mk::kVarForward) && a.gran_nseg == 0);
}

int main() {
  launch_limit();
  row_shapes();
  backward_scratch();
  equal_rows();
  if (g_fail == 0) std::printf("all checks passed\n");
  return g_fail ? 1 : 0;
}
