// Checks of the default schedule's rule (tg_columns.h) on the CPU.
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "tg_columns.h"

struct Graph {
  std::vector<std::vector<uint32_t>> preds;
  std::vector<uint64_t> cost;
  uint32_t add(std::vector<uint32_t> p, uint64_t c) {
    preds.push_back(std::move(p));
    cost.push_back(c);
    return (uint32_t)cost.size() - 1;
  }
};

static int failures = 0;

static void check(const char* what, const Graph& g, uint64_t nw, bool want) {
  std::vector<uint32_t> level(g.cost.size(), 0);
  for (uint32_t v = 0; v < level.size(); ++v)
    for (uint32_t p : g.preds[v]) level[v] = std::max(level[v], level[p] + 1);
  const bool got = tg::columns_hold(
      level, nw, [&](uint32_t v) { return g.cost[v]; },
      [&](uint32_t u, uint32_t v) { return std::find(g.preds[v].begin(), g.preds[v].end(), u) != g.preds[v].end(); });
  std::printf("%s %s: %s\n", got == want ? "ok  " : "FAIL", what, got ? "columns" : "levels");
  failures += got != want;
}

// W lanes, T levels; a task depends on its lane (shifted by `shift` lanes) and the next one.
template <class Cost>
static Graph rectangle(uint32_t W, uint32_t T, uint32_t shift, Cost cost) {
  Graph g;
  for (uint32_t t = 0; t < T; ++t)
    for (uint32_t i = 0; i < W; ++i) {
      std::vector<uint32_t> p;
      if (t) p = {(t - 1) * W + (i + shift) % W, (t - 1) * W + (i + shift + 1) % W};
      g.add(p, cost(t, i));
    }
  return g;
}

// A chain of tasks of cost a, each releasing k leaves of cost b.
static Graph leaves(uint32_t T, uint32_t k, uint64_t a, uint64_t b) {
  Graph g;
  uint32_t last = 0;
  for (uint32_t t = 0; t < T; ++t) {
    last = g.add(t ? std::vector<uint32_t>{last} : std::vector<uint32_t>{}, a);
    for (uint32_t i = 0; i < k; ++i) g.add({last}, b);
  }
  return g;
}

int main() {
  std::mt19937 rng(1);
  std::lognormal_distribution<double> ln(5, 1);
  auto same = [](uint32_t, uint32_t) { return (uint64_t)80; };
  auto by_level = [](uint32_t t, uint32_t) { return (uint64_t)(80 + 1000 * (t % 7)); };
  auto uneven = [&](uint32_t, uint32_t) { return (uint64_t)(64 + ln(rng)); };
  auto slightly = [&](uint32_t, uint32_t) { return (uint64_t)(80 + rng() % 60); };
  check("no task", Graph{}, 8192, true);
  check("one task", rectangle(1, 1, 0, uneven), 8192, true);
  check("one task, no worker counted", rectangle(1, 1, 0, uneven), 0, true);
  for (uint32_t W : {1u, 7u, 63u, 64u, 300u, 8191u, 8192u, 8193u, 20000u}) {
    check("equal costs", rectangle(W, 12, 0, same), 8192, true);
    check("costs equal in each level", rectangle(W, 12, 0, by_level), 8192, true);
    check("equal costs, shifted lanes", rectangle(W, 12, 1, same), 8192, true);
  }
  check("one level", rectangle(1000, 1, 0, same), 64, true);
  check("small differences", rectangle(300, 40, 2, slightly), 8192, true);
  check("uneven costs along dependent columns", rectangle(300, 40, 0, uneven), 8192, true);
  check("uneven costs across columns", rectangle(300, 40, 2, uneven), 8192, false);
  check("uneven costs, several of a level to a worker", rectangle(300, 40, 0, uneven), 64, false);
  check("uneven chain", rectangle(1, 500, 0, uneven), 8192, true);
  check("cheap leaves", leaves(500, 1, 72, 72), 8192, true);
  check("leaves of a hand-off's cost", leaves(500, 1, 72, 160), 8192, true);
  check("leaves that cost more", leaves(500, 1, 72, 300), 8192, false);
  check("expensive leaves", leaves(1000, 3, 72, 4160), 8192, false);
  check("expensive leaves, few workers", leaves(1000, 3, 72, 4160), 2, false);
  if (!failures) std::printf("all cases pass\n");
  return failures != 0;
}
