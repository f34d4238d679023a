// When one graph runs in column order by default (plain C++, so the rule can be
// checked on a machine without a GPU).
//
// Column order gives the i-th task of every dependence level to worker i mod nw,
// so a task and its successor of the same lane share a worker: their edge needs no
// signal, and waits between other pairs find the worker awake.  Level order deals
// the tasks over all workers, so every edge is a hand-off, about 1.8 us more a level
// than in a column.  But a column runs one after another, and where its tasks do
// not depend on each other that can cost more than the hand-offs: the leaves that a
// chain of cheap tasks releases one by one are all in column 1.
//
// Column order is chosen if
//  (a) the busiest worker's estimated cost is at most what the cheapest task of
//      every level would make it, plus kSlack a level.  A graph whose level mates
//      cost the same always is such a graph, and its columns then take no longer
//      than a path through its levels (times the tasks of a level each worker gets);
//  (b) or every list entry depends on the one before it: then a column is a path
//      of the graph, which no order runs any faster.
// Both sides measured (us, level / column, 256-word tasks, 8192 workers).  A chain of
// 500 empty tasks releasing leaves of R rounds: R = 0 1353 / 605, R = 24 (95 units of
// cost a level more than the chain) 1391 / 1046, R = 40 (159) 1354 / 1409, R = 96 (382)
// 1374 / 2660, R = 1024 (4079) 1385 / 23456.  Random DAGs of 5000 tasks in 120
// levels, log-normal rounds: sigma 0.3 (39) 394 / 358, 0.7 (82) 416 / 461, 1.2 (188) 694 /
// 862, 2 (701) 2534 / 3007.  Under (b) alone, a stencil of 300 x 40 with log-normal
// rounds about 64: sigma 1 (671) 790 / 723.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <vector>

namespace tg {

constexpr uint64_t kSlack = 96;  // cost units (about 11 ns each)

// level[v]: dependence levels of a graph's tasks; cost(v): estimated cost of a task;
// joined(u, v): whether task v depends on task u.
template <class Cost, class Joined>
bool columns_hold(const std::vector<uint32_t>& level, uint64_t nworkers, Cost&& cost, Joined&& joined) {
  const uint32_t N = (uint32_t)level.size();
  if (N == 0) return true;
  struct Level {
    uint64_t least = ~0ull;  // cost of the cheapest task
    uint32_t width = 0, seen = 0;
  };
  std::vector<Level> at;
  // level mates mostly follow each other: one run of equal levels at a time, in
  // registers (61,440 tasks 0.15 ms, a task at a time 0.35)
  auto runs = [&](auto&& f) {
    for (uint32_t v = 0, e; v < N; v = e) {
      for (e = v + 1; e < N && level[e] == level[v];) ++e;
      f(v, e, level[v]);
    }
  };
  uint32_t widest = 0;
  runs([&](uint32_t v, uint32_t e, uint32_t lv) {
    if (lv >= at.size()) at.resize((size_t)lv + 1);
    widest = std::max(widest, at[lv].width += e - v);
  });
  const uint32_t nw = (uint32_t)std::min<uint64_t>(nworkers ? nworkers : 1, widest);
  std::vector<uint64_t> load(nw, 0);
  runs([&](uint32_t v, uint32_t e, uint32_t lv) {
    Level& a = at[lv];
    uint64_t least = a.least;
    uint32_t w = a.seen % nw;
    a.seen += e - v;
    for (; v < e; ++v) {
      const uint64_t c = cost(v);
      least = std::min(least, c);
      load[w] += c;
      if (++w == nw) w = 0;
    }
    a.least = least;
  });
  uint64_t even = 0;
  for (const Level& a : at) even += a.least * ((a.width + nw - 1) / nw);
  if (*std::max_element(load.begin(), load.end()) <= even + kSlack * at.size()) return true;
  if (nw < widest) return false;  // two tasks of the widest level follow each other
  std::vector<std::vector<uint32_t>> by_level(at.size());
  for (uint32_t v = 0; v < N; ++v) by_level[level[v]].push_back(v);
  std::vector<uint32_t> last(nw, 0xFFFFFFFFu);
  for (const std::vector<uint32_t>& l : by_level)
    for (uint32_t i = 0; i < l.size(); ++i) {
      if (last[i] != 0xFFFFFFFFu && !joined(last[i], l[i])) return false;
      last[i] = l[i];
    }
  return true;
}

}  // namespace tg
