// Checks of the inference's bucket width (tg_buckets.h) on the CPU: the entries
// and comparisons that the chosen width gives a program, counted interval by
// interval, against every other width.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "tg_buckets.h"

struct Iv {
  uint64_t lo, hi;
};

static int failures = 0;

// Entries and comparisons (the sum over buckets of the square of their entries)
// at one shift.
static void count(const std::vector<Iv>& iv, uint64_t space, uint32_t shift, double* entries, double* work) {
  // +1 / -1 at the first bucket and past the last: running sums are list lengths
  std::vector<long> d((size_t)((space - 1) >> shift) + 2, 0);
  *entries = *work = 0;
  for (const Iv& x : iv) {
    d[x.lo >> shift]++;
    d[((x.hi - 1) >> shift) + 1]--;
    *entries += (double)(((x.hi - 1) >> shift) - (x.lo >> shift) + 1);
  }
  long n = 0;
  for (long v : d) {
    n += v;
    *work += (double)n * (double)n;
  }
}

// The chosen width's comparisons are at most `factor` times the least over all
// widths, and `most` entries an interval are enough for it.
static void check(const char* what, const std::vector<Iv>& iv, uint64_t space, uint64_t max_buckets, double factor,
                  double most) {
  uint64_t cls[64] = {};
  long double length = 0;
  for (const Iv& x : iv) {
    cls[63 - __builtin_clzll(x.hi - x.lo)]++;
    length += (long double)(x.hi - x.lo);
  }
  const uint32_t s = tg::entry_shift(cls, iv.size(), length, space, max_buckets);
  double e, w, least = 1e300;
  for (uint32_t t = 0; t <= 40; ++t) {
    if (((space - 1) >> t) + 1 > max_buckets) continue;
    count(iv, space, t, &e, &w);
    if (w < least) least = w;
  }
  count(iv, space, s, &e, &w);
  const bool ok = w <= factor * least && e <= most * (double)iv.size();
  std::printf("%s %s: shift %u, %.3g entries, %.3g comparisons, least %.3g\n", ok ? "ok  " : "FAIL", what, s, e, w, least);
  failures += !ok;
}

// P subregions of S elements, each rewritten in every sweep with a halo of up to
// 32 elements on either side, and `readers` whole-array readers a sweep.
static std::vector<Iv> halo(uint64_t P, uint64_t S, int sweeps, int readers) {
  std::vector<Iv> v;
  for (int k = 0; k < sweeps; ++k) {
    for (uint64_t p = 0; p < P; ++p) {
      v.push_back({p * S, p * S + S});
      if (p) v.push_back({p * S - 1 - (uint64_t)rand() % 32, p * S});
      if (p + 1 < P) v.push_back({p * S + S, p * S + S + 1 + (uint64_t)rand() % 32});
    }
    for (int r = 0; r < readers; ++r) v.push_back({0, P * S});
  }
  return v;
}

int main() {
  constexpr uint64_t kMany = 1ull << 25, kFew = 1ull << 17;  // buckets that the two entry points allow
  srand(1);
  for (uint64_t b : {kMany, kFew}) {
    for (int readers : {0, 1, 2, 3, 8}) check("halo 1024 x 64", halo(1024, 16384, 64, readers), 1024 * 16384, b, 4, 3);
    check("halo of ragged subregions", halo(700, 10000, 30, 4), 700 * 10000, b, 4, 3);
    {  // many short writers, whole-array readers
      std::vector<Iv> v;
      for (uint64_t i = 0; i < 200000; ++i) v.push_back({16 * i, 16 * i + 16});
      for (int r = 0; r < 200; ++r) v.push_back({0, 16 * 200000});
      check("200 readers of 200,000 writers", v, 16 * 200000, b, 4, 4);
      v.push_back({0, 16 * 200000});
      v.resize(200001);
      check("one reader of 200,000 writers", v, 16 * 200000, b, 4, 4);
    }
    {  // lengths over five orders of magnitude
      std::vector<Iv> v;
      const uint64_t space = 1 << 22;
      for (int i = 0; i < 20000; ++i) {
        const uint64_t len = 1ull << (rand() % 20), lo = (uint64_t)rand() % (space - len);
        v.push_back({lo, lo + len});
      }
      check("lengths of all classes", v, space, b, 4, 60);
    }
    {  // one element each, and one interval of everything
      std::vector<Iv> v;
      for (uint64_t i = 0; i < 100000; ++i) v.push_back({i, i + 1});
      check("single elements", v, 100000, b, 4, 3);
      v.push_back({0, 100000});
      check("single elements and one fill", v, 100000, b, 4, 3);
      check("one interval", {{5, 6}}, 100, b, 1e9, 1);
      check("the whole space", {{0, 100}, {0, 100}}, 100, b, 4, 2);
    }
  }
  if (!failures) std::printf("all cases pass\n");
  return failures != 0;
}
