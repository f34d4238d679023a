// Bucket width of the dependence inference (plain C++, so the rule can be checked
// on a machine without a GPU).
//
// An interval has one entry in every bucket it overlaps, and an entry is
// compared with the others of its bucket.  Wide buckets put unrelated intervals
// together, narrow ones cut long intervals into many entries.
#pragma once
#include <stdint.h>

namespace tg {

// The shift (buckets of width 2^shift) of the sorted entries, for `count`
// non-empty intervals of `length` elements in all, cls[c] of them of length
// [2^c, 2^(c + 1)).
//
// It is the length class that holds the median element of all intervals (half of
// the length, rounded down to the class, lies in shorter classes or this one): most
// elements then belong to intervals of one to three entries, and short intervals
// beside long ones (halos) do not shrink the buckets.  But at most four times the
// mean length m: about count + length / width entries, each compared with the
// entries per bucket, make (count + length / width)^2 x width comparisons per
// element of the index space, which is least at width m and 1.6 times that at 4 m.
// Where a few intervals over much of the index space hold most of the elements (a
// global read, a checkpoint, a reduction), the median's class is theirs and would
// put all others into a handful of buckets.  Halo program of 65,536 tasks: 2^14 by
// either rule; with two whole-array readers a sweep 2^16 and 2e8 comparisons, where
// the median alone takes 2^24, one bucket and 3.9e10 (the inference: 1.2 and 39 ms).
inline uint32_t entry_shift(const uint64_t* cls, uint64_t count, long double length, uint64_t space,
                            uint64_t max_buckets) {
  long double total = 0, upto = 0;
  for (int c = 0; c < 64; ++c) total += (long double)cls[c] * (long double)(1ull << c);
  uint32_t shift = 0;
  for (; shift < 63; ++shift) {
    upto += (long double)cls[shift] * (long double)(1ull << shift);
    if (2 * upto >= total) break;
  }
  while (shift && (long double)(1ull << shift) * (long double)count > 4 * length) --shift;
  while (shift < 63 && ((space - 1) >> shift) + 1 > max_buckets) ++shift;
  return shift;
}

}  // namespace tg
