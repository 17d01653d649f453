// Searches in sorted keys: range starts of a catalogue.  Also compiles for the
// CPU.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pgx {

// first index of the sorted keys with key >= t (binary search)
__device__ __forceinline__ int64_t lower_bound_key(const int32_t* __restrict__ key, int64_t n, int64_t t) {
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((int64_t)key[mid] < t)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

// starts[k] = first index of the sorted keys with key >= k div, for k in [0, nkeys]:
// the entries of thread t < nkeys / run + 1.  A search for the first of its `run`
// entries, then steps of doubling length from each entry to the next: one launch
// takes the place of a fill, a histogram and a two-launch scan, however the keys
// are spread.  us per launch with runs of 1, 4 and 8 (n keys over the entries):
// 1.3e6 entries 22, 18, 27 (n = 4e5) and 23, 33, 55 (2.6e6); 2.6e6 entries 38, 26,
// 28 (4e5) and 40, 41, 52 (2.6e6); 5.2e6 entries 65, 35, 39 (4e5), 99, 84, 119
// (1.1e7), 128, 120, 166 (3.1e7) and 174, 201, 255 (3.7e8); 1.0e7 entries 118, 55,
// 52 (4e5), 234, 171, 198 (4.4e7) and 271, 213, 261 (1.1e8); 5.2e7 entries 650, 280,
// 234 (3.6e6).  So runs of 4 above 2^21 entries, fewer than which leave wavefronts
// idle and the chain of searches as the time, and up to 16 keys per entry, where
// the steps get long.
__host__ __device__ constexpr int starts_run(int64_t n, int64_t nkeys) {
  return nkeys <= (1 << 21) || n > 16 * nkeys ? 1 : 4;
}
__device__ __forceinline__ void range_starts(const int32_t* __restrict__ key, int64_t n, int32_t div, int64_t nkeys,
                                             int run, int64_t t, int32_t* __restrict__ starts) {
  const int64_t k0 = t * run;
  if (k0 > nkeys) return;
  int64_t lo = lower_bound_key(key, n, k0 * div);
  for (int r = 0; r < run && k0 + r <= nkeys; ++r) {
    const int64_t v = (k0 + r) * div;
    // keys before lo are < v; step past those that still are
    int64_t step = 1;
    while (lo + step <= n && (int64_t)key[lo + step - 1] < v) {
      lo += step;
      step *= 2;
    }
    const int64_t m = step - 1 < n - lo ? step - 1 : n - lo;  // key[lo + step - 1] >= v, or past the end
    lo += lower_bound_key(key + lo, m, v);
    starts[k0 + r] = (int32_t)lo;
  }
}

}  // namespace pgx
