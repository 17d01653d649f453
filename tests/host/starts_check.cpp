// Range starts (csrc/pgx_starts.hpp) on the CPU, thread by thread, against
// std::lower_bound: every run length, divisors above 1, keys sparse, dense, all
// equal, at the ends and absent.  Built with AddressSanitizer, which stops at a
// read past the keys or a write past the entries.  Exits non-zero on the first
// failed check.
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>

#include "../../paper_1705_03464_amd/csrc/pgx_starts.hpp"

int main() {
  std::mt19937_64 rng(7);
  for (int trial = 0; trial < 6000; ++trial) {
    const int64_t nkeys = 1 + (int64_t)(rng() % 300);
    const int32_t div = trial % 3 == 0 ? 1 + (int32_t)(rng() % 70) : 1;
    const int64_t span = nkeys * div;
    const size_t n = trial % 7 == 0 ? rng() % 3 : rng() % 5000;
    std::vector<int32_t> key(n);
    const int kind = trial % 5;
    const int32_t one = (int32_t)(rng() % (uint64_t)span);
    for (auto& k : key) {
      k = (int32_t)(rng() % (uint64_t)span);
      if (kind == 1) k = one;                              // one range holds everything
      if (kind == 2) k = rng() % 2 ? 0 : (int32_t)span - 1;  // the ends only
      if (kind == 3) k = k % 13 * (int32_t)(span / 13 + 1) % (int32_t)span;  // long gaps
    }
    std::sort(key.begin(), key.end());
    for (int run : {1, 2, 4, 8, 16}) {
      std::vector<int32_t> starts((size_t)nkeys + 1, -1);
      for (int64_t t = 0; t < nkeys / run + 1 + 5; ++t)  // (threads past the last entry do nothing)
        pgx::range_starts(key.data(), (int64_t)n, div, nkeys, run, t, starts.data());
      for (int64_t k = 0; k <= nkeys; ++k) {
        const int64_t want = std::lower_bound(key.begin(), key.end(), k * div,
                                              [](int32_t a, int64_t b) { return (int64_t)a < b; }) - key.begin();
        if (starts[(size_t)k] != want) {
          std::fprintf(stderr, "trial %d run %d entry %lld: %d, not %lld\n", trial, run, (long long)k,
                       starts[(size_t)k], (long long)want);
          return 1;
        }
      }
    }
  }
  static_assert(pgx::starts_run(1, 1 << 21) == 1 && pgx::starts_run(1, (1 << 21) + 1) == 4, "");
  static_assert(pgx::starts_run(16 * 3000000ll, 3000000) == 4 && pgx::starts_run(16 * 3000000ll + 1, 3000000) == 1, "");
  std::printf("range start checks passed\n");
  return 0;
}
