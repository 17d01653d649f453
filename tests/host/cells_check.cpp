// The cell list's size (cells_per_side, csrc/pgx_host.hpp) over box sizes and
// largest separations of every ratio: the last cell's 32-bit index does not
// wrap (UndefinedBehaviorSanitizer stops at it), every cell is at least the
// largest separation wide, and lists that fit are as fine as the separation
// allows.  Exits non-zero on the first failed check.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "../../paper_1705_03464_amd/csrc/pgx_host.hpp"

int main() {
  std::mt19937_64 rng(5);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  for (int i = 0; i < 200000; ++i) {
    const double L = std::pow(10.0, 4.0 * u(rng)), smax = L / 3.0 * std::pow(10.0, -12.0 * u(rng) * u(rng));
    const int nc = pgx::cells_per_side(L, smax), c = nc - 1;
    const int last = (c * nc + c) * nc + c;
    const double want = std::floor(L / (smax * (1.0 + 1e-12)));
    const bool ok = last >= 0 && (int64_t)last + 1 == (int64_t)nc * nc * nc && L / nc >= smax &&
                    (want > pgx::kMaxCellsPerSide || nc == (int)want);
    if (!ok) {
      std::fprintf(stderr, "L %g, largest separation %g: %d cells per side, last index %d\n", L, smax, nc, last);
      return 1;
    }
  }
  std::printf("cell list checks passed\n");
  return 0;
}
