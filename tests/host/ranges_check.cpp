// The shared point ranges of the x-direction passes (csrc/pgx_ranges.hpp) run
// on the CPU: every thread of the wavefront or block is a std::thread, the
// synchronisations and the lane shuffles std::barriers around a host array.
// The real build, find and Walk are compared with 64-bit sums in order, for
// ordinary ranges and for ranges as long as a catalogue of 2^31 - 1 points
// makes them, each point once per line of the group that it reaches (16 times
// with TSC): totals of up to 2^35.  Built with UndefinedBehaviorSanitizer, which
// also stops at a signed sum that wraps, and AddressSanitizer.  Exits non-zero
// on the first failed check.
#include <barrier>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <random>
#include <thread>
#include <vector>

#include <hip/hip_runtime.h>

// one emulated block: lanes' shuffle slots and the barriers
struct Emu {
  int nt;
  std::barrier<> block;
  std::vector<std::unique_ptr<std::barrier<>>> wave;
  std::vector<int64_t> slot;
  explicit Emu(int n) : nt(n), block(n), slot((size_t)n) {
    for (int w = 0; w < n / 64; ++w) wave.push_back(std::make_unique<std::barrier<>>(64));
  }
};
static Emu* emu = nullptr;
static thread_local struct { unsigned x; } threadIdx;

namespace pgx {
inline void block_sync() { emu->block.arrive_and_wait(); }
inline void wave_sync() { emu->wave[threadIdx.x / 64]->arrive_and_wait(); }
}  // namespace pgx
template <typename V> V lane_value(V v, int src) {
  emu->slot[threadIdx.x] = (int64_t)v;
  pgx::wave_sync();
  const V r = (V)emu->slot[threadIdx.x / 64 * 64 + (unsigned)src];
  pgx::wave_sync();
  return r;
}
template <typename V> V __shfl_up(V v, int d, int) {
  const int lane = (int)(threadIdx.x & 63u);
  return lane_value(v, lane >= d ? lane - d : lane);
}
template <typename V> V __shfl(V v, int src, int) { return lane_value(v, src); }

#include "../../paper_1705_03464_amd/csrc/pgx_ranges.hpp"

#define CHECK(c, ...)                                              \
  do {                                                             \
    if (!(c)) {                                                    \
      std::fprintf(stderr, "check failed: %s: ", #c);              \
      std::fprintf(stderr, __VA_ARGS__);                           \
      std::fprintf(stderr, "\n");                                  \
      std::exit(1);                                                \
    }                                                              \
  } while (0)

// ranges [s, e) of one group; NT threads build, then one walks
template <int NR, int NT> void check(const std::vector<int>& s, const std::vector<int>& e, std::mt19937_64& rng) {
  Emu block(NT);
  emu = &block;
  pgx::PointRanges<NR, NT> pr;
  std::vector<int64_t> totals(NT);
  std::vector<std::thread> lanes;
  for (int t = 0; t < NT; ++t)
    lanes.emplace_back([&, t] {
      threadIdx.x = (unsigned)t;
      totals[t] = (int64_t)pr.build([&](int r, int& a, int& b) {
        a = s[r];
        b = e[r];
      });
    });
  for (auto& l : lanes) l.join();
  std::vector<int64_t> at(NR + 1, 0);
  for (int r = 0; r < NR; ++r) at[r + 1] = at[r] + (e[r] - s[r]);
  const int64_t total = at[NR];
  for (int t = 0; t < NT; ++t)
    CHECK(totals[t] == total, "<%d, %d> thread %d: total %lld of %lld", NR, NT, t, (long long)totals[t], (long long)total);
  CHECK((int64_t)pr.count == total, "<%d, %d>: count", NR, NT);
  // the ends of every range and some points inside, ascending as a walk has them
  std::vector<int64_t> idx;
  std::vector<int> of;
  for (int r = 0; r < NR; ++r) {
    const int64_t n = at[r + 1] - at[r];
    if (n == 0) continue;
    std::vector<int64_t> in = {0, n - 1, (int64_t)(rng() % (uint64_t)n)};
    if (in[2] < in[1]) std::swap(in[1], in[2]);
    for (int64_t k : in) {
      idx.push_back(at[r] + k);
      of.push_back(r);
    }
  }
  typename pgx::PointRanges<NR, NT>::Walk walk;
  for (size_t k = 0; k < idx.size(); ++k) {
    const int r = of[k];
    const int64_t p = s[r] + (idx[k] - at[r]);
    CHECK(pr.find(idx[k]) == r, "<%d, %d>: find(%lld)", NR, NT, (long long)idx[k]);
    CHECK((int64_t)walk.point(pr, idx[k]) == p && walk.r == r, "<%d, %d>: point %lld", NR, NT, (long long)idx[k]);
  }
}

template <int NR, int NT> void check_all(std::mt19937_64& rng) {
  const int most = 0x7FFFFFFE;  // points of the largest catalogue
  for (int kind = 0; kind < 6; ++kind) {
    std::vector<int> s(NR), e(NR);
    for (int r = 0; r < NR; ++r) {
      int n = 0;
      if (kind == 0) n = (int)(rng() % 40);
      if (kind == 1) n = rng() % 4 ? 0 : (int)(rng() % 3000);
      if (kind == 2) n = r == NR / 2 ? most : 0;              // one line holds everything
      if (kind == 3) n = r % 16 < 9 ? most / 16 : (int)(rng() % 3);  // 1.3e8 points, every source
      if (kind == 4) n = r % (NR > 16 ? NR / 16 : 1) == 0 ? most : 0;  // every line of the group reads all
      if (kind == 5) n = (int)(rng() % (uint64_t)(most / (NR > 16 ? NR / 16 : 1)));
      s[r] = (int)(rng() % (uint64_t)(most - n + 1));
      e[r] = s[r] + n;
    }
    check<NR, NT>(s, e, rng);
  }
}

template <int NW> void check_together(std::mt19937_64& rng) {
  typedef pgx::PointRanges<4, 64> R;
  std::vector<R> w(NW);
  for (int trial = 0; trial < 400; ++trial) {
    int64_t most = 0, trips = 0;
    for (int g = 0; g < NW; ++g) {
      const int bits = (int)(rng() % 35);
      const int64_t n = (int64_t)(rng() % ((uint64_t)1 << bits));
      w[g].count = (decltype(R::count))n;
      most = n > most ? n : most;
      trips += n / (64 * NW) + 4;
    }
    CHECK((pgx::scatter_together<4, NW>(w.data())) == (trips < most / 64), "scatter_together<%d>", NW);
  }
}

int main() {
  std::mt19937_64 rng(11);
  // gathers: the sources of a block's lines (CIC, TSC) at 64^3, 256^3 and 512^3
  check_all<256, 256>(rng);
  check_all<1024, 256>(rng);
  check_all<64, 256>(rng);
  check_all<128, 256>(rng);
  // scatters: the sources of a wavefront's lines
  check_all<64, 64>(rng);
  check_all<256, 64>(rng);
  check_all<8, 64>(rng);
  check_all<32, 64>(rng);
  // dual form
  check_all<72, 64>(rng);
  check_all<9, 64>(rng);
  check_all<4, 64>(rng);
  check_together<4>(rng);
  std::printf("point range checks passed\n");
  return 0;
}
