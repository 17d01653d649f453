// The points that a wavefront or block of the x-direction passes shares among
// its threads, as one index range.  Nothing here touches a point: only the
// ranges' bounds, so the header also compiles for the CPU.  Included by
// pgx_kernels.hpp after block_sync and wave_sync.
#pragma once
#include <stdint.h>

namespace pgx {

// The points of several ranges of a catalogue as one index range that NT
// threads walk together: one wavefront (NT = 64) or the whole block.  The
// x-direction passes give a line TPL threads, few on small grids, while a
// clustered catalogue puts most of a block's points on one or two lines.  The
// gathers share the points of a block's lines among all its threads; the
// scatters share those of a wavefront's lines within it, so that a line's LDS
// additions come from one wavefront and keep their order from run to run.
// build(range): range(r, s, e) gives the bounds of range r < NR; returns the
// number of points.  A Walk follows ascending combined indices, searching only
// when it leaves a range.  Combined indices have 64 bits: a point counts once
// for every line of the group that it reaches (up to 16 of a block's lines with
// TSC), so a catalogue below 2^31 points, which point indices fit, can have 2^35
// of them.  (Against 32-bit ones, which wrap there, the scatters take up to 2.4%
// longer: 504 and 515 us at 256^3, 7.45 and 7.51 ms with 3.6e8 HOD pairs; whole
// passes up to 0.4%.  A walk by steps with the point and the rest of its range in
// 32 bits took 8.4 ms there.)
template <int NR, int NT> struct PointRanges {
  int64_t off[NR];     // combined index of the range's first point
  uint32_t first[NR];  // its first point minus that, modulo 2^32
  int64_t part[NT / 64];
  int64_t count;       // all points
  __device__ __forceinline__ static void sync() {
    if constexpr (NT == 64) wave_sync();
    else block_sync();
  }
  template <typename Fn> __device__ __forceinline__ int64_t build(Fn&& range) {
    constexpr int PER = (NR + NT - 1) / NT;
    const int tid = threadIdx.x % NT, lane = tid & 63;
    int s[PER], c[PER];
    int64_t sum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      s[k] = c[k] = 0;
      const int r = tid * PER + k;
      if (r < NR) {
        int e = 0;
        range(r, s[k], e);
        c[k] = e - s[k];
      }
      sum += c[k];
    }
    int64_t inc = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int64_t u = __shfl_up(inc, d, 64);
      if (lane >= d) inc += u;
    }
    int64_t base = inc - sum, total = __shfl(inc, 63, 64);
    if constexpr (NT > 64) {
      if (lane == 63) part[tid >> 6] = inc;
      block_sync();
      total = 0;
#pragma unroll
      for (int w = 0; w < NT / 64; ++w) {
        const int64_t v = part[w];
        if (w < tid >> 6) base += v;
        total += v;
      }
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int r = tid * PER + k;
      if (r < NR) {
        off[r] = base;
        first[r] = (uint32_t)s[k] - (uint32_t)base;
      }
      base += c[k];
    }
    if (tid == 0) count = total;
    sync();
    return total;
  }
  __device__ __forceinline__ int find(int64_t i) const {
    int r = 0;
    constexpr int TOP = NR <= 1 ? 0 : 1 << (31 - __builtin_clz(NR - 1));
#pragma unroll
    for (int step = TOP; step > 0; step >>= 1)
      if (((NR & (NR - 1)) == 0 || r + step < NR) && off[r + step] <= i) r += step;
    return r;
  }
  struct Walk {
    int r = 0;
    int64_t next = 0;
    uint32_t shift = 0;
    // point of combined index i (ascending from call to call); its range is r
    __device__ __forceinline__ int point(const PointRanges& b, int64_t i) {
      if (i >= next) {
        r = b.find(i);
        next = r + 1 < NR ? b.off[r + 1] : INT64_MAX;
        shift = b.first[r];
      }
      return (int)((uint32_t)i + shift);
    }
  };
};

// Whether the NW wavefronts of a scatter block take the wavefronts' points one
// after another together, each into its own copy of the lines, instead of each
// its own: trips of 64 NW points plus the copies' sum and two barriers per
// wavefront (about three trips), against the trips of the most crowded one.
// Depends on the points only, so every run adds in the same order.
template <int NR, int NW>
__device__ __forceinline__ bool scatter_together(const PointRanges<NR, 64>* wave_ranges) {
  int64_t most = 0, trips = 0;
#pragma unroll
  for (int g = 0; g < NW; ++g) {
    const int64_t n = wave_ranges[g].count;
    most = n > most ? n : most;
    trips += n / (64 * NW) + 4;
  }
  return trips < most / 64;
}

}  // namespace pgx
