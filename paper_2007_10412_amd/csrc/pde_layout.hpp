// Sizes and step counts of the reaction-diffusion kernels, shared by the entry points and the launch.  Plain host code and
// constexpr functions: it compiles without HIP as well.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>

namespace rad {

constexpr int kPdeRuns = 16;        // runs that a problem's workspace has room for, and counters
constexpr int kPdeWaves = 4;        // stencil waves at most, and sampling waves of each of the two sets
constexpr int kPdeCells = 256;      // cells of a stencil wave, or of a sampling wave, at most

// Entries that a run of `total` draws at fraction p has room for: eight standard deviations above the mean.
inline int64_t pde_run_capacity(double total, double p) {
  return (int64_t)std::min(std::ceil(total * p + 8.0 * std::sqrt(total * p * (1.0 - p))) + 64.0, total);
}

// What a problem's workspace is sized for: kPdeRuns runs of 62 cells each at steps + 1 times.  (Two grid rows have 62 cells at
// most, the whole grid 961 = 15.5 x 62; the runs below take less: fewer cells together, and eight deviations of longer runs.)
inline int64_t pde_workspace_run(int64_t steps, double p) { return pde_run_capacity(62.0 * ((double)steps + 1.0), p); }

// A run for each sampling wave: the 256 cells of its stencil wave (the last one less) at the even or at the odd times.
struct PdeRunLayout { int64_t at[2][kPdeWaves], cap[2][kPdeWaves], total; };
inline PdeRunLayout pde_run_layout(int cells, int64_t steps, double p) {
  PdeRunLayout l{};
  for (int odd = 0; odd < 2; ++odd)
    for (int w = 0; w < kPdeWaves; ++w) {
      const int own = std::min(kPdeCells, std::max(0, cells - w * kPdeCells));
      l.at[odd][w] = l.total;
      l.cap[odd][w] = pde_run_capacity(own * (double)((steps + 2 - odd) / 2), p);
      l.total += l.cap[odd][w];
    }
  return l;
}

// Whether two steps or more are left after t <= steps of them.  (steps goes up to 2^32 - 2, where t + 2 would be 0.)
constexpr bool pde_pair_left(uint32_t t, uint32_t steps) { return steps - t >= 2u; }

}  // namespace rad
