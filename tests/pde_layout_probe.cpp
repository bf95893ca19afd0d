// With step counts: prints where the forward pass leaves its loop over pairs of steps when it enters it four steps (or all of
// them) before the end.  With "runs": for all grids and several step counts and fractions, cells, steps, 10^6 p, the entries that
// the runs of the sampling waves have room for, their overlaps and those of the workspace.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "pde_layout.hpp"

static void runs() {
  const double fractions[] = {1e-6, 1e-4, 0.01, 0.1, 0.25, 0.5, 0.9, 0.999, 1.0};
  for (int n = 2; n <= 32; ++n)
    for (int64_t steps : {1ll, 2ll, 3ll, 10ll, 63ll, 1000ll, 40960ll, 4000000ll})
      for (double p : fractions) {
        const int cells = (n - 1) * (n - 1);
        const rad::PdeRunLayout l = rad::pde_run_layout(cells, steps, p);
        int64_t at = 0, wrong = 0, draws = 0;
        for (int odd = 0; odd < 2; ++odd)
          for (int w = 0; w < rad::kPdeWaves; ++w) {
            wrong += l.at[odd][w] < at || l.cap[odd][w] < 0;
            at = l.at[odd][w] + l.cap[odd][w];
            draws += l.cap[odd][w];
          }
        std::printf("%d %lld %.0f %lld %lld %lld\n", cells, (long long)steps, p * 1e6, (long long)draws,
                    (long long)(wrong + (at > l.total)), (long long)(rad::kPdeRuns * rad::pde_workspace_run(steps, p)));
      }
}

int main(int argc, char** argv) {
  if (argc == 2 && !std::strcmp(argv[1], "runs")) { runs(); return 0; }
  for (int k = 1; k < argc; ++k) {
    const uint32_t steps = (uint32_t)std::strtoul(argv[k], nullptr, 10);
    uint32_t t = steps < 4u ? 0u : steps - 4u, turns = 0;
    for (; turns < 10u && rad::pde_pair_left(t, steps); t += 2) ++turns;
    std::printf("%u %u %u\n", steps, turns, t);
  }
  return 0;
}
