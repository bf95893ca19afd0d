// Prints, for the step counts given, where the forward pass leaves its loop over pairs of steps when it enters it four
// steps (or all of them) before the end.
#include <cstdio>
#include <cstdlib>

#include "pde_layout.hpp"

int main(int argc, char** argv) {
  for (int k = 1; k < argc; ++k) {
    const uint32_t steps = (uint32_t)std::strtoul(argv[k], nullptr, 10);
    uint32_t t = steps < 4u ? 0u : steps - 4u, turns = 0;
    for (; turns < 10u && rad::pde_pair_left(t, steps); t += 2) ++turns;
    std::printf("%u %u %u\n", steps, turns, t);
  }
  return 0;
}
