// Step counts of the reaction-diffusion kernels.  Plain constexpr code: it compiles without HIP as well.
#pragma once
#include <cstdint>

namespace rad {

// Whether two steps or more are left after t <= steps of them.  (steps goes up to 2^32 - 2, where t + 2 would be 0.)
constexpr bool pde_pair_left(uint32_t t, uint32_t steps) { return steps - t >= 2u; }

}  // namespace rad
