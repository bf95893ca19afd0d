// Waits of the recurrent kernels that take a chunk of time steps per launch.  Plain constexpr code: it compiles without HIP as well.
#pragma once
#include <cstdint>

namespace rad {

// Looks at the flags before a launch gives up, for chunks of `chunk` steps.  A look takes 0.3 us or more: 0.6 ms for chunks of 32
// steps, several times what the other kernels of a training step hold a CU and what another context's chunk takes, and a
// quarter of what the stand-in takes for a chunk; longer chunks wait longer, in whole multiples of that.  `own`, 0 to 7, is the
// context's part and decides which of two launches gives way: bounds of different contexts are 256 looks apart or more,
// whatever the chunks of their models.
constexpr uint32_t rnn_wide_polls(int chunk, uint32_t own) {
  return 2048u * (uint32_t)(chunk < 48 ? 1 : (chunk + 16) / 32) + 256u * own;
}

// Launches that go to the stand-in without trying after the (fails + 1)-th one in a row gave up: none after the first, then about
// 32, 96, 224 and up to 480 time steps' worth.
constexpr uint32_t rnn_wide_skip(uint32_t fails, int chunk) {
  const uint32_t steps = 32u * ((1u << (fails < 4u ? fails : 4u)) - 1u), per = chunk < 32 ? 32u : (uint32_t)chunk;
  return (steps + per / 2u) / per;
}

}  // namespace rad
