// Prints "chunk own bound" for the chunks of 1 to 128 steps and the parts of a context.
#include <cstdio>

#include "rnn_chunk.hpp"

int main() {
  for (int chunk = 1; chunk <= 128; ++chunk)
    for (uint32_t own = 0; own < 8; ++own) std::printf("%d %u %u\n", chunk, own, rad::rnn_wide_polls(chunk, own));
  return 0;
}
