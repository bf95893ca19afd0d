// Prints, for the chunks of 1 to 128 steps, "chunk own bound" for the parts of a context, or, with an argument, "chunk fails skip".
#include <cstdio>

#include "rnn_chunk.hpp"

int main(int argc, char**) {
  for (int chunk = 1; chunk <= 128; ++chunk)
    for (uint32_t k = 0; k < 8; ++k)
      std::printf("%d %u %u\n", chunk, k, argc > 1 ? rad::rnn_wide_skip(k, chunk) : rad::rnn_wide_polls(chunk, k));
  return 0;
}
