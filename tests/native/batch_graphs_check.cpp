// Reads batches "variant work by_wave", one a line, and prints for each the graph it replays, whether
// that is captured again, and what it launches.
#include <cstdio>

#include "batch_graphs.h"

int main() {
  mknn::BatchGraphs g;
  int variant;
  unsigned work, by_wave;
  while (std::scanf("%d %u %u", &variant, &work, &by_wave) == 3) {
    const mknn::BatchGraphs::Choice c = g.choose(variant, work, by_wave);
    std::printf("%d %d %u\n", c.graph, c.grown ? 1 : 0, c.launch);
  }
  return 0;
}
