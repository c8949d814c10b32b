// Which captured graph a batch replays.  Plain host code, so that it can be checked without a GPU.
#pragma once
#include <cstdint>

namespace mknn {

// A register class of more than 16 neighbours goes by rows or by waves, from batch to batch.  A
// graph launches a class by one of them only: the other's launch would dispatch its whole grid
// for nothing (a plan of 64 requests and 262144 queries, batches of 4 x 4096 queries: 7-15 us
// of 410-480).  So there is a graph for every division of the three classes that has
// occurred, and it gains a class when one first has work in it.
struct BatchGraphs {
  static constexpr int kDivisions = 8;
  uint32_t waves = 0;                         // classes (bit c) whose last work went by waves
  uint32_t classes[2][kDivisions] = {};       // per variant: the classes each graph launches

  struct Choice {
    int graph;         // which of the variant's graphs
    bool grown;        // it gains a class: to be captured again
    uint32_t launch;   // what it launches: bit c by rows, bit c + 4 by waves
  };
  // work: the classes with work in this batch; by_wave: those of them that go by waves.  A class
  // without work keeps its side, so that it opens no division of its own.
  Choice choose(int variant, uint32_t work, uint32_t by_wave) {
    waves = (waves & ~work) | (by_wave & work);
    Choice c;
    c.graph = (int)((waves >> 1) & (kDivisions - 1));
    uint32_t &have = classes[variant][c.graph];
    c.grown = (work & ~have) != 0;
    have |= work;
    c.launch = (have & ~waves) | ((have & waves) << 4);
    return c;
  }
};

}  // namespace mknn
