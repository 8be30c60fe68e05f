// Prints the shape that the stencil's planner (csrc/stencil_plan.h) takes for
// each "N steps" pair of the command line on a device of 256 CUs at 2.4 GHz.
#include <stdio.h>
#include <stdlib.h>

#include "../../paper_2004_05371_amd/csrc/stencil_plan.h"

int main(int argc, char** argv) {
  for (int i = 1; i + 1 < argc; i += 2) {
    const redsum::TilePlan t = redsum::plan_tiles(atoll(argv[i]), atoi(argv[i + 1]), 256, 2400000);
    printf("%d %d %d %d %lld\n", t.v, t.launches, t.k, t.m, (long long)t.waves);
  }
  return 0;
}
