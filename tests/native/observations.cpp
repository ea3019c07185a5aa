// Pinned allocations after each of six calls of one sweep and its observables on
// a lattice of L = argv[1] (fake_hip.hpp).
#include <stdio.h>

#include "fake_hip.hpp"

#include "potts.h"

int main(int argc, char **argv) {
  potts_state *s = nullptr;
  if (argc != 2 || potts_init(atoi(argv[1]), 6, 1, POTTS_RANDOM, &s)) return 1;
  const long before = fake::host_allocations;
  for (int k = 0; k < 6; ++k) {
    potts_obs o;
    if (potts_sweep(s, 1.0, 1) || potts_observables(s, &o)) return 1;
    printf("%ld\n", fake::host_allocations - before);
  }
  potts_free(s);
  return 0;
}
