// Launches of the sweep calls argv[4..] (sweeps each) of one lattice without a
// GPU (fake_hip.hpp): argv[1] "square", "buffers" (the same in the caller's
// buffers), "heat bath" or "cube", L, q.  Prints, per call, plain and cooperative launches.  A colour-split sweep is two launches, the pack and
// the unpack one each; 64 band sweeps are one cooperative launch and a fold.
#include <stdio.h>

#include "fake_hip.hpp"

#include "potts.h"

int main(int argc, char **argv) {
  if (argc < 5) return 2;
  const bool cube = argv[1][0] == 'c';
  potts_state *s = nullptr;
  potts3d_state *c = nullptr;
  const int L = atoi(argv[2]), q = atoi(argv[3]);
  void *mine[2] = {nullptr, nullptr};
  for (int k = 0; k < 2 && argv[1][0] == 'b'; ++k)
    if (hipMalloc(&mine[k], (size_t)L * L)) return 1;
  if (cube ? potts3d_init(L, q, 1, POTTS_RANDOM, &c)
           : potts_init_ex(L, q, 1, POTTS_RANDOM, mine[0], mine[1], (size_t)L * L, nullptr, 0, &s))
    return 1;
  for (int k = 4; k < argc; ++k) {
    fake::launches = fake::cooperative = 0;
    const int n = atoi(argv[k]);
    if (cube ? potts3d_sweep(c, 0.5, n) : argv[1][0] == 'h' ? potts_sweep_heatbath(s, 1.0, n) : potts_sweep(s, 1.0, n)) return 1;
    printf("%ld+%ld\n", fake::launches, fake::cooperative);
  }
  if (cube)
    potts3d_free(c);
  else
    potts_free(s);
  return 0;
}
