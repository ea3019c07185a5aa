// Sweep calls in which one allocation after another fails (fake_hip.hpp), on
// lattices that some kernel sweeps without any memory of its own: argv[1] "square",
// "heat bath", "cube" or "nnn", L, q, sweeps.  Prints the calls that ended well out
// of all, and the launches of the last one, after every allocation has failed.
#include <stdio.h>

#include "fake_hip.hpp"

#include "potts.h"

int main(int argc, char **argv) {
  if (argc != 5) return 2;
  const char kind = argv[1][0];
  const int L = atoi(argv[2]), q = atoi(argv[3]), n = atoi(argv[4]);
  int calls = 0, good = 0;
  for (long fail = 0; fail <= 6; ++fail) {
    potts_state *s = nullptr;
    potts3d_state *c = nullptr;
    potts_nnn_state *d = nullptr;
    if (kind == 'c' ? potts3d_init(L, q, 1, POTTS_RANDOM, &c)
                    : kind == 'n' ? potts_nnn_init(L, q, 1, POTTS_RANDOM, &d) : potts_init(L, q, 1, POTTS_RANDOM, &s))
      return 1;
    fake::fail_at = fake::allocations + fail;
    fake::fail_all = fail == 6;
    for (int k = 0; k < 2; ++k, ++calls) {
      fake::launches = 0;
      good += (kind == 'c'   ? potts3d_sweep(c, 0.5, n)
               : kind == 'n' ? potts_nnn_sweep(d, 0.8, 0.5, n)
               : kind == 'h' ? potts_sweep_heatbath(s, 1.0, n)
                             : potts_sweep(s, 1.0, n)) == 0;
    }
    fake::fail_at = -1;
    fake::fail_all = false;
    potts_free(s);
    potts3d_free(c);
    potts_nnn_free(d);
  }
  printf("%d/%d %ld\n", good, calls, fake::launches);
  return 0;
}
