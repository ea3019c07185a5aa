// Prints every L % 16 == 0 up to 65520 and q for which the multi-sweep tile
// kernel has no automatic shape (none is expected), then the number of sizes
// looked at.
#include <stdio.h>

#include "tiles.hpp"

int main() {
  unsigned n = 0;
  for (uint32_t q : {2u, 16u, 17u, 64u, 65u, 128u, 256u})
    for (uint32_t L = 16; L <= potts::kTileMaxL; L += 16, ++n)
      for (int64_t nsweeps : {(int64_t)1, (int64_t)5, (int64_t)200}) {
        potts::TileParams p{};
        p.L = L;
        p.q = q;
        if (!potts::auto_tile_shape(p, nsweeps) || !p.tx || !p.ty)
          printf("none %u %u %lld\n", L, q, (long long)nsweeps);
      }
  printf("sizes %u\n", n);
  return 0;
}
