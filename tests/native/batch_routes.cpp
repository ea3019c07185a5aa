// Kernel launches of a run of `count` jobs of L, q and n sweeps (argv) without a
// GPU (fake_hip.hpp): one where the LDS-resident kernel takes them all, several
// where the multi-sweep tiles do, two a sweep in the strip kernel.
#include <stdio.h>

#include "fake_hip.hpp"

#include "potts.h"

int main(int argc, char **argv) {
  if (argc != 5) return 2;
  potts_job job = {};
  job.L = atoi(argv[2]);
  job.q = atoi(argv[3]);
  job.seed = 1;
  job.beta = 1.0;
  job.nsweeps = atoi(argv[4]);
  const std::vector<potts_job> jobs((size_t)atoi(argv[1]), job);
  potts_batch *b = nullptr;
  if (potts_batch_create(jobs.data(), (int32_t)jobs.size(), nullptr, &b)) return 1;
  fake::launches = 0;
  if (potts_batch_run(b)) return 1;
  printf("%ld\n", fake::launches);
  potts_batch_free(b);
  return 0;
}
