// Runs of a batch in which one allocation after another fails (fake_hip.hpp).
// Every device-to-device copy of a run has to go to the lattice of a job of that
// size.  Prints the runs that ended well and the copies that did not.
#include <stdio.h>

#include "fake_hip.hpp"

#include "potts.h"

int main() {
  // the larger lattice is of another class of q than the smaller one
  potts_job jobs[2] = {};
  jobs[0].L = 512;
  jobs[0].q = 6;
  jobs[1].L = 64;
  jobs[1].q = 200;
  for (int j = 0; j < 2; ++j) {
    jobs[j].seed = 1;
    jobs[j].beta = 1.0;
    jobs[j].nsweeps = 1;
  }
  const potts_batch_opts opts = {};
  int good = 0, bad = 0;
  for (long fail = 0; fail < 6; ++fail) {
    potts_batch *b = nullptr;
    if (potts_batch_create(jobs, 2, &opts, &b)) return 1;
    const void *lattice[2];
    for (int j = 0; j < 2; ++j) {
      std::vector<uint8_t> spins((size_t)jobs[j].L * jobs[j].L);
      if (potts_batch_spins(b, j, spins.data())) return 1;
      lattice[j] = fake::host_copies.back().src;
    }
    fake::device_copies.clear();
    fake::fail_at = fake::allocations + fail;
    good += potts_batch_run(b) == 0;
    fake::fail_at = -1;
    for (const fake::Copy &c : fake::device_copies) {
      const int j = c.dst == lattice[0] ? 0 : c.dst == lattice[1] ? 1 : -1;
      bad += j < 0 || c.bytes != (size_t)jobs[j].L * jobs[j].L;
    }
    potts_batch_free(b);
  }
  printf("runs %d misplaced %d\n", good, bad);
  return 0;
}
