// Device memory of a server of four L = 512 jobs (fake_hip.hpp) with a budget of
// their lattices and rings times argv[1] / 4: prints what the peak exceeded the
// budget by, in KiB, and the kernel launches.
#include <stdio.h>

#include "fake_hip.hpp"

#include "potts.h"

int main(int argc, char **argv) {
  if (argc != 2) return 2;
  const int L = 512, q = 6, n = 24, slots = 32;  // ring slots: a power of two above n
  const size_t job = (size_t)L * L + (size_t)slots * (q + 1) * 8, budget = job * (size_t)atoi(argv[1]);
  potts_server_cfg cfg = {};
  cfg.hbm_budget = (int64_t)budget;
  potts_server *s = nullptr;
  if (potts_server_start(&cfg, &s)) return 1;
  double betas[3] = {1.0, 1.1, 1.2};
  int64_t sweeps[3] = {n, n, n};
  potts_request req = {};
  req.L = L;
  req.q = q;
  req.seed = 1;
  req.npoints = 3;
  req.betas = betas;
  req.sweeps = sweeps;
  for (int i = 0; i < 4; ++i) {
    int64_t ticket;
    if (potts_server_submit(s, &req, &ticket)) return 1;
  }
  if (potts_server_drain(s, 60000)) return 1;
  const size_t peak = fake::peak;
  potts_server_stop(s);
  printf("%zu %ld\n", peak > budget ? (peak - budget + 1023) / 1024 : 0, fake::launches);
  return 0;
}
