// A served job of L = 256 whose tile launches lack their second lattice, totals or
// one of their tables: the four allocations after the job's own two fail one after
// the other (fake_hip.hpp).  Prints the status of each job.
#include <stdio.h>

#include "fake_hip.hpp"

#include "potts.h"

int main() {
  for (long fail = 0; fail < 4; ++fail) {
    potts_server *s = nullptr;
    if (potts_server_start(nullptr, &s)) return 1;
    double beta = 1.0;
    int64_t n = 64, ticket;
    potts_request req = {};
    req.L = 256;
    req.q = 6;
    req.seed = 1;
    req.npoints = 1;
    req.betas = &beta;
    req.sweeps = &n;
    fake::fail_at = fake::allocations + 2 + fail;
    if (potts_server_submit(s, &req, &ticket)) return 1;
    const int rc = potts_server_drain(s, 60000);
    fake::fail_at = -1;
    potts_served info = {};
    potts_summary sum = {};
    if (!rc) potts_server_collect(s, ticket, &info, &sum, nullptr);
    printf("%d\n", rc ? rc : info.status);
    potts_server_stop(s);
  }
  return 0;
}
