"""Batches and the serving loop on multi-sweep tile launches (few small
lattices), bit for bit against the oracle: lattices of several sizes, classes
of q and sweep counts in one launch (some end turns before others, some on an
odd number of turns), rings shorter than a turn, several runs of one batch,
with and without a graph, and sets that are too large for the tiles."""
import math

import numpy as np
import pytest

from tests.inputs import beta_c

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def potts():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1101_0876_amd as p

    p.load()
    return p


# L, q, sweeps; q in every class, zero thresholds at beta = 30
SMALL = [(16, 3, 1), (32, 16, 2), (48, 17, 5), (64, 9, 13), (96, 129, 7), (128, 6, 24), (144, 64, 3), (256, 5, 11),
         (240, 2, 9), (80, 65, 40), (16, 256, 8)]


def _jobs(scale):
    return [dict(L=L, q=q, seed=100 + i, start=i % 2, beta=30.0 if i == 3 else beta_c(q), nsweeps=n * scale)
            for i, (L, q, n) in enumerate(SMALL)]


@pytest.mark.parametrize("graph,extra", [(True, 0), (False, 0), (True, 1), (True, 140)])
def test_batch_runs(potts, oracle_lib, graph, extra):
    """extra: 1 adds a lattice for the streaming kernels, 140 lattices of L =
    256 leave the small ones to the LDS-resident kernel."""
    print(f"tile batch graph={graph} extra={extra}", flush=True)
    jobs = _jobs(1)
    if extra == 1:
        jobs.append(dict(L=512, q=6, seed=7, start=1, beta=beta_c(6), nsweeps=6))
    jobs += [dict(L=256, q=4, seed=500 + i, start=1, beta=beta_c(4), nsweeps=2) for i in range(extra if extra > 1 else 0)]
    with potts.Batch(jobs, graph=graph, tune=False) as b:
        for _ in range(2):
            b.run()
        for i, j in enumerate(jobs[:14]):
            n = 2 * j["nsweeps"]
            want_spins, want_rec = oracle_lib.run(j["L"], j["q"], j["seed"], j["start"], j["beta"], n)
            assert np.array_equal(b.spins(i), want_spins), i
            keep = min(n, j["nsweeps"])
            assert np.array_equal(b.records(i, n - keep, keep), want_rec[n - keep:]), i


@pytest.mark.parametrize("quantum,large", [(0, False), (5, False), (32, True)])
def test_served_ramps(potts, oracle_lib, quantum, large):
    print(f"tile serve quantum={quantum} large={large}", flush=True)
    jobs = [(L, q, 40 + i, i % 2, [1, n, 2 * n]) for i, (L, q, n) in enumerate(SMALL)] + [(512, 6, 3, 1, [4, 9])]
    if large:
        jobs.append((2064, 6, 4, 1, [3]))  # too large for the tiles
    srv = potts.Server(quantum=quantum)
    try:
        tickets = []
        for L, q, seed, start, sweeps in jobs:
            betas = [beta_c(q) * (0.98 + 0.02 * k) for k in range(len(sweeps))]
            tickets.append((srv.submit(L, q, seed, start, betas, sweeps, keep_spins=True), betas))
        srv.drain()
        for (ticket, betas), (L, q, seed, start, sweeps) in zip(tickets, jobs):
            got = srv.collect(ticket, spins=True)
            s = oracle_lib.init(L, q, seed, start)
            t = 0
            for b, n, point in zip(betas, sweeps, got["points"]):
                rec = oracle_lib.sweeps(s, q, seed, t, n, oracle_lib.threshold_table(b))
                t += n
                w = (n + 1) // 2
                assert point["n"] == w
                assert math.isclose(point["e"], -rec[-w:, 0].mean() / (L * L), rel_tol=1e-12)
            assert got["status"] == 0 and got["e_sat"] == rec[-1, 0]
            assert np.array_equal(got["spins"], s)
    finally:
        srv.stop()


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("Ls", [(512, 560, 64), (1024, 528), (2048, 16), (320, 272, 608, 304)])
def test_batches_whole_on_tiles(potts, oracle_lib, Ls, graph):
    """Small batches with lattices beyond the LDS-resident sizes, of both strip
    layouts: tiles take all of it, unless the sites are too many or the caller
    asks for a strip height, and give the same bits; twice, so that the second
    run continues from the first."""
    jobs = [dict(L=L, q=q, seed=40 + i, start=i % 2, beta=beta_c(q), nsweeps=n)
            for i, (L, q, n) in enumerate(zip(Ls, (6, 40, 3, 200), (5, 9, 8, 3)))]
    want = []
    for j in jobs:
        s = oracle_lib.init(j["L"], j["q"], j["seed"], j["start"])
        rec = oracle_lib.sweeps(s, j["q"], j["seed"], 0, 2 * j["nsweeps"], oracle_lib.threshold_table(j["beta"]))
        want.append((s, rec))
    for rows in (0, 4):
        with potts.Batch(jobs, graph=graph, tune=False, strip_rows=rows) as b:
            b.run()
            b.run()
            for i, (j, (s, rec)) in enumerate(zip(jobs, want)):
                assert np.array_equal(b.spins(i), s)
                n = j["nsweeps"]
                assert np.array_equal(b.records(i, n, n), rec[n:])
