"""A served job that changes between the multi-sweep tile launches and the strip
launches as other jobs come and go: the strip launches add into record slots
that the tiles have not cleared.  Spins are exact; the points' statistics are
those of the same job alone."""
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


@pytest.mark.parametrize("L,q", [(1040, 6), (2048, 40)])
def test_points_of_a_job_that_leaves_the_tiles(potts, L, q):
    # points of one and two sweeps: every second record, at least, is in a window
    betas, sweeps = [beta_c(q) * (0.98 + 0.001 * k) for k in range(40)], [1, 2, 1, 1] * 10
    # two at a time: the short job keeps the first on tiles until its ring has
    # been round, then L = 2064 takes it to strips, and afterwards it is alone
    with potts.Server(quantum=4, max_slots=2) as srv:
        a = srv.submit(L, q, 3, 1, betas, sweeps, keep_spins=True)
        srv.submit(64, q, 4, 1, [beta_c(q)], [45])
        srv.submit(2064, q, 5, 1, [beta_c(q)], [30])
        srv.drain(120000)
        got = srv.collect(a, spins=True)
    with potts.Lattice(L, q, 3, 1) as lat:
        for k, (b, n) in enumerate(zip(betas, sweeps)):
            lat.sweep(b, n)
            st = lat.stats(lat.t - (n + 1) // 2, (n + 1) // 2, b)
            for key in ("e", "C", "V_L", "m", "chi"):
                assert got["points"][k][key] == st[key], (k, key)
        assert np.array_equal(lat.spins(), got["spins"])
