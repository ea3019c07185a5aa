"""The multi-sweep tile kernel asked for where a lattice cut into 32 equal
parts has parts too large for a workgroup (L = 6672 .. 8192) or above, against
the oracle and the strip kernel.  Integers throughout, so equality is exact."""
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


def test_matches_oracle(potts, oracle_lib):
    L, q, n = 6672, 6, 2
    want_spins, want_rec = oracle_lib.run(L, q, 3, 1, beta_c(q), n)
    with potts.Lattice(L, q, 3, 1) as lat:
        lat.tune(5)
        lat.sweep(beta_c(q), n)
        assert np.array_equal(lat.records(0, n), want_rec)
        assert np.array_equal(lat.spins(), want_spins)


@pytest.mark.parametrize("L,q", [(6672, 200), (7504, 17), (8192, 9), (8208, 6)])
def test_matches_strip_kernel(potts, L, q):
    got = []
    for kernel in (5, 1):
        with potts.Lattice(L, q, 3, 1) as lat:
            lat.tune(kernel)
            lat.sweep(beta_c(q), 3)
            lat.sweep(beta_c(q), 1)
            got.append((lat.records(0, 4), lat.spins()))
    assert np.array_equal(got[0][0], got[1][0])
    assert np.array_equal(got[0][1], got[1][1])
