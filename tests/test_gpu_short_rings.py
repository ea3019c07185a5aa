"""Records of the LDS-resident kernel with drawn words on rings of fewer slots
than the eight sweeps whose records it stores at once: the records that the
ring keeps are the last sweeps', whatever the group they fell in.  Integers
throughout, so equality is exact."""
from __future__ import annotations

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


@pytest.mark.parametrize("kernel,L,q", [(0, 16, 3), (6, 16, 200), (0, 64, 9), (6, 64, 9), (0, 64, 200), (0, 96, 16),
                                        (0, 96, 24)])
@pytest.mark.parametrize("cap", [2, 4, 8])
def test_last_records_of_a_short_ring(potts, oracle_lib, kernel, L, q, cap):
    thr = oracle_lib.threshold_table(beta_c(q))
    s = oracle_lib.init(L, q, 5, 1)
    t = 0
    with potts.Lattice(L, q, 5, 1) as lat:
        lat.reserve_records(cap)
        lat.tune(kernel)
        for n in (3, 8, 23, 1, 5, 12):
            lat.sweep_thr(thr, n)
            rec = oracle_lib.sweeps(s, q, 5, t, n, thr)
            t += n
            k = min(cap - 1, n)
            assert np.array_equal(lat.records(t - k, k), rec[-k:]), (n, k)
            assert lat.observables()["e_sat"] == rec[-1][0]
        assert np.array_equal(lat.spins(), s)
