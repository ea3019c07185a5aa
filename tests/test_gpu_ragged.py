"""Colour-split kernels on lattices whose plane rows end inside a 16-byte item
(L % 32 != 0), bit for bit against the oracle: every remainder of L/2 by 16
(2 .. 14 sites in the last item, the last site in byte 1 or 3 of its dword),
every class of q, the narrow and the wide acceptance table, walks of every
length, and kernel switches and reads in the middle of a chain.  Integers
throughout, so equality is exact."""
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


# L / 2 % 16 = 2, 4, 6, 8, 10, 12, 14
CUBES = [(68, 3, 0), (72, 16, 4), (76, 17, 2), (80, 64, 16), (84, 65, 0), (88, 129, 8), (92, 256, 0), (100, 6, 4)]


@pytest.mark.parametrize("L,q,rows", CUBES)
def test_cubes(potts, oracle_lib, L, q, rows):
    print(f"ragged cube L={L} q={q} rows={rows}", flush=True)
    tables = [oracle_lib.threshold_table6(0.55), np.array([9, 0, 7, 0, 3, 0], dtype=np.uint32)]
    s = oracle_lib.init3d(L, q, 5, 1)
    t, recs = 0, []
    with potts.Cube(L, q, 5, 1) as c:
        c.tune(0, rows)
        for thr, n in zip(tables, (2, 1)):
            c.sweep_thr(thr, n)
            recs.append(oracle_lib.sweeps3d(s, q, 5, t, n, thr))
            t += n
            assert np.array_equal(c.spins(), s)
        c.tune(2)  # the chunk kernel, in place
        c.sweep_thr(tables[0], 1)
        recs.append(oracle_lib.sweeps3d(s, q, 5, t, 1, tables[0]))
        c.tune(0)
        c.sweep_thr(tables[0], 1)
        recs.append(oracle_lib.sweeps3d(s, q, 5, t + 1, 1, tables[0]))
        assert np.array_equal(c.records(0, t + 2), np.concatenate(recs))
        assert np.array_equal(c.spins(), s)
