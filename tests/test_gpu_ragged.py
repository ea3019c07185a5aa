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


# L / 2 % 16 = 2 .. 14, rows per item from 2 to 32
PLANES = [(4740, 6, 0), (4744, 16, 4), (4748, 17, 2), (4752, 64, 16), (4756, 65, 0), (4760, 129, 8), (4764, 256, 2)]


@pytest.mark.parametrize("L,q,rows", PLANES)
def test_lattices(potts, oracle_lib, L, q, rows):
    """Above the tiles' range: two sweeps of the colour-split kernel under the
    narrow and the wide table, a strip or chunk sweep in between, a heat-bath
    sweep after them."""
    print(f"ragged lattice L={L} q={q} rows={rows}", flush=True)
    thr, zeros = oracle_lib.threshold_table(beta_c(q)), np.array([9, 0, 7, 0], dtype=np.uint32)
    s = oracle_lib.init(L, q, 5, 1)
    recs = []
    with potts.Lattice(L, q, 5, 1) as lat:
        lat.tune(0, rows)
        for t, (table, kernel) in enumerate([(thr, 0), (zeros, 0), (thr, 2), (thr, 0)]):
            lat.tune(kernel, rows)
            lat.sweep_thr(table, 1)
            recs.append(oracle_lib.sweeps(s, q, 5, t, 1, table))
        lat.sweep_heatbath_thr(thr, 1)
        recs.append(oracle_lib.heatbath_sweeps(s, q, 5, 4, 1, thr))
        assert np.array_equal(lat.records(0, 5), np.concatenate(recs))
        assert np.array_equal(lat.spins(), s)


def test_caller_buffers(potts, oracle_lib):
    """The caller's buffer is current after each call, and a write into it is
    where the next call starts."""
    import torch

    L, q = 4748, 7
    thr = oracle_lib.threshold_table(beta_c(q))
    s = oracle_lib.init(L, q, 8, 1)
    with potts.Lattice.from_torch(L, q, 8, 1) as lat:
        lat.sweep_thr(thr, 1)
        oracle_lib.sweeps(s, q, 8, 0, 1, thr, record=False)
        torch.cuda.synchronize()
        assert np.array_equal(lat._keep[0].cpu().numpy().reshape(L, L), s)
        s[:] = np.random.default_rng(5).integers(0, q, (L, L), dtype=np.uint8)
        lat._keep[0].copy_(torch.from_numpy(s.reshape(-1)))
        torch.cuda.synchronize()
        lat.sweep_thr(thr, 2)
        oracle_lib.sweeps(s, q, 8, 1, 2, thr, record=False)
        torch.cuda.synchronize()
        assert np.array_equal(lat._keep[0].cpu().numpy().reshape(L, L), s)
