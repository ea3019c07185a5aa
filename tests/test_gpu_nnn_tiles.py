"""Second-neighbour sweeps on LDS tiles with recomputed halos, bit for bit
against the oracle: regions that wrap around the lattice, cut tiles, one to
three items per lane, calls shorter than a launch, every class of q, tables
with zeros and tables no temperature gives, and switches to and from the other
kernels in the middle of a chain.  Integers throughout, so equality is exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def potts():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1101_0876_amd as p

    p.load()
    return p


def _tables(oracle_lib):
    rng = np.random.default_rng(7)
    wild = rng.integers(0, 2**32 + 1, size=81, dtype=np.uint64)
    wild[::5] = 0
    return [oracle_lib.nnn_table(0.8, 0.5), oracle_lib.nnn_table(1.1, -0.25), wild]


# the last three: one, two and three items per lane
CASES = [(12, 2, (1, 4)), (24, 16, (7,)), (36, 17, (2, 5)), (60, 128, (9,)), (84, 129, (4,)), (132, 256, (3, 6)),
         (252, 9, (13,)), (1020, 6, (1, 8)), (3072, 9, (5,)), (4500, 6, (3,))]


@pytest.mark.parametrize("L,q,calls", CASES)
def test_sweeps_match_oracle(potts, oracle_lib, L, q, calls):
    print(f"nnn tiles L={L} q={q} calls={calls}", flush=True)
    # row- and segment-keyed words: the chain of a large lattice in the oracle takes seconds, so one table there
    tables = _tables(oracle_lib) if L < 1000 else _tables(oracle_lib)[:1]
    with potts.NnnLattice(L, q, 3, 1) as lat:
        s = lat.spins()
        t, recs = 0, []
        for thr in tables:
            for n in calls:
                lat.sweep_thr(thr, n)
                recs.append(oracle_lib.nnn_sweeps(s, q, 3, t, n, thr))
                t += n
        assert np.array_equal(lat.records(0, t), np.concatenate(recs))
        assert np.array_equal(lat.spins(), s)
        obs = lat.observables()
        assert obs["e1"] == recs[-1][-1, 0] and obs["e2"] == recs[-1][-1, 1]


def test_switches_between_kernels(potts, oracle_lib):
    L, q = 156, 5
    thr = oracle_lib.nnn_table(0.9, 0.5)
    with potts.NnnLattice(L, q, 8, 1) as lat:
        s = lat.spins()
        t, recs = 0, []
        for kernel, n in [(0, 3), (1, 2), (0, 5), (2, 1), (0, 1), (1, 1), (0, 4)]:
            lat.tune(kernel)
            lat.sweep_thr(thr, n)
            recs.append(oracle_lib.nnn_sweeps(s, q, 8, t, n, thr))
            t += n
        assert np.array_equal(lat.records(0, t), np.concatenate(recs))
        assert np.array_equal(lat.spins(), s)
