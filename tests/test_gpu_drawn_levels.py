"""The LDS-resident kernel with pre-drawn words where its pieces have edges, bit
for bit against the oracle: one or two groups a lane, lanes without one, calls
that draw their words in the kernel (up to 4 sweeps), whole and part groups of
eight sweeps, every class of q, tables that do not fall with the gap or hold
zeros, and captured calls.  Integers throughout, so equality is exact."""
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


CASES = [(16, 2, (1, 8, 5)), (16, 256, (4, 9)), (32, 16, (3, 16)), (48, 17, (2, 7)), (48, 129, (17,)), (64, 9, (1, 5, 24)),
         (64, 128, (4, 8)), (64, 200, (11,)), (80, 6, (1, 3, 10)), (80, 64, (8,)), (96, 12, (2, 3, 12)), (96, 255, (9,))]


@pytest.mark.parametrize("table", ["falling", "rising", "zeros"])
@pytest.mark.parametrize("L,q,calls", CASES)
def test_levels_match_oracle(potts, oracle_lib, L, q, calls, table):
    print(f"drawn levels L={L} q={q} calls={calls} {table}", flush=True)
    thr = {"falling": oracle_lib.threshold_table(beta_c(q)),
           "rising": np.array([1 << 28, 1 << 31, 3, 0xFFFFFFFF], dtype=np.uint32),
           "zeros": np.array([1 << 30, 1 << 29, 0, 0], dtype=np.uint32)}[table]
    s = oracle_lib.init(L, q, 21, 1)
    want = oracle_lib.sweeps(s, q, 21, 0, sum(calls), thr)
    with potts.Lattice(L, q, 21, 1) as lat:
        for n in calls:
            lat.sweep_thr(thr, n)
        assert np.array_equal(lat.records(0, sum(calls)), want)
        assert np.array_equal(lat.spins(), s)


@pytest.mark.parametrize("L,k", [(64, 10), (64, 3), (96, 5)])
def test_captured_after_a_short_call(potts, oracle_lib, L, k):
    """The captured call may not allocate the words' buffer that the short call
    before it had no need of."""
    import torch

    q = 6
    thr = oracle_lib.threshold_table(beta_c(q))
    s = oracle_lib.init(L, q, 9, 1)
    oracle_lib.sweeps(s, q, 9, 0, 1, thr)
    stream = torch.cuda.Stream()
    with potts.Lattice.on_stream(L, q, 9, 1, stream=stream) as lat:
        lat.sweep_thr(thr, 1)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            lat.sweep_thr(thr, k)
        for _ in range(3):
            with torch.cuda.stream(stream):
                g.replay()
            torch.cuda.synchronize()
            oracle_lib.sweeps(s, q, 9, 1, k, thr)
            assert np.array_equal(lat.spins(), s)


@pytest.mark.parametrize("L,q", [(16, 5), (64, 200), (100, 9), (1000, 40), (4740, 3)])
def test_observables_after_every_kind_of_call(potts, oracle_lib, L, q):
    """The last record's host copy belongs to the last call, whichever kernel
    took it, and to none after the lattice has been replaced."""
    thr = oracle_lib.threshold_table(beta_c(q))
    s = oracle_lib.init(L, q, 4, 1)
    t = 0
    with potts.Lattice(L, q, 4, 1) as lat:
        for kind, n in (("m", 1), ("m", 2), ("h", 1), ("m", 9), ("set", 0), ("m", 1), ("chunk", 1), ("m", 1)):
            if L > 4000 and n > 2:
                continue
            if kind == "set":
                lat.set_spins(s, t)
                continue
            if kind == "chunk":
                lat.tune(2)
            (lat.sweep_heatbath_thr if kind == "h" else lat.sweep_thr)(thr, n)
            rec = (oracle_lib.heatbath_sweeps if kind == "h" else oracle_lib.sweeps)(s, q, 4, t, n, thr)
            t += n
            lat.tune(0)
            for _ in range(2):
                o = lat.observables()
                assert (o["t"], o["e_sat"]) == (t, rec[-1][0])
                assert np.array_equal(o["hist"], rec[-1][1:])
