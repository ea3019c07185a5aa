"""The multi-sweep tile kernel where its geometry has edges, bit for bit
against the oracle (spins and every record): lattices that are no multiple of
16 or of the tile (cut tiles, items whose second half is another tile's),
regions wider than the lattice, one to six items per lane, calls shorter than
a launch, every class of q, caller-owned buffers, and rings shorter than a
launch.  Integers throughout, so equality is exact."""
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


# L, q, start, calls: 4 .. 60 wrap around, 68 .. 500 one item per lane, 1280
# two, 2000 four, 3584 six
CASES = [
    (4, 2, 1, (1, 5, 9)), (8, 16, 1, (7, 2)), (12, 17, 0, (9,)), (20, 256, 1, (8, 1)), (28, 65, 1, (3, 6)),
    (36, 9, 1, (17,)), (60, 128, 1, (6,)), (68, 129, 0, (1, 2, 10)), (100, 64, 1, (13,)), (252, 5, 1, (6, 6)),
    (256, 16, 0, (12,)), (260, 3, 1, (9,)), (500, 6, 1, (4, 11)), (516, 24, 1, (8,)), (1000, 12, 1, (11,)),
    (1280, 200, 1, (5,)), (1284, 6, 1, (9,)), (2000, 6, 1, (9,)), (3584, 6, 1, (3,)),
]


@pytest.mark.parametrize("L,q,start,calls", CASES)
def test_automatic_tiles_match_oracle(potts, oracle_lib, L, q, start, calls):
    print(f"tile edges L={L} q={q} start={start} calls={calls}", flush=True)
    n, beta = sum(calls), beta_c(q)
    want_spins, want_rec = oracle_lib.run(L, q, 31, start, beta, n)
    with potts.Lattice(L, q, 31, start) as lat:
        for k in calls:
            lat.sweep(beta, k)
        assert np.array_equal(lat.records(0, n), want_rec)
        assert np.array_equal(lat.spins(), want_spins)


@pytest.mark.parametrize("L,q", [(52, 7), (300, 33)])
def test_caller_buffers_wide_table_and_short_ring(potts, oracle_lib, L, q):
    """Zero thresholds (the 64-bit acceptance table), odd numbers of launches on
    the caller's buffers, and a ring of four slots, fewer than a launch's
    sweeps."""
    import torch

    tables = [oracle_lib.threshold_table(beta_c(q)), np.array([5, 0, 9, 0], dtype=np.uint32)]
    s = oracle_lib.init(L, q, 3, 1)
    t, recs = 0, []
    with potts.Lattice.from_torch(L, q, 3, 1, records_capacity=4) as lat:
        for thr, n in zip(tables * 2, (3, 10, 1, 6)):
            lat.sweep_thr(thr, n)
            recs.append(oracle_lib.sweeps(s, q, 3, t, n, thr))
            t += n
            torch.cuda.synchronize()
            assert np.array_equal(lat._keep[0].cpu().numpy().reshape(L, L), s)
            k = min(3, n)
            assert np.array_equal(lat.records(t - k, k), recs[-1][-k:])


@pytest.mark.parametrize("L,q,k", [(128, 6, 3), (100, 6, 2), (512, 9, 10)])
def test_sweeps_in_a_captured_graph(potts, oracle_lib, L, q, k):
    """A captured call works on the lattice in place: every replay runs its
    sweeps on what the one before left, with eager work between them."""
    import torch

    beta, warm = beta_c(q), 5
    thr = oracle_lib.threshold_table(beta)
    s = oracle_lib.init(L, q, 9, 1)
    oracle_lib.sweeps(s, q, 9, 0, warm, thr)
    stream = torch.cuda.Stream()
    with potts.Lattice.on_stream(L, q, 9, 1, stream=stream) as lat:
        lat.sweep(beta, warm)
        assert np.array_equal(lat.spins(), s)
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            lat.sweep(beta, k)
        busy = torch.ones(1 << 20, device="cuda")
        for _ in range(3):
            graph.replay()
            torch.cuda.synchronize()
            oracle_lib.sweeps(s, q, 9, warm, k, thr)
            assert np.array_equal(lat.spins(), s)
            busy = busy * 0.5 + 1.0
