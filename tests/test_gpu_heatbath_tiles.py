"""Heat-bath sweeps on multi-sweep tiles and on colour planes whose rows end
inside a 16-byte item, bit for bit against the oracle (spins and every record):
regions wider than the lattice, cut tiles, one to six items per lane, every
class of q, the narrow and the wide draw table, calls shorter than a launch,
caller-owned buffers, rings shorter than a launch, Metropolis sweeps and
kernel switches in between, and captured calls.  Integers throughout, so
equality is exact."""
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


# L, q, start, calls: 4 .. 60 wrap around, 100 .. 512 one item per lane, 1284
# two, 2004 four, 3580 six
CASES = [
    (4, 2, 1, (1, 5, 9)), (8, 16, 1, (7, 2)), (20, 256, 1, (8, 1)), (36, 9, 0, (11,)), (60, 128, 1, (6,)),
    (64, 17, 1, (3, 4)), (100, 64, 1, (9,)), (252, 129, 0, (1, 2, 8)), (256, 3, 1, (12,)), (500, 6, 1, (9,)),
    (512, 65, 1, (4,)), (1284, 24, 1, (5,)), (2004, 6, 1, (4,)), (3580, 5, 1, (2,)),
]


@pytest.mark.parametrize("L,q,start,calls", CASES)
def test_tiles_match_oracle(potts, oracle_lib, L, q, start, calls):
    print(f"heatbath tiles L={L} q={q} calls={calls}", flush=True)
    thr = oracle_lib.threshold_table(beta_c(q))
    s = oracle_lib.init(L, q, 13, start)
    want = oracle_lib.heatbath_sweeps(s, q, 13, 0, sum(calls), thr)
    with potts.Lattice(L, q, 13, start) as lat:
        for n in calls:
            lat.sweep_heatbath(beta_c(q), n)
        assert np.array_equal(lat.records(0, sum(calls)), want)
        assert np.array_equal(lat.spins(), s)


# L / 2 % 16 = 2 .. 14 above the tiles' range
PLANES = [(4100, 6, 0), (4104, 16, 4), (4108, 17, 2), (4112, 64, 16), (4116, 65, 0), (4120, 129, 8), (4124, 256, 0)]


@pytest.mark.parametrize("L,q,rows", PLANES)
def test_partial_items_match_oracle(potts, oracle_lib, L, q, rows):
    print(f"heatbath ragged planes L={L} q={q} rows={rows}", flush=True)
    thr = oracle_lib.threshold_table(beta_c(q)) if q != 17 else np.array([5, 0, 9, 0], dtype=np.uint32)
    s = oracle_lib.init(L, q, 3, 1)
    with potts.Lattice(L, q, 3, 1) as lat:
        lat.tune(0, rows)
        lat.sweep_heatbath_thr(thr, 1)
        a = oracle_lib.heatbath_sweeps(s, q, 3, 0, 1, thr)
        lat.sweep_thr(thr, 1)  # tiles or planes
        b = oracle_lib.sweeps(s, q, 3, 1, 1, thr)
        lat.sweep_heatbath_thr(thr, 1)
        c = oracle_lib.heatbath_sweeps(s, q, 3, 2, 1, thr)
        assert np.array_equal(lat.records(0, 3), np.concatenate([a, b, c]))
        assert np.array_equal(lat.spins(), s)


@pytest.mark.parametrize("L,q", [(52, 7), (128, 12), (300, 33)])
def test_caller_buffers_and_short_ring(potts, oracle_lib, L, q):
    """Changing tables, the wide one among them, odd numbers of launches on the
    caller's buffers, Metropolis sweeps between, and a ring of four slots."""
    import torch

    tables = [oracle_lib.threshold_table(beta_c(q)), np.array([5, 0, 9, 0], dtype=np.uint32)]
    s = oracle_lib.init(L, q, 3, 1)
    t = 0
    with potts.Lattice.from_torch(L, q, 3, 1, records_capacity=4) as lat:
        for i, (thr, n) in enumerate(zip(tables * 3, (3, 10, 1, 6, 2, 5))):
            hb = i % 3 != 2
            (lat.sweep_heatbath_thr if hb else lat.sweep_thr)(thr, n)
            rec = (oracle_lib.heatbath_sweeps if hb else oracle_lib.sweeps)(s, q, 3, t, n, thr)
            t += n
            torch.cuda.synchronize()
            assert np.array_equal(lat._keep[0].cpu().numpy().reshape(L, L), s)
            k = min(3, n)
            assert np.array_equal(lat.records(t - k, k), rec[-k:])


@pytest.mark.parametrize("L,q,heatbath", [(512, 6, True), (100, 6, True), (100, 6, False), (500, 9, False), (4740, 6, False)])
def test_captured_calls_with_eager_work_between(potts, oracle_lib, L, q, heatbath):
    """Replays and eager calls take turns on one lattice: whatever buffer or
    plane an eager call would prefer, a replay continues from what it left."""
    import torch

    thr = oracle_lib.threshold_table(beta_c(q))
    s = oracle_lib.init(L, q, 9, 1)
    run = oracle_lib.heatbath_sweeps if heatbath else oracle_lib.sweeps
    stream = torch.cuda.Stream()
    with potts.Lattice.on_stream(L, q, 9, 1, stream=stream) as lat:
        sweep = lat.sweep_heatbath_thr if heatbath else lat.sweep_thr
        warm = 9 if L < 4000 else 2
        sweep(thr, warm)
        run(s, q, 9, 0, warm, thr)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            sweep(thr, 2)
        t = warm + 2
        for eager in (1, warm, 2):
            with torch.cuda.stream(stream):
                g.replay()
            run(s, q, 9, warm, 2, thr)
            torch.cuda.synchronize()
            assert np.array_equal(lat.spins(), s)
            sweep(thr, eager)
            run(s, q, 9, t, eager, thr)
            t += eager
            torch.cuda.synchronize()
        assert np.array_equal(lat.spins(), s)
