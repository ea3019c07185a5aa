"""A captured sweep call replayed with eager calls between, at the sizes where
the kernel depends on the length of a call: replays and eager calls work on one
lattice, wherever the call before left it (rows or colour planes), and reading
it gives what the last of them left.  Integers throughout, so equality is
exact."""
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


def kinds(lat, oracle_lib, heatbath):
    if heatbath:
        return lat.sweep_heatbath_thr, oracle_lib.heatbath_sweeps
    return lat.sweep_thr, oracle_lib.sweeps


# (L, heat bath, eager sweeps before the capture, captured sweeps, eager calls
# between the replays); 0 sweeps before: nothing has run on the lattice
CASES = [
    (4128, False, 5, 1, (1, 5)),   # on tiles before, one sweep captured
    (4128, False, 1, 5, (5, 1)),   # on the planes before
    (4128, False, 0, 1, (5,)),
    (4864, False, 0, 1, (1,)),     # a size that is always on the planes
    (4864, False, 1, 1, (1,)),
    (2048, False, 48, 2, (1, 48)),  # bands before and between
    (2048, False, 2, 2, (48, 2)),
    (4096, False, 2, 2, (1, 2)),   # bands, captured too
    (4096, False, 1, 1, (1,)),
    (3616, True, 4, 1, (4,)),
    (3616, True, 1, 4, (1,)),
    (1024, True, 1, 1, (2, 1)),
    (4740, False, 1, 1, (1,)),     # partial items, on planes of their own
    (4740, False, 0, 1, (2,)),
    (4100, False, 1, 5, (5,)),
    (4100, False, 5, 1, (1,)),
    (3620, True, 1, 1, (4,)),
]


@pytest.mark.parametrize("L,heatbath,warm,n,eager", CASES)
def test_replays_and_eager_calls_share_the_lattice(potts, oracle_lib, L, heatbath, warm, n, eager):
    import torch

    q = 6
    thr = oracle_lib.threshold_table(beta_c(q))
    s = oracle_lib.init(L, q, 9, 1)
    stream = torch.cuda.Stream()
    with potts.Lattice.on_stream(L, q, 9, 1, stream=stream) as lat:
        sweep, run = kinds(lat, oracle_lib, heatbath)
        if warm:
            sweep(thr, warm)
            run(s, q, 9, 0, warm, thr)
        elif heatbath:
            raise AssertionError("the heat bath's table has to be there")
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            sweep(thr, n)
        t = warm + n
        for k in eager:
            for _ in range(2):
                with torch.cuda.stream(stream):
                    g.replay()
                run(s, q, 9, warm, n, thr)
                torch.cuda.synchronize()
                assert np.array_equal(lat.spins(), s)
            sweep(thr, k)
            rec = run(s, q, 9, t, k, thr)
            t += k
            torch.cuda.synchronize()
            assert np.array_equal(lat.records(t - k, k), rec)
            assert np.array_equal(lat.spins(), s)


@pytest.mark.parametrize("first", [1, 4])
def test_other_kernels_and_writes_after_a_capture(potts, oracle_lib, first):
    """Kernel choices, the other update and a new configuration between replays,
    the lattice on rows (4 sweeps before) or planes (1) when captured."""
    import torch

    L, q = 3648, 6
    thr = oracle_lib.threshold_table(beta_c(q))
    s = oracle_lib.init(L, q, 9, 1)
    stream = torch.cuda.Stream()
    with potts.Lattice.on_stream(L, q, 9, 1, stream=stream) as lat:
        lat.sweep_heatbath_thr(thr, first)
        oracle_lib.heatbath_sweeps(s, q, 9, 0, first, thr)
        lat.sweep_thr(thr, first)
        oracle_lib.sweeps(s, q, 9, first, first, thr)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            lat.sweep_thr(thr, 1)
        t = 2 * first + 1

        def replay():
            with torch.cuda.stream(stream):
                g.replay()
            torch.cuda.synchronize()
            oracle_lib.sweeps(s, q, 9, 2 * first, 1, thr)

        for kernel in (1, 4, 5, 2, 0):
            replay()
            lat.tune(kernel)
            lat.sweep_thr(thr, 1)
            oracle_lib.sweeps(s, q, 9, t, 1, thr)
            replay()
            assert np.array_equal(lat.spins(), s), kernel
            t += 1
        lat.sweep_heatbath_thr(thr, 4)
        oracle_lib.heatbath_sweeps(s, q, 9, t, 4, thr)
        replay()
        assert np.array_equal(lat.spins(), s)
        s = oracle_lib.init(L, q, 10, 1)
        lat.set_spins(s, t)
        replay()
        assert np.array_equal(lat.spins(), s)
