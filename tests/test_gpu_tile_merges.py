"""Tile maxima of tiles that no wave or segment lies in: the candidates, and the
time of merging them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from sps_inputs.workloads import Workload  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sps():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_02328_amd import sps as mod
    mod.library()
    return mod


@pytest.mark.parametrize("widths", [[1, 2, 4, 8, 16], [1, 3, 5, 10]])
def test_per_thread_merges(sps, widths):
    # An atomic for each thread's maximum, whether or not it can raise the
    # tile's: 512 x 4096 outputs in tiles of 64 x 1000 take 25 times as long as
    # in tiles of 64 x 1024; without those that cannot, 7 times.
    ndm, nout = 512, 4096
    wl = Workload("m", 256, 1000.0, 1500.0, 1e-4, nout, ndm, 0.0, 1.0, tuple(widths))
    rng = np.random.Generator(np.random.PCG64(len(widths)))
    Y = torch.from_numpy(rng.integers(30000, 31000, (ndm, nout)).astype(np.int32)).cuda()
    snr = torch.empty((ndm, nout), dtype=torch.float32, device="cuda")
    best = torch.empty((ndm, nout), dtype=torch.uint8, device="cuda")
    st = torch.empty((ndm, 2), dtype=torch.int32, device="cuda")
    ends = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    with sps.plan_for(wl) as plan:
        def ms(tile_t):
            times = []
            for _ in range(9):
                ends[0].record()
                got = sps.sps_search(plan, Y, nout, widths, None, None, st, 1.0, 64, tile_t, 0, 5)
                ends[1].record()
                ends[1].synchronize()
                times.append(ends[0].elapsed_time(ends[1]))
            return np.median(times), got

        for planes in ((snr, best), (None, None)):
            c, n = sps.sps_search(plan, Y, nout, widths, *planes, st, 1.0, 64, 1000, 0, 5)
            if planes[0] is not None:
                want = sps.sps_detect(plan, snr, best, nout, widths, 1.0, 64, 1000, 0, 5)
            assert n == want[1] > 0 and np.array_equal(c, want[0])
        t, (c, n) = ms(1000)
        whole, _ = ms(1024)
        print("any", t, "whole waves", whole)
        assert n == want[1] and np.array_equal(c, want[0])
        assert t < 13 * whole
