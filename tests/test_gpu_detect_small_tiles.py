"""Tile maxima where a tile's rows have fewer vectors than a workgroup has
threads: tile lengths around the sharing of threads among rows, ragged last
tiles, rows at any dword, and the time of small tiles."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from _checks import check_candidates_exact  # noqa: E402
from sps_inputs.workloads import Workload  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sps():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_02328_amd import sps as mod
    mod.library()
    return mod


def _plan(sps, ndm, nout):
    return sps.plan_for(Workload("t", 8, 1000.0, 1500.0, 1e-4, nout, ndm, 0.0, 10.0, (1,)))


@pytest.mark.parametrize("tt", [1, 3, 4, 5, 15, 16, 17, 19, 33, 64, 129, 255, 257, 511, 512, 515,
                                516, 600])
@pytest.mark.parametrize("ndm,td", [(37, 5), (70, 70), (9, 1), (300, 130)])
def test_tile_lengths(sps, tt, ndm, td):
    nout, widths = 3 * tt + max(1, tt // 3), [1, 2, 4]
    rng = np.random.Generator(np.random.PCG64(ndm * tt))
    snr = (rng.standard_normal((ndm, nout)) * 1.5).astype(np.float32)
    k = min(60, ndm * nout // 4)
    snr[rng.integers(0, ndm, k), rng.integers(0, nout, k)] = 9.5  # exact ties
    snr[rng.integers(0, ndm, k), rng.integers(0, nout, k)] = -np.inf
    best = rng.integers(0, 3, (ndm, nout)).astype(np.uint8)
    co = oracle.detect(snr, best, 1.0, td, tt, 1, 2, cap=1 << 14)
    pad = torch.empty(ndm * nout + 1, dtype=torch.float32, device="cuda")
    planes = [torch.from_numpy(snr).cuda(), pad[1:].view(ndm, nout)]  # aligned, one dword on
    planes[1].copy_(planes[0])
    with _plan(sps, ndm, nout) as plan:
        for s in planes:
            c, n = sps.sps_detect(plan, s, torch.from_numpy(best).cuda(), nout, widths, 1.0, td,
                                  tt, 1, 2, cap=1 << 14)
            check_candidates_exact(c, n, co, widths)


def test_small_tiles_take_about_as_long_as_large_ones(sps):
    # 512 x 262,147 outputs, tiles of 16 x 256 to tiles of 64 x 4096: 3.3 with a
    # row at a time, 1.5 with several
    ndm, nout = 512, 262147
    ends = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    snr = torch.randn((ndm, nout), device="cuda")
    best = torch.zeros((ndm, nout), dtype=torch.uint8, device="cuda")
    with _plan(sps, ndm, nout) as plan:
        def ms(td, tt):
            times = []
            for _ in range(9):
                ends[0].record()
                sps.sps_detect(plan, snr, best, nout, [1], 20.0, td, tt, 0, 0)
                ends[1].record()
                ends[1].synchronize()
                times.append(ends[0].elapsed_time(ends[1]))
            return np.median(times)

        small, large = ms(16, 256), ms(64, 4096)
        print("small", small, "large", large)
        assert small < 2.4 * large
