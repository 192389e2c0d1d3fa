"""Boxcar for any width list where a segment ends early: rows and last segments
around the 512 and 1536 outputs of the short forms, with planes and without, and the time
of short rows."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from _checks import check_candidates_exact, check_snr  # noqa: E402
from sps_inputs.workloads import Workload  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sps():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_02328_amd import sps as mod
    mod.library()
    return mod


def _plan(sps, ndm, nchan=4096):
    return sps.plan_for(Workload("r", nchan, 1000.0, 1500.0, 1e-4, 4096, ndm, 0.0, 1.0, (1,)))


@pytest.mark.parametrize("nout", [7, 255, 256, 257, 511, 512, 513, 1025, 4096 + 1, 4096 + 511,
                                  4096 + 512, 4096 + 513, 8192 + 200, 1535,
                                  1536, 1537, 4096 + 1536, 4096 + 1537])
@pytest.mark.parametrize("widths", [[3], [2, 3, 7], [1, 2, 3, 257], [5, 300]])
def test_short_segments(sps, nout, widths):
    widths = [w for w in widths if w <= nout]
    rng = np.random.Generator(np.random.PCG64(nout + len(widths)))
    Y = rng.integers(400000, 400400, size=(7, nout)).astype(np.int64)
    Y[1] = rng.integers(0, 255 * 4096 + 1, size=nout)      # prefixes past 2^24
    Y[2] = 77                                              # MAD 0
    Y[3] = rng.integers(1000, 1003, size=nout)
    Y = Y.astype(np.uint32)
    sto = oracle.stats(Y)
    with _plan(sps, len(Y)) as plan:
        Yd = torch.from_numpy(Y.view(np.int32)).cuda()
        snr = torch.full(Y.shape, -7.0, dtype=torch.float32, device="cuda")
        best = torch.full(Y.shape, 99, dtype=torch.uint8, device="cuda")
        st = torch.empty((len(Y), 2), dtype=torch.int32, device="cuda")
        sps.sps_boxcar_snr(plan, Yd, nout, widths, snr, best, st)
        g, b = snr.cpu().numpy(), best.cpu().numpy()
        check_snr(Y, sto, widths, g, b)
        # tile columns of one segment, of whole waves and of any length
        for tt in (4096, 64, 100):
            co = oracle.detect(g, b, 1.0, 2, tt, 0, 5, cap=1 << 14)
            for s, w in ((snr, best), (None, None)):
                c, n = sps.sps_search(plan, Yd, nout, widths, s, w, st, 1.0, 2, tt, 0, 5,
                                      cap=1 << 14)
                check_candidates_exact(c, n, co, widths, f"tiles of {tt}")


def test_short_rows_take_less_than_whole_segments(sps):
    # 512 rows of 250 outputs to 512 rows of 4096, 64 widths: 0.9 when every
    # thread works through 16 outputs, 0.36 in the short form
    widths = list(range(1, 65))
    ends = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    with _plan(sps, 512) as plan:
        def us(nout):
            Y = torch.randint(400000, 400400, (512, nout), dtype=torch.int32, device="cuda")
            snr = torch.empty((512, nout), dtype=torch.float32, device="cuda")
            best = torch.empty((512, nout), dtype=torch.uint8, device="cuda")
            st = torch.empty((512, 2), dtype=torch.int32, device="cuda")
            times = []
            for _ in range(5):
                ends[0].record()
                for _ in range(20):
                    sps.sps_boxcar_snr(plan, Y, nout, widths, snr, best, st)
                ends[1].record()
                ends[1].synchronize()
                times.append(ends[0].elapsed_time(ends[1]))
            return np.median(times)

        short, whole = us(250), us(4096)
        print("short", short, "whole", whole)
        assert short < 0.6 * whole
