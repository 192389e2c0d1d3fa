"""GPU parity of the plane passes on rows that start at any dword: statistics,
the boxcar for arbitrary width lists (pairs of widths, odd lists, first width
above 1, windows shorter and longer than the scan held in registers, prefixes
about +-2^24), detection with tiles shared by several workgroups, and the
search's tile keys and candidate read-back at the edges of their forms."""
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


# lists: one width; a pair; odd; first above 1; w_max 257 and 258 (the longest
# scan in registers and one more); rows: within a segment, at its end, past it,
# each length modulo 4
@pytest.mark.parametrize("widths,nout", [
    ([3], 4097), ([2, 5], 4099), ([1, 3, 6], 8191), ([7, 20, 21], 4102),
    ([1, 2, 3, 257], 4096 + 256), ([1, 2, 3, 257], 2 * 4096 + 257), ([5, 258], 4096 + 257),
    ([1, 6, 1000, 2001], 3 * 4096 + 1), ([2, 3], 5), ([4, 9], 9)])
def test_any_widths_on_unaligned_rows(sps, widths, nout):
    nchan, med = 4096, 500000
    rng = np.random.Generator(np.random.PCG64(nout + len(widths)))
    Y = rng.integers(0, 255 * nchan + 1, size=(6, nout)).astype(np.int64)
    Y[1] = rng.integers(1000, 1003, size=nout)
    Y[2] = 77  # MAD 0
    # prefixes of Y - med that cross +-2^24 inside a segment; MAD 1
    for r, lift in ((3, 400000), (4, -400000)):
        Y[r] = med + np.tile([1, -1, 0], nout // 3 + 1)[:nout]
        if nout > 4500:
            Y[r, 900:900 + 42] = med + lift
    Y = Y.astype(np.uint32)
    sto = oracle.stats(Y)
    wl = Workload("u", nchan, 1000.0, 1500.0, 1e-4, nout, len(Y), 0.0, 1.0, tuple(widths))
    td, tt = 2, 1500
    with sps.plan_for(wl) as plan:
        Yd = torch.from_numpy(Y.view(np.int32)).cuda()
        snr = torch.empty(Y.shape, dtype=torch.float32, device="cuda")
        best = torch.empty(Y.shape, dtype=torch.uint8, device="cuda")
        st = torch.empty((len(Y), 2), dtype=torch.int32, device="cuda")
        sps.sps_boxcar_snr(plan, Yd, nout, widths, snr, best, st)
        c, n = sps.sps_detect(plan, snr, best, nout, widths, 3.0, td, tt, 1, 300, cap=8192)
    assert np.array_equal(st.cpu().numpy().astype(np.int64), sto)
    g, b = snr.cpu().numpy(), best.cpu().numpy()
    check_snr(Y, sto, widths, g, b)
    check_candidates_exact(c, n, oracle.detect(g, b, 3.0, td, tt, 1, 300, cap=8192), widths)


# tiles of at least 65536 outputs, fewer than 1024: shared, with row counts
# that do not divide by the parts; below that size, or of few rows: not
@pytest.mark.parametrize("ndm,nout,td,tt", [
    (37, 70001, 37, 4096), (130, 9999, 64, 4099), (9, 200003, 5, 20001), (3, 100003, 3, 100003),
    (64, 1023, 64, 1023), (64, 1025, 64, 1024)])
def test_detect_with_shared_tiles(sps, ndm, nout, td, tt):
    rng = np.random.Generator(np.random.PCG64(ndm * nout))
    snr = (rng.standard_normal((ndm, nout)) * 1.5).astype(np.float32)
    snr[rng.integers(0, ndm, 60), rng.integers(0, nout, 60)] = 9.5  # exact ties
    best = rng.integers(0, 3, (ndm, nout)).astype(np.uint8)
    widths = [1, 2, 4]
    co = oracle.detect(snr, best, 4.0, td, tt, 3, 50, cap=8192)
    wl = Workload("d", 8, 1000.0, 1500.0, 1e-4, nout, ndm, 0.0, 10.0, (1,))
    pad = torch.empty(ndm * nout + 1, dtype=torch.float32, device="cuda")
    planes = [torch.from_numpy(snr).cuda(), pad[1:].view(ndm, nout)]  # aligned, one dword on
    planes[1].copy_(planes[0])
    with sps.plan_for(wl) as plan:
        for s in planes:
            c, n = sps.sps_detect(plan, s, torch.from_numpy(best).cuda(), nout, widths, 4.0, td,
                                  tt, 3, 50, cap=8192)
            check_candidates_exact(c, n, co, widths)


# tile counts: one, a few, the most that the selection decodes itself (8192)
# and one column more; read-back around the 256 records of the first copy
@pytest.mark.parametrize("nout,td,tt,thr,cap", [
    (4096, 64, 4096, 2.0, 10), (4099, 16, 1000, 2.0, 8192), (4096, 1, 32, 1.0, 8192),
    (4097, 1, 32, 1.0, 16384), (4097, 1, 32, 1.0, 255), (4097, 1, 32, 1.0, 256),
    (4097, 1, 32, 1.0, 257)])
def test_search_tile_counts_and_read_back(sps, nout, td, tt, thr, cap):
    widths = [1, 2, 4]
    rng = np.random.Generator(np.random.PCG64(nout + cap))
    Y = rng.integers(30000, 31000, size=(64, nout)).astype(np.uint32)
    wl = Workload("s", 256, 1000.0, 1500.0, 1e-4, nout, 64, 0.0, 1.0, tuple(widths))
    with sps.plan_for(wl) as plan:
        Yd = torch.from_numpy(Y.view(np.int32)).cuda()
        snr = torch.empty(Y.shape, dtype=torch.float32, device="cuda")
        best = torch.empty(Y.shape, dtype=torch.uint8, device="cuda")
        st = torch.empty((64, 2), dtype=torch.int32, device="cuda")
        runs = [sps.sps_search(plan, Yd, nout, widths, s, b, st, thr, td, tt, 0, 5, cap=cap,
                               allow_truncated=True) for s, b in ((snr, best), (None, None))]
    co = oracle.detect(snr.cpu().numpy(), best.cpu().numpy(), thr, td, tt, 0, 5, cap=1 << 16)
    assert co["n_found"] > (cap if 255 <= cap <= 257 else 0)
    for c, n in runs:
        assert len(c) == min(n, cap)
        check_candidates_exact(c, n, co, widths)
