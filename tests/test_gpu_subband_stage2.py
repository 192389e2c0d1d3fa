"""The second stage of subband dedispersion at the edges of its forms,
bit-exact against the oracle: shifts up to and past the 1024 samples that the
LDS form stages, outputs around its tiles of 1024, fine trials that do not
fill a coarse group or its eights, and single subbands."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from sps_inputs import synth  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sps():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_02328_amd import sps as mod
    mod.library()
    return mod


def rmax_of(nchan, f, ndm, n0, nsub, ts, ddm):
    R, _, _ = oracle.subband_residuals(f, 1500.0, ts, oracle.equal_subbands(nchan, nsub), ndm, 0.0,
                                       ddm, n0)
    return int(R.max()), R


# the step that puts the largest shift at `rmax` samples is found from the table
@pytest.mark.parametrize("rmax", [0, 1, 255, 1023, 1024, 1025, 2500])
@pytest.mark.parametrize("ndm,n0,nsub,nout", [
    (17, 8, 4, 1023), (16, 16, 1, 1024), (21, 9, 3, 1025), (10, 3, 2, 3000), (5, 8, 16, 7)])
def test_stage2_edges(sps, rmax, ndm, n0, nsub, nout):
    nchan, ts = 16, 1e-4
    f = 1500.0 - (np.arange(nchan) + 0.5) * 500.0 / nchan
    lo, hi = 0.0, 1e4
    for _ in range(100):  # bisection on the DM step
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if rmax_of(nchan, f, ndm, n0, nsub, ts, mid)[0] < rmax else (lo, mid)
    ddm = hi if rmax else 1e-9
    got, R = rmax_of(nchan, f, ndm, n0, nsub, ts, ddm)
    assert got == rmax
    with sps.sps_subband_plan_create(f, 1500.0, ts, ndm, 0.0, ddm, n0, nsub) as plan:
        Dc, _, _, mx = sps.sps_subband_tables(plan)
        nsamp = nout + mx
        X = synth.random_bytes(nchan, nsamp, seed=rmax + nout)
        Xd = torch.full((nchan, (nsamp + 15) // 16 * 16 + 16), 0x5A, dtype=torch.uint8, device="cuda")
        Xd[:, :nsamp] = torch.from_numpy(X).cuda()
        Y = torch.full((ndm, nout), -1, dtype=torch.int32, device="cuda")
        sps.sps_dedisperse_subband(plan, Xd, nsamp, Y, nout)
        Yo = oracle.subband_dedisperse(X, Dc, oracle.equal_subbands(nchan, nsub), R, n0, nout, nsamp)
        assert np.array_equal(Y.cpu().numpy().view(np.uint32), Yo)
