"""Detection on more tiles than the selection holds on chip (8192): none, one
and a few tile peaks at or above the threshold, and their reading back."""
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


@pytest.mark.parametrize("offers", [0, 1, 2, 3, 200])
@pytest.mark.parametrize("nout,td,tt", [(4100, 1, 30), (4096, 2, 8), (4099, 1, 4)])
def test_few_offers_beyond_8192_tiles(sps, offers, nout, td, tt):
    ndm, widths = 64, [1, 2, 4]
    assert -(-ndm // td) * -(-nout // tt) > 8192
    rng = np.random.Generator(np.random.PCG64(offers + nout))
    snr = rng.standard_normal((ndm, nout)).astype(np.float32)
    np.clip(snr, -5.0, 5.0, out=snr)
    at = rng.choice(ndm * nout, offers, replace=False)
    snr.reshape(-1)[at] = 7.0 + rng.integers(0, 3, offers)  # with ties
    best = rng.integers(0, 3, (ndm, nout)).astype(np.uint8)
    co = oracle.detect(snr, best, 7.0, td, tt, 2, 20, cap=1 << 14)
    wl = Workload("t", 8, 1000.0, 1500.0, 1e-4, nout, ndm, 0.0, 10.0, (1,))
    S, B = torch.from_numpy(snr).cuda(), torch.from_numpy(best).cuda()
    with sps.plan_for(wl) as plan:
        for call in (sps.sps_detect, sps.sps_detect):  # the second on used scratch
            c, n = call(plan, S, B, nout, widths, 7.0, td, tt, 2, 20, cap=1 << 14)
            assert (n > 0) == (offers > 0)
            check_candidates_exact(c, n, co, widths)


@pytest.mark.parametrize("td,tt", [(64, 1024), (64, 4096), (40, 3999)])
def test_hundreds_of_large_tiles(sps, td, tt):
    """512 to 1023 tiles: shared by two workgroups below 2^18 outputs, else not."""
    nd = 16 if tt == 1024 else 8
    ndm, nout, widths = nd * td - 3, (520 // nd + 1) * tt - 5, [1, 2, 4]
    assert 512 <= -(-ndm // td) * -(-nout // tt) < 1024
    g = torch.Generator(device="cuda")
    g.manual_seed(tt)
    S = torch.randn((ndm, nout), generator=g, device="cuda").clamp_(-5.0, 5.0)
    rng = np.random.Generator(np.random.PCG64(tt))
    at = torch.from_numpy(rng.choice(ndm * nout, 900, replace=False)).cuda()
    S.view(-1)[at] = torch.from_numpy(7.0 + rng.integers(0, 3, 900)).float().cuda()
    B = torch.zeros((ndm, nout), dtype=torch.uint8, device="cuda")
    B.view(-1)[at] = torch.from_numpy(rng.integers(0, 3, 900).astype(np.uint8)).cuda()
    co = oracle.detect(S.cpu().numpy(), B.cpu().numpy(), 6.5, td, tt, 2, 20, cap=1 << 12)
    wl = Workload("t", 8, 1000.0, 1500.0, 1e-4, nout, ndm, 0.0, 10.0, (1,))
    with sps.plan_for(wl) as plan:
        c, n = sps.sps_detect(plan, S, B, nout, widths, 6.5, td, tt, 2, 20, cap=1 << 12)
    assert n > 100
    check_candidates_exact(c, n, co, widths)
