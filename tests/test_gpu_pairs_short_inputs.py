"""Channels in pairs on inputs of less than one 16-byte vector, down to none:
sums as the oracle's, whatever lies behind the samples."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from test_gpu_dedisperse_pairs import distances  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sps():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_02328_amd import sps as mod
    mod.library()
    return mod


@pytest.mark.parametrize("nsamp", [0, 1, 15, 16, 17, 31, 33])
@pytest.mark.parametrize("m", [4, 3])
def test_short_inputs(sps, nsamp, m):
    nchan, ndm, nouts = 271, 17, (4, 40, 2100)
    f, dms = np.linspace(1500.0, 1400.0, nchan), np.linspace(0.0, 10.0, ndm)
    D = oracle.delays(f, 1500.0, 1e-4, dms)
    assert (np.concatenate(distances(D)) > 2).mean() <= 0.125  # summed in pairs
    rng = np.random.Generator(np.random.PCG64(nsamp))
    X = rng.integers(0, 256, (nchan, nsamp), dtype=np.uint8)
    pitch = max(16, (nsamp + 15) // 16 * 16)  # rows of no more than they need
    Xd = torch.full((nchan, pitch), 0xA5, dtype=torch.uint8, device="cuda")
    Xd[:, :nsamp] = torch.from_numpy(X).cuda()
    host = np.full((nchan, pitch), 0xA5, np.uint8)
    host[:, :nsamp] = X
    with sps.sps_plan_create(f, 1500.0, 1e-4, dms) as plan:
        sps.sps_plan_set_tiling(plan, m, 1, 16, 16, 4)
        want = [oracle.dedisperse(host, D, n, nsamp) for n in nouts]
        beams = []
        for n, Yo in zip(nouts, want):
            Y = torch.full((ndm, n), -1, dtype=torch.int32, device="cuda")
            sps.sps_dedisperse(plan, Xd, nsamp, Y, n, sps.SPS_ZERO_PAD)
            assert np.array_equal(Y.cpu().numpy().view(np.uint32), Yo), n
            beams.append(dict(X=Xd, nsamp_in=nsamp, nout=n, snr=None, best_w=None,
                              Y=torch.full((ndm, n), -1, dtype=torch.int32, device="cuda"),
                              stats=torch.zeros((ndm, 2), dtype=torch.int32, device="cuda")))
        with sps.sps_batch_create(plan, beams, [1, 2, 4], threshold=7.0, tile_dm=16, tile_t=1024,
                                  nms_dm=8, nms_t=64, flags=sps.SPS_ZERO_PAD) as batch:
            sps.sps_batch_enqueue(batch)
            torch.cuda.synchronize()
        for b, Yo in zip(beams, want):
            assert np.array_equal(b["Y"].cpu().numpy().view(np.uint32), Yo), b["nout"]
