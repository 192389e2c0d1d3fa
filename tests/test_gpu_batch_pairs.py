"""Batches whose channels are summed in pairs, bit-exact against the oracle on
every beam: beams of unequal length with lengths around whole time tiles,
windows that end past a beam's input, and beams whose rows hold pair sums next
to beams whose rows do not, eagerly and replayed from a graph."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from test_gpu_dedisperse_pairs import data, distances  # noqa: E402

pytestmark = pytest.mark.gpu

FREF, TS = 1500.0, 1e-4
SETUPS = [  # channels, trials, DM range, first and last channel's frequency
    (256, 16, 300.0, 305.0, 1500.0, 1400.0), (320, 33, 100.0, 115.0, 1500.0, 1100.0),
    (333, 40, 80.0, 100.0, 1100.0, 1500.0), (512, 48, 0.0, 30.0, 1500.0, 1000.0)]
# outputs and how far a beam's input falls short of its last window
BEAMS = [(2033, 0), (700, 31), (4064, 0), (1520, 5), (4, 3), (4500, 40), (2032, 17), (1521, 0)]
KINDS = ("noise", "bytes", "edges", "channels", "noise", "late", "full", "edges")


@pytest.fixture(scope="module")
def sps():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_02328_amd import sps as mod
    mod.library()
    return mod


@pytest.mark.parametrize("nchan,ndm,dm0,dm1,f0,f1", SETUPS)
@pytest.mark.parametrize("m", [4, 3])
def test_batch_pairs_match_oracle(sps, nchan, ndm, dm0, dm1, f0, f1, m):
    f, dms = np.linspace(f0, f1, nchan), np.linspace(dm0, dm1, ndm)
    D = oracle.delays(f, FREF, TS, dms)
    assert nchan >= 256 and (np.concatenate(distances(D)) > 2).mean() <= 0.125  # in pairs
    stream = torch.cuda.Stream()
    with sps.sps_plan_create(f, FREF, TS, dms) as plan:
        sps.sps_plan_set_tiling(plan, m, 1, 16, 16, 4)
        beams, lengths = [], []
        for nout, short in BEAMS:
            ns = nout + int(D.max()) - short
            beams.append(dict(
                X=torch.full((nchan, (ns + 15) // 16 * 16 + 16), 0xA5, dtype=torch.uint8,
                             device="cuda"), nsamp_in=ns, nout=nout, snr=None, best_w=None,
                Y=torch.zeros((ndm, nout), dtype=torch.int32, device="cuda"),
                stats=torch.zeros((ndm, 2), dtype=torch.int32, device="cuda")))
            lengths.append(ns)
        batch = sps.sps_batch_create(plan, beams, [1, 2, 4], threshold=7.0, tile_dm=16,
                                     tile_t=1024, nms_dm=8, nms_t=64, flags=sps.SPS_ZERO_PAD)
        with batch:
            for rep in range(3):  # eagerly, then replays with new data in between
                X = [data(KINDS[(i + rep) % len(KINDS)], nchan, ns, D, seed=10 * i + rep)
                     for i, ns in enumerate(lengths)]
                with torch.cuda.stream(stream):
                    for b, x in zip(beams, X):
                        b["X"][:, :x.shape[1]] = torch.from_numpy(x).cuda()
                        b["Y"].fill_(-1)
                    if rep == 0:
                        sps.sps_batch_enqueue(batch, stream)
                    else:
                        sps.sps_batch_launch_graph(batch, stream)
                stream.synchronize()
                for i, (b, x) in enumerate(zip(beams, X)):
                    Yo = oracle.dedisperse(x, D, b["nout"], b["nsamp_in"])
                    assert np.array_equal(b["Y"].cpu().numpy().view(np.uint32), Yo), (rep, i)
