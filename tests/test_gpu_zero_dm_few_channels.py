"""Zero-DM filter of few channels: byte for byte against the oracle at the
edges of the tiles and row counts of each form, and no workgroup per handful of
samples."""
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


@pytest.mark.parametrize("nchan", [2, 7, 8, 9, 15, 16, 17, 63, 64, 65, 126, 128, 129])
@pytest.mark.parametrize("inplace", [False, True])
def test_tile_edges(sps, nchan, inplace):
    for nsamp in (1, 3, 15, 16, 17, 511, 512, 513, 1022, 1024, 1029, 2060, 5000):
        X = synth.random_bytes(nchan, nsamp, seed=nchan + nsamp)
        if nsamp > 100:
            X[:, 40:60] = 255       # largest sums and both clips
            X[::2, 60:80] = 0
        pitch = (nsamp + 15) // 16 * 16 + 16
        Xd = torch.full((nchan, pitch), 0xA5, dtype=torch.uint8, device="cuda")
        Xd[:, :nsamp] = torch.from_numpy(X).cuda()
        Xo = Xd if inplace else torch.full((nchan, pitch + 32), 0x5A, dtype=torch.uint8,
                                           device="cuda")
        rest = Xo[:, nsamp:].clone()
        sps.sps_zero_dm(Xd, nsamp, Xo)
        assert np.array_equal(Xo[:, :nsamp].cpu().numpy(), oracle.zero_dm(X, nsamp)), nsamp
        assert torch.equal(Xo[:, nsamp:], rest)     # nothing past the samples is written


def test_few_channels_take_less_than_many(sps):
    # 4 channels move a 32nd of the bytes of 128: 0.17 of their time, launch
    # included, and 0.83 where the samples of a workgroup did not follow the channels
    nsamp = 1 << 20
    ends = [torch.cuda.Event(enable_timing=True) for _ in range(2)]

    def us(nchan):
        X = torch.randint(0, 256, (nchan, nsamp), dtype=torch.uint8, device="cuda")
        Xo = torch.empty_like(X)
        best = []
        for _ in range(5):
            ends[0].record()
            for _ in range(20):
                sps.sps_zero_dm(X, nsamp, Xo)
            ends[1].record()
            ends[1].synchronize()
            best.append(ends[0].elapsed_time(ends[1]))
        return np.median(best)

    few, many = us(4), us(128)
    print("few", few, "many", many)
    assert few < 0.5 * many
