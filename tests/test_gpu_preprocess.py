"""Zero-DM filter and square-law downsampling at the edges of their tiles and
variants, byte for byte against the oracle."""
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


# channels around the row counts that stay in registers (128 rows per step)
@pytest.mark.parametrize("nchan", [1, 127, 128, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4111])
@pytest.mark.parametrize("nsamp", [1, 16, 127, 129, 300])
@pytest.mark.parametrize("inplace", [False, True])
def test_zero_dm_edges(sps, nchan, nsamp, inplace):
    X = synth.random_bytes(nchan, nsamp, seed=nchan + nsamp)
    if nsamp > 100:
        X[:, 40:60] = 255       # largest sums and both clips
        X[::2, 60:80] = 0
    pitch = (nsamp + 15) // 16 * 16 + 16
    Xd = torch.full((nchan, pitch), 0xA5, dtype=torch.uint8, device="cuda")
    Xd[:, :nsamp] = torch.from_numpy(X).cuda()
    Xo = Xd if inplace else torch.full((nchan, pitch + 32), 0x5A, dtype=torch.uint8, device="cuda")
    rest = Xo[:, nsamp:].clone()
    sps.sps_zero_dm(Xd, nsamp, Xo)
    assert np.array_equal(Xo[:, :nsamp].cpu().numpy(), oracle.zero_dm(X, nsamp))
    assert torch.equal(Xo[:, nsamp:], rest)     # nothing past the samples is written


@pytest.mark.parametrize("factor", list(range(1, 19)) + [32, 100, 4095, 4096, 4097, 70001])
def test_downsample_factors(sps, factor):
    rng = np.random.default_rng(factor)
    for nb, extra, shift in ((1, 0, 0), (3, factor - 1, 1), (17, 1, 2), (1037 if factor < 100 else 5, 0, 3)):
        nsamp = nb * factor + min(extra, factor - 1)
        X = rng.integers(0, 256, (3, nsamp), dtype=np.uint8)
        X[1] = 255
        X[2] = rng.integers(0, 3, nsamp, dtype=np.uint8)
        # rows at any byte address
        buf = torch.full((3, nsamp + 9), 0xA5, dtype=torch.uint8, device="cuda")
        Xd = buf[:, shift:]
        Xd[:, :nsamp] = torch.from_numpy(X).cuda()
        out = torch.full((3, nb + 7), 0x5A, dtype=torch.uint8, device="cuda")
        sps.sps_downsample_sqrt(Xd, nsamp, factor, out[:, shift:])
        assert np.array_equal(out[:, shift:shift + nb].cpu().numpy(),
                              oracle.downsample_sqrt(X, factor, nsamp))
        assert bool((out[:, shift + nb:] == 0x5A).all()) and bool((out[:, :shift] == 0x5A).all())
