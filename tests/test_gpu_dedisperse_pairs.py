"""Dedispersion with channels summed in pairs, bit-exact against the oracle:
sums inside and just outside the range of a signed byte, rows and slabs where
some or all pairs leave it, pairs with more than two distances in a block,
channel orders of either sign, channels past the last whole slab, partial
blocks and tiles, and windows that end past the input."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sps():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_02328_amd import sps as mod
    mod.library()
    return mod


def distances(D):
    """Distances of each channel pair over each block of 16 trials."""
    pairs = D[:, 1::2].astype(np.int64) - D[:, :D.shape[1] // 2 * 2:2]
    return [np.ptp(pairs[i:i + 16], axis=0) + 1 for i in range(0, len(D), 16)]


def data(kind, nchan, nsamp, D, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    X = np.clip(np.rint(rng.normal(128, 16, (nchan, nsamp))), 0, 255).astype(np.uint8)
    if kind == "edges":       # sums of a pair of -128, -129, 127 and 128
        X[:] = rng.choice(np.array([64, 191], np.uint8), (nchan, 1))
        X[1::2] = X[:nchan // 2 * 2:2]        # 64 + 64 - 256 = -128; 191 + 191 - 256 = 126
        for c in rng.integers(0, nchan, 6):
            X[c, rng.integers(0, nsamp, 3)] += 1
        for c in rng.integers(0, nchan, 6):
            X[c, rng.integers(0, nsamp, 3)] -= 1
    elif kind == "channels":  # a tenth of the channels far off, a broadband burst
        X[rng.random(nchan) < 0.1] = rng.integers(0, 256, nsamp)
        X[:, nsamp // 3:nsamp // 3 + 3] = 255
    elif kind == "late":      # every pair from the tenth slab on
        X[160:] = rng.integers(0, 256, X[160:].shape)
    elif kind == "bytes":     # every pair
        X = rng.integers(0, 256, X.shape, dtype=np.uint8)
    elif kind == "full":
        X[:] = 255
    return X


SETUPS = [  # channels, trials, DM range, outputs, first and last channel's frequency
    (256, 1, 100.0, 100.0, 100, 1500.0, 1450.0), (257, 16, 300.0, 305.0, 2033, 1500.0, 1400.0),
    (271, 17, 90.0, 105.0, 2032, 1500.0, 1400.0), (320, 33, 100.0, 115.0, 4500, 1500.0, 1100.0),
    (333, 40, 80.0, 100.0, 700, 1100.0, 1500.0), (2048, 17, 100.0, 135.0, 2200, 1500.0, 1000.0),
    (512, 48, 0.0, 30.0, 2500, 1500.0, 1000.0)]


@pytest.mark.parametrize("nchan,ndm,dm0,dm1,nout,f0,f1", SETUPS)
@pytest.mark.parametrize("kind", ["noise", "edges", "channels", "late", "bytes", "full"])
def test_pairs_match_oracle(sps, nchan, ndm, dm0, dm1, nout, f0, f1, kind):
    f = np.linspace(f0, f1, nchan)
    fref, ts = 1500.0, 1e-4
    dms = np.linspace(dm0, dm1, ndm)
    D = oracle.delays(f, fref, ts, dms)
    more = np.concatenate(distances(D)) > 2
    assert nchan >= 256 and more.mean() <= 0.125  # summed in pairs
    with sps.sps_plan_create(f, fref, ts, dms) as plan:
        for short in (0, 31):
            nsamp = nout + int(D.max()) - short
            X = data(kind, nchan, nsamp, D, seed=nchan + ndm)
            Yo = oracle.dedisperse(X, D, nout, nsamp)
            Xd = torch.full((nchan, (nsamp + 15) // 16 * 16 + 16), 0xA5, dtype=torch.uint8,
                            device="cuda")
            Xd[:, :nsamp] = torch.from_numpy(X).cuda()
            for t in (t for i in range(sps.sps_tiling_count())
                      for t in [sps.sps_tiling_describe(i)] if t["nw"] == 16):
                sps.sps_plan_set_tiling(plan, t["m"], t["dpw"], t["nw"], t["cs"],
                                        t["waves_per_eu"])
                Y = torch.full((ndm, nout), -1, dtype=torch.int32, device="cuda")
                sps.sps_dedisperse(plan, Xd, nsamp, Y, nout, sps.SPS_ZERO_PAD)
                assert np.array_equal(Y.cpu().numpy().view(np.uint32), Yo), (t, short)


def test_the_last_setup_reaches_three_distances():
    nchan, ndm, dm0, dm1, _, f0, f1 = SETUPS[-1]
    D = oracle.delays(np.linspace(f0, f1, nchan), 1500.0, 1e-4, np.linspace(dm0, dm1, ndm))
    assert max(int(v.max()) for v in distances(D)) > 2
