"""Dedispersion on the matrix cores at the edges of its tiles, bit-exact
against the oracle: outputs around whole time tiles, channels around whole
slabs, trials around whole blocks, delays with every remainder mod 16 and the
longest rows of each tiling, on uniform random bytes and on all-255 input."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from sps_inputs import synth  # noqa: E402

pytestmark = pytest.mark.gpu

K_DM, F, FREF, TSAMP = 4.148808e3, 1000.0, 1500.0, 1e-4


@pytest.fixture(scope="module")
def sps():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_02328_amd import sps as mod
    mod.library()
    return mod


def plan_with_delays(sps, lowest, nchan):
    """A plan whose lowest channel has the delays `lowest` (non-decreasing)."""
    unit = TSAMP / (K_DM * (1 / F**2 - 1 / FREF**2))
    f = np.linspace(1400.0, F, nchan) if nchan > 1 else np.array([F])
    dm = np.asarray(lowest, np.float64) * unit
    D = oracle.delays(f, FREF, TSAMP, dm)
    assert np.array_equal(D[:, -1], lowest)
    return sps.sps_plan_create(f, FREF, TSAMP, dm), D


def check(sps, plan, D, nout, short=0, full=False, seed=1):
    nsamp = nout + int(D.max()) - short
    X = np.full((D.shape[1], nsamp), 255, np.uint8) if full else \
        synth.random_bytes(D.shape[1], nsamp, seed=seed)
    Yo = oracle.dedisperse(X, D, nout, nsamp)
    Xd = torch.full((D.shape[1], (nsamp + 15) // 16 * 16 + 16), 0xA5, dtype=torch.uint8,
                    device="cuda")
    Xd[:, :nsamp] = torch.from_numpy(X).cuda()
    Y = torch.full((D.shape[0], nout), -1, dtype=torch.int32, device="cuda")
    sps.sps_dedisperse(plan, Xd, nsamp, Y, nout, sps.SPS_ZERO_PAD)
    assert np.array_equal(Y.cpu().numpy().view(np.uint32), Yo)


def set_tiling(sps, plan, t):
    sps.sps_plan_set_tiling(plan, t["m"], t["dpw"], t["nw"], t["cs"], t["waves_per_eu"])


@pytest.mark.parametrize("index", range(16))
def test_tile_slab_and_block_edges(sps, index):
    if index >= sps.sps_tiling_count():
        pytest.skip("fewer tilings are compiled")
    t = sps.sps_tiling_describe(index)
    nt, nd, cs = 512 * t["m"] - 16, t["dpw"] * t["nw"], t["cs"]
    for ndm, nchan in ((1, 1), (nd, cs), (nd + 1, cs + 1), (2 * nd - 1, 3 * cs - 1)):
        # consecutive delays: every remainder mod 16
        plan, D = plan_with_delays(sps, 3 + np.arange(ndm), nchan)
        with plan:
            set_tiling(sps, plan, t)
            for nout in (1, nt - 1, nt, nt + 1, 2 * nt + 15):
                check(sps, plan, D, nout, short=min(nout - 1, 21), seed=nout)
            check(sps, plan, D, nt + 5, full=True)


# (name of an earlier tiling, trials of its block, largest delay spread its
# staged rows held)
EARLIER = (((5, 1, 16, 16, 8), 16, 749), ((5, 1, 16, 16, 4), 16, 2797), ((5, 1, 16, 16, 0), 16, 2797),
           ((3, 1, 16, 16, 8), 16, 1261), ((3, 1, 16, 16, 0), 16, 1261),
           ((7, 1, 16, 16, 4), 16, 1261), ((7, 1, 16, 16, 0), 16, 1261),
           ((5, 1, 8, 8, 4), 8, 6893), ((5, 1, 8, 8, 0), 8, 6893))


@pytest.mark.parametrize("name,nd,spread", EARLIER)
def test_earlier_tilings_are_still_taken(sps, name, nd, spread):
    plan, D = plan_with_delays(sps, 15 + np.round(np.linspace(0, spread, nd)).astype(np.int64), 5)
    with plan:
        sps.sps_plan_set_tiling(plan, *name)
        check(sps, plan, D, 4100)


def test_longest_rows_and_beyond(sps):
    # spreads up to and past what any tiling stages: the widest row of 8
    # trials, one more (the plain kernel), and tilings refused for them
    limits = [(8, 1024 * 9 - 2048), (8, 1024 * 9 - 2048 + 16)]
    for nd, spread in limits:
        low = np.round(np.linspace(0, spread, nd)).astype(np.int64)
        plan, D = plan_with_delays(sps, low, 3)
        with plan:
            got = sps.sps_plan_get_tiling(plan)
            assert (got["m"] == 0) == (spread > limits[0][1])
            check(sps, plan, D, 2100)
            with pytest.raises(sps.SpsError) as e:
                sps.sps_plan_set_tiling(plan, 4, 1, 16, 16, 4)
            assert e.value.name == "SPS_ERR_RANGE"
            with pytest.raises(sps.SpsError) as e:
                sps.sps_plan_set_tiling(plan, 9, 1, 16, 16, 4)
            assert e.value.name == "SPS_ERR_INVALID_ARG"


@pytest.mark.parametrize("ndm,nouts", [(40, (1, 496, 497, 1009, 2033, 4064, 4065, 4600)),
                                       (1500, (4096, 16384))])
def test_default_tile_by_span(sps, ndm, nouts):
    # no tiling set: the time tile follows the span, on the same staged table
    plan, D = plan_with_delays(sps, np.arange(ndm) * 5 // 2, 33)
    with plan:
        for nout in nouts:
            check(sps, plan, D, nout, short=min(nout - 1, 9), seed=nout)
