"""Delay spreads whose rows leave room for two workgroups on a CU run two: the
default tilings and the names of earlier ones at the ends of the row lengths,
bit-exact against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_gpu_dedisperse_matrix import check, plan_with_delays  # noqa: E402

pytestmark = pytest.mark.gpu

LDS, SIMDS = 160 * 1024, 4


@pytest.fixture(scope="module")
def sps():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_02328_amd import sps as mod
    mod.library()
    return mod


# spreads over 8 trials; rows of 5 KiB held 3840 at most when a tile was 1280 outputs long
@pytest.mark.parametrize("spread", [2048, 2049, 2064, 2310, 3072, 3073, 3088, 3584, 3585, 3600,
                                    3840, 4096])
@pytest.mark.parametrize("name", [None, (5, 1, 8, 8, 4)])
def test_two_workgroups_per_cu(sps, spread, name):
    low = 15 + np.round(np.linspace(0, spread, 8)).astype(np.int64)
    for nchan in (1, 8, 13):
        plan, D = plan_with_delays(sps, np.concatenate([low, low[-1] + low[:5]]), nchan)
        with plan:
            if name:
                sps.sps_plan_set_tiling(plan, *name)
            t = sps.sps_plan_get_tiling(plan)
            assert 2 * t["lds_bytes"] <= LDS and SIMDS * t["waves_per_eu"] >= 2 * t["nw"], t
            for nout in (1, 1009, 2100, 4100):
                check(sps, plan, D, nout, short=min(nout - 1, 21), seed=nout)


@pytest.mark.parametrize("spread", [4112, 5000, 7168])
def test_wider_spreads_run_one(sps, spread):
    low = 15 + np.round(np.linspace(0, spread, 8)).astype(np.int64)
    plan, D = plan_with_delays(sps, low, 9)
    with plan:
        assert sps.sps_plan_get_tiling(plan)["nw"] == 8
        check(sps, plan, D, 4100)
