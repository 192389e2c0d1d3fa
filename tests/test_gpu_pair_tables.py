"""The tables for summing channels in pairs are held only by tilings that read
them: time tiles of at least three steps."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

NCHAN, NDM = 4096, 2048
TABLES = 64 * (NCHAN // 16) * (NDM + NDM // 16)
SLACK = 8 << 20  # four allocations, each rounded up to 2 MiB at most


@pytest.fixture(scope="module")
def sps():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_02328_amd import sps as mod
    mod.library()
    return mod


def test_tables_are_held_by_the_tilings_that_read_them(sps):
    assert TABLES > 2 * SLACK
    f = np.linspace(1500.0, 1000.0, NCHAN)
    with sps.sps_plan_create(f, 1500.0, 49.152e-6, np.linspace(0.0, 100.0, NDM)) as plan:
        free = {}
        for m in (4, 2, 1, 3, 2, 4):
            sps.sps_plan_set_tiling(plan, m, 1, 16, 16, 4)
            torch.cuda.synchronize()
            free.setdefault(m, []).append(torch.cuda.mem_get_info()[0])
        base = free[4][0]
        for m, v in free.items():
            for x in v:
                assert abs(x - base - (TABLES if m < 3 else 0)) <= SLACK, (m, x - base)
