"""The tables for summing channels in pairs in the server's account: counted
while they are held, and given up where a stream or a detector would not fit
beside them, with the same planes and candidates."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from test_gpu_dedisperse_pairs import data, distances  # noqa: E402

pytestmark = pytest.mark.gpu

MIB = 1 << 20
DET = dict(threshold=7.0, tile_dm=16, tile_t=512, nms_dm=8, nms_t=64)
# channels, trials, DM range, sampling: set-ups summed in pairs
SMALL, OTHER = (512, 48, 0.0, 30.0, 1e-4), (320, 33, 100.0, 115.0, 1e-4)
LARGE = (4096, 2048, 0.0, 100.0, 49.152e-6)


@pytest.fixture(scope="module")
def sps():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_02328_amd import sps as mod
    mod.library()
    return mod


def _band(setup):
    return np.linspace(1500.0, 1000.0, setup[0]), np.linspace(setup[2], setup[3], setup[1])


def _add(sps, server, setup, chunk):
    f, dms = _band(setup)
    return sps.sps_server_add_stream(server, f, 1500.0, setup[4], dms, [1, 2, 4, 8],
                                     chunk_len=chunk, **DET)


def _tables(setup):
    """Bytes of one plan's tables: a 64-byte entry per trial and per block of 16 trials for each
    16 channels."""
    return 64 * (setup[0] // 16) * (setup[1] + (setup[1] + 15) // 16)


def _paired(setup):
    f, dms = _band(setup)
    D = oracle.delays(f, 1500.0, setup[4], dms)
    return setup[0] >= 256 and (np.concatenate(distances(D)) > 2).mean() <= 0.125


def _used(sps, setups, chunk, workers):
    with sps.sps_server_create(1 << 40, workers) as server:
        for s in setups:
            _add(sps, server, s, chunk)
        return sps.sps_server_memory(server)["used"]


def test_account_covers_what_is_held(sps):
    assert _paired(LARGE)
    _used(sps, [LARGE], 4096, 2)  # code and runtime allocations of a first use
    free0 = torch.cuda.mem_get_info()[0]
    with sps.sps_server_create(1 << 40, 2) as server:
        _add(sps, server, LARGE, 4096)
        held = free0 - torch.cuda.mem_get_info()[0]
        used = sps.sps_server_memory(server)["used"]
    print("held", held, "accounted", used, "tables", 2 * _tables(LARGE))
    # each allocation is rounded up, to 2 MiB at most; 2 workers x 11 and a ring
    assert held <= used + 23 * 2 * MIB and 2 * _tables(LARGE) > 23 * 2 * MIB


@pytest.mark.parametrize("short", [1, 2])  # of the tables of one worker, of both
def test_tables_give_way_to_a_stream(sps, short):
    workers, chunk, T = 2, 2500, _tables(SMALL)
    assert _paired(SMALL)
    full = _used(sps, [SMALL], chunk, workers)
    f, dms = _band(SMALL)
    D = oracle.delays(f, 1500.0, SMALL[4], dms)
    X = data("noise", SMALL[0], 2 * chunk, D, seed=3)
    got = []
    for budget in (full, full - short * T):
        with sps.sps_server_create(budget, workers) as server:
            sid = _add(sps, server, SMALL, chunk)
            assert sps.sps_server_memory(server)["used"] == budget
            for k in range(2):
                Y = torch.zeros((SMALL[1], chunk), dtype=torch.int32, device="cuda")
                c, n = sps.sps_server_push(server, sid, X[:, k * chunk:(k + 1) * chunk], Y_copy=Y)
                torch.cuda.synchronize()
                got.append((Y.cpu().numpy(), c, n))
    for (Ya, ca, na), (Yb, cb, nb) in zip(got[:2], got[2:]):
        assert np.array_equal(Ya, Yb) and na == nb and np.array_equal(ca, cb)
    with sps.sps_server_create(full - workers * T - 1, workers) as server:
        with pytest.raises(sps.SpsError) as e:
            _add(sps, server, SMALL, chunk)
        assert e.value.name == "SPS_ERR_NOMEM"
        assert sps.sps_server_memory(server)["used"] == 0


def test_held_tables_give_way_to_another_set_up(sps):
    chunk, T, T2 = 2500, _tables(SMALL), _tables(OTHER)
    assert _paired(SMALL) and _paired(OTHER)
    both, first = _used(sps, [SMALL, OTHER], chunk, 1), _used(sps, [SMALL], chunk, 1)
    with sps.sps_server_create(both - T2 - 1, 1) as server:
        _add(sps, server, SMALL, chunk)
        assert sps.sps_server_memory(server)["used"] == first
        sid = _add(sps, server, OTHER, chunk)
        assert sps.sps_server_memory(server)["used"] == both - T2 - T
        f, dms = _band(OTHER)
        D = oracle.delays(f, 1500.0, OTHER[4], dms)
        X = data("edges", OTHER[0], chunk, D, seed=5)
        Y = torch.zeros((OTHER[1], chunk), dtype=torch.int32, device="cuda")
        sps.sps_server_push(server, sid, X, Y_copy=Y)
        torch.cuda.synchronize()
        lead = (int(D.max()) + 15) // 16 * 16
        series = np.concatenate([np.zeros((OTHER[0], lead), np.uint8), X], axis=1)
        assert np.array_equal(Y.cpu().numpy().view(np.uint32), oracle.dedisperse(series, D, chunk))
    # not enough even so: nothing is given up
    with sps.sps_server_create(both - T2 - T - 1, 1) as server:
        _add(sps, server, SMALL, chunk)
        with pytest.raises(sps.SpsError):
            _add(sps, server, OTHER, chunk)
        assert sps.sps_server_memory(server)["used"] == first


def test_held_tables_give_way_to_a_detector(sps):
    setup, chunk = (320, 512, 100.0, 160.0, 1e-4), 4096
    assert _paired(setup)
    tile = 256 * 512 * 2
    full = _used(sps, [setup], chunk, 1)
    net = sps.sps_cnn_create(1)
    with net, sps.sps_server_create(full + tile - 1, 1) as server:
        _add(sps, server, setup, chunk)
        sps.sps_server_set_detector(server, net)
        assert sps.sps_server_memory(server)["used"] == full + tile - _tables(setup)
        sps.sps_server_set_detector(server, None)
