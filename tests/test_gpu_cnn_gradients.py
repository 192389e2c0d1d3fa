"""Gradients of a batch of distinct tiles against the mean of the gradients of
its tiles one at a time, parameter tensor by parameter tensor."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402

cnn = oracle.cnn()

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sps():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_02328_amd import sps as mod
    mod.library()
    return mod


def _flat(params):
    return np.concatenate([np.asarray(params[k], np.float32).ravel()
                           for k in cnn.param_names()])


def _tensors(vec, like):
    out, o = {}, 0
    for k in cnn.param_names():
        out[k] = np.asarray(vec[o:o + like[k].size], np.float64)
        o += like[k].size
    return out


def _tiles(n, seed):
    """Pooled S/N of noise times the detector's scale of 0.125, a pulse in two tiles of three."""
    rng = np.random.Generator(np.random.PCG64(seed))
    t = rng.normal(0.3, 0.09, (n, cnn.TILE_DM, cnn.TILE_T))
    pulses = [None] * n
    for i in range(n):
        if i % 3:
            r, c = rng.uniform(8, cnn.TILE_DM - 8), rng.uniform(8, cnn.TILE_T - 8)
            pulses[i] = (r, c)
            t[i, int(r) - 3:int(r) + 4, int(c) - 3:int(c) + 4] += rng.uniform(0.6, 4.0)
    return cnn.bf16_bits(cnn.bf16(t)).view(np.int16), cnn.labels_for(n, pulses).astype(np.float32)


@pytest.fixture(scope="module")
def singles(sps):
    """130 tiles, labels, parameters, and each tile's loss and gradients alone."""
    params = cnn.init_params(43)
    tiles, y = _tiles(130, 17)
    T, Y = torch.from_numpy(tiles).cuda(), torch.from_numpy(y).cuda()
    out = []
    with sps.sps_cnn_create(1) as net:
        sps.sps_cnn_set_params(net, _flat(params))
        loss = torch.zeros(1, dtype=torch.float32, device="cuda")
        for i in range(len(tiles)):
            sps.sps_cnn_loss_grad(net, T[i:i + 1].contiguous(), Y[i:i + 1].contiguous(), 1, loss)
            torch.cuda.synchronize()
            out.append((float(loss.cpu()[0]), _tensors(sps.sps_cnn_get_grads(net), params)))
    return params, T, Y, out


# A batch scales every loss by 1 / n.  For a power of two each bfloat16 signal
# rounds as it does alone, and gradients differ by the order of float32 sums: at
# most 2^20 terms of mixed sign, whose sum is about 2^-10 of their magnitudes',
# so about 2^-24 x 2^10 = 2^-14 of a tensor's norm.  Otherwise each of the six layers'
# signals may round the other way: 2^-9 each, at most 6 x 2^-9 together.  One
# tile of 128 left out or taken twice is 2^-7 at least.
@pytest.mark.parametrize("n,tol", [(2, 2.0 ** -11), (4, 2.0 ** -11), (8, 2.0 ** -11),
                                   (16, 2.0 ** -11), (32, 2.0 ** -11), (64, 2.0 ** -11),
                                   (128, 2.0 ** -11), (3, 2.0 ** -6), (33, 2.0 ** -6),
                                   (63, 2.0 ** -6), (65, 2.0 ** -6), (130, 2.0 ** -6)])
def test_batch_gradients_are_the_mean_of_single_tiles(sps, singles, n, tol):
    params, T, Y, one = singles
    with sps.sps_cnn_create(n) as net:
        sps.sps_cnn_set_params(net, _flat(params))
        loss = torch.zeros(1, dtype=torch.float32, device="cuda")
        sps.sps_cnn_loss_grad(net, T[:n].contiguous(), Y[:n].contiguous(), n, loss)
        torch.cuda.synchronize()
        got = _tensors(sps.sps_cnn_get_grads(net), params)
        L = float(loss.cpu()[0])
    mean = np.mean([l for l, _ in one[:n]])
    assert abs(L - mean) <= 2.0 ** -16 * mean  # positive terms
    for k in cnn.param_names():
        want = np.mean([g[k] for _, g in one[:n]], axis=0)
        norm = np.linalg.norm(want)
        assert norm > 0, k
        err = np.linalg.norm(got[k] - want) / norm
        print(n, k, err)
        assert err <= tol, (k, err)
