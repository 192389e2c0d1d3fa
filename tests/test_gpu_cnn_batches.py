"""The detector's forward pass and gradients do not depend on the batch that a
tile is in: batches around the sizes where the layers change their blocks, and
the smallest, against the same tiles in batches of three."""
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


@pytest.mark.parametrize("n", [1, 63, 64, 65, 130])
def test_forward_is_the_same_in_any_batch(sps, n):
    rng = np.random.Generator(np.random.PCG64(n))
    tiles = cnn.bf16_bits(cnn.bf16(rng.standard_normal((n, 256, 512))))
    T = torch.from_numpy(tiles.view(np.int16)).cuda()
    with sps.sps_cnn_create(n) as net, sps.sps_cnn_create(3) as small:
        heads = []
        for c, step in ((net, n), (small, 3)):
            sps.sps_cnn_set_params(c, _flat(cnn.init_params(41)))
            for run in (sps.sps_cnn_forward, sps.sps_cnn_infer):
                head = torch.zeros((n, 3, 8, 16), dtype=torch.float32, device="cuda")
                for i in range(0, n, step):
                    m = min(step, n - i)
                    run(c, T[i:i + m].contiguous(), m, head[i:i + m])
                heads.append(head.cpu().numpy())
        # the products of an output are summed in the order of K alone
        for h in heads[1:]:
            assert np.array_equal(heads[0], h)


# n copies of one tile against 4 copies: the mean over tiles is the same.  At 64
# the loss scale 1 / n differs by a power of two, so every rounded signal is the
# same but for it, and gradients differ by the order of float32 sums of up to
# 2^19 terms (about 2^-24 x 2^9.5 of their spread); at 63 every bfloat16 signal
# may also round the other way (2^-9 each).  A wrong block is off by its share.
@pytest.mark.parametrize("n,tol", [(63, 2.0 ** -6), (64, 2.0 ** -10)])
def test_gradients_are_the_same_in_any_batch(sps, n, tol):
    rng = np.random.Generator(np.random.PCG64(7))
    tile = cnn.bf16_bits(cnn.bf16(rng.standard_normal((1, 256, 512))))
    y = np.zeros((1, 3, 8, 16), np.float32)
    y[0, :, 3, 5] = 1.0, 0.4, 0.6
    grads = []
    for m in (n, 4):
        T = torch.from_numpy(np.repeat(tile, m, axis=0).view(np.int16)).cuda()
        Y = torch.from_numpy(np.repeat(y, m, axis=0)).cuda()
        loss = torch.zeros(1, dtype=torch.float32, device="cuda")
        with sps.sps_cnn_create(m) as net:
            sps.sps_cnn_set_params(net, _flat(cnn.init_params(41)))
            sps.sps_cnn_loss_grad(net, T, Y, m, loss)
            torch.cuda.synchronize()
            grads.append(np.asarray(sps.sps_cnn_get_grads(net), np.float64))
    a, b = grads
    assert np.abs(b).max() > 0
    assert np.all(np.abs(a - b) <= tol * np.abs(b).max())
