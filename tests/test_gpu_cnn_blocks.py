"""The convolution kernels' 256-pixel blocks, which serve batches of about 128 images (second layer), 512 (third) and 1,024
(fourth, four images a block) on: outputs and gradients at batches whose last block is partial, against the FP64
reference and against the same images in the smaller batches that the 128-pixel blocks serve."""
import numpy as np
import pytest

from oracle import cnn
from synth.surrogate import init_params
from test_gpu_cnn_batches import BOUND, _reference

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1611_03404_amd import celeste as cb
    p = init_params(37)
    c = cb.Context(0)
    net = cb.Net(c, p, np.zeros(27), np.ones(27))
    yield net, p
    net.close()
    c.close()


def _inputs(B):
    import torch
    rng = np.random.default_rng(B)
    x = rng.normal(size=(B, 5, 32, 32)).astype(np.float32)
    t = rng.normal(size=(B, 27)).astype(np.float32)
    return x, t, torch.from_numpy(x).to(torch.bfloat16).cuda(), torch.from_numpy(t).cuda()


@pytest.mark.parametrize("B", [129, 515, 1027])
def test_forward(env, B):
    import torch
    net, p = env
    x, _, xg, _ = _inputs(B)
    print("forward", B, flush=True)
    y = net.forward(xg).cpu().numpy()
    few = np.array([0, 1, B // 2, B - 4, B - 3, B - 2, B - 1])
    q, o = p.copy(), 0
    for k, s in enumerate(cnn.param_shapes()):        # weights are used in BF16, biases in FP32
        n = int(np.prod(s))
        if k % 2 == 0:
            q[o:o + n] = torch.from_numpy(p[o:o + n]).to(torch.bfloat16).float().numpy()
        o += n
    ref, _ = cnn.forward(q, xg[few].double().cpu().numpy())
    scale = np.abs(ref).max()
    assert np.abs(y[few] - ref).max() <= 2e-2 * scale       # the bound of the network's own forward test
    small = np.concatenate([net.forward(xg[a:a + 41].contiguous()).cpu().numpy() for a in range(0, B, 41)])
    assert np.abs(y - small).max() <= 2e-2 * scale


def _check(g, ref, what):
    o = 0
    for k, s in enumerate(cnn.param_shapes()):
        n = int(np.prod(s))
        err = np.linalg.norm(g[o:o + n] - ref[o:o + n]) / np.linalg.norm(ref[o:o + n])
        o += n
        print(what, "layer", k, "relative L2", err, flush=True)
        assert err <= BOUND, (what, k, err)


@pytest.mark.parametrize("B", [131, 515])
def test_gradient(env, B):
    net, p = env
    x, t, xg, tg = _inputs(B)
    loss, g = net.loss_grad(xg, tg)
    print("gradient", B, loss, flush=True)
    ref_loss, ref = _reference(p, x, t)
    assert abs(loss - ref_loss) <= 1e-3 * ref_loss
    _check(g, np.concatenate(ref), B)


def test_gradient_of_parts(env):
    """A batch of 1,027 against its parts of 103 (the last of 100), weighted by their sizes."""
    net, _ = env
    B, part = 1027, 103
    _, _, xg, tg = _inputs(B)
    loss, g = net.loss_grad(xg, tg)
    total, want = 0.0, np.zeros(g.size)
    for a in range(0, B, part):
        n = min(part, B - a)
        l1, g1 = net.loss_grad(xg[a:a + n].contiguous(), tg[a:a + n].contiguous())
        total += l1 * n / B
        want += g1.astype(np.float64) * (n / B)
    assert abs(loss - total) <= 1e-3 * total
    _check(g, want, "parts")
