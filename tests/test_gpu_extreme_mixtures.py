"""Mixture components at the ends of FP32 under the whole-tile skips: a PSF so narrow that its derivatives' polynomials
overflow away from its centre, where the density is 0, and shapes whose constants are not finite."""
import numpy as np
import pytest

import synth
from synth.generate import perturb_theta
from helpers import assert_derivs_close, assert_elbo_close, oracle_eval

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1611_03404_amd import celeste as cb
    c = cb.Context(0)
    yield cb, c
    c.close()


@pytest.mark.parametrize("tile_w", [8, 16])
@pytest.mark.parametrize("var", [1e-4, 1e-8, 1e-10, 1e-20, 1e-40])
def test_narrow_psf(env, var, tile_w):
    """The source's light falls between the pixels, so every term of it is 0: finite derivatives, the oracle's."""
    cb, ctx = env
    sb = synth.make_config(0)
    sb.img_psf[:, :, 3] = sb.img_psf[:, :, 5] = var
    sb.img_psf[:, :, 4] = 0.0
    th = perturb_theta(sb.theta_truth, 1)
    th[:, 6] = 1e-3 * np.sqrt(var)
    v, g, H = oracle_eval(sb, 0, th[0])
    b = cb.Batch.from_synth(sb)
    print("narrow psf", var, tile_w, flush=True)
    try:
        ctx.set_option(cb.OPT_TILE_W, tile_w)
        e1, g1, _ = ctx.elbo_eval(b, th, want="grad")
        e2, g2, H2 = ctx.elbo_eval(b, th, want="hess")
    finally:
        ctx.set_option(cb.OPT_TILE_W, 8)
    for e in (e1, e2):
        assert_elbo_close(e[0], v)
    assert np.isfinite(H2).all()
    assert_derivs_close(g1[0], H2[0], g, H)
    assert_derivs_close(g2[0], H2[0], g, H)


def test_constants_that_are_not_finite_are_not_skipped(env):
    """A scale whose square leaves FP64: the galaxy's densities are NaN, and so are the ELBO and the rendered patch."""
    import torch
    cb, ctx = env
    sb = synth.make_config(0)
    th = perturb_theta(sb.theta_truth, 1)
    th[:, 6] = 1e200
    e = ctx.elbo_eval(cb.Batch.from_synth(sb), th, want="value")[0]
    assert np.isnan(e).all()
    one = np.array([1], np.int32)
    b = cb.Batch(np.array([0, 1], np.int64), 2 * one, 9 * one, 9 * one, 9 * one, np.array([[3.0, 4.0]]),
                 np.array([[1.0, 0, 0, 1.0, 0, 0]]), np.array([90.0]), np.ones(1), sb.img_psf[:1], sb.img_npsf[:1],
                 torch.ones(81, device="cuda"), np.zeros(1, np.int64), sb.prior, sb.profiles)
    th[:, 0:2] = 8.0
    f = ctx.render_fields(b, torch.from_numpy(th).cuda(), np.zeros(1, np.int32), 1, 20, 20)
    for x in f:
        x = x.reshape(20, 20)
        assert bool(torch.isnan(x[4:13, 3:12]).all()) and int(torch.isnan(x).sum()) == 81
