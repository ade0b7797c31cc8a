"""Host batches whose pixels and results go through the two pinned pieces in one, exactly two and many turns, in a context
whose pieces grow, equal the same batch in device memory, bit for bit."""
import numpy as np
import pytest

import synth
from synth.generate import perturb_theta

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cb():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1611_03404_amd import celeste
    return celeste


def _batches(cb, n_img, side, pitch, nbr, seed):
    """One source's n_img images of side x side pixels: in host memory with rows `pitch` apart, and in device memory as
    the host ones are laid there, without gaps (the pixel constants of rows with gaps are summed in another order)."""
    import torch
    z = synth.make_config(0)
    rng = np.random.default_rng(seed)
    rep = np.arange(n_img) % 5
    px = rng.poisson(100.0, n_img * side * pitch).astype(np.float32)
    nb = rng.uniform(0, 9, (2, n_img * side * pitch)).astype(np.float32)

    def make(f, pitch):
        kw = dict(nbr_mean=f(nb[0]), nbr_var=f(nb[1])) if nbr else {}
        return cb.Batch(np.array([0, n_img], np.int64), z.img_band[rep], np.full(n_img, side), np.full(n_img, side),
                        np.full(n_img, pitch), z.img_origin[rep], z.img_wcs[rep], z.img_sky[rep], z.img_calib[rep],
                        z.img_psf[rep], z.img_npsf[rep], f(px), np.arange(n_img, dtype=np.int64) * side * pitch, z.prior,
                        z.profiles, **kw)

    def dense(a):
        return torch.from_numpy(np.ascontiguousarray(a.reshape(n_img, side, pitch)[:, :, :side]).ravel()).cuda()

    return make(lambda a: a, pitch), make(dense, side), perturb_theta(z.theta_truth, seed)


def _same(ctx, host, dev, th, want):
    import torch
    a = ctx.elbo_eval(host, th, want=want)
    b = ctx.elbo_eval(dev, torch.from_numpy(th).cuda(), want=want)
    for x, y in zip(a, b):
        assert (x is None) == (y is None)
        if x is not None:
            assert np.array_equal(x, y.cpu().numpy())


@pytest.mark.parametrize("want", ["value", "grad", "hess"])
def test_pixels_in_pieces(cb, want):
    ctx = cb.Context(0)
    # 16 images of 64 x 64 are one piece of 256 KB; the pieces grow at 4 MB and stay grown
    for n_img, side, pitch, nbr in ((1, 1, 1, False), (15, 64, 64, False), (16, 64, 64, False), (17, 64, 64, False),
                                    (32, 64, 64, False), (33, 64, 64, False), (20, 63, 70, True), (70, 61, 61, True),
                                    (300, 64, 64, False), (513, 65, 67, False), (3, 40, 41, True)):
        print("pieces", n_img, side, pitch, nbr, want, flush=True)
        host, dev, th = _batches(cb, n_img, side, pitch, nbr, n_img + side)
        _same(ctx, host, dev, th, want)
    ctx.close()


def test_results_in_pieces(cb):
    """Hessians of 1, 100 and 1,300 sources: less and more than the ring holds (5.8 KB each), 7.9 MB in the last."""
    ctx = cb.Context(0)
    sb = synth.make_config(0)
    for n in (1, 100, 1300):
        print("results", n, flush=True)
        host, dev, th = _batches(cb, 1, 5, 5, False, n)
        th = perturb_theta(np.repeat(sb.theta_truth, n, axis=0), n)
        many = []
        for b in (host, dev):
            m = b.subset(np.zeros(n, np.int64))[0]
            many.append(m)
        _same(ctx, *many, th, "hess")
    ctx.close()


@pytest.mark.parametrize("n", [46, 47, 93, 94, 186, 187, 400])
def test_results_beside_few_pixels(cb, n):
    """Hessians (5,624 bytes a source) of one image of 5 x 5 pixels each, on either side of 256 KB, 512 KB and 1 MB, in a
    new context and in one whose ring has come to be mapped whole meanwhile."""
    ctx = cb.Context(0)
    host, dev, th = _batches(cb, 1, 5, 5, False, n)
    th = perturb_theta(np.repeat(th, n, axis=0), n)
    host, dev = (b.subset(np.zeros(n, np.int64))[0] for b in (host, dev))
    for k in range(8):
        print("few pixels", n, k, flush=True)
        _same(ctx, host, dev, th, "hess")
    ctx.close()


def test_no_error_is_left_behind(cb):
    """While a call waits for its kernels it asks the stream whether it is done: the answer "not yet" must not
    come up as the error of somebody's next launch."""
    ctx = cb.Context(0)
    host, _, th = _batches(cb, 300, 64, 64, False, 1)
    hip_last_error = cb.load().hipGetLastError
    for k in range(6):
        print("call", k, flush=True)
        ctx.elbo_eval(host, th, want="hess")
        assert hip_last_error() == 0
    ctx.close()
