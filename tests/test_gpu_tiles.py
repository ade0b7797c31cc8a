"""Tile walks and whole-tile skips of the pixel kernels at the sizes where they can go wrong: images
narrower than a tile, bands of fewer than 64 pixels, partial last bands and tiles, work items of one
band, subsampled items of blocks that do not adjoin.  The skips change no bit against the option that
skips nothing, and the results meet the FP64 oracle."""
import numpy as np
import pytest

import synth
from synth.generate import perturb_theta
from helpers import assert_derivs_close, assert_elbo_close, oracle_eval

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (3, 2), (7, 1), (9, 3), (8, 8), (17, 7), (16, 9), (31, 5), (40, 23), (33, 64)]   # (h, w)


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1611_03404_amd import celeste as cb
    c = cb.Context(0)
    yield cb, c
    c.close()


def _one(h, w, seed, far):
    """One five-band source with h x w patches, its centre in the patch or `far` pixels to its right."""
    sb = synth.make_config(0)
    rng = np.random.default_rng(seed)
    sb.img_h[:], sb.img_w[:], sb.img_pitch[:] = h, w, w
    n = h * w
    sb.img_pix_off = np.arange(5, dtype=np.int64) * n
    sb.pixels = rng.poisson(100.0, 5 * n).astype(np.float32)
    sb.img_origin[:] = np.rint(sb.u_cat[0]) - np.array([w // 2 + far, h // 2])
    return sb


@pytest.mark.parametrize("want", ["hess", "grad", "value"])
@pytest.mark.parametrize("shape", SHAPES)
def test_small_shapes_skips_and_oracle(env, shape, want):
    cb, ctx = env
    for far in (0, 14):
        sb = _one(*shape, seed=shape[0] * 100 + shape[1], far=far)
        th = perturb_theta(sb.theta_truth, 3)
        b = cb.Batch.from_synth(sb)
        ref = oracle_eval(sb, 0, th[0])
        try:
            for chunk, tw in ((4096, 8), (64, 8), (4096, 16)):
                print("shape", shape, "far", far, "chunk", chunk, "tile", tw, want, flush=True)
                ctx.set_option(cb.OPT_CHUNK_PX, chunk)
                ctx.set_option(cb.OPT_TILE_W, tw)
                ctx.set_option(cb.OPT_VALUE_TILE_W, tw)
                ctx.set_option(cb.OPT_EXACT_ZERO, 1)
                e0, g0, H0 = ctx.elbo_eval(b, th, want=want)
                ctx.set_option(cb.OPT_EXACT_ZERO, 0)
                e1, g1, H1 = ctx.elbo_eval(b, th, want=want)
                assert np.array_equal(e0, e1)
                assert_elbo_close(e1[0], ref[0])
                if want != "value":
                    assert np.array_equal(g0, g1)
                if want == "hess":
                    assert np.array_equal(H0, H1)
                    assert_derivs_close(g1[0], H1[0], ref[1], ref[2])
        finally:
            ctx.set_option(cb.OPT_CHUNK_PX, 4096)
            ctx.set_option(cb.OPT_TILE_W, 8)
            ctx.set_option(cb.OPT_VALUE_TILE_W, 8)
            ctx.set_option(cb.OPT_EXACT_ZERO, 0)


@pytest.mark.parametrize("shape", [(40, 3), (41, 7), (64, 23), (23, 61)])
def test_kept_blocks_skips(env, shape):
    cb, ctx = env
    sb = _one(*shape, seed=5, far=0)
    th = perturb_theta(sb.theta_truth, 4)
    b = cb.Batch.from_synth(sb)
    nb = (shape[0] + 7) // 8
    keep = np.tile(np.array([1, 0, 1, 1, 0, 1, 0, 1], np.uint8)[:nb], 5)
    off = np.arange(6, dtype=np.int64) * nb
    try:
        for chunk in (64, 4096):
            print("kept", shape, "chunk", chunk, flush=True)
            ctx.set_option(cb.OPT_CHUNK_PX, chunk)
            ctx.set_option(cb.OPT_EXACT_ZERO, 1)
            r0 = [ctx.elbo_eval_sampled(b, th, keep, off, 0.5, want=w) for w in ("value", "grad", "hess")]
            ctx.set_option(cb.OPT_EXACT_ZERO, 0)
            r1 = [ctx.elbo_eval_sampled(b, th, keep, off, 0.5, want=w) for w in ("value", "grad", "hess")]
            for x, y in zip(r0, r1):
                for p, q in zip(x, y):
                    assert (p is None and q is None) or np.array_equal(p, q)
            assert_elbo_close(r1[0][0][0], r1[2][0][0], rtol=1e-9)
    finally:
        ctx.set_option(cb.OPT_CHUNK_PX, 4096)
        ctx.set_option(cb.OPT_EXACT_ZERO, 0)


@pytest.mark.parametrize("pitch", [0, 5])
@pytest.mark.parametrize("nbr", [False, True])
@pytest.mark.parametrize("kind", ["counts", "fractional", "large"])
@pytest.mark.parametrize("shape", [(9, 1), (31, 5), (40, 23), (65, 66)])
def test_pixel_constants(env, shape, kind, nbr, pitch):
    """The theta-independent sums over runs, remainders and strided rows, counts of the log n! table and
    others, against the oracle; a bad value anywhere is found."""
    cb, ctx = env
    h, w = shape
    sb = _one(h, w, seed=h + w, far=0)
    rng = np.random.default_rng(h * w + len(kind))
    x = rng.poisson(100.0, (5, h, w)).astype(np.float32)
    if kind == "fractional":
        x += rng.random((5, h, w)).astype(np.float32)
    if kind == "large":
        x[:, h // 2, w // 2] = [65535.0, 65536.0, 65537.0, 1e6, 0.0]
    e, v = rng.uniform(0, 20, (2, 5, h, w)).astype(np.float32)
    th = perturb_theta(sb.theta_truth, 6)

    def batch(x, e, v):
        buf = np.full((3, 5, h, w + pitch), np.nan, np.float32)   # the gaps between rows are never read
        for k, a in enumerate((x, e, v)):
            buf[k, :, :, :w] = a
        buf[:, :, -1, w:] = 0
        n = h * (w + pitch)
        off = np.arange(5, dtype=np.int64) * n
        kw = dict(nbr_mean=buf[1].ravel(), nbr_var=buf[2].ravel(), nbr_pitch=w + pitch) if nbr else {}
        return cb.Batch(sb.src_img_off, sb.img_band, sb.img_h, sb.img_w, sb.img_w + pitch, sb.img_origin, sb.img_wcs,
                        sb.img_sky, sb.img_calib, sb.img_psf, sb.img_npsf, _device(buf[0]), off, sb.prior,
                        sb.profiles, **{k: _device(a) if k != "nbr_pitch" else a for k, a in kw.items()})

    sb.pixels = x.ravel()
    onbr = {i: (e[i], v[i]) for i in range(5)} if nbr else None
    ref = oracle_eval(sb, 0, th[0], nbr=onbr, want="value")[0]
    print("constants", shape, kind, nbr, pitch, flush=True)
    el = ctx.elbo_eval(batch(x, e, v), th, want="value")[0]
    # FP64 sums of the same terms: what differs is the FP32 theta-dependent rest
    assert_elbo_close(float(el[0]), ref, rtol=1e-6)
    for k, bad in ((0, -1.0), (0, np.nan), (0, np.inf)) + (((1, -1.0), (2, np.inf), (1, np.nan)) if nbr else ()):
        a = [x.copy(), e.copy(), v.copy()]
        a[k][4, h - 1, w - 1] = bad
        with pytest.raises(cb.CelesteError) as err:
            ctx.elbo_eval(batch(*a), th, want="value")
        assert err.value.code == cb.E_INVALID


def _device(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a).ravel()).cuda()
