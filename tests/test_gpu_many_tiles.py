"""Rendering more tiles than one launch can hold: a launch of 2^32 threads or more runs a part of its blocks only."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_render_more_tiles_than_a_launch_holds():
    import torch
    from paper_1611_03404_amd import celeste as cb
    sb = synth.make_config(0)
    nf = (1 << 23) + 1000                     # one-pixel fields, a tile each; two blocks of 256 threads a tile
    at = np.array([0, (1 << 22) - 1, 1 << 22, (1 << 23) - 1, 1 << 23, nf - 1], np.int32)   # each lit by a source
    n = len(at)
    one = np.ones(n, np.int32)
    b = cb.Batch(np.arange(n + 1, dtype=np.int64), 2 * one, one, one, one, np.zeros((n, 2)),
                 np.tile([1.0, 0, 0, 1.0, 0, 0], (n, 1)), np.full(n, 90.0), np.ones(n), np.repeat(sb.img_psf[:1], n, axis=0),
                 np.repeat(sb.img_npsf[:1], n), torch.ones(n, device="cuda"), np.arange(n, dtype=np.int64), sb.prior,
                 sb.profiles)
    th = np.repeat(sb.theta_truth, n, axis=0)
    th[:, 0:2] = 0.0
    t = torch.from_numpy(th).cuda()
    ctx = cb.Context(0)
    print("render", nf, "tiles", flush=True)
    few = ctx.render_fields(b, t, np.arange(n, dtype=np.int32), n, 1, 1)
    many = ctx.render_fields(b, t, at, nf, 1, 1)
    ctx.close()
    for x, y in zip(few, many):
        x, y = x.ravel(), y.ravel()
        assert float(x.min()) > 0.0
        assert torch.equal(y[torch.from_numpy(at.astype(np.int64)).cuda()], x)
        assert int((y != 0).sum()) == n
