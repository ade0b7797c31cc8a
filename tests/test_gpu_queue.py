"""Fits that draw their work items from the device list: more items than every persistent grid has blocks, at its default
size, one and four blocks per compute unit, both block sizes and register budgets, replayed and eager, with and without
derivatives at trial points; ragged sources.  Every bit is that of one block per item."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

CHUNK = 64   # an item is 8 rows of an image


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1611_03404_amd import celeste as cb
    c = cb.Context(0)
    c.set_option(cb.OPT_CHUNK_PX, CHUNK)
    sets = {}
    for n in (2, 110):
        sb = synth.make_config(1, n_sources=n)
        th = np.zeros((n, 27))
        th[:, 0:2] = sb.u_cat
        sets[n] = (cb.Batch.from_synth(sb), th, int(((sb.img_h + 7) // 8).sum()))
    yield cb, c, sets
    c.close()


def _fit(env, n, persistent, graph=1, trial=1):
    cb, ctx, sets = env
    b, th, items = sets[n]
    ctx.set_option(cb.OPT_PERSISTENT, persistent)
    ctx.set_option(cb.OPT_USE_GRAPH, graph)
    ctx.set_option(cb.OPT_TRIAL_DERIVATIVES, trial)
    ctx.stats(reset=True)
    t, r = ctx.batch_fit(b, th, cb.default_opts(init_mode=cb.INIT_PLAIN, max_iter=8))
    return t, r, ctx.stats()["fit_grid_blocks"], items


@pytest.mark.parametrize("trial", [1, 0])
@pytest.mark.parametrize("block,variant", [(256, 3), (256, 2), (128, 3), (128, 2)])
def test_list_equals_one_block_per_item(env, block, variant, trial):
    cb, ctx, _ = env
    try:
        ctx.set_option(cb.OPT_BLOCK, block)
        ctx.set_option(cb.OPT_VARIANT, variant)
        for n, listed in ((110, True), (2, False)):   # 2 sources: fewer items than blocks, no list
            t0, r0, g0, _ = _fit(env, n, 0, trial=trial)
            assert g0 == 0
            for persistent in (-1, 1, 4):
                for graph in (1, 0):
                    print("list", block, variant, trial, n, persistent, graph, flush=True)
                    t, r, grid, items = _fit(env, n, persistent, graph, trial)
                    assert (items > grid) == listed and grid > 0
                    assert np.array_equal(t, t0)
                    for k in ("elbo", "iters", "status", "n_full_evals", "n_accepted"):
                        assert np.array_equal(r[k], r0[k])
    finally:
        for o, v in ((cb.OPT_BLOCK, 256), (cb.OPT_VARIANT, 3), (cb.OPT_PERSISTENT, -1), (cb.OPT_USE_GRAPH, 1),
                     (cb.OPT_TRIAL_DERIVATIVES, 1)):
            ctx.set_option(o, v)
