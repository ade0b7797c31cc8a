"""Field calls check estimates where they lie, in device memory: the first one out of range is named, and nothing is
written."""
import numpy as np
import pytest

import synth
from synth.generate import perturb_theta

pytestmark = pytest.mark.gpu

N, SIZE = 700, 96   # more sources than two blocks of the check take


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1611_03404_amd import celeste as cb
    z = synth.make_config(0)
    one = np.ones(N, np.int32)
    xy = np.stack([np.arange(N) % 32, np.arange(N) // 32], axis=1) * 3.0      # disjoint patches of 3 x 3
    b = cb.Batch(np.arange(N + 1, dtype=np.int64), 2 * one, 3 * one, 3 * one, 3 * one, xy,
                 np.tile([1.0, 0, 0, 1.0, 0, 0], (N, 1)), np.full(N, 90.0), np.ones(N), np.repeat(z.img_psf[:1], N, axis=0),
                 np.repeat(z.img_npsf[:1], N), torch.ones(9 * N, device="cuda"), np.arange(N, dtype=np.int64) * 9, z.prior,
                 z.profiles)
    th = perturb_theta(np.repeat(z.theta_truth, N, axis=0), 3)
    th[:, 0:2] = xy + 1.0
    c = cb.Context(0)
    yield cb, c, b, th
    c.close()


@pytest.mark.parametrize("call", ["render", "neighbours", "update old", "update new", "elbo"])
@pytest.mark.parametrize("s,i,v", [(0, 4, 1.5), (257, 0, float("inf")), (N - 1, 26, float("nan")), (600, 6, 0.0)])
def test_bad_estimate_is_named(env, call, s, i, v):
    import torch
    cb, ctx, b, th = env
    bad = th.copy()
    bad[s, i] = v
    bad[N - 1, 9] = -1.0 if s != N - 1 else bad[N - 1, 9]     # another one behind it
    good, bad = torch.from_numpy(th).cuda(), torch.from_numpy(bad).cuda()
    meta = (np.zeros(N, np.int32), 1, SIZE, SIZE)
    f = [torch.full((1, SIZE, SIZE), 7.0, device="cuda") for _ in range(2)]
    nb = [torch.full((9 * N,), 7.0, device="cuda") for _ in range(2)]
    off = np.arange(N, dtype=np.int64) * 9
    print("refused", call, s, i, v, flush=True)
    with pytest.raises(cb.CelesteError) as e:
        if call == "render":
            ctx.render_fields(b, bad, *meta, out=f)
        elif call == "neighbours":
            ctx.neighbour_arrays(b, bad, *meta, f, off, *nb)
        elif call == "elbo":
            ctx.field_elbo(b, bad, *meta, f, torch.ones(1, SIZE, SIZE, device="cuda"), np.full(1, 90.0))
        else:
            ctx.update_fields(b, *((bad, good) if call == "update old" else (good, bad)), *meta, f)
    assert e.value.code == cb.E_INVALID and f"theta[{s}]" in str(e.value)
    for x in f + nb:
        assert bool((x == 7.0).all())
