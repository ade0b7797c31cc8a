"""The bound by which the pixel kernels decide, for a whole tile, that a mixture component is exactly 0
on it (CPU only).

A component's log2 density at offset d is e(d) = c0 - (A dx^2 + B dx dy + C dy^2).  The kernels bound e
over the box of a tile's pixels: the form's minimum over a box that does not hold the origin lies on
the nearest edge in x or the nearest edge in y, at the best clamped coordinate along it, with a slack of
2^-20 of the largest terms on the box plus 0.01 for the rounding of the FP32 exponents.  This restates
the bound in FP32 and checks that it is never below the FP32 exponent of any pixel of the box (the
pixels' offsets formed by the kernels' own operations), and that it is tight where the exact minimum
is attained on a pixel.
"""
import numpy as np
import pytest

F = np.float32


def _bound(c0, A, B, C, xl, xh, yl, yh):
    med = lambda v, lo, hi: np.minimum(np.maximum(v, lo), hi)  # noqa: E731
    bc = F(0.5) * B / C if C > 0 else F(0)
    ba = F(0.5) * B / A if A > 0 else F(0)
    xn, yn = med(F(0), xl, xh), med(F(0), yl, yh)
    ys, xs = med(-bc * xn, yl, yh), med(-ba * yn, xl, xh)
    q1 = A * xn * xn + ys * (B * xn + C * ys)
    q2 = C * yn * yn + xs * (B * yn + A * xs)
    X, Y = np.maximum(abs(xl), abs(xh)), np.maximum(abs(yl), abs(yh))
    M = X * (A * X + abs(B) * Y) + C * Y * Y
    return (c0 - np.minimum(q1, q2)) + (M * F(2.0 ** -20) + F(0.01))


@pytest.mark.parametrize("far", [10.0, 200.0, 30000.0])
def test_bound_dominates_every_pixel(far):
    rng = np.random.default_rng(int(far))
    loose = []
    for _ in range(3000):
        t = rng.uniform(0, np.pi)
        l1 = np.exp(rng.uniform(np.log(0.05), np.log(2000.0)))
        l2 = l1 * np.exp(rng.uniform(np.log(1e-4), 0.0))
        R = np.array([[np.cos(t), -np.sin(t)], [np.sin(t), np.cos(t)]])
        P = R @ np.diag([1 / l1, 1 / l2]) @ R.T
        k = 0.5 / np.log(2.0)
        A, B, C = F(k * P[0, 0]), F(2 * k * P[0, 1]), F(k * P[1, 1])
        c0 = F(rng.uniform(-20, 5))
        x0, y0 = int(rng.uniform(0, far)), int(rng.uniform(0, far))
        nx, ny = int(rng.integers(1, 65)), int(rng.integers(1, 9))
        psx, psy = F(rng.uniform(0, far)), F(rng.uniform(0, far))
        if rng.random() < 0.3:
            psx, psy = F(x0 + rng.uniform(-3, nx + 3)), F(y0 + rng.uniform(-3, ny + 3))
        xi, yi = F(rng.normal(0, 0.5)), F(rng.normal(0, 0.5))
        off = lambda c, ps, o: (F(c) - ps) - o  # noqa: E731
        e_max = _bound(c0, A, B, C, off(x0, psx, xi), off(x0 + nx - 1, psx, xi), off(y0, psy, yi),
                       off(y0 + ny - 1, psy, yi))
        dx = (np.arange(x0, x0 + nx).astype(F) - psx) - xi
        dy = (np.arange(y0, y0 + ny).astype(F) - psy) - yi
        DX, DY = np.meshgrid(dx, dy)
        e32 = -A * (DX * DX) + (-B * (DX * DY) + (-C * (DY * DY) + c0))
        assert e_max >= e32.max(), (A, B, C, c0, x0, y0, nx, ny, psx, psy, e_max, e32.max())
        if l2 > 0.5 and e32.max() > -300:
            loose.append(float(e_max - e32.max()))
    # the continuous box holds at most half a pixel of slack along each axis around a pixel's minimum
    if loose:
        assert np.median(loose) < 2.0


def test_component_without_weight_is_skipped():
    assert not _bound(F(-np.inf), F(1), F(0), F(1), F(-1), F(1), F(-1), F(1)) >= F(-127)
