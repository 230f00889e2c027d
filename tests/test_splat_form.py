"""The rasterizers' decisions about a splat's quadratic form (raster_common.h),
redone here in float32 with one rounding per operation: a splat walked without
the test on a positive power never has one, and a splat culled for a rectangle
of pixels reaches 1/255 at none of them."""
import numpy as np
import pytest

F = np.float32
LOG2_ALPHA_MIN_LOOSE = F(-7.994353436858858 - 0.01)   # kLog2AlphaMinLoose


def fma(a, b, c):
    return (a.astype(np.float64) * b + c).astype(F)


def p2(A, B, C, dx, dy):
    """splat_p2: fma(fma(C, dy, B dx), dy, (A dx) dx)"""
    return fma(fma(C, dy, dx * B), dy, (dx * A) * dx)


def forms(rng, n, slack):
    """Base-2 conics with B^2 = 4 A C (1 - slack), extents from a fraction of a
    pixel to thousands, both signs of B."""
    A = -np.exp2(rng.uniform(-24, 1.3, n)).astype(F)
    C = -np.exp2(rng.uniform(-24, 1.3, n)).astype(F)
    B = (np.sqrt(4.0 * A.astype(np.float64) * C * (1 - slack)) * rng.choice([-1, 1], n)).astype(F)
    return A, B, C


@pytest.mark.parametrize("slack", [1e-4, 1.01e-4, 1e-3, 0.1, 1.0])
def test_plain_splats_have_no_positive_power(slack):
    rng = np.random.default_rng(5)
    n = 500_000
    A, B, C = forms(rng, n, slack)
    plain = (A < 0) & (C < 0) & (B * B <= F(3.9996) * (A * C))
    assert plain.mean() > (0.3 if slack == 1e-4 else 0.99)
    # offsets along the form's long axis, where it is closest to zero, and off it
    dy = (rng.uniform(-1, 1, n) * np.exp2(rng.uniform(-12, 11, n))).astype(F)
    along = -0.5 * B.astype(np.float64) * dy / A
    dx = (along * (1 + rng.choice([0, 1e-7, 1e-5, 1e-3, 0.5], n) * rng.standard_normal(n))).astype(F)
    assert (p2(A, B, C, dx, dy)[plain] <= 0).all()


@pytest.mark.parametrize("w,h", [(8, 8), (16, 4)])
@pytest.mark.parametrize("slack", [-1e-6, 0.0, 1e-4, 0.05, 1.0])
def test_culled_splats_reach_no_pixel(w, h, slack):
    rng = np.random.default_rng(6)
    n = 60_000
    A, B, C = forms(rng, n, slack)
    lo = np.log2(rng.uniform(1 / 255, 1, n)).astype(F)
    # centres from inside the rectangle to some extents away from it
    ext = np.sqrt(8.0 / np.minimum(-A, -C).astype(np.float64))
    far = rng.choice([0, 1], n) * np.minimum(ext, 4000)
    u = (rng.uniform(-1, w, n) + rng.uniform(-1, 1, n) * far).astype(F)
    v = (rng.uniform(-1, h, n) + rng.uniform(-1, 1, n) * far).astype(F)
    xa, xb, ya, yb = u - F(w - 1), u, v - F(h - 1), v
    thr = LOG2_ALPHA_MIN_LOOSE - lo
    zero = F(0)
    kx, ky = F(-0.5) * B * (F(1) / A), F(-0.5) * B * (F(1) / C)
    x0 = np.minimum(np.maximum(zero, xa), xb)
    y0 = np.minimum(np.maximum(zero, ya), yb)
    ys = np.minimum(np.maximum(ky * x0, ya), yb)
    xs = np.minimum(np.maximum(kx * y0, xa), xb)
    fx = fma(fma(C, ys, B * x0), ys, A * x0 * x0)
    fy = fma(fma(A, xs, B * y0), xs, C * y0 * y0)
    xm, ym = np.maximum(abs(xa), abs(xb)), np.maximum(abs(ya), abs(yb))
    mag = abs(A) * xm * xm + abs(B) * xm * ym + abs(C) * ym * ym
    keep = np.maximum(fx, fy) + fma(F(1e-5) * np.ones_like(mag), mag, F(0.02)) >= thr
    assert 0.02 < keep.mean() < 0.98
    hit = np.zeros(n, bool)
    for j in range(h):
        for i in range(w):
            p = p2(A, B, C, u - F(i), v - F(j))
            hit |= (p <= 0) & (p + lo >= LOG2_ALPHA_MIN_LOOSE)
    assert hit.any() and not (hit & ~keep).any()
