"""Stages whose work can be uneven, timed against the same amount of even work on
the same card: the least of several runs of each, with a factor between them that
holds easily where the work is shared out and fails where one workgroup, or a
slower way for all, has it."""
import numpy as np
import pytest
import torch

from paper_2410_08743_amd import render as R
from paper_2410_08743_amd import synthetic as S

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _params(means, scales, opacity=0.7):
    n = len(means)
    f = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float32, device=DEV)
    quats = np.zeros((n, 4))
    quats[:, 0] = 1.0
    return R.GaussianParams(f(means), f(scales), f(quats), f(np.full(n, opacity)),
                            f(S.rng_for(n, 8).random((n, 1, 3))), 0)


def _stage_us(g, cam, names, views=1, runs=12):
    """Least time of the stages together, over forwards of the same view."""
    pose = torch.tensor(np.stack([S.identity_pose()] * views), dtype=torch.float32, device=DEV).contiguous()
    cams = [cam] * views
    rast = R.Rasterizer(0)
    rast.forward(g, cams, pose)
    rast.capacity = int(1.5 * rast.instances()[0]) + 4096
    rast.ws = None
    rast.forward(g, cams, pose)
    best = np.inf
    R.profile_enable(0, R.PROFILE_TIMING)
    try:
        R.profile_read(0)
        for _ in range(runs):
            rast.forward(g, cams, pose, check=False)
            st = R.profile_read(0)
            best = min(best, sum(st[k][1] for k in names))
    finally:
        R.profile_enable(0, 0)
    return 1e3 * best


def test_depth_order_of_walls():
    """Three walls that face the camera, 70 splats of each in every tile: with
    equal depths, and with depths that differ."""
    w, h, f, step = 1200, 680, 600.0, 2
    y, x = np.mgrid[0:h:step, 0:w:step]
    z0 = np.concatenate([np.full(x.size, z) for z in (2.5, 3.0, 3.5)])
    spread = z0 * (1 + 0.06 * S.rng_for(1, 8).uniform(-1, 1, len(z0)))
    cam = S.Camera(w, h, f, f, w / 2, h / 2)
    us = []
    for z in (z0, spread):
        means = np.stack([(np.tile(x.ravel(), 3) + 0.5 - w / 2) / f * z, (np.tile(y.ravel(), 3) + 0.5 - h / 2) / f * z,
                          z], 1)
        us.append(_stage_us(_params(means, np.repeat((1.1 * step / f * z)[:, None], 3, 1)), cam, ["depth_order"]))
    print(f"depth order: equal {us[0]:.1f}, different {us[1]:.1f} us")
    assert us[0] < 5.5 * us[1]


def test_binning_of_many_small_views():
    """32 views fit the chip side by side: they take hardly longer than one."""
    cam = S.Camera(128, 128, 100.0, 100.0, 64.0, 64.0)
    rng = S.rng_for(3, 8)
    z = rng.uniform(1.5, 8.0, 1000)
    means = np.stack([rng.uniform(-0.7, 0.7, 1000) * z, rng.uniform(-0.7, 0.7, 1000) * z, z], 1)
    g = _params(means, np.exp(rng.uniform(np.log(0.01), np.log(0.1), (1000, 3))))
    us = [_stage_us(g, cam, ["duplicate", "ranges", "tile_sort"], views) for views in (1, 32)]
    print(f"binning: one view {us[0]:.1f}, 32 views {us[1]:.1f} us")
    assert us[1] < 2.0 * us[0]


@pytest.mark.parametrize("first", [True, False])
def test_binning_of_neighbouring_large_splats(first):
    """300 splats over the whole view, in front of or behind 100k small ones: next
    to each other and spread over the scene."""
    w, h, f, n, big = 1008, 756, 815.0, 100_000, 300
    rng = S.rng_for(4, 8)
    z = rng.uniform(1.5, 8.0, n)
    means = np.stack([rng.uniform(-0.6, 0.6, n) * z, rng.uniform(-0.45, 0.45, n) * z, z], 1)
    scales = np.exp(rng.uniform(np.log(0.01), np.log(0.05), (n, 3)))
    at = slice(0, big) if first else slice(n - big, n)
    means[at, :2] *= 0.2
    scales[at] = 5.0
    cam = S.Camera(w, h, f, f, w / 2, h / 2)
    us = []
    for order in (np.arange(n), rng.permutation(n)):
        us.append(_stage_us(_params(means[order], scales[order], 0.02), cam, ["duplicate", "ranges", "tile_sort"]))
    print(f"binning: together {us[0]:.1f}, spread {us[1]:.1f} us")
    assert us[0] < 4.0 * us[1]


@pytest.mark.parametrize("kind,factor", [("none", 30.0), ("octaves", 170.0)])
def test_unprojection_without_near_neighbours(kind, factor):
    """A frame without any depth, and one whose depths are spread over forty octaves
    pixel by pixel, against a smooth one."""
    from paper_2410_08743_amd import relpose as RP
    w, h = 1200, 680
    cam = S.Camera(w, h, 600.0, 600.0, w / 2, h / 2)
    image = torch.rand(3, h, w, device=DEV)
    y, x = torch.meshgrid(torch.arange(h, device=DEV), torch.arange(w, device=DEV), indexing="ij")
    smooth = (3.0 + 0.001 * x + 0.002 * y).contiguous()
    gen = torch.Generator(device=DEV)
    gen.manual_seed(5)
    depth = {"none": torch.zeros(h, w, device=DEV),
             "octaves": torch.exp2(40 * torch.rand(h, w, device=DEV, generator=gen) - 20)}[kind]
    us = []
    R.profile_enable(0, R.PROFILE_TIMING)
    try:
        for d in (depth, smooth):
            best = np.inf
            R.profile_read(0)
            for _ in range(8):
                RP.unproject(cam, d, image, 4)
                best = min(best, 1e3 * R.profile_read(0)["unproject"][1])
            us.append(best)
    finally:
        R.profile_enable(0, 0)
    print(f"unproject: {kind} {us[0]:.1f}, smooth {us[1]:.1f} us")
    assert us[0] < factor * us[1]
