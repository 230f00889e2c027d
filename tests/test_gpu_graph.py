"""The pose step (forward, L1, backward with the pose gradient, guarded Adam)
captured once in a HIP graph and replayed: every replay must give the same
pose as the eager step it stands for.  The library's kernels allocate
nothing and clear buffers with kernels (no memset nodes), so the step is
capturable as is."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2410_08743_amd import render as R
from paper_2410_08743_amd import synthetic as S

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _state(wl, g, cam):
    rast = R.Rasterizer(0)
    tgt, _ = rast.forward(g, [cam], torch.tensor(wl.pose[None], device=DEV))
    st = {"tgt": tgt.clone(), "pose": torch.tensor(wl.init_pose[None], device=DEV),
          "m": torch.zeros((1, 6), device=DEV), "v": torch.zeros((1, 6), device=DEV),
          "k": torch.zeros(1, dtype=torch.int32, device=DEV),
          "img": torch.empty(3 * cam.width * cam.height, device=DEV),
          "dpose": torch.empty((1, 6), device=DEV), "rast": rast}
    st["dl"] = torch.empty_like(st["img"])
    rast.forward(g, [cam], st["pose"], images=st["img"])
    rast.capacity = int(2 * rast.instances()[0]) + 1024
    rast.ws = None
    rast._ensure(g, R.N.view_array([cam]))
    return st


def _step(g, cam, st):
    rast = st["rast"]
    rast.forward(g, [cam], st["pose"], check=False, images=st["img"])
    R.loss_l1([cam], st["img"], st["tgt"], grad=st["dl"], with_loss=False)
    rast.backward(g, [cam], st["pose"], st["dl"], want=(), pose=True, out={"pose": st["dpose"]})
    R.pose_adam(st["pose"], st["dpose"], st["m"], st["v"], st["k"], 1e-2, 1e-4, 40,
                guard=rast.ws)


def test_graph_replays_match_eager_steps():
    wl = S.tiny()
    cam = wl.camera
    g = R.GaussianParams.from_set(wl.scene, DEV)
    K = 12
    eager = _state(wl, g, cam)
    ref = []
    for _ in range(K):
        _step(g, cam, eager)
        ref.append(eager["pose"].cpu().numpy().copy())

    st = _state(wl, g, cam)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        _step(g, cam, st)           # recorded, not run
    torch.cuda.synchronize()
    assert np.array_equal(st["pose"].cpu().numpy(), wl.init_pose[None])   # nothing ran at capture
    for k in range(K):
        graph.replay()
        torch.cuda.synchronize()
        got = st["pose"].cpu().numpy()
        assert np.array_equal(got, ref[k]), f"replay {k}"
        assert not np.array_equal(got, wl.init_pose[None])
        # eager work between replays must not disturb the graph's buffers
        _ = (st["img"] * 2).sum().item()
    assert not st["rast"].overflowed()


@pytest.mark.parametrize("views,masked", [(1, False), (3, False), (2, True)])
def test_graph_replayed_solve_equals_eager_solve(views, masked):
    wl = S.tiny()
    cam = wl.camera
    g = R.GaussianParams.from_set(wl.scene, DEV)
    rast = R.Rasterizer(0)
    tgt, _ = rast.forward(g, [cam], torch.tensor(wl.pose[None], device=DEV))
    targets = [tgt.clone()] * views
    rng = S.rng_for(31, 1)
    inits = torch.tensor(np.stack([wl.init_pose] + [S.perturb_pose(wl.pose, 3.0, 0.05, rng)
                                                    for _ in range(views - 1)]).astype(np.float32),
                         device=DEV)
    eager = R.solve_poses(g, [cam] * views, targets, inits, steps=30, masked=masked)
    graphed = R.solve_poses(g, [cam] * views, targets, inits, steps=30, masked=masked, graph=True)
    assert torch.equal(eager, graphed)
    assert not torch.equal(eager, inits)


def _keys(rast, g, cam):
    """The tile ids of the last forward, as the region of the workspace that
    gsp_inspect names (no copy)."""
    p, cnt = ctypes.c_void_p(), ctypes.c_int64()
    gs, views = g.struct(), R.N.view_array([cam])
    nbytes = rast._ws_bytes(g.n, g.sh_degree, views, rast.capacity)
    R.N.check(R.N.lib().gsp_inspect(R.context(0), ctypes.byref(gs), 1, views, R._ptr(rast.ws), nbytes, rast.capacity,
                                    b"keys", ctypes.byref(p), ctypes.byref(cnt)), "gsp_inspect")
    off = p.value - rast.ws.data_ptr()
    return rast.ws[off:off + 4 * cnt.value].view(torch.int32)


def _expected_keys(rast, g, cam):
    rg = rast.inspect(g, [cam], "ranges", torch.int32).cpu().numpy().view(np.uint32).reshape(-1, 2)
    return np.repeat(np.arange(len(rg), dtype=np.int32), (rg[:, 1] - rg[:, 0]).astype(np.int64))


def test_inspected_keys_follow_every_forward():
    """gsp_inspect names a region; what lies there is the last forward's."""
    wl = S.tiny()
    cam = wl.camera
    g = R.GaussianParams.from_set(wl.scene, DEV)
    rast = R.Rasterizer(0)
    pose = torch.tensor(wl.pose[None], device=DEV)
    rast.forward(g, [cam], pose)
    keys = _keys(rast, g, cam)
    for p in (wl.pose, wl.init_pose):
        rast.forward(g, [cam], torch.tensor(p[None], device=DEV), check=False)
        ref = _expected_keys(rast, g, cam)
        assert len(ref) == rast.instances()[0] and np.array_equal(keys[:len(ref)].cpu().numpy(), ref)


def test_keys_are_inspected_while_a_stream_captures():
    wl = S.tiny()
    cam = wl.camera
    g = R.GaussianParams.from_set(wl.scene, DEV)
    st = _state(wl, g, cam)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        _step(g, cam, st)
        keys = _keys(st["rast"], g, cam)
    for _ in range(3):   # the pose moves from replay to replay
        graph.replay()
        torch.cuda.synchronize()
        ref = _expected_keys(st["rast"], g, cam)
        assert len(ref) > 0 and np.array_equal(keys[:len(ref)].cpu().numpy(), ref)
