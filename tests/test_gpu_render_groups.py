"""Depth rendering at the edges of the hierarchy's layout against the FP64 brute-force oracle: surfaces of one
leaf (2 triangles), of one node level, just below and above one refit workgroup's 1024 triangles, and with two
levels of nodes above the subtrees, all as envs of one renderer (different hierarchies side by side).
Bars of test_gpu_render.py: ids equal off silhouettes and depth ties, depth and points within 1e-5."""
import numpy as np
import pytest

from oracle import render_oracle as RO
from paper_2604_17513_amd import scenes
from test_gpu_render import _compare, _look_at, _ties

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(2,), (3, 2, 24), (23, 70)])
def test_surfaces_at_the_edges_of_the_hierarchy(sizes):
    import torch
    from paper_2604_17513_amd import flash as F
    W, H = 40, 33
    rng = np.random.default_rng(len(sizes))
    envs, xs = [], []
    for n in sizes:
        rest, tris = scenes.cloth_grid(n, 0.6, (-0.3, -0.3), 0.0)
        envs.append(scenes.EnvDesc(scenes.TRI, rest, tris))
        x = rest.copy()
        x[:, 1] += 0.05 + 0.03 * np.sin(9.0 * x[:, 0] + rng.uniform(0, 6)) * np.cos(8.0 * x[:, 2])
        xs.append(x.astype(np.float32))
    x = torch.tensor(np.concatenate(xs).T.copy(), device="cuda")
    cams = [_look_at((0.3, 0.5, -0.4), (0.0, 0.03, 0.0), 45.0, W, H)] * len(sizes)
    obs = [[scenes.ground()]] * len(sizes)
    R = F.Renderer(envs)
    for _ in range(2):   # a second frame over the first one's boxes
        out = R.render(x, cams, W, H, obstacles=obs, points=True)
    depth, inst, pts = (out[k].cpu().numpy() for k in ("depth", "instance", "points"))
    for e, env in enumerate(envs):
        tris = RO.surface_triangles(env.elem, env.elements)
        xe = xs[e].astype(np.float64)
        rd, ri, rp = RO.render(xe, tris, obs[e], cams[e], W, H)
        assert (ri == 0).sum() > 100
        _compare(f"sheet {sizes[e]}", depth[e], inst[e], pts[e], rd, ri, rp, _ties(xe, tris, obs[e], cams[e], W, H))
    R.close()


@pytest.mark.parametrize("view", ["inside", "grazing", "behind", "sheared"])
def test_views_where_boxes_do_not_project(view):
    """A tile picks the subtrees whose boxes project onto it: cameras inside the surface's box (boxes around and
    behind the camera's plane), along the sheet, looking away, and with a matrix that is no rotation (nothing may
    be dropped)."""
    import torch
    from paper_2604_17513_amd import flash as F
    W, H, n = 271, 249, 29   # 17 x 16 tiles
    rest, tris = scenes.cloth_grid(n, 0.6, (-0.3, -0.3), 0.0)
    env = scenes.EnvDesc(scenes.TRI, rest, tris)
    x = rest.copy()
    x[:, 1] += 0.08 + 0.05 * np.sin(11.0 * x[:, 0]) * np.cos(9.0 * x[:, 2])
    x = x.astype(np.float32)
    cam = {"inside": _look_at((0.02, 0.081, 0.01), (0.3, 0.07, 0.2), 160.0, W, H),
           "grazing": _look_at((-0.5, 0.1, 0.013), (0.3, 0.08, 0.0), 320.0, W, H),
           "behind": _look_at((0.0, 0.5, 0.013), (0.1, 0.9, 0.0), 210.0, W, H),
           "sheared": _look_at((0.3, 0.5, -0.4), (0.0, 0.03, 0.0), 240.0, W, H)}[view]
    if view == "sheared":
        cam["rot"] = cam["rot"] @ np.array([[1.2, 0.3, 0.0], [0.0, 0.7, 0.0], [0.1, 0.0, 1.0]])
    obs = [scenes.ground()]
    R = F.Renderer([env])
    out = R.render(torch.tensor(x.T.copy(), device="cuda"), [cam], W, H, obstacles=[obs], points=True)
    depth, inst, pts = (out[k].cpu().numpy()[0] for k in ("depth", "instance", "points"))
    xe = x.astype(np.float64)
    rd, ri, rp = RO.render(xe, tris, obs, cam, W, H)
    assert view == "behind" or (ri == 0).sum() > 50
    _compare(view, depth, inst, pts, rd, ri, rp, _ties(xe, tris, obs, cam, W, H))
    R.close()
