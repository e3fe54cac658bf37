"""The splat's passes over a wave (box pixels, queued covered pixels, queued
owned pixels) at the sizes where they change: triangles around and far above
the 124-pixel span of the 32-bit edge functions, slivers, splat boxes a lane
walks alone and boxes the whole wave walks, view counts around the queue's view
groups (64, and fewer at large views), frames of so few points that the views
are split over waves, and quilt tiles with and without room for the queues.
Views, depth and written pixels equal the oracle's bit for bit."""
import dataclasses

import numpy as np
import pytest

from oracle import oracle as O
from paper_2601_19901_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _soup(seed, n, W, H, tex_size, pbr=False):
    """n random triangles in front of the rig, edges log-uniform from 1 px to twice the view, some nearly
    degenerate, some reaching far off the view."""
    rng = np.random.default_rng(seed)
    fx, fy = W / 2 / (1.6 * np.tan(np.radians(15.0))), H / 2 / np.tan(np.radians(15.0))
    z = rng.uniform(6.0, 14.0, n)
    c = np.stack([rng.uniform(-0.6, 0.6, n) * W * z / fx, rng.uniform(-0.6, 0.6, n) * H * z / fy, z], 1)
    size = np.exp(rng.uniform(0.0, np.log(2.0 * max(W, H)), n))
    size[: n // 4] = rng.uniform(118.0, 130.0, n // 4)  # spans around the 32-bit limit
    d = rng.normal(size=(n, 3, 3)) * (size * z / max(fx, fy) / 2.0)[:, None, None]
    d[..., 2] *= 0.3
    thin = rng.random(n) < 0.2
    d[thin, 2] = d[thin, 0] * 0.4 + d[thin, 1] * 0.6 + 1e-3 * d[thin, 2]
    pos = (c[:, None, :] + d)
    pos[..., 2] = np.maximum(pos[..., 2], 1.0)
    uv = rng.uniform(0.0, 2.0, (n * 3, 2))
    texs = [scenes.value_noise_texture(tex_size, rng), scenes.checker_texture(2 * tex_size, rng)]
    idx = np.arange(n * 3).reshape(n, 3)
    idx = np.concatenate([idx, idx[:, ::-1]])  # one of the two faces the rig
    tid = rng.integers(0, 2, 2 * n)
    s = scenes.Scene((pos.reshape(-1, 3) - [0, 0, 10.0]).astype(np.float32), uv.astype(np.float32), idx.astype(np.uint32),
                     tid.astype(np.uint16), texs, "soup")
    if pbr:
        s = dataclasses.replace(s, materials=np.stack([tid, 1 - tid, tid], 1).astype(np.uint16))
    return s.check()


@pytest.mark.parametrize("W,H,V,tex,quilt", [
    (130, 70, 3, 4, None), (130, 70, 3, 64, None), (300, 41, 70, 8, None), (64, 64, 65, 4, (0, 0)), (1, 1, 5, 4, None),
    (2100, 1030, 5, 4, None), (4096, 37, 9, 8, None), (37, 2049, 9, 8, None),
    (512, 64, 40, 8, (4, 9)), (512, 64, 40, 8, (1, 38)), (512, 64, 40, 8, (1, 39)), (256, 64, 20, 16, (4, 9)), (2048, 24, 6, 8, (1, 9))])
@pytest.mark.parametrize("pbr", [False, True])
def test_splat_passes_match_the_oracle(torch_cuda, W, H, V, tex, quilt, pbr):
    from paper_2601_19901_amd import lfdpr
    scene = _soup(W * 7 + V, 60 if W * H * V < 2_000_000 else 24, W, H, tex, pbr)
    vp = scenes.ViewParams(V=V, W=W, H=H, fovy_deg=30.0, aspect=1.6, D=10.0, cone_deg=40.0, znear=0.5)
    light = scenes.default_light() if pbr else None
    model = scenes.model_matrix(3, 10.0)
    o = O.render(scene, vp, model, shading=light) if pbr else O.render(scene, vp, model)
    R = lfdpr.Renderer(0)
    sid = R.upload_scene(scene)
    R.set_views(vp)
    R.set_shading(light)
    if quilt:
        R.set_splat_order(lfdpr.SPLAT_QUILT)
        R.set_quilt_tile(*quilt)
    views, depth = R.alloc_views(with_depth=True)
    R.render_frame(sid, model, views, depth)
    st = R.stats()
    print(f"[{W}x{H}x{V} tex {tex} quilt {quilt} pbr {pbr}] {st}", flush=True)
    assert st["points"] == int(o["stats"]["points"])
    assert st["written_px"] == o["stats"]["fragments"] - o["stats"]["misses"]
    np.testing.assert_array_equal(views.cpu().numpy().view(np.uint32), o["rgba"])
    np.testing.assert_array_equal(depth.cpu().numpy().view(np.uint32), o["depth"].view(np.uint32))


@pytest.mark.parametrize("blocks", [1, 5, 15, 16, 17, 1024, 5000])
def test_every_work_queue_is_drawn(torch_cuda, blocks):
    """Frames of one chunk of points and of many, under grids with fewer waves than work queues and with more."""
    from paper_2601_19901_amd import lfdpr
    R = lfdpr.Renderer(0)
    R.set_launch(blocks, 0)
    for scene, V in ((_soup(5, 1, 40, 30, 4), 3), (_soup(6, 60, 130, 70, 64), 13)):
        vp = scenes.ViewParams(V=V, W=130, H=70, fovy_deg=30.0, aspect=1.6, D=10.0, cone_deg=40.0, znear=0.5)
        model = scenes.model_matrix(3, 10.0)
        o = O.render(scene, vp, model)
        R.set_views(vp)
        views, depth = R.alloc_views(with_depth=True)
        R.render_frame(R.upload_scene(scene), model, views, depth)
        assert R.stats()["written_px"] == o["stats"]["fragments"] - o["stats"]["misses"]
        np.testing.assert_array_equal(views.cpu().numpy().view(np.uint32), o["rgba"])
        np.testing.assert_array_equal(depth.cpu().numpy().view(np.uint32), o["depth"].view(np.uint32))
