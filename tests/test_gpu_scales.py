"""The same frame in units from 2^-30 to 2^30 of a scene's: the set-up takes its
quotients and roots by the fast forms in the middle of the binary32 range and by
the plain operators outside it, where products of areas underflow or overflow;
sample densities, counts, points, views and depth equal the oracle's bit for bit
either way, and in rigs of extreme focal lengths."""
import dataclasses

import numpy as np
import pytest

from oracle import oracle as O
from paper_2601_19901_amd import scenes

pytestmark = pytest.mark.gpu



def check(scene, vp, model, label):
    import torch
    from paper_2601_19901_amd import lfdpr
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    o = O.render(scene, vp, model)
    R = lfdpr.Renderer(0)
    sid = R.upload_scene(scene)
    R.set_views(vp, 1 << 20)
    views, depth = R.alloc_views(with_depth=True)
    nt = scene.n_tris
    df = torch.zeros(nt * 8, dtype=torch.float32, device="cuda")
    di = torch.zeros(nt * 8, dtype=torch.int32, device="cuda")
    R.set_debug_records(df, di)
    R.render_frame(sid, model, views, depth)
    st = R.stats(allow_overflow=True)
    print(f"[{label}] {st['active_tris']} active, {st['points']} points, {st['written_px']} pixels", flush=True)
    np.testing.assert_array_equal(R.counts(nt), o["count"].astype(np.uint32))
    assert st["points"] == o["n_points"] and st["point_views"] == o["stats"]["point_views"]
    np.testing.assert_array_equal(df.cpu().numpy().reshape(nt, 8), o["trif"])
    np.testing.assert_array_equal(di.cpu().numpy().reshape(nt, 8), o["trii"])
    np.testing.assert_array_equal(views.cpu().numpy().view(np.uint32), o["rgba"])
    np.testing.assert_array_equal(depth.cpu().numpy().view(np.uint32), o["depth"].view(np.uint32))
    return o


@pytest.mark.parametrize("k,fovy,aspect", [(0, 30.0, 1.6), (-24, 30.0, 1.6), (-28, 30.0, 1.6), (-30, 30.0, 1.6), (12, 30.0, 1.6),
                                           (30, 30.0, 1.6), (0, 0.01, 1.0), (0, 170.0, 0.02), (0, 30.0, 500.0)])
def test_any_unit_gives_the_oracles_frame(k, fovy, aspect):
    u = 2.0 ** k
    w = scenes.small_display(seed=9, V=7, W=80, H=64, hf_quads=24)
    scene = dataclasses.replace(w.scene, pos=(w.scene.pos * np.float32(u)).astype(np.float32))
    vp = dataclasses.replace(w.views, D=w.views.D * u, znear=w.views.znear * u, fovy_deg=fovy, aspect=aspect)
    check(scene, vp, scenes.model_matrix(2, vp.D, w.tilt_deg), f"2^{k}, {fovy} deg, aspect {aspect}")


def facing(k, px, n, seed):
    """n triangles, px pixels wide, that eyes of a 7-view rig look at head-on: the foot of the eye's perpendicular is
    inside the triangle, whose plane leans by less than its width over the distance."""
    rng = np.random.default_rng(seed)
    u = 2.0 ** k
    vp = scenes.ViewParams(V=7, W=80, H=64, fovy_deg=30.0, aspect=1.6, D=10.0 * u, cone_deg=40.0, znear=0.5 * u)
    eye = vp.D * np.tan(np.radians(20.0)) * (2.0 * (np.arange(7) + 0.5) / 7 - 1.0)
    fy = 32.0 / np.tan(np.radians(15.0))
    dist = vp.D * np.exp(rng.uniform(-1.0, 0.5, n))
    size = np.exp(rng.uniform(np.log(px / 8), np.log(px), n)) * dist / fy
    lean = rng.uniform(-0.5, 0.5, (n, 2)) * (size / dist)[:, None]
    nrm = np.concatenate([lean, -np.ones((n, 1))], 1)
    nrm /= np.linalg.norm(nrm, axis=1, keepdims=True)
    s = np.cross(nrm, [0.0, 1.0, 0.0])
    s /= np.linalg.norm(s, axis=1, keepdims=True)
    t = np.cross(nrm, s)
    e = np.stack([rng.choice(eye, n), np.zeros(n), np.zeros(n)], 1)
    foot = e - nrm * dist[:, None]
    a = rng.uniform(0, 2 * np.pi, (n, 1)) + np.array([0.0, 2.1, 4.2]) + rng.uniform(-0.3, 0.3, (n, 3))
    pos = foot[:, None] + size[:, None, None] * (np.cos(a)[..., None] * s[:, None] + np.sin(a)[..., None] * t[:, None])
    idx = np.arange(3 * n).reshape(n, 3)
    idx = np.concatenate([idx, idx[:, ::-1]])  # one of the two faces the rig
    tex = scenes.value_noise_texture(64, rng)
    scene = scenes.Scene(pos.reshape(-1, 3).astype(np.float32), rng.uniform(0, 2, (3 * n, 2)).astype(np.float32),
                         idx.astype(np.uint32), np.zeros(2 * n, np.uint16), [tex], "facing").check()
    return scene, vp, np.eye(3, 4, dtype=np.float32)


@pytest.mark.parametrize("k,px", [(0, 4.0), (-20, 4.0), (-26, 1.0), (-27, 1.0), (-28, 0.5), (-28, 2.0), (-31, 4.0)])
def test_microscopic_triangles_seen_head_on(k, px):
    """Their areas' reciprocal overflows below some 2^-28: the nearest point is infinite, and so may be a sample
    density, whatever form the quotients after it take."""
    scene, vp, model = facing(k, px, 3000, 5)
    check(scene, vp, model, f"2^{k}, {px} px")
