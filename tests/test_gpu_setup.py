"""The triangle set-up and the emission at the sizes where they change: scenes
of one triangle, around a workgroup of the eight-lane form (32 triangles), an
emission tile (256), and the 131,072 triangles above which one lane takes a
triangle; lattices of very many rows beside tiny ones; rigs whose view loop
takes the general quotients (focal lengths below one pixel, a z_near near
zero).  Records, counts, points, views, depth and statistics equal the oracle's
bit for bit."""
import dataclasses

import numpy as np
import pytest

from oracle import oracle as O
from paper_2601_19901_amd import scenes
from test_gpu_parity import assert_parity, run_gpu
from test_gpu_splat_wave import _soup

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _first(scene, n):
    return dataclasses.replace(scene, idx=scene.idx[:n].copy(), tex=scene.tex[:n].copy())


@pytest.mark.parametrize("n,W,H,V,fovy,znear,tex", [
    (1, 64, 48, 5, 30.0, 0.5, 8), (31, 64, 48, 5, 30.0, 0.5, 8), (32, 64, 48, 9, 30.0, 0.5, 64), (33, 64, 48, 8, 30.0, 0.5, 64),
    (257, 200, 150, 17, 30.0, 0.5, 64), (300, 600, 40, 3, 30.0, 0.5, 512), (300, 1, 1, 7, 150.0, 0.5, 4),
    (120, 64, 48, 6, 30.0, 1e-12, 16), (131071, 96, 80, 4, 30.0, 0.5, 8), (131072, 96, 80, 4, 30.0, 0.5, 8)])
def test_setup_and_emission_match_the_oracle(torch_cuda, n, W, H, V, fovy, znear, tex):
    from paper_2601_19901_amd import lfdpr
    if n < 10000:
        scene = _first(_soup(n + W, (n + 1) // 2, W, H, tex), n)
    else:
        scene = _first(scenes.display_scene(5, hf_quads=250, levels=(2, 1), counts=(57, 143), tex_size=tex, n_tex=2), n)
    assert scene.n_tris == n
    vp = scenes.ViewParams(V=V, W=W, H=H, fovy_deg=fovy, aspect=1.6, D=10.0, cone_deg=40.0, znear=znear)
    model = scenes.model_matrix(3, 10.0, -55.0 if n >= 10000 else 0.0)
    o = O.render(scene, vp, model)
    R = lfdpr.Renderer(0)
    sid = R.upload_scene(scene)
    R.set_views(vp)
    w = scenes.Workload("setup", scene, vp, None)
    g = run_gpu(R, sid, w, model, n)
    print(f"[n {n} {W}x{H}x{V}] {g['stats']}", flush=True)
    assert_parity(g, o, n, f"set-up n {n}")
    assert g["stats"]["active_tris"] == o["stats"]["active_tris"]
    assert g["stats"]["point_views"] == o["stats"]["point_views"]
    assert g["stats"]["overflow_tris"] == o["stats"]["overflow_tris"]
    # covered pixels but those of triangles without points (overflowed lattices) and those outside their splat
    assert g["stats"]["written_px"] == o["stats"]["fragments"] - o["stats"]["misses"] - o["stats"]["orphans"]


@pytest.mark.parametrize("n", [8160, 8192, 8193, 8225])
def test_totals_around_the_scan_in_the_set_up(torch_cuda, n):
    """Up to 256 set-up workgroups (8,192 triangles) the last one scans the
    point counts; from there on a launch of its own does.  Frames one after the
    other on one context give the oracle's points and statistics each time."""
    from paper_2601_19901_amd import lfdpr
    scene = _first(scenes.display_scene(5, hf_quads=70, levels=(2, 1), counts=(57, 143), tex_size=8, n_tex=2), n)
    assert scene.n_tris == n
    vp = scenes.ViewParams(V=5, W=96, H=80, fovy_deg=30.0, aspect=1.6, D=10.0, cone_deg=40.0, znear=0.5)
    w = scenes.Workload("scan", scene, vp, None)
    R = lfdpr.Renderer(0)
    sid = R.upload_scene(scene)
    R.set_views(vp)
    for angle in (-55.0, 20.0, -55.0):
        model = scenes.model_matrix(3, 10.0, angle)
        o = O.render(scene, vp, model)
        g = run_gpu(R, sid, w, model, n)
        print(f"[n {n} angle {angle}] {g['stats']}", flush=True)
        assert_parity(g, o, n, f"scan n {n}")
        for key in ("active_tris", "point_views", "overflow_tris"):
            assert g["stats"][key] == o["stats"][key]
