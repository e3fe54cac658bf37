"""Quilt tiles that leave no LDS for the queues of covered pixels hold them in
registers: the frame equals the oracle's where few and many pixels wait at once,
and costs no more than with a tile of fewer views that has room for them."""
import time

import numpy as np
import pytest

from oracle import oracle as O
from paper_2601_19901_amd import scenes

pytestmark = pytest.mark.gpu

LDS, QUEUES = 160 * 1024, 16 * 191 * 4  # of a compute unit; of a tile's sixteen waves


def tile_bytes(rows, views, W, H):
    return rows * views * W * 8 + (W + H) * 4 + 16


def renderer():
    import torch
    from paper_2601_19901_amd import lfdpr
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    R = lfdpr.Renderer(0)
    R.set_splat_order(lfdpr.SPLAT_QUILT)
    return R


# few points per tile, boxes of many pixels, textures of one texel (points that
# cover dozens of pixels), and frames with a last view subset of one view
@pytest.mark.parametrize("W,H,V,tile,tex,pbr", [(600, 24, 8, (4, 8), 64, False), (600, 24, 9, (4, 8), 1, False),
                                               (800, 30, 13, (2, 12), 256, False), (600, 24, 8, (4, 8), 8, True),
                                               (317, 33, 31, (2, 31), 64, True), (2048, 16, 10, (1, 9), 16, False)])
def test_held_queue_matches_the_oracle(W, H, V, tile, tex, pbr):
    assert LDS - QUEUES < tile_bytes(*tile, W, H) <= LDS  # fits, but not with its queues
    R = renderer()
    rng = np.random.default_rng(W + tex)
    w = scenes.small_display(seed=5, V=V, W=W, H=H)
    scene = w.scene
    scene.textures = [rng.integers(0, 256, (tex, tex, 4), dtype=np.uint8) for _ in scene.textures]
    light = scenes.default_light() if pbr else None
    if pbr:
        scene.materials = rng.integers(0, len(scene.textures), (scene.n_tris, 3)).astype(np.uint16)
    model = w.model(2)
    o = O.render(scene, w.views, model, shading=light) if pbr else O.render(scene, w.views, model)
    R.set_shading(light)
    R.set_views(w.views)
    R.set_quilt_tile(*tile)
    views, depth = R.alloc_views(with_depth=True)
    R.render_frame(R.upload_scene(scene), model, views, depth)
    st = R.stats()
    assert (st["quilt_rows"], st["quilt_views"]) == tile
    assert st["written_px"] == o["stats"]["fragments"] - o["stats"]["misses"]
    np.testing.assert_array_equal(views.cpu().numpy().view(np.uint32), o["rgba"])
    np.testing.assert_array_equal(depth.cpu().numpy().view(np.uint32), o["depth"].view(np.uint32))


def test_held_queue_is_no_slower_than_a_smaller_tile():
    """48 views of 600 x 512: the automatic tile (4 rows x 8 views) has no room for queues, 4 x 6 has.  Both take the
    frame in 6 and 8 view subsets; taking covered pixels one lane at a time made the first twice as slow."""
    import torch
    R = renderer()
    w = scenes.display(hf_quads=160, levels=(3, 2), tex_size=256, n_tex=4, W=600, H=512)
    sid = R.upload_scene(w.scene)
    R.set_views(w.views)
    views, _ = R.alloc_views()
    model = w.model(0)

    def fastest(tile):
        R.set_quilt_tile(*tile)
        best = np.inf
        for _ in range(12):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            R.render_frame(sid, model, views)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        st = R.stats()
        assert st["quilt_rows"] == 4 and st["quilt_views"] == (tile[1] or 8)
        return best * 1e6

    auto, roomy = fastest((0, 0)), fastest((4, 6))
    print(f"4 x 8 without room {auto:.0f} us, 4 x 6 with room {roomy:.0f} us")
    assert auto < 1.3 * roomy


@pytest.mark.parametrize("W,H,V,tile,tex", [(512, 24, 12, (4, 6), (4, 4)), (512, 24, 13, (4, 6), (4, 128)), (600, 24, 8, (4, 8), (2, 256)),
                                            (130, 40, 70, (1, 70), (1, 64)), (128, 40, 9, (40, 2), (1, 32))])
def test_points_shaded_ahead_match_the_oracle(W, H, V, tile, tex):
    """Points of many pixels beside points of few: views shaded ahead and pixel by pixel follow each other."""
    R = renderer()
    rng = np.random.default_rng(W + V)
    w = scenes.small_display(seed=6, V=V, W=W, H=H, hf_quads=20)
    scene = w.scene
    scene.textures = [rng.integers(0, 256, (tex[k % 2],) * 2 + (4,), dtype=np.uint8) for k in range(len(scene.textures))]
    part = (scene.tex % 2)[:, None] + 2 * rng.integers(0, len(scene.textures) // 2, (scene.n_tris, 3))
    scene.materials = part.astype(np.uint16)  # a triangle's four textures are all coarse or all fine
    light = scenes.default_light()
    model = w.model(2)
    o = O.render(scene, w.views, model, shading=light)
    R.set_shading(light)
    R.set_views(w.views)
    R.set_quilt_tile(*tile)
    views, depth = R.alloc_views(with_depth=True)
    R.render_frame(R.upload_scene(scene), model, views, depth)
    st = R.stats()
    print(f"{st['points']} points, {st['point_views']} point-views, {st['written_px']} pixels")
    assert st["quilt_rows"] == tile[0] and st["written_px"] == o["stats"]["fragments"] - o["stats"]["misses"]
    np.testing.assert_array_equal(views.cpu().numpy().view(np.uint32), o["rgba"])
    np.testing.assert_array_equal(depth.cpu().numpy().view(np.uint32), o["depth"].view(np.uint32))


def test_points_of_many_pixels_are_shaded_once():
    """3,232 triangles with textures of 8 texels: a point covers dozens of pixels of a view, so shading costs the frame
    little; shading every pixel made it 1.6 times as long as the unlit one."""
    import torch
    R = renderer()
    rng = np.random.default_rng(4)
    scene = scenes.display_scene(3, hf_quads=16, levels=(2, 1), counts=(6, 10), tex_size=8, n_tex=4)
    scene.materials = rng.integers(0, 4, (scene.n_tris, 3)).astype(np.uint16)
    sid = R.upload_scene(scene)
    w = scenes.display(hf_quads=8, levels=(1, 1), counts=(1, 1), tex_size=8, n_tex=2)
    R.set_views(w.views)
    views, _ = R.alloc_views()

    def fastest(light):
        R.set_shading(light)
        best = np.inf
        for _ in range(12):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            R.render_frame(sid, w.model(0), views)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        return best * 1e6

    unlit, shaded = fastest(None), fastest(scenes.default_light())
    print(f"unlit {unlit:.0f} us, shaded {shaded:.0f} us")
    assert shaded < 1.2 * unlit
