"""Timing cases of the library's public entry points, from the smallest frame to the largest.

Five kinds of work, each through the calls a program makes:

* ``frame``    one frame: render every view of a rig, filter sub-views where the rig has them, interleave the
               panel.  Options that programs use: physically based shading, depth output, two frames in flight,
               the row-band quilt, the allocation-free call, every panel reconstruction mode.
* ``batch``    several scenes of uneven sizes in one launch sequence, replayed from its graph, with panels.
* ``panel``    reconstruction alone: sub-views to views (angular filter), views to the panel.
* ``network``  the learned reconstruction's forward pass from rendered views and depth.
* ``training`` one training step's forward and backward pass on image crops.

Sizes are those of the repository's workloads (``scenes.py``, ``bench.py``) or generic ones of the same ranges.
"""
import dataclasses
import math

import numpy as np
import torch

from paper_2601_19901_amd import lfdpr, scenes

TEX_TILE = 256  # textures above this edge repeat a seeded tile: quick to make, the same texel addresses


def listed():
    return [
        # A light field of a few thousand triangles (a preview, an icon, a unit of an interactive editor): the
        # workload `tiny`, where launches and latency are all there is.
        _frame("frame-tiny", scene="tiny", V=8, W=128, H=128, Wp=512, Hp=512, depth=True),
        # A serving loop that may not allocate: a small scene at odd sizes through render_frame_noalloc.
        _frame("frame-noalloc", quads=96, levels=(2, 1), tex=128, n_tex=4, V=12, W=97, H=89, Wp=321, Hp=203, noalloc=True),
        # A mid-size scene on an odd-sized rig with depth for a compositor and the full panel reconstruction.
        _frame("frame-mid-odd", quads=181, levels=(3, 2), tex=512, n_tex=8, V=25, W=317, H=253, Wp=1283, Hp=797,
               mode=scenes.RECON_BOTH, depth=True),
        # The headline: one million triangles, 48 views of 512^2, a 2560x1600 panel, one frame at a time ...
        _frame("frame-display-1M"),
        # ... and as the benchmark streams it, with two frames in flight.
        _frame("frame-display-1M-stream", in_flight=2),
        # The same scene physically shaded (four textures per triangle, a light that moves with the seed).
        _frame("frame-display-1M-pbr", pbr=True, n_tex=8),
        # 2x spatial supersampling: views of 1024^2, spatial taps.
        _frame("frame-spatial2x", quads=256, levels=(3, 2), V=48, W=1024, H=1024, mode=scenes.RECON_SPATIAL, capacity=16 << 20),
        # 4x angular supersampling: 192 sub-views through the quilt, filtered to 48 views.
        _frame("frame-ss4-quilt", quads=512, S=4, order=lfdpr.SPLAT_QUILT),
        # Independent scenes of uneven sizes per call, cones of 30 to 50 degrees, with their panels.
        {"name": "batch-uneven", "kind": "batch", "n": 5, "lo": 50e3, "hi": 1e6, "tex": 1024, "n_tex": 4, "V": 48,
         "W": 512, "H": 512, "Wp": 2560, "Hp": 1600},
        # Reconstruction of views that exist already (a recorded light field, a panel calibration).
        {"name": "panel-ss4-both", "kind": "panel", "V": 48, "S": 4, "W": 512, "H": 512, "Wp": 2560, "Hp": 1600,
         "mode": scenes.RECON_BOTH},
        # The learned reconstruction of a whole display frame ...
        {"name": "network-display", "kind": "network", "V": 48, "W": 512, "H": 512},
        # ... and its training on crops, as learned.py trains it.
        {"name": "training-crops", "kind": "training", "V": 48, "W": 128, "H": 128},
    ]


def draw(rng):
    kind = rng.choices(("frame", "batch", "panel", "network", "training"), (8, 2, 2, 2, 2))[0]
    logi = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))  # noqa: E731
    panel = {"Wp": logi(200, 2560), "Hp": logi(150, 1600), "mode": rng.choice((0, 0, 1, 2, 3))}
    if kind == "network":
        return {"kind": kind, "V": rng.randint(5, 48), "W": logi(48, 512), "H": logi(48, 512)}
    if kind == "training":
        return {"kind": kind, "V": rng.randint(5, 48), "W": logi(33, 160), "H": logi(33, 160)}
    if kind == "panel":
        return {"kind": kind, "V": rng.randint(4, 48), "S": rng.choice((1, 2, 3, 4)), "W": logi(64, 600), "H": logi(64, 600), **panel}
    if kind == "batch":
        return {"kind": kind, "n": rng.randint(2, 5), "lo": 5e3, "hi": float(logi(2e4, 1e6)), "tex": 2 ** rng.randint(7, 10),
                "n_tex": 4, "V": rng.randint(6, 48), "W": logi(96, 512), "H": logi(96, 512), **panel}
    noalloc = rng.random() < 0.15
    if noalloc:  # within the limits of that call
        return _frame(None, quads=logi(8, 110), levels=(2, 1), tex=2 ** rng.randint(6, 10), n_tex=4, V=rng.randint(3, 16),
                      W=logi(48, 160), H=logi(48, 160), noalloc=True, depth=rng.random() < 0.5, **panel)
    S = rng.choice((1, 1, 1, 2, 3, 4))
    V = rng.randint(4, 48)
    W, H = logi(64, 600), logi(64, 512)
    if V * S * W * H > 192 * 512 * 512:
        W = 512
    quads = logi(16, 512)
    return _frame(None, quads=quads, levels=(2, 1) if quads < 100 else (3, 2) if quads < 300 else (4, 3), tex=2 ** rng.randint(6, 11),
                  n_tex=rng.choice((4, 8, 16)), V=V, S=S, W=W, H=H, pbr=rng.random() < 0.25,
                  depth=rng.random() < 0.5, in_flight=rng.choice((1, 2)), mip=rng.random() < 0.9,
                  order=lfdpr.SPLAT_QUILT if V * S > 100 or rng.random() < 0.25 else lfdpr.SPLAT_POINT, **panel)


def _frame(name, scene="display", quads=512, levels=(4, 3), tex=2048, n_tex=16, V=48, S=1, W=512, H=512, Wp=2560, Hp=1600,
           mode=scenes.RECON_NONE, pbr=False, depth=False, in_flight=1, order=lfdpr.SPLAT_POINT, noalloc=False, mip=True,
           capacity=0):
    c = {"kind": "frame", "scene": scene, "quads": quads, "level_a": levels[0], "level_b": levels[1], "tex": tex, "n_tex": n_tex,
         "V": V, "S": S, "W": W, "H": H, "Wp": Wp, "Hp": Hp, "mode": mode, "pbr": pbr, "depth": depth, "in_flight": in_flight,
         "order": order, "noalloc": noalloc, "mip": mip, "capacity": capacity}
    return {"name": name, **c} if name else c


# ---------------------------------------------------------------------------------------------------- inputs


def _textures(ts, size):
    """The scene's seeded texture tiles repeated to the asked edge."""
    return [np.tile(t, (size // t.shape[0], size // t.shape[0], 1)) for t in ts]


def _display_scene(seed, quads, levels, tex, n_tex):
    counts = (57, 143) if quads >= 100 else (6, 10)
    s = scenes.display_scene(seed, hf_quads=quads, levels=levels, counts=counts, tex_size=min(tex, TEX_TILE), n_tex=n_tex)
    return dataclasses.replace(s, textures=_textures(s.textures, tex))


def _with_materials(scene, seed, tex):
    """Two material sets (normal map, roughness, metallic) picked by the albedo texture, the first with a normal
    map twice as large as the albedo."""
    rng = np.random.default_rng(seed + 900)
    textures, sets = list(scene.textures), []
    for m in range(2):
        size = min(4096, tex * (2 if m == 0 else 1))
        made = ((scenes.normal_map_texture(min(size, TEX_TILE), rng), size),
                (scenes.scalar_texture(min(size // 2, TEX_TILE), rng, 0.15, 0.95), size // 2),
                (scenes.metallic_texture(min(size // 4, TEX_TILE), rng), size // 4))
        sets.append([len(textures) + k for k in range(3)])
        textures += [_textures([t], s)[0] for t, s in made]
    mats = np.asarray(sets, np.uint16)[scene.tex.astype(np.int64) % 2]
    return dataclasses.replace(scene, textures=textures, materials=np.ascontiguousarray(mats))


def _lens(case, seed):
    S = 2 if case["W"] >= 1024 else 1  # the taps keep their footprint when the views are supersampled
    taps = scenes.gaussian_taps(seed + 200, sigma_s=0.5625 * S, trunc_s=1.125 * S)
    return scenes.LensParams(Wp=case["Wp"], Hp=case["Hp"], pitch_subpx=3.0 * 3840.0 / 479.36,
                             slope=-math.tan(math.radians(9.66)), offset=0.13, mode=case.get("mode", 0), taps=taps)


def _views(case, seed, cone=40.0):
    S = case.get("S", 1)
    return scenes.ViewParams(V=case["V"], W=case["W"], H=case["H"], fovy_deg=30.0, aspect=1.6, D=10.0, cone_deg=cone, znear=0.5,
                             S=S, jitter=scenes.subview_jitter(seed + 100, case["V"] * S) if S > 1 else None,
                             mip=case.get("mip", True))


def _images(seed, n, H, W, dev):
    """n smooth pictures with depth, as a renderer leaves them: RGBA8 in int32, depth in float32, +inf where empty."""
    g = torch.Generator(device=dev).manual_seed(seed)
    grid = torch.rand((n, 5, 9, 9), generator=g, device=dev)
    f = torch.nn.functional.interpolate(grid, size=(H, W), mode="bilinear", align_corners=True)
    f = f + 0.08 * (torch.rand((n, 5, H, W), generator=g, device=dev) - 0.5)
    rgb = (f[:, :3].clamp(0.0, 1.0) * 255.0 + 0.5).to(torch.int32)
    views = rgb[:, 0] | (rgb[:, 1] << 8) | (rgb[:, 2] << 16) | (255 << 24)
    empty = f[:, 4] < 0.2
    depth = torch.where(empty, torch.full_like(f[:, 3], math.inf), 6.0 + 8.0 * f[:, 3])
    return torch.where(empty, torch.zeros_like(views), views).contiguous(), depth.contiguous()


def _params(seed):
    """The network's parameters as a training run starts from them, the last layer already moved off zero."""
    rng = np.random.default_rng(seed + 77)
    out = []
    for k, (ci, co) in enumerate(lfdpr.NET_SHAPES):
        std = math.sqrt(2.0 / (9 * ci)) * (0.1 if k == 3 else 1.0)
        out.append((rng.normal(0.0, std, (9, co, ci)).astype(np.float32), rng.normal(0.0, 0.02, co).astype(np.float32)))
    return out


def prepare(case, seed):
    dev, kind = "cuda:0", case["kind"]
    R = lfdpr.Renderer(0)
    s = {"case": case, "R": R}
    if kind in ("frame", "batch"):
        rng = np.random.default_rng(seed + 5)
        frames = rng.integers(0, 1000, 16)
    if kind in ("frame", "batch", "panel"):
        R.set_lens(_lens(case, seed))
        s["panel"] = torch.empty((case.get("n", 1), case["Hp"], case["Wp"], 3), dtype=torch.uint8, device=dev)
    if kind == "frame":
        if case["scene"] == "tiny":
            w = scenes.tiny(seed)
            scene, vp, tilt = w.scene, w.views, w.tilt_deg
        else:
            scene = _display_scene(seed, case["quads"], (case["level_a"], case["level_b"]), case["tex"], case["n_tex"])
            vp, tilt = _views(case, seed), -55.0
        if case["pbr"]:
            scene = _with_materials(scene, seed, case["tex"])
            light = rng.normal(size=3) * 0.2 + np.array([0.35, -0.55, -0.75])
            light = (light / np.linalg.norm(light)).astype(np.float32)
            R.set_shading(dataclasses.replace(scenes.default_light(), light_dir=tuple(float(x) for x in light)))
        s["sid"] = R.upload_scene(scene)
        R.set_views(vp, case["capacity"])
        R.set_splat_order(case["order"])
        R.set_frames_in_flight(1 if case["noalloc"] else case["in_flight"])
        s["model"] = scenes.model_matrix(int(frames[0]), vp.D, tilt)
        s["views"], s["depth"] = R.alloc_views(case["depth"])
        if case["S"] > 1:
            s["filtered"] = torch.empty((case["V"], case["H"], case["W"]), dtype=torch.int32, device=dev)
    elif kind == "batch":
        sizes = np.exp(np.linspace(math.log(case["lo"]), math.log(case["hi"]), case["n"]))
        ids, vps = [], []
        for k, tris in enumerate(sizes):
            quads = max(8, int(round(math.sqrt(tris / 4.0))))
            levels = (2, 1) if tris < 1e5 else (3, 2) if tris < 5e5 else (4, 3)
            ids.append(R.upload_scene(_display_scene(seed + k, quads, levels, case["tex"], case["n_tex"])))
            vps.append(_views(case, seed + k, cone=float(rng.uniform(30.0, 50.0))))
        s["batch"] = lfdpr.Batch(R, ids, vps)
        s["models"] = np.stack([scenes.model_matrix(int(f), 10.0, -55.0) for f in frames[: case["n"]]])
        s["views"] = s["batch"].alloc_views()
    elif kind == "panel":
        R.set_views(_views(case, seed), 1024)
        s["views"], _ = _images(seed, case["V"] * case["S"], case["H"], case["W"], dev)
        if case["S"] > 1:
            s["filtered"] = torch.empty((case["V"], case["H"], case["W"]), dtype=torch.int32, device=dev)
    else:
        V, H, W = case["V"], case["H"], case["W"]
        s["net"] = net = lfdpr.Net(R, V, H, W)
        net.set_rig(_views({**case, "W": 512, "H": 512}, seed))
        net.set_params(lfdpr.params_to_flat(_params(seed)))
        s["views"], s["depth"] = _images(seed, V, H, W, dev)
        s["x"] = torch.empty((V, H, W, 4), dtype=torch.int16, device=dev)
        s["y"] = torch.empty_like(s["x"])
        if kind == "training":
            s["target"] = torch.empty_like(s["x"])
            s["grad"] = torch.empty(net.n_params, dtype=torch.float32, device=dev)
            net.pack_input(s["views"], s["depth"], s["x"], 10.0)
            net.pack_input(_images(seed + 1, V, H, W, dev)[0], None, s["target"])
    return s


def run(s):
    R, case, kind = s["R"], s["case"], s["case"]["kind"]
    if kind == "frame":
        if case["noalloc"]:
            R.render_frame_noalloc(s["sid"], s["model"], s["views"], s["depth"])
        else:
            R.render_frame(s["sid"], s["model"], s["views"], s["depth"])
        out = {"views": s["views"], "panel": s["panel"]}
        if case["depth"]:
            out["depth"] = s["depth"]
        if case["S"] > 1:
            R.angular_filter(s["views"], s["filtered"])
            out["filtered"] = s["filtered"]
        R.reconstruct(s["filtered"] if case["S"] > 1 else s["views"], s["panel"][0])
        return out
    if kind == "batch":
        s["batch"].render(s["models"], s["views"], s["panel"])
        return {"views": s["views"], "panels": s["panel"]}
    if kind == "panel":
        if case["S"] == 1:
            R.reconstruct(s["views"], s["panel"][0])
            return {"panel": s["panel"]}
        R.angular_filter(s["views"], s["filtered"])
        R.reconstruct(s["filtered"], s["panel"][0])
        return {"filtered": s["filtered"], "panel": s["panel"]}
    net = s["net"]
    if kind == "network":
        net.pack_input(s["views"], s["depth"], s["x"], 10.0)
        net.forward(s["x"], s["y"])
        return {"y": s["y"].view(torch.bfloat16)}
    net.forward(s["x"], s["y"])
    loss = net.backward(s["target"])
    net.copy_state(20, s["grad"])
    return {"loss": loss, "grad": s["grad"]}


def work(case):
    """Bytes read and written once: meshes, views, panels, activations that the call keeps; flops where the work is a
    contraction (the frame's own arithmetic depends on the scene and is not counted here)."""
    kind = case["kind"]
    if kind in ("network", "training"):
        px = case["V"] * case["W"] * case["H"]
        flops = 2.0 * 9 * sum(ci * co for ci, co in lfdpr.NET_SHAPES) * px
        acts = 3 * 64 * px  # three hidden layers of 32 bfloat16 channels, kept for the backward pass
        if kind == "network":
            return {"bytes": px * (8 + 8 + 8) + acts, "flops": flops}
        return {"bytes": px * (8 + 8 + 8) + 2 * acts, "flops": 3.0 * flops - 2.0 * 9 * 24 * 32 * px}
    S = case.get("S", 1)
    vpx = case["V"] * case["W"] * case["H"]
    panel = 3 * case["Wp"] * case["Hp"]
    if kind == "panel":
        return {"bytes": 4 * vpx * (S + 2 if S > 1 else 1) + panel, "flops": 0}
    filt = 8 * vpx if S > 1 else 0
    if kind == "batch":
        tris = sum(np.exp(np.linspace(math.log(case["lo"]), math.log(case["hi"]), case["n"])))
        return {"bytes": case["n"] * (4 * vpx + panel) + 24 * float(tris), "flops": 0}
    tris = 1280 if case["scene"] == "tiny" else 2 * case["quads"] ** 2
    if case["scene"] != "tiny":
        ca, cb = (57, 143) if case["quads"] >= 100 else (6, 10)
        tris += 20 * (ca * 4 ** case["level_a"] + cb * 4 ** case["level_b"])
    return {"bytes": vpx * S * (8 if case["depth"] else 4) + filt + panel + 24 * tris, "flops": 0}


# ---------------------------------------------------------------------------------- the network in 64 bits


def _network64(x, k, params, kept=None):
    """The network of a frame in float64: x (V, H, W, 4) = (R, G, B, D/Z - 1), k the pixels per view step and unit of
    disparity; y (V, H, W, 3)."""
    V, H, W, _ = x.shape
    dev = x.device
    t = torch.arange(-4, 5, device=dev, dtype=torch.float64) / 4.0
    w = torch.round(65535.0 * torch.exp(-2.0 * t * t))
    w = w / w.sum()
    blur = torch.zeros((V, H, W, 3), dtype=torch.float64, device=dev)
    col = torch.arange(W, device=dev, dtype=torch.float64)
    d = x[..., 3]
    step = torch.where(d > -1.0, k * d, torch.zeros_like(d))
    for j in range(9):
        u = (col + t[j] * step).clamp(-1.0, float(W))
        i0 = u.floor()
        f = (u - i0).unsqueeze(-1)
        a, b = i0.long().clamp(0, W - 1), (i0.long() + 1).clamp(0, W - 1)
        take = lambda i: torch.gather(x[..., :3], 2, i.unsqueeze(-1).expand(-1, -1, -1, 3))  # noqa: E731
        blur += w[j] * ((1.0 - f) * take(a) + f * take(b))

    def conv(h, wt, bias, dil):  # (V, H, W, ci) -> (V, H, W, co): nine shifted products
        p = torch.nn.functional.pad(h, (0, 0, dil, dil, 1, 1))
        out = bias.expand(*h.shape[:3], bias.numel())
        for tap in range(9):
            r, c = tap // 3, (tap % 3) * dil
            out = out + (p[:, r:r + H, c:c + W].reshape(-1, h.shape[3]) @ wt[tap].t()).reshape(*h.shape[:3], -1)
        return out

    zero = torch.zeros((2, H, W, 4), dtype=torch.float64, device=dev)
    near = torch.cat([zero, x, zero])
    out = []
    for v in range(V):  # a view at a time keeps the memory small
        h = torch.cat([*(near[v + o] for o in range(5)), blur[v], zero[0, ..., :1]], dim=-1).unsqueeze(0)
        for layer, dil in enumerate((1, 3, 9, 1)):
            h = conv(h, *params[layer], dil)
            h = torch.relu(h) if layer < 3 else h
        out.append(h[0] + blur[v])
        if kept is not None:
            kept(v, out[-1])
            out[-1] = None
    return None if kept is not None else torch.stack(out)


def _input64(views, depth):
    rgb = torch.stack([((views >> (8 * c)) & 255).double() / 255.0 for c in range(3)], dim=-1)
    d = torch.zeros_like(rgb[..., 0]) if depth is None else torch.where(torch.isfinite(depth), 10.0 / depth.double() - 1.0, -1.0)
    return torch.cat([rgb, d.unsqueeze(-1)], dim=-1)


def exact(case, seed):
    """The network and its gradients in 64 bits.  Views and panels are whole numbers; a frame's depth is defined by
    fixed binary32 steps (which pixels a splat owns included) and has no 64-bit counterpart."""
    if case["kind"] not in ("network", "training"):
        return None
    dev, V, H, W = "cuda:0", case["V"], case["H"], case["W"]
    params = [(torch.tensor(w, dtype=torch.float64, device=dev), torch.tensor(b, dtype=torch.float64, device=dev)) for w, b in _params(seed)]
    fx = 256.0 / (1.6 * math.tan(math.radians(15.0)))
    k = fx * 2.0 * math.tan(math.radians(20.0)) / V
    views, depth = _images(seed, V, H, W, dev)
    x = _input64(views, depth)
    if case["kind"] == "network":
        y = _network64(x, k, params)
        return {"y": torch.cat([y, torch.zeros_like(y[..., :1])], dim=-1)}
    target = _input64(_images(seed + 1, V, H, W, dev)[0], None)[..., :3]
    for w, b in params:
        w.requires_grad_()
        b.requires_grad_()
    loss = torch.zeros((), dtype=torch.float64, device=dev)

    def one(v, yv):
        part = ((yv - target[v]) ** 2).sum() / target.numel()
        part.backward()
        loss.add_(part.detach())

    _network64(x, k, params, one)
    grad = torch.cat([torch.cat([w.grad.reshape(-1), b.grad]) for w, b in params])
    return {"loss": loss.reshape(1), "grad": grad}
