"""The bench's roofline names the kernel that takes longest by itself: with two
frames in flight the set-up's events span the splat that runs beside it."""
import importlib.util
import os

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_roofline_takes_stages_of_single_frames():
    spec = importlib.util.spec_from_file_location("bench_stages", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    overlapped = {"setup": 1.13, "scan": 0.03, "emit": 0.2, "splat": 1.11, "resolve": 0.06, "interleave": 0.02}
    alone = {"setup": 0.17, "scan": 0.006, "emit": 0.14, "splat": 1.02, "resolve": 0.04}
    shape = dict(nt=999168, views=48, points=3.0e6, pixels=48 * 512 * 512, out_pixels=48 * 512 * 512, panel_px=2560 * 1600,
                 tris_with_points=4.8e5, written_px=4.8e7, quilt=False)
    r = bench.roofline(bench.stages_alone(overlapped, alone), 1.47e8, shape, traffic=1.0e9)
    assert r["kernel"] == "k_splat" and r["launch_ms"] == 1.02 and r["traffic"] == 1.0e9
    assert bench.stages_alone(overlapped, alone)["interleave"] == 0.02  # not part of a rendered frame
