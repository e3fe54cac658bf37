"""Views of a few columns: the disparity blur steps from row to row at the same
cost as in wide views (a loop over the rows of a step took up to 256 turns a
thread and step), so a forward pass takes as long as one of as many pixels in a
square."""
import numpy as np
import pytest

from oracle import net_oracle as N

pytestmark = pytest.mark.gpu


def forward_us(V, H, W):
    import torch
    from paper_2601_19901_amd import lfdpr
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    net = lfdpr.Net(lfdpr.Renderer(0), V, H, W)
    x = torch.zeros((V, H, W, 4), dtype=torch.int16, device="cuda")
    y = torch.empty_like(x)
    best = np.inf
    for _ in range(8):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        for _ in range(100):
            net.forward(x, y)
        t1.record()
        t1.synchronize()
        best = min(best, t0.elapsed_time(t1) * 10.0)
    net.close()
    return best


def test_one_column_costs_what_a_square_does():
    narrow, square = forward_us(5, 64, 1), forward_us(5, 8, 8)
    print(f"64 x 1 {narrow:.1f} us, 8 x 8 {square:.1f} us")
    assert narrow < 1.2 * square


@pytest.mark.parametrize("V,H,W", [(48, 96, 1), (48, 70, 2), (31, 150, 3), (48, 64, 85), (48, 64, 253), (48, 64, 256)])
def test_narrow_rows_match_the_oracle(V, H, W):
    """Several rows a group where the block's step is whole rows, a row more, or less than a (padded) row."""
    import torch
    from paper_2601_19901_amd import lfdpr
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(V + W)
    x = rng.random((V, H, W, 4)) * 2 - 0.5
    x[..., 3] = rng.uniform(-0.5, 3.0, (V, H, W))
    x = N.bf16(x)
    bits = (x.astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    net = lfdpr.Net(lfdpr.Renderer(0), V, H, W)
    net.set_disparity_scale(2.5)
    net.forward(torch.from_numpy(bits.view(np.int16)).cuda(), torch.empty((V, H, W, 4), dtype=torch.int16, device="cuda"))
    blur = torch.zeros((V, H, W, 4), dtype=torch.int16, device="cuda")
    net.copy_state(4, blur)
    got = (blur.cpu().numpy().view(np.uint16).astype(np.uint32) << 16).view(np.float32)
    np.testing.assert_array_equal(got, N.disparity_blur(x, np.float32(2.5)))
