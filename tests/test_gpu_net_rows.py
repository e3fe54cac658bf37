"""The disparity blur stages groups of rows in LDS when a frame has many: it
matches the oracle bit for bit at the widths where a group, its padding or its
last pass can go wrong, and the rows after the first group are the rows they
should be."""
import numpy as np
import pytest

from oracle import net_oracle as N

pytestmark = pytest.mark.gpu


# groups of 6 rows of one pixel; 4 rows, the last group cut short; 2 rows; one
# row with a last pass of one thread; the widest row that is staged
@pytest.mark.parametrize("V,H,W,k", [(48, 201, 1, 3.0), (47, 131, 7, 2.75), (48, 65, 258, 9.05), (3, 5, 257, 4.4),
                                     (2, 2, 4096, 40.0)])
def test_blur_in_groups_of_rows(V, H, W, k):
    import torch
    from paper_2601_19901_amd import lfdpr
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(V + W)
    x = rng.random((V, H, W, 4)) * 2 - 0.5
    x[..., 3] = rng.uniform(-0.5, 3.0, (V, H, W))
    x[..., 3][rng.random((V, H, W)) < 0.1] = -1.0
    x = N.bf16(x)
    bits = (x.astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    net = lfdpr.Net(lfdpr.Renderer(0), V, H, W)
    net.set_disparity_scale(k)
    xt = torch.from_numpy(bits.view(np.int16)).cuda()
    y = torch.zeros((V, H, W, 4), dtype=torch.int16, device="cuda")
    net.forward(xt, y)
    blur = torch.zeros((V, H, W, 4), dtype=torch.int16, device="cuda")
    net.copy_state(4, blur)
    got = (blur.cpu().numpy().view(np.uint16).astype(np.uint32) << 16).view(np.float32)
    np.testing.assert_array_equal(got, N.disparity_blur(x, np.float32(k)))
