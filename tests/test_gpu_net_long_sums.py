"""Sums over every pixel of a large training batch (64 views of 1024 x 1024, the
most a network takes) keep the small terms that follow large ones: 512
workgroups share the tiles of 4 x 64 pixels, and the first tile of each, the
first 128 rows, holds terms so large that a single running sum in binary32
would drop all later ones, or a fifth of them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

V, H, W = 64, 1024, 1024
PX = V * H * W
HEAD = 128  # rows of view 0


@pytest.fixture(scope="module")
def net():
    """Output 0 everywhere, third activation 1 everywhere: zero weights and inputs, third bias 1."""
    import torch
    from paper_2601_19901_amd import lfdpr
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    net = lfdpr.Net(lfdpr.Renderer(0), V, H, W)
    params = [(np.zeros((9, co, ci), np.float32), np.full(co, float(k == 2), np.float32))
              for k, (ci, co) in enumerate(lfdpr.NET_SHAPES)]
    net.set_params(lfdpr.params_to_flat(params))
    x = torch.zeros((V, H, W, 4), dtype=torch.int16, device="cuda")
    y = torch.ones_like(x)
    net.forward(x, y)
    assert int(y.abs().max()) == 0
    yield net, x, y  # the backward pass reads both
    net.close()


def backward(net, head, tail):
    """Loss and gradients for a target of -head in the first rows and -tail after them."""
    import torch
    from paper_2601_19901_amd import lfdpr
    t = torch.full((V, H, W, 4), -tail, dtype=torch.bfloat16, device="cuda")
    t[0, :HEAD] = -head
    loss = float(net.backward(t.view(torch.int16)))
    g = torch.empty(net.n_params, dtype=torch.float32, device="cuda")
    net.copy_state(20, g)
    return loss, lfdpr.flat_to_params(g.double().cpu().numpy())


# dZ = 2 * 3 * 2^k / (3 * 2^26), a power of two in the head; 1.25 * 2^-18 of it after the head: below half a unit in
# the last place of the 128 head terms that one lane adds, and 2.5 units of a whole head tile per 16 products
DZ_HEAD, DZ_TAIL = 3.0, 3.0 * 1.25 * 2.0 ** -18


def test_bias_gradient_keeps_small_terms(net):
    """128 terms of a tile, 512 tiles, two halves, 64 rows and 8 phases of partial sums: at most 714 roundings."""
    _, G = backward(net[0], DZ_HEAD, DZ_TAIL)
    want = (HEAD * W + (PX - HEAD * W) * 1.25 * 2.0 ** -18) * 2.0 / PX
    err = np.abs(G[3][1] - want) / want
    print("bias gradient, relative errors", err)
    assert (err < 714 * 2.0 ** -24).all()


def test_weight_gradient_keeps_small_terms(net):
    """128 products of eight tiles (two roundings each), 64 such sums, 64 rows and 8 phases of partial sums: at most 392
    roundings, which a matrix accumulator may do towards zero."""
    _, G = backward(net[0], DZ_HEAD, DZ_TAIL)
    dz = np.zeros((2, 3, 3))  # pixels that tap (r, c) sees inside the view: in the head, after it
    for r in range(3):
        for c in range(3):
            w = W - abs(c - 1)
            head = (HEAD - 1 if r == 0 else HEAD) * w
            dz[:, r, c] = head, V * (H - abs(r - 1)) * w - head
    want = ((dz[0] + dz[1] * 1.25 * 2.0 ** -18) * 2.0 / PX).reshape(9, 1, 1)
    err = np.abs(G[3][0] - want) / want
    print("weight gradient, largest relative error", err.max())
    assert err.max() < 392 * 2.0 ** -23


def test_loss_keeps_small_terms(net):
    """2,048 workgroups, a lane per pixel: its first is in the head, with squares 2^24 times those of the 511 after it.
    Three squares of a pixel, 16 pixels, 32 such sums, then halves of 64 lanes, 8 workgroups and halves of 256: at most
    72 roundings, and those of the division by the number of terms."""
    head = 4096.0
    loss, _ = backward(net[0], head, 1.0)
    n_head = HEAD * W
    want = (n_head * head ** 2 + (PX - n_head)) / PX
    print("loss, relative error", loss / want - 1.0)
    assert abs(loss / want - 1.0) < 74 * 2.0 ** -24
