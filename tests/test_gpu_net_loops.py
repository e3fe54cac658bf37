"""The persistent convolutions' steady state: at most 512 workgroups share the
tiles of 8 x 64 pixels, and here each takes three or four of them (1,920 tiles,
ragged in both directions), so that a tile is fetched two ahead while one is
staged behind the previous one's stores.  Views whose tiles come first, in the
middle and last in a workgroup's run equal the oracle's, layer by layer, forward
and backward."""
import numpy as np
import pytest

from oracle import net_oracle as N
from test_gpu_net import assert_bf16_close, bits_to_f, f_to_bits, get16, make_net, random_input, random_params, t16

pytestmark = pytest.mark.gpu

V, H, W = 48, 75, 200
# Each XCD's 64 workgroups take an eighth of the order, six views of 40 tiles: the first, second, third and fourth tile
# of a workgroup lie in the views at places 0-1, 1-3, 3-4 and 4-5 of an eighth.
CHECKED = (0, 11, 25, 26, 38, 39, 47)


def test_three_and_four_tiles_per_workgroup():
    import torch
    from paper_2601_19901_amd import lfdpr
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    R, net = make_net(torch, V, H, W)
    net.set_disparity_scale(3.1)
    flat = lfdpr.params_to_flat(random_params(12))
    net.set_params(flat)
    P = lfdpr.flat_to_params(flat.astype(np.float64))
    rng = np.random.default_rng(12)
    xb = random_input(rng, V, H, W)
    tb = f_to_bits(np.concatenate([rng.random((V, H, W, 3)), np.zeros((V, H, W, 1))], axis=-1))
    x, t = t16(xb, torch), t16(tb, torch)
    y = torch.zeros((V, H, W, 4), dtype=torch.int16, device="cuda")
    net.forward(x, y)
    net.backward(t)

    def state(which):
        a = torch.zeros((V, H, W, 32), dtype=torch.int16, device="cuda")
        net.copy_state(which, a)
        return get16(a)

    views = list(CHECKED)
    blur = N.disparity_blur(bits_to_f(xb), np.float32(3.1))
    acts = [N.assemble(bits_to_f(xb), blur)] + [state(k) for k in (1, 2, 3)]
    for k in range(4):
        w, d = N.bf16(P[k][0]), N.DILATION[k]
        conv = np.stack([N.conv3x3(acts[k][v], w, P[k][1], d) for v in views])
        S = np.stack([N.conv3x3(np.abs(acts[k][v]), np.abs(w), np.abs(P[k][1]), d) for v in views])
        if k < 3:
            assert_bf16_close(acts[k + 1][views], N.bf16(np.maximum(conv, 0)), f"layer {k + 1}", abs_sum=S)
        else:
            got = get16(y)[views]
            assert (got[..., 3] == 0).all()
            assert_bf16_close(got[..., :3], N.bf16(conv + blur[views][..., :3]), "output", abs_sum=S + np.abs(blur[views][..., :3]))
    dz = {4: state(14)}
    for k in (3, 2, 1):
        dz[k] = state(10 + k)
        w, d = N.bf16(P[k][0]), N.DILATION[k]
        src = dz[k + 1][..., :w.shape[1]]
        want = N.bf16(np.stack([N.conv3x3_xgrad(src[v], w, d) for v in views]) * (acts[k][views] > 0))
        S = np.stack([N.conv3x3_xgrad(np.abs(src[v]), np.abs(w), d) for v in views])
        assert_bf16_close(dz[k][views], want, f"dZ{k}", abs_sum=S)
