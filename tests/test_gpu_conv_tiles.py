"""Convolution kernels at the edges of their bricks and of their address
arithmetic, against the oracle and plain float64 sums (bounds as for the other
convolution tests: 2e-5 of the same sum of absolute terms, FP32 accumulation)."""
import numpy as np
import pytest

from oracle import nn_oracle as N

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _setup():
    import torch
    assert torch.cuda.is_available()
    from paper_1511_04633_amd import unet
    unet.nn()


def rnd(shape, seed):
    return N.bf16_round(np.random.default_rng(seed).standard_normal(shape))


def to_bf(a):
    import torch
    return torch.tensor(np.asarray(a, np.float32)).cuda().to(torch.bfloat16)


def wgrad(x, g):
    """(gw, gb) of device tensors x [B, D, H, W, ci], g [B, D, H, W, co]."""
    import torch
    from paper_1511_04633_amd import unet
    B, D, H, W, ci = x.shape
    co = g.shape[-1]
    gw = torch.zeros((co, 27, ci), dtype=torch.float32, device="cuda")
    gb = torch.zeros(co, dtype=torch.float32, device="cuda")
    unet.call("lbmx_nn_conv3d_wgrad", unet.P(x), unet.P(g), unet.P(gw), unet.P(gb), B, D, H, W, ci, co,
              unet.stream_ptr())
    torch.cuda.synchronize()
    return gw, gb


# one brick (16 x 8 x 8) exactly, one voxel less and more per axis, two bricks
# with a one-voxel second one, quarters (4 x 4 of y, z) partly and wholly empty
@pytest.mark.parametrize("shape", [(1, 8, 8, 16), (1, 7, 9, 15), (2, 9, 7, 17), (1, 1, 1, 1), (1, 4, 5, 33),
                                   (3, 12, 16, 32), (1, 17, 3, 16)])
@pytest.mark.parametrize("ci,co", [(16, 16), (32, 48)])
def test_weight_gradient_brick_edges(shape, ci, co):
    print(f"case: wgrad bricks {shape} {ci}->{co}", flush=True)
    B, D, H, W = shape
    x, g = rnd((B, D, H, W, ci), 21), rnd((B, D, H, W, co), 22)
    ref, bound = N.conv3d_wgrad(x, g), N.conv3d_wgrad(np.abs(x), np.abs(g))
    got = wgrad(to_bf(x), to_bf(g))
    for a, r, b in zip(got, ref, bound):
        err = np.abs(a.cpu().numpy() - r)
        assert np.all(err <= 2e-5 * b + 1e-6), (err.max(), shape)


def test_weight_gradient_planes_beyond_32_bit_offsets():
    """Planes so large that a brick's halo spans more than 2^32 bytes: gout is
    zero except at seeded voxels, whose neighbourhoods give the sums."""
    import torch
    B, D, H, W, ci, co = 1, 2, 1024, 1024, 192, 16
    print(f"case: wgrad far offsets {D}x{H}x{W} {ci}->{co}", flush=True)
    assert 2 * 11 * (H + 1) * (W + 2) * ci >= 2 ** 32 and 6 * (H + 1) * (W + 2) * ci < 2 ** 31
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = torch.empty((B, D, H, W, ci), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    g = torch.zeros((B, D, H, W, co), dtype=torch.bfloat16, device="cuda")
    r = np.random.default_rng(4)
    pts = {(0, 0, 0), (1, H - 1, W - 1), (1, 0, W - 1), (0, H - 1, 0)}
    pts |= {(int(r.integers(D)), int(r.integers(H)), int(r.integers(W))) for _ in range(500)}
    ref = np.zeros((co, 27, ci))
    bound = np.zeros((co, 27, ci))
    for z, y, xx in sorted(pts):
        v = rnd((co,), z * H * W + y * W + xx)
        g[0, z, y, xx] = to_bf(v)
        for t in range(27):
            q = (z + t // 9 - 1, y + t // 3 % 3 - 1, xx + t % 3 - 1)
            if 0 <= q[0] < D and 0 <= q[1] < H and 0 <= q[2] < W:
                u = x[0, q[0], q[1], q[2]].double().cpu().numpy()
                ref[:, t] += np.outer(v, u)
                bound[:, t] += np.outer(np.abs(v), np.abs(u))
    gw, gb = wgrad(x, g)
    err = np.abs(gw.cpu().numpy() - ref)
    assert np.all(err <= 2e-5 * bound + 1e-6), err.max()
    gsum = g.double().sum((0, 1, 2, 3)).cpu().numpy()
    assert np.all(np.abs(gb.cpu().numpy() - gsum) <= 2e-5 * g.double().abs().sum((0, 1, 2, 3)).cpu().numpy() + 1e-6)
