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


# volumes of two chunks (16 x 8 x 4) in a column exactly, one voxel less and more per
# axis, columns of one voxel and row, teams (two rows) partly and wholly outside
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


def forward(x, w, b, kind, gate=None, split=0):
    """Outputs of the forward convolution: FP32, BF16, with its SiLU, times SiLU' at gate, or split."""
    import torch
    from paper_1511_04633_amd import unet
    B, D, H, W, ci = x.shape
    co = w.shape[0]
    new = lambda c, t=torch.bfloat16: torch.full((B, D, H, W, c), 7.0, dtype=t, device="cuda")
    out = new(split or co, torch.float32 if kind == "f32" else torch.bfloat16)
    act = new(co) if kind == "act" else None
    out2 = new(co - split) if split else None
    p = unet.P
    if kind == "f32":
        unet.call("lbmx_nn_conv3d_fwd", p(x), p(w), p(b), p(out), 1, B, D, H, W, ci, co, unet.stream_ptr())
    else:
        unet.call("lbmx_nn_conv3d_fwd_ep", p(x), p(w), p(b), p(out), p(act), p(gate), p(out2), split, B, D, H, W,
                  ci, co, unet.stream_ptr())
    torch.cuda.synchronize()
    return [t for t in (out, act, out2) if t is not None]


# voxel counts on both sides of every tile choice: two and three channel tiles, bricks of
# 8 planes (whole, one plane and one row more, x and y remainders), several rounds of channels
@pytest.mark.parametrize("shape,ci,co", [
    ((1, 64, 32, 64), 16, 32), ((1, 61, 33, 65), 48, 32), ((1, 64, 32, 64), 32, 48), ((2, 33, 31, 66), 16, 48),
    ((1, 64, 64, 64), 16, 16), ((1, 65, 61, 67), 48, 16), ((4, 57, 36, 33), 32, 16), ((1, 72, 64, 49), 16, 80),
    ((2, 69, 61, 67), 16, 16), ((1, 33, 30, 66), 48, 80), ((3, 8, 8, 8), 32, 32)])
def test_forward_tile_choices(shape, ci, co):
    print(f"case: forward tiles {shape} {ci}->{co}", flush=True)
    x, w, b = rnd(shape + (ci,), 31), rnd((co, 27, ci), 32), np.random.default_rng(33).standard_normal(co)
    tx, tw = to_bf(x), to_bf(w)
    import torch
    tb = torch.tensor(b.astype(np.float32)).cuda()
    r = np.random.default_rng(34)
    edge = [[0, 0, 0, 0], [shape[0] - 1, *(n - 1 for n in shape[1:])]]
    pts = np.concatenate([edge, np.stack([r.integers(0, n, 4000) for n in shape], 1)])
    z8 = pts[r.integers(0, len(pts), 500)]
    z8[:, 1] = (z8[:, 1] // 8 * 8 + 7 * r.integers(0, 2, 500)).clip(0, shape[1] - 1)  # first and last planes of bricks
    pts = np.concatenate([pts, z8])
    b32 = b.astype(np.float32).astype(np.float64)
    ref = N.conv3d_at(x, w, b32, pts)
    bound = 2e-5 * N.conv3d_at(np.abs(x), np.abs(w), np.abs(b32), pts) + 1e-6
    at = tuple(torch.tensor(pts.T).cuda())
    f32, = forward(tx, tw, tb, "f32")
    assert np.all(np.abs(f32[at].double().cpu().numpy() - ref) <= bound)
    # the other outputs are roundings of the same sums
    z, a = forward(tx, tw, tb, "act")
    assert torch.equal(z, f32.to(torch.bfloat16))
    assert torch.equal(forward(tx, tw, tb, "plain")[0], z)
    s = torch.nn.functional.silu(z.float())
    assert torch.all((a.float() - s).abs() <= 2 ** -8 * s.abs() + 1e-6)
    gate = to_bf(rnd(shape + (co,), 35))
    q = gate.double()
    sg = torch.sigmoid(q)
    want = z.double() * sg * (1 + q * (1 - sg))
    got = forward(tx, tw, tb, "gate", gate)[0].double()
    assert torch.all((got - want).abs() <= 2 ** -8 * want.abs() + 1e-5 * z.double().abs() + 1e-6)
    if co > 16:
        lo, hi = forward(tx, tw, tb, "split", split=16)
        assert torch.equal(torch.cat([lo, hi], -1), z)


@pytest.mark.parametrize("shape,ci,co", [((1, 9, 10, 17), 32, 16), ((1, 24, 20, 40), 16, 32)])
def test_operands_off_16_bytes_give_the_same(shape, ci, co):
    """Views that start 2 bytes (FP32 output: 4) off a 16-byte boundary."""
    import torch
    from paper_1511_04633_amd import unet
    print(f"case: misaligned {shape} {ci}->{co}", flush=True)

    def off(t):
        flat = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")
        flat[1:] = t.flatten()
        return flat[1:].view(t.shape)

    x, w = to_bf(rnd(shape + (ci,), 41)), to_bf(rnd((co, 27, ci), 42))
    b = to_bf(rnd((co,), 43)).float()
    gate = to_bf(rnd(shape + (co,), 44))
    for kind, g in (("f32", None), ("act", None), ("gate", gate), ("plain", None)):
        for p, q in zip(forward(x, w, b, kind, g), forward(off(x), off(w), b, kind, None if g is None else off(g))):
            assert torch.equal(p, q), kind
    gw, gb = wgrad(x, gate)
    for o in (wgrad(off(x), gate), wgrad(x, off(gate))):
        assert torch.allclose(o[0], gw, rtol=1e-4, atol=1e-2) and torch.allclose(o[1], gb, rtol=1e-4, atol=1e-2)
    K = 3
    tgt = torch.randn(shape + (K,), device="cuda")
    res = []
    for f in (lambda t: t, off):
        pred, grad = f(torch.zeros(shape + (co,), device="cuda")), f(torch.zeros_like(gate))
        part = torch.zeros(4096, dtype=torch.float64, device="cuda")
        xx, ww = f(x), f(w)
        unet.call("lbmx_nn_conv3d_mse", unet.P(xx), unet.P(ww), unet.P(b), unet.P(tgt), K, unet.P(grad),
                  unet.P(part), 4096, unet.P(pred), *shape, ci, co, unet.stream_ptr())
        torch.cuda.synchronize()
        res.append((pred.clone(), grad.clone(), part.sum().item()))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])
    assert abs(res[0][2] - res[1][2]) <= 1e-12 * res[0][2]


# many channel pairs leave few blocks each: long ranges of chunks (the rings wrap several
# times), ranges that start and end inside a column, several columns per block
@pytest.mark.parametrize("shape,ci,co", [((1, 30, 9, 17), 256, 256), ((2, 19, 10, 20), 96, 128),
                                         ((1, 45, 8, 16), 160, 128)])
def test_weight_gradient_long_ranges(shape, ci, co):
    print(f"case: wgrad ranges {shape} {ci}->{co}", flush=True)
    B, D, H, W = shape
    x, g = rnd((B, D, H, W, ci), 51), rnd((B, D, H, W, co), 52)
    ref, bound = N.conv3d_wgrad(x, g), N.conv3d_wgrad(np.abs(x), np.abs(g))
    for a, r, b in zip(wgrad(to_bf(x), to_bf(g)), ref, bound):
        err = np.abs(a.cpu().numpy() - r)
        assert np.all(err <= 2e-5 * b + 1e-6), (err.max(), shape)


def test_weight_gradient_upsampled_input():
    """A decoder layer's input read in place, against its concatenation."""
    import torch
    from paper_1511_04633_amd import unet
    B, D, H, W, cu, cs, co = 2, 22, 10, 34, 32, 16, 32
    print(f"case: wgrad upcat {B}x{D}x{H}x{W} {cu}+{cs}->{co}", flush=True)
    low, skip, g = rnd((B, D // 2, H // 2, W // 2, cu), 61), rnd((B, D, H, W, cs), 62), rnd((B, D, H, W, co), 63)
    tl, ts, tg = to_bf(low), to_bf(skip), to_bf(g)
    gw = torch.zeros((co, 27, cu + cs), device="cuda")
    gb = torch.zeros(co, device="cuda")
    unet.call("lbmx_nn_conv3d_wgrad_upcat", unet.P(tl), unet.P(ts), unet.P(tg), unet.P(gw), unet.P(gb), B, D, H, W,
              cu, cs, co, unet.stream_ptr())
    torch.cuda.synchronize()
    x = np.concatenate([N.up2(low), skip], -1)
    ref, bound = N.conv3d_wgrad(x, g), N.conv3d_wgrad(np.abs(x), np.abs(g))
    for a, r, b in zip((gw, gb), ref, bound):
        assert np.all(np.abs(a.cpu().numpy() - r) <= 2e-5 * b + 1e-6)


# chunks of 16 x 8 x 4 voxels down columns: depths about whole chunks with remainders in x and
# y, rows of one to four teams, plain and 2 bytes off a 16-byte boundary (loads through registers)
@pytest.mark.parametrize("shape", [(1, 3, 1, 15), (2, 4, 2, 17), (1, 5, 3, 16), (1, 8, 6, 31), (2, 9, 7, 33),
                                   (1, 13, 8, 1), (1, 16, 9, 18), (3, 12, 4, 16)])
@pytest.mark.parametrize("aligned", [True, False])
def test_weight_gradient_chunks_of_a_column(shape, aligned):
    import torch
    print(f"case: wgrad chunks {shape} aligned {aligned}", flush=True)
    ci, co = 32, 16
    x, g = rnd(shape + (ci,), 71), rnd(shape + (co,), 72)
    ref, bound = N.conv3d_wgrad(x, g), N.conv3d_wgrad(np.abs(x), np.abs(g))
    t = []
    for a in (to_bf(x), to_bf(g)):
        if not aligned:
            flat = torch.empty(a.numel() + 1, dtype=a.dtype, device="cuda")
            flat[1:] = a.flatten()
            a = flat[1:].view(a.shape)
        t.append(a)
    for a, r, b in zip(wgrad(*t), ref, bound):
        assert np.all(np.abs(a.cpu().numpy() - r) <= 2e-5 * b + 1e-6), shape


@pytest.mark.parametrize("H", [2, 4, 6, 12])
def test_weight_gradient_leaves_rows_outside_alone(H):
    """An infinite input in the last row enters no tap that pairs it with a row
    outside the volume, where the output gradient counts as zero (rows are taken
    in pairs: of an odd number the last has one outside beside it)."""
    import torch
    print(f"case: wgrad non-finite input, {H} rows", flush=True)
    shape, ci, co = (1, 4, H, 16), 16, 16
    x, g = to_bf(rnd(shape + (ci,), 81)), to_bf(rnd(shape + (co,), 82))
    want = wgrad(x, g)[0]
    x[0, 1, H - 1, 5, 3] = float("inf")
    got = wgrad(x, g)[0]
    # taps with y offset -1 pair input row y with output row y + 1
    assert torch.equal(got[:, [t for t in range(27) if t // 3 % 3 == 0]],
                       want[:, [t for t in range(27) if t // 3 % 3 == 0]])
    assert not torch.isfinite(got[:, 13, 3]).any()
