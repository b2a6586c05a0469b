"""The lattice's plane layout behind the public calls: the default launch
(planes in storage order) against explicit block shapes on ragged sizes, and
the slab layout of checkpoint files, which the planes are converted to and
from."""
import os

import numpy as np
import pytest

from oracle import oracle as O
from paper_1511_04633_amd import inputs
from paper_1511_04633_amd import lbmx as L

pytestmark = pytest.mark.gpu

STORAGES = ("f64", "f32", "f16", "bf16", "f16_f32", "bf16_f32", "f16_i16")


@pytest.fixture(scope="module", autouse=True)
def _setup():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    L.load()


@pytest.mark.parametrize("storage", STORAGES)
@pytest.mark.parametrize("n", [4, 5, 17, 67, 130])
def test_default_launch_equals_explicit_shapes(storage, n):
    """Each node's update does not depend on which lane runs it: bitwise equal."""
    print(f"case: default launch {storage} n={n}", flush=True)
    th = inputs.theta_noise(n, 7, 0.3)
    out = []
    for shape in ((0, 0), (n if n < 64 else 64, 3)):
        c = L.Cavity(n=n, wall_type=2, ra=1e4, storage=storage, theta0=th).set_launch(*shape)
        c.step(3)
        out.append(c.get_populations())
        c.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("storage,n", [("f32", 16), ("f32", 37), ("f64", 11), ("f16_f32", 9)])
def test_checkpoint_file_holds_slabs(tmp_path, storage, n):
    """A file holds slabs of 2^L nodes: 19 flow segments (offsets f - w, over w
    in 16 bits), then 7 energy segments.  Streaming the file's populations by
    one node gives the state's, away from the walls."""
    print(f"case: checkpoint slabs {storage} n={n}", flush=True)
    c = L.Cavity(n=n, wall_type=3, ra=1e4, storage=storage, theta0=inputs.theta_noise(n, 3, 0.2))
    c.step(5)
    path = os.path.join(tmp_path, "c.ckpt")
    c.save(path)
    f, g = (a.reshape(-1, n, n, n) for a in c.get_populations())
    c.close()
    ft, gt, shift = {"f32": ("f4", "f4", 11), "f64": ("f8", "f8", 10), "f16_f32": ("f2", "f4", 12)}[storage]
    per, cells = 1 << shift, n ** 3
    slab = np.dtype([("f", ft, (19, per)), ("g", gt, (7, per))])
    raw = np.fromfile(path, dtype=slab, offset=376)
    assert raw.size == -(-cells // per) and os.path.getsize(path) == 376 + raw.nbytes
    fs = raw["f"].transpose(1, 0, 2).reshape(19, -1)
    gs = raw["g"].transpose(1, 0, 2).reshape(7, -1)
    assert not fs[:, cells:].any() and not gs[:, cells:].any()
    fs, gs = fs[:, :cells].reshape(19, n, n, n), gs[:, :cells].reshape(7, n, n, n)
    e = O.velocities()[0].astype(int)
    w = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)
    inner = slice(1, n - 1)
    for i in range(19):
        up = tuple(slice(1 - int(k), n - 1 - int(k)) for k in e[i][::-1])
        off = fs[i][up].astype(np.float64)
        if storage == "f16_f32":
            off = (fs[i][up].astype(np.float32) * np.float32(w[i])).astype(np.float64)
        assert np.array_equal(f[i][inner, inner, inner], w[i] + off), i
        if i < 7:
            assert np.array_equal(g[i][inner, inner, inner], gs[i][up].astype(np.float64)), i


@pytest.mark.parametrize("storage", STORAGES)
@pytest.mark.parametrize("n", [5, 33, 66])
def test_guo_forcing_does_not_depend_on_the_block(storage, n):
    """Flat blocks, explicit ones up to 256 threads and above it, bitwise."""
    print(f"case: Guo blocks {storage} n={n}", flush=True)
    th = inputs.theta_noise(n, 7, 0.3)
    out = []
    for shape in ((0, 0), (min(n, 64), 4), (33, 31)):
        c = L.Cavity(n=n, wall_type=3, ra=1e4, storage=storage, theta0=th, force_model=2).set_launch(*shape)
        c.step(4)
        out.append(c.get_populations())
        c.close()
    for f, g in out[1:]:
        assert np.array_equal(out[0][0], f) and np.array_equal(out[0][1], g)


# one size for each policy of the step kernel's stores and loads, by lattice bytes, rows of
# whole lines and blocks per plane; `other` brings a batch's total across the 132 MB at which
# its stores change
@pytest.mark.parametrize("storage,n,other", [
    ("f64", 30, 90), ("f64", 34, 90), ("f64", 38, 90), ("f64", 43, 90), ("f64", 90, 24), ("f64", 96, 24),
    ("f32", 38, 112), ("f32", 42, 112), ("f32", 44, 112), ("f32", 60, 112), ("f32", 111, 24), ("f32", 128, 24),
    ("f16", 56, 140), ("f16", 150, 24), ("f16", 192, 24), ("bf16_f32", 50, 132), ("bf16_f32", 132, 24),
    ("f16_i16", 56, 140), ("f16_i16", 150, 24)])
def test_access_policies_give_the_same_steps(storage, n, other):
    print(f"case: access policy {storage} n={n}", flush=True)
    th = inputs.theta_noise(n, 9, 0.3)
    kw = dict(wall_type=3, ra=1e5)
    out = []
    for shape in ((0, 0), (min(n, 256), max(1, 256 // n)), (64, 3)):
        c = L.Cavity(n=n, storage=storage, theta0=th, **kw).set_launch(*shape)
        for _ in range(3):  # one at a time: no step by the kernels that take two
            c.step(1)
        out.append(c.read_macro())
        c.close()
    for sizes in ([n], [n, other]):
        b = L.Batch([dict(n=m, **kw) for m in sizes], storage=storage)
        b.init_rest(0, th)
        b.step(3)
        out.append(b.read_macro(0))
        b.close()
    for fields in out[1:]:
        assert all(np.array_equal(p, q) for p, q in zip(out[0], fields))
