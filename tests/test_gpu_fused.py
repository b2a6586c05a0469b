"""The kernels that take two steps per pass against the one-step kernel, which
an explicit launch shape selects: the same node update on the same values, so
the populations are equal bit for bit.  Sizes: the tiles' and marching columns'
edges and remainders, every wall type, odd step counts (a one-step launch ends
the run)."""
import numpy as np
import pytest

from paper_1511_04633_amd import inputs
from paper_1511_04633_amd import lbmx as L

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _setup():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    L.load()


def both(steps, read=L.Cavity.get_populations, **kw):
    n = kw["n"]
    out = []
    for shape in ((0, 0), (min(n, 256), 1)):
        c = L.Cavity(theta0=inputs.theta_noise(n, 5, 0.3), **kw).set_launch(*shape)
        c.step(steps)
        assert c.t == steps
        out.append(read(c))
        c.close()
    return out


# tiles (up to 40^3 FP32, 32^3 FP64) and the sizes just above
SMALL = [4, 5, 7, 16, 17, 31, 32, 33, 39, 40, 41]
# marching columns: FP32 64 x 13 (112, 127, 170, 176, 257) and 32 x 13 (144),
# FP64 32 x 13; 144 = 11 x 13 + 1, 170 = 13 x 13 + 1 and 257 = 4 x 64 + 1 end a
# column one node before the wall (its halo lies on the wall)
LARGE = [("f32", 112), ("f32", 127), ("f32", 144), ("f32", 170), ("f32", 176), ("f32", 257), ("f64", 96),
         ("f64", 144)]


@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("n", SMALL)
def test_tiles_equal_single_steps(storage, n):
    for wall_type in (1, 2, 3):
        print(f"case: two-step tiles {storage} n={n} T{wall_type}", flush=True)
        a, b = both(7, n=n, wall_type=wall_type, ra=1e4, storage=storage)
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), (n, wall_type)


@pytest.mark.parametrize("storage,n", LARGE)
def test_marching_columns_equal_single_steps(storage, n):
    wall_type = 2 + n % 2
    print(f"case: two-step columns {storage} n={n} T{wall_type}", flush=True)
    # the fields alone where the populations would take gigabytes on the host
    read = L.Cavity.get_populations if n < 200 else L.Cavity.read_macro
    a, b = both(5, read, n=n, wall_type=wall_type, ra=1e5, storage=storage)
    assert all(np.array_equal(p, q) for p, q in zip(a, b)), n


@pytest.mark.parametrize("force_model,aniso", [(1, None), (2, None), (0, (1.2, 0.9, 1.1, 0.1, -0.2, 0.05))])
def test_variants_equal_single_steps(force_model, aniso):
    for n in (20, 112):
        print(f"case: two steps, force {force_model} aniso {aniso} n={n}", flush=True)
        a, b = both(4, n=n, wall_type=2, ra=1e4, storage="f32", force_model=force_model, aniso=aniso)
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), n


# both sides of the lattice sizes at which the steps' store policy changes
@pytest.mark.parametrize("n,storage", [(45, "f32"), (48, "f32"), (51, "f32"), (108, "f32"), (112, "f32"),
                                       (86, "f64"), (88, "f64"), (135, "f16_i16"), (140, "f16_i16")])
def test_store_policies_give_the_same_steps(n, storage):
    """The state after several steps equals the batch's (another kernel) bit for bit."""
    print(f"case: store policy n={n} {storage}", flush=True)
    th = inputs.theta_noise(n, 3, 0.3)
    cav = L.Cavity(n=n, wall_type=1, ra=1e5, storage=storage)
    cav.init_rest(th)
    b = L.Batch([dict(n=n, wall_type=1, ra=1e5)], storage=storage)
    b.init_rest(0, th)
    cav.step(5)
    b.step(5)
    for p, q in zip(cav.read_macro(), b.read_macro(0)):
        assert np.array_equal(p, q)


def test_the_compared_launches_differ():
    """The default launch takes two steps per pass at the sizes compared above and
    explicit shapes one; sizes between the tiles and the columns take one."""
    two = [("f32", n) for n in SMALL if n <= 40] + [("f64", n) for n in SMALL if n <= 32] + LARGE
    for storage, n in two + [("f32", 41), ("f64", 33), ("f32", 64), ("f64", 64), ("f16", 112)]:
        print(f"case: steps per pass {storage} n={n}", flush=True)
        c = L.Cavity(n=n, wall_type=1, ra=1e4, storage=storage)
        assert c.steps_per_pass() == (2 if (storage, n) in two else 1), (storage, n)
        assert c.set_launch(min(n, 256), 1).steps_per_pass() == 1
        c.close()
    guo = L.Cavity(n=112, wall_type=1, ra=1e4, storage="f32", force_model=2)
    assert guo.steps_per_pass() == 1
