"""Lattices above 4 GiB, which the step, pull, read, Nu and initialisation
kernels address by 64-bit plane bases and 32-bit offsets in them.  FP64 at
328^3 (7.3 GB per lattice) and FP32 at 416^3 (7.5 GB per lattice), started
from smooth random fields so that every population carries a distinct value,
are checked one step at a time on sampled nodes against the oracle (as the
256^3 test does), including nodes whose populations lie beyond the first
4 GiB; the Nu family of the state against the oracle's; and the macroscopic
read-back against the populations it is defined from (Eqs. 20, 25, 30)."""
import gc

import numpy as np
import pytest

from oracle import oracle as O
from paper_1511_04633_amd import inputs
from paper_1511_04633_amd import lbmx as L

pytestmark = pytest.mark.gpu

@pytest.fixture(scope="module", autouse=True)
def _setup():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    L.load()
    O.build(force=False)


def sample_nodes(n, seed=11):
    pts = {(x, y, z) for x in (0, n - 1) for y in (0, n - 1) for z in (0, n - 1)}
    m = n // 2
    pts.update({(m, m, 0), (m, m, n - 1), (0, m, m), (n - 1, m, m), (m, 0, m), (m, n - 1, m)})
    rng = np.random.default_rng(seed)
    for _ in range(400):
        pts.add(tuple(int(v) for v in rng.integers(0, n, 3)))
    for _ in range(200):  # the last eighth of the lattice: offsets beyond 4 GiB
        pts.add((int(rng.integers(0, n)), int(rng.integers(0, n)), int(rng.integers(7 * n // 8, n))))
    return sorted(pts)


@pytest.mark.parametrize("storage,n", [("f64", 328), ("f32", 416)])
def test_step_beyond_4gib(storage, n):
    import torch
    print(f"case: {storage} {n}^3 (lattice > 4 GiB), sampled one-step parity", flush=True)
    bpc = L.bytes_per_cell(storage)
    assert n ** 3 * bpc / 2 > 2 ** 32
    cav = L.Cavity(n=n, wall_type=2, ra=1e5, storage=storage)
    fld = torch.from_numpy(inputs.random_fields(8, 20151115)).cuda()
    cav.init_fields(fld[0], fld[1], fld[2], fld[3])
    cav.step(2)
    f0, g0 = cav.get_populations()
    cav.step(1)
    f1, g1 = cav.get_populations()
    nu_gpu = cav.nusselt()
    rho, ux, uy, uz, th = (a.reshape(-1) for a in cav.read_macro())
    cav.close()
    del fld
    torch.cuda.empty_cache()

    tol_f, tol_g = (1e-14, 1e-14) if storage == "f64" else (2e-8, 4e-8)
    e19 = O.velocities()[0]
    ora = O.Oracle(n, 2, ra=1e5, state=False)
    worst = 0.0
    for (x, y, z) in sample_nodes(n):
        c = x + n * (y + n * z)
        fo, go = ora.step_node(f0, g0, x, y, z)
        df, dg = np.abs(f1[:, c] - fo).max(), np.abs(g1[:, c] - go).max()
        assert df <= tol_f and dg <= tol_g, ((x, y, z), df, dg)
        worst = max(worst, df, dg)
        # read-back: rho = sum f, u = sum e f / rho, theta = sum g (Eqs. 20, 25, 30)
        r = f1[:, c].sum()
        assert abs(rho[c] - r) <= 1e-12
        assert np.abs(np.array([ux[c], uy[c], uz[c]]) - e19.T @ f1[:, c] / r).max() <= 1e-12
        assert abs(th[c] - g1[:, c].sum()) <= 1e-12
    print({"storage": storage, "n": n, "worst": worst})
    nu_ora = ora.nusselt_of(g1)
    for k in ("nu3d", "nu2d", "numax"):
        assert abs(nu_gpu[k] - nu_ora[k]) <= 1e-12 * abs(nu_ora[k]), (k, nu_gpu[k], nu_ora[k])
    del f0, g0, f1, g1
    gc.collect()
