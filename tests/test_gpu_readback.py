"""Large results travel to the host in chunks by several threads: each array
equals the same array read alone, which is copied in one piece."""
import ctypes
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def alone(cav, k):
    """Field k of the five, read without the others."""
    from paper_1511_04633_amd import lbmx
    out = np.full(cav.n ** 3, np.nan)
    ptr = [None] * 5
    ptr[k] = out.ctypes.data_as(ctypes.POINTER(ctypes.c_double))
    assert lbmx.load().lbmx_read_macro(cav._h, *ptr) == 0
    return out.reshape((cav.n,) * 3)


def started(n, storage, seed):
    from paper_1511_04633_amd import lbmx
    cav = lbmx.Cavity(n=n, wall_type=1, ra=1e5, storage=storage)
    cav.init_rest(np.random.default_rng(seed).uniform(-0.5, 0.5, n ** 3))
    cav.step(3)
    return cav


# below and above the size from which threads copy; chunks that end inside an array
@pytest.mark.parametrize("n,storage", [(74, "f32"), (75, "f32"), (76, "f64"), (97, "f16_i16"), (128, "f32")])
def test_fields_and_populations(n, storage):
    print(f"case: readback n={n} {storage}", flush=True)
    cav = started(n, storage, n)
    for _ in range(2):  # the first read allocates the staging memory
        for k, a in enumerate(cav.read_macro()):
            assert np.array_equal(a, alone(cav, k)), k
    f, g = cav.get_populations()
    rho = f.reshape(19, n, n, n).sum(0)
    assert np.allclose(rho, alone(cav, 0), rtol=0, atol=1e-12 * 19)
    assert np.allclose(g.reshape(7, n, n, n).sum(0), alone(cav, 4), rtol=0, atol=1e-12 * 7)


def test_handles_read_from_several_threads():
    print("case: readback from four threads", flush=True)
    cavs = [started(75 + k, "f32", k) for k in range(4)]
    got = [None] * 4

    def read(k):
        got[k] = cavs[k].read_macro()

    ts = [threading.Thread(target=read, args=(k,)) for k in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for k, c in enumerate(cavs):
        for q in range(5):
            assert np.array_equal(got[k][q], alone(c, q)), (k, q)


def test_large_reads_on_a_per_thread_stream():
    """hipStreamPerThread (handle 2) is another stream in every thread."""
    from types import SimpleNamespace

    from paper_1511_04633_amd import lbmx
    n = 80
    print(f"case: readback on a per-thread stream n={n}", flush=True)
    th = np.random.default_rng(1).uniform(-0.5, 0.5, n ** 3)
    got = []
    for stream in (None, SimpleNamespace(cuda_stream=2)):
        cav = lbmx.Cavity(n=n, wall_type=1, ra=1e5, storage="f32", stream=stream)
        cav.init_rest(th)
        for _ in range(3):
            cav.step(50)
            fields = cav.read_macro()
        got.append(fields + cav.get_populations())
        cav.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)


def test_fields_at_the_largest_single_copy():
    """One field of 127^3 is copied in one piece, the five together by threads."""
    n = 127
    assert 8 * n ** 3 < 16 << 20 < 5 * 8 * n ** 3
    print(f"case: readback n={n}", flush=True)
    cav = started(n, "f32", n)
    for k, a in enumerate(cav.read_macro()):
        assert np.array_equal(a, alone(cav, k)), k


def test_a_batch_is_read_by_several_threads():
    """Fields and resampled fields of different cavities and of the same one."""
    from paper_1511_04633_amd import inputs, lbmx
    print("case: batch readback from eight threads", flush=True)
    sizes = (76, 80, 64)
    b = lbmx.Batch([dict(n=n, wall_type=1, ra=1e5) for n in sizes])
    for k, n in enumerate(sizes):
        b.init_rest(k, inputs.theta_noise(n, k, 0.3))
    b.step(5)
    jobs = [(b.read_macro, (k,)) for k in range(3)] + [(b.resample, (k, m)) for k in range(3) for m in (20, 112)]
    want = [f(*a) for f, a in jobs]
    got = [[None] * len(jobs) for _ in range(8)]

    def run(t):
        for i in range(len(jobs)):
            j = (i + t) % len(jobs)
            got[t][j] = jobs[j][0](*jobs[j][1])

    ts = [threading.Thread(target=run, args=(t,)) for t in range(8)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for row in got:
        for a, w in zip(row, want):
            assert all(np.array_equal(p, q) for p, q in zip(a, w))
