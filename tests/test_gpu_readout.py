"""Large results to the program's own pages: the same bytes as the device holds,
about the size where several threads take over, at every start address of the
destination, to pinned memory, and from two threads at once."""
import ctypes
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_1203_6350_amd import lbm, workloads as wl  # noqa: E402


def lattice(nx, ny, storage="f32", seed=0):
    g = np.random.default_rng(seed)
    rho = 1.0 + 1e-3 * g.standard_normal((ny, nx))
    u = 0.05 + 1e-3 * g.standard_normal((ny, nx))
    return lbm.Lattice(nx, ny, s=wl.S_MRT_DEFAULT, storage=storage, variant="II", ux_base=0.05,
                       rho=rho, ux=u, uy=0.1 * u)


def on_device(lat, ny, nx):
    out = [torch.empty(ny, nx, dtype=torch.float64, device="cuda") for _ in range(3)]
    torch.cuda.synchronize()
    lbm.lbm_moments_dev(lat.h, *out)
    lat.sync()
    return [o.cpu().numpy() for o in out]


# 3 x 8 bytes a cell: 64 MiB lie at 2796203 cells; chunks are 2 MiB
@pytest.mark.parametrize("nx,ny", [(2796202, 1), (1, 2796203), (1699, 1647), (2049, 2047), (4096, 1024)])
def test_moments_and_state(nx, ny):
    lat = lattice(nx, ny)
    want = on_device(lat, ny, nx)
    for got, w in zip(lat.moments(), want):
        assert np.array_equal(got, w)
    for _ in range(2):  # again, into pages and pinned memory that are there
        for got, w in zip(lat.moments(), want):
            assert np.array_equal(got, w)
    f = lat.populations()
    assert np.allclose(f.reshape(9, ny, nx).sum(0), want[0], rtol=0, atol=1e-6)
    state = lbm.lbm_save_state(lat.h)
    twin = lattice(nx, ny, seed=1)
    lbm.lbm_load_state(twin.h, state)
    for got, w in zip(twin.moments(), want):
        assert np.array_equal(got, w)
    lat.close()
    twin.close()


@pytest.mark.parametrize("off", [0, 1, 3])
@pytest.mark.parametrize("pinned", [False, True])
@pytest.mark.parametrize("which", ["rho", "rho uy", "ux"])
def test_destinations(off, pinned, which):
    nx, ny = 3001, 3000  # one field alone is above 64 MiB
    lat = lattice(nx, ny)
    want = dict(zip(("rho", "ux", "uy"), on_device(lat, ny, nx)))
    buf = {k: torch.zeros(nx * ny * 8 + 64, dtype=torch.uint8, pin_memory=pinned) for k in which.split()}
    ptr = [ctypes.cast(buf[k].data_ptr() + 8 * off, lbm._DP) if k in buf else None
           for k in ("rho", "ux", "uy")]
    lbm._check(lbm.load().lbm_moments(lat.h, *ptr))
    for k, b in buf.items():
        raw = b.numpy()
        got = raw[8 * off:8 * off + nx * ny * 8].view(np.float64).reshape(ny, nx)
        assert np.array_equal(got, want[k])
        assert not raw[:8 * off].any() and not raw[8 * off + nx * ny * 8:].any()
    lat.close()


def test_three_dimensions_and_two_threads():
    def case(seed, out):
        g = np.random.default_rng(seed)
        shp = (150, 141, 139)
        f = [1.0 + 1e-3 * g.standard_normal(shp)] + [1e-2 * g.standard_normal(shp) for _ in range(3)]
        lat = lbm.Lattice3(shp[2], shp[1], shp[0], rho=f[0], ux=f[1], uy=f[2], uz=f[3], storage="f64",
                           variant="none")
        got = [lat.moments() for _ in range(2)]
        pop = lat.populations()
        # FP64 storage of deviations from the base state: a few roundings
        out[seed] = all(np.allclose(a, b, rtol=0, atol=1e-14) for m in got for a, b in zip(m, f))
        out[seed] &= np.allclose(pop.reshape(15, -1).sum(0), f[0].ravel(), rtol=0, atol=1e-14)
        lat.close()
    out = {}
    threads = [threading.Thread(target=case, args=(s, out)) for s in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert out == {0: True, 1: True}
