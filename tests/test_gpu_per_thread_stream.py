"""Handles on hipStreamPerThread: large read-outs, which elsewhere several threads
copy, are in order behind the steps and kernels that the calling thread enqueued."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_1203_6350_amd import lbm  # noqa: E402

PER_THREAD = 2  # hipStreamPerThread


def test_large_readouts():
    nx, ny, n = 2049, 2047, 40
    g = np.random.default_rng(0)
    rho = 1.0 + 1e-3 * g.standard_normal((ny, nx))
    lats = [lbm.Lattice(nx, ny, rho=rho, storage="f64", stream=s) for s in (PER_THREAD, None)]
    for _ in range(3):
        for lat in lats:
            lat.step(n)
        for a, b in zip(lats[0].moments(), lats[1].moments()):
            assert np.array_equal(a, b)
        lats[0].step(n)
        lats[1].step(n)
        assert np.array_equal(lats[0].populations(), lats[1].populations())
    cubes = [lbm.Lattice3(151, 150, 149, rho=1.0 + 1e-3 * g.standard_normal((149, 150, 151)),
                          storage="f64", stream=PER_THREAD)]
    cubes.append(lbm.Lattice3(151, 150, 149, storage="f64"))
    cubes[1].set_populations(cubes[0].populations())
    for _ in range(3):
        for c in cubes:
            c.step(n)
        # (restoring from populations costs a rounding; the same state would be equal)
        for a, b in zip(cubes[0].moments(), cubes[1].moments()):
            assert np.allclose(a, b, rtol=0, atol=1e-12)
