"""Replays of captured steps with a running-mean reference, with calls of other
lengths between them: state and mean as single steps give them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_1203_6350_amd import lbm  # noqa: E402


@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("shape,captured,between", [(None, (4, 2), (3, 5)), (None, (10,), (7, 1)),
                                                    ((4, 0), (9, 1), (9, 1)), ((4, 0), (8,), (5, 5))])
@pytest.mark.parametrize("nx,ny", [(96, 80), (2000, 1003)])
def test_replays(nx, ny, shape, captured, between, storage):
    print("case", storage, shape, captured, between, nx, ny, flush=True)
    g = np.random.default_rng(3)
    f = [1.0 + 1e-3 * g.standard_normal((ny, nx)), 0.05 + 1e-3 * g.standard_normal((ny, nx)),
         1e-3 * g.standard_normal((ny, nx))]
    s = torch.cuda.Stream()
    a, r = (lbm.Lattice(nx, ny, rho=f[0], ux=f[1], uy=f[2], storage=storage, variant="II", ux_base=0.05,
                        stream=st) for st in (s, None))
    for lat in (a, r):
        lat.set_sponge_separable(np.full(nx, 0.05), None, "max", (1.0, 0.05, 0.0))
        lat.set_qref_field(*f)
        lat.set_qref_average(0.02)
    r.set_tuning(kernel=0, block=256)
    if shape:
        a.set_tuning(kernel=shape[0], block=128, rows=shape[1])
        a.step(shape[0])  # the second buffer is there before the capture
        r.step(shape[0])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        for n in captured:
            a.step(n)
    for eager in ((), between, (), between):
        for n in eager:
            a.step(n)
            r.step(n)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for n in captured:
            r.step(n)
        assert np.array_equal(a.populations(), r.populations())
        for p, q in zip(a.qref_field(), r.qref_field()):
            assert np.array_equal(p, q)
