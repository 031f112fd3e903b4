"""The tile kernel (several steps per launch on regions held in LDS) and the
rule that takes it: bit for bit the one-cell kernel's results, at the sizes
where tiles, halos and the periodic wrap can go wrong, and the same detector
trips, buffers and captured replays as one-step launches."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_1203_6350_amd import lbm, workloads as wl  # noqa: E402


def say(*a):
    print(*a, flush=True)


def noisy(nx, ny, seed, u0=0.1):
    g = np.random.default_rng(seed)
    return (1.0 + 1e-3 * g.standard_normal((ny, nx)), u0 + 1e-3 * g.standard_normal((ny, nx)),
            1e-3 * g.standard_normal((ny, nx)))


def make(nx, ny, storage, variant, sponge, seed=0, one_step=False, **kw):
    rho, ux, uy = noisy(nx, ny, seed)
    lat = lbm.Lattice(nx, ny, rho=rho, ux=ux, uy=uy, storage=storage, variant=variant,
                      ux_base=0.1, **kw)
    g = np.random.default_rng(seed + 1)
    top = 1.0 if variant == "visc" else 0.3
    cx, cy = (top * g.random(n) * (g.random(n) < 0.4) for n in (nx, ny))
    q = (1.001, 0.11, 0.002)
    if sponge == "field":
        lat.set_sponge(np.maximum(cx[None, :], cy[:, None]), q)
    elif sponge != "zero":
        if variant == "visc":
            sponge = "max"
        lat.set_sponge_separable(cx, cy, sponge, q)
    if one_step:
        lat.set_tuning(kernel=0, block=256)
    return lat


SIZES = [(1, 1), (2, 3), (5, 40), (7, 7), (23, 25), (24, 24), (33, 31), (48, 47), (64, 96),
         (129, 65), (250, 131)]


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("size", SIZES)
def test_tiles_equal_the_one_cell_kernel(size, storage):
    """Every variant and sponge form on a small lattice as created (tiles) and
    with the one-cell kernel set: populations equal bit for bit after calls of
    every length up to two launches and over."""
    nx, ny = size
    case = 0
    for variant in ("none", "I", "II", "III", "visc"):
        for sponge in ("zero", "field", "max", "sum"):
            for steps in ((2, 3, 4), (5, 6, 9), (13, 14, 15), (29, 40))[case % 4]:
                say("case", size, storage, variant, sponge, steps)
                a = make(nx, ny, storage, variant, sponge, seed=case)
                b = make(nx, ny, storage, variant, sponge, seed=case, one_step=True)
                a.step(steps)
                b.step(steps)
                assert np.array_equal(a.populations(), b.populations(), equal_nan=True)  # Type I may overflow
                a.close()
                b.close()
            case += 1


@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_general_parameters(storage):
    """Conserved rates other than 0 and n != m (the collision's general form)."""
    kw = dict(s=(1.2, 0.3, 0.4, 1.7, 1.6, 1.5, 1.4, 1.9, 1.8), shift_n=0.5, shift_m=0.3)
    for variant in ("I", "II", "III", "visc"):
        say("case", storage, variant)
        a = make(41, 29, storage, variant, "max", seed=3, **kw)
        b = make(41, 29, storage, variant, "max", seed=3, one_step=True, **kw)
        a.step(23)
        b.step(23)
        assert np.array_equal(a.populations(), b.populations(), equal_nan=True)  # Type I may overflow


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("alpha", [0.0, 0.05])
@pytest.mark.parametrize("general", [False, True])
def test_reference_fields(storage, alpha, general):
    """Per-cell references, fixed and running, in every variant: state and field."""
    kw = dict(shift_n=0.5, shift_m=0.25) if general else {}
    for k, variant in enumerate(("none", "I", "II", "III", "visc")):
        for steps in (3, 14, 31):
            say("case", storage, alpha, general, variant, steps)
            lats = [make(37, 58, storage, variant, "max", seed=k, one_step=one, **kw)
                    for one in (False, True)]
            g = np.random.default_rng(k)
            f = [1.0 + 1e-3 * g.random((58, 37)), 0.1 + 1e-3 * g.random((58, 37)),
                 1e-3 * g.random((58, 37))]
            for lat in lats:
                lat.set_qref_field(*f)
                lat.set_qref_average(alpha)
                lat.step(steps)
            assert np.array_equal(lats[0].populations(), lats[1].populations(), equal_nan=True)
            for p, q in zip(lats[0].qref_field(), lats[1].qref_field()):
                assert np.array_equal(p, q, equal_nan=True)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("size", [(3, 1), (4, 7), (9, 30), (25, 24), (47, 16), (64, 33), (201, 50)])
def test_channel(size, storage):
    """A line source with and without outflow: one call against single steps
    (a call of one step runs the one-cell kernel)."""
    nx, ny = size
    for outflow in (False, True):
        for variant, steps in (("II", 30), ("visc", 13), ("none", 7), ("I", 14), ("III", 2)):
            say("case", size, storage, outflow, variant, steps)
            pair = [make(nx, ny, storage, variant, "max", seed=5) for _ in range(2)]
            for lat in pair:
                lat.set_line_source((1.0, 1e-3, 0.013, 0.4, 0.1, 0.01), outflow)
            pair[0].step(steps)
            for _ in range(steps):
                pair[1].step(1)
            assert np.array_equal(pair[0].populations(), pair[1].populations(), equal_nan=True)


@pytest.mark.parametrize("size", [(64, 64), (700, 500), (513, 200)])
def test_detector_trips_at_the_same_step(size):
    """An unstable Type I layer trips at the step at which one-step launches
    see it, also where the period does not divide the steps per launch."""
    nx, ny = size
    for every in (1, 7, 50):
        got = []
        for one in (False, True):
            say("case", size, every, one)
            lat = make(nx, ny, "f32", "I", "zero", seed=9, one_step=one)
            prof = wl.quadratic_ramp_1d(nx, 12, 0.8)
            lat.set_sponge_separable(prof, None, "max", (1.0, 0.1, 0.0))
            lat.set_detector(every, 0.05)
            for n in (33, 200, 400):
                lat.step(n)
            got.append(lat.detector_status())
        assert got[0] == got[1]


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("n", [2, 7, 10, 64])
def test_current_buffer_and_captured_replays(storage, n):
    """The buffer that is current after a call is the one that n one-step
    launches leave current, so a captured even number of steps replays."""
    nx, ny = 96, 80
    cfg = lbm.make_config(nx, ny, storage=storage, ux_base=0.1)
    each = (lbm.lbm_required_bytes(cfg) // 2 + 255) // 256 * 256
    bufs = [torch.zeros(each, dtype=torch.uint8, device="cuda") for _ in range(2)]
    rho, ux, uy = noisy(nx, ny, 2)
    h = lbm.lbm_create_ext(cfg, bufs[0], bufs[1], rho, ux, uy)
    ref = lbm.Lattice(nx, ny, rho=rho, ux=ux, uy=uy, storage=storage, ux_base=0.1)
    ref.set_tuning(kernel=0, block=256)
    lbm.lbm_step(h, n)
    lbm.lbm_sync(h)
    ref.step(n)
    state = ref.save_state()[:-8]
    assert np.array_equal(bufs[n & 1].cpu().numpy()[:state.size], state)
    lbm.lbm_destroy(h)
    if n & 1:
        return
    s = torch.cuda.Stream()
    cap = lbm.Lattice(nx, ny, rho=rho, ux=ux, uy=uy, storage=storage, ux_base=0.1, stream=s)
    ref = lbm.Lattice(nx, ny, rho=rho, ux=ux, uy=uy, storage=storage, ux_base=0.1)
    ref.set_tuning(kernel=0, block=256)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        cap.step(n)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        ref.step(n)
        assert np.array_equal(cap.populations(), ref.populations())


@pytest.mark.parametrize("variant", ["I", "II", "III", "visc"])
@pytest.mark.parametrize("value", [1e18, 3e19, 1e25, 3e38, float("inf"), float("nan")])
def test_overflow_outside_the_layer(variant, value):
    """Values at and past the end of the range, in cells clear of the layer:
    tiles and FP16 strips leave the damping out there and still reach the
    one-cell kernel's values (NaN = NaN, +0 = -0)."""
    nx, ny = 150, 60
    for storage in ("f64", "f32", "f16"):
        base = make(nx, ny, storage, variant, "zero", seed=4, one_step=True)
        prof = wl.quadratic_ramp_1d(nx, 10, 0.3)
        state = base.save_state()
        dt = {"f64": np.float64, "f32": np.float32, "f16": np.float16}[storage]
        planes = state[:-8].view(dt)
        ps = planes.size // 9
        g = np.random.default_rng(8)
        with np.errstate(over="ignore"):
            for k in range(40):
                i, y, x = int(g.integers(9)), int(g.integers(ny)), int(g.integers(40, nx - 40))
                planes[i * ps + y * nx + x] = dt(value if k % 2 else -value)
        for steps in (1, 2, 4):
            out = []
            for tuning in (dict(kernel=0, block=256), None, dict(kernel=4, block=128, rows=8)):
                say("case", variant, value, storage, steps, tuning)
                lat = make(nx, ny, storage, variant, "zero", seed=4)
                lat.set_sponge_separable(prof, None, "max", (1.0, 0.1, 0.0))
                lat.load_state(state)
                if tuning:
                    lat.set_tuning(**tuning)
                lat.step(steps)
                out.append(lat.save_state()[:-8].view(dt).copy())
            for o in out[1:]:
                assert np.array_equal(out[0], o, equal_nan=True)
