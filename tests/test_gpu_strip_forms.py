"""Four steps per launch of a single lattice in strips of a set height (fitted
heights mean square tiles on small lattices): every variant and sponge form, the
collision's general form against single steps and the oracle, and large lattices
of the general form as created."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import oracle  # noqa: E402
from paper_1203_6350_amd import lbm, workloads as wl  # noqa: E402

RATES = {"bgk": dict(s=(1.7,) * 9), "mixed": dict(s=(0.0, 0.6, 0.0, 1.1, 1.2, 1.3, 1.4, 1.5, 1.6)),
         "n != m": dict(s=(0.0, 0.0, 0.0, 1.1, 1.2, 1.3, 1.4, 1.5, 1.6), shift_n=0.3, shift_m=0.8)}
Q = (1.0005, 0.045, -0.003)


def fields(nx, ny, seed, variant):
    g = np.random.default_rng(seed)
    f = [1.0 + 1e-3 * g.standard_normal((ny, nx)), 0.04 + 1e-3 * g.standard_normal((ny, nx)),
         1e-3 * g.standard_normal((ny, nx))]
    top = {"I": 0.05, "visc": 0.5}.get(variant, 0.3)
    cx, cy = (top * g.random(n) * (g.random(n) < 0.4) for n in (nx, ny))
    return f, cx, cy


def stepped(f, cx, cy, form, steps, storage, variant, tuning, **kw):
    ny, nx = f[0].shape
    lat = lbm.Lattice(nx, ny, rho=f[0], ux=f[1], uy=f[2], storage=storage, variant=variant, ux_base=0.04,
                      f16_scale=1e-3, **kw)
    if form == "field":
        lat.set_sponge(np.maximum(cx[None, :], cy[:, None]), Q)
    elif form == "zero":
        lat.set_sponge(None, Q)
    else:
        lat.set_sponge_separable(cx, cy, form, Q)
    if tuning:
        lat.set_tuning(**tuning)
    lat.step(steps)
    return lat


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("variant", ["none", "I", "II", "III", "visc"])
def test_variants_and_sponge_forms(storage, variant):
    f, cx, cy = fields(133, 29, 3, variant)
    for form in ("zero", "field", "max", "sum"):
        if variant == "visc" and form == "sum":
            continue  # the ramp combines by max
        print("case", storage, variant, form, flush=True)
        want = stepped(f, cx, cy, form, 9, storage, variant, dict(kernel=0, block=64)).save_state()
        for block in (64, 128, 256):
            got = stepped(f, cx, cy, form, 9, storage, variant, dict(kernel=4, block=block, rows=5))
            assert np.array_equal(got.save_state(), want)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("rates", list(RATES))
@pytest.mark.parametrize("variant", ["I", "II", "III"])
def test_general_form(storage, rates, variant):
    """Against single steps bit for bit, and in FP64 the oracle to 1e-12 of the
    populations, as for the other kernels (ten steps of some 120 roundings each)."""
    f, cx, cy = fields(97, 23, 13, variant)
    kw = RATES[rates]
    print("case", storage, rates, variant, flush=True)
    want = stepped(f, cx, cy, "field", 10, storage, variant, dict(kernel=0, block=64), **kw)
    got = stepped(f, cx, cy, "field", 10, storage, variant, dict(kernel=4, block=64, rows=5), **kw)
    assert np.array_equal(got.save_state(), want.save_state())
    if storage == "f64":
        ref = oracle.step(oracle.feq_field(*f), 10, s=kw["s"], chi=np.maximum(cx[None, :], cy[:, None]), qref=Q,
                          variant=variant, n=kw.get("shift_n", 0.5), m=kw.get("shift_m", 0.5))
        pops = got.populations()
        assert np.abs(pops - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("rates", ["bgk", "n != m"])
def test_large_lattices_of_the_general_form_as_created(storage, rates):
    f, cx, cy = fields(1003, 1009, 17, "II")
    for form in ("max", "field"):
        for steps in (4, 7, 11):
            print("case", storage, rates, form, steps, flush=True)
            a = stepped(f, cx, cy, form, steps, storage, "II", None, **RATES[rates])
            b = stepped(f, cx, cy, form, steps, storage, "II", dict(kernel=0, block=256), **RATES[rates])
            assert np.array_equal(a.save_state(), b.save_state())
