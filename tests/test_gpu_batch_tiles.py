"""Small batches on square tiles: bit for bit each member stepped alone by
one-step launches, with members of every variant and sponge form, narrower
than a region and uneven, uneven step counts in a tick, ticks of every parity, and
a changing member list."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_1203_6350_amd import lbm, workloads as wl  # noqa: E402

SIZES = [(64, 64), (131, 77), (5, 40), (1, 1), (96, 33), (200, 150)]
VARIANTS = ["none", "I", "II", "III", "visc", "II"]
SPONGES = ["max", "sum", "field", "max", "max", None]


def member(i, storage, one, conserved=0.0):
    nx, ny = SIZES[i % len(SIZES)]
    g = np.random.default_rng(40 + i)
    f = [1.0 + 1e-3 * g.standard_normal((ny, nx))] + [0.05 + 1e-3 * g.standard_normal((ny, nx))
                                                      for _ in range(2)]
    s = (conserved,) * 3 + tuple(wl.S_MRT_DEFAULT[3:])
    var = VARIANTS[i % len(VARIANTS)]
    lat = lbm.Lattice(nx, ny, s=s, storage=storage, variant=var, ux_base=0.05, uy_base=0.05,
                      rho=f[0], ux=f[1], uy=f[2])
    top = 0.5 if var == "visc" else 0.05 if var == "I" else 0.3
    cx, cy = (top * g.random(n) * (g.random(n) < 0.5) for n in (nx, ny))
    how = SPONGES[i % len(SPONGES)]
    if how == "field" and var != "none":
        lat.set_sponge(np.maximum(cx[None, :], cy[:, None]), (1.001, 0.06, 0.04))
    elif how and var != "none":
        lat.set_sponge_separable(cx, cy, "max" if var == "visc" else how, (1.001, 0.06, 0.04))
    if one:
        lbm.lbm_set_tuning(lat.h, 0, 256)
    return lat


def same(a, b):
    return np.array_equal(a.populations(), b.populations(), equal_nan=True)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("ticks", [[2], [3, 1, 2], [14, 15], [47, 30]])
def test_uniform_ticks(storage, ticks):
    lats = [member(i, storage, False) for i in range(6)]
    ref = [member(i, storage, True) for i in range(6)]
    b = lbm.Batch(lats)
    for n in ticks:
        b.step(n)
    b.sync()
    for i, (a, r) in enumerate(zip(lats, ref)):
        r.step(sum(ticks))
        assert same(a, r), i
    b.close()


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
def test_uneven_steps_and_members(storage):
    lats = [member(i, storage, False) for i in range(9)]
    ref = [member(i, storage, True) for i in range(9)]
    done = [0] * 9
    b = lbm.Batch(lats[:4])
    plan = [(range(4), [7, 0, 12, 5]), (range(2, 9), [1, 2, 3, 9, 17, 0, 16]),
            (range(9), [20, 19, 18, 1, 2, 3, 0, 11, 13]), (range(3), [2, 1, 0])]
    for who, steps in plan:
        b.set_members([lats[i] for i in who])
        b.tick(max(steps), steps)
        b.sync()
        for i, s in zip(who, steps):
            done[i] += s
    for i in range(9):
        ref[i].step(done[i])
        assert same(lats[i], ref[i]), i
    b.close()


def test_members_of_the_general_form():
    """Conserved rates that are not 0: one-step launches, as before."""
    lats = [member(i, "f32", False, 0.5 if i == 1 else 0.0) for i in range(3)]
    ref = [member(i, "f32", True, 0.5 if i == 1 else 0.0) for i in range(3)]
    b = lbm.Batch(lats)
    b.step(11)
    b.sync()
    for a, r in zip(lats, ref):
        r.step(11)
        assert same(a, r)
    b.close()


def test_a_tick_in_which_no_member_steps():
    lats = [member(i, "f32", False) for i in range(6)]
    ref = [member(i, "f32", True) for i in range(6)]
    b = lbm.Batch(lats)
    for n in (14, 0, 14, 0):
        b.tick(14, [n] * 6)
    b.sync()
    for a, r in zip(lats, ref):
        r.step(28)
        assert same(a, r)
    b.close()
