"""The level-wise QR sweeps of the Von Neumann kernel: lanes that converge at
different speeds, spectra that are defective or zero, and a lane that never
converges beside lanes that do."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1203_6350_amd import lbm, workloads as wl  # noqa: E402

SETS = {"mrt flow": dict(s=wl.S_MRT_DEFAULT, chi=0.2, qref=(1, 0.1, 0.03), variant="II"),
        "relaxed at once": dict(s=(1.0,) * 9, chi=0.0, qref=(1, 0.0, 0.0), variant="II"),
        "undamped": dict(s=(1.9,) * 9, chi=0.0, qref=(1, 0.0, 0.0), variant="II"),
        "large": dict(s=(1.99,) * 9, chi=50.0, qref=(1, 0.2, 0.1), variant="I"),
        "type III": dict(s=wl.S_MRT_DEFAULT, chi=0.05, qref=(1, 0.15, 0.0), variant="III")}


def waves():
    """Axis and diagonal waves, zero, and random ones, shuffled over the lanes."""
    g = np.random.default_rng(7)
    k = np.linspace(-np.pi, np.pi, 33)
    kx = np.concatenate([k, k, 0 * k, g.uniform(-np.pi, np.pi, 94)])
    ky = np.concatenate([0 * k, k, k, g.uniform(-np.pi, np.pi, 94)])
    p = g.permutation(len(kx))
    return kx[p], ky[p]


@pytest.mark.parametrize("name", list(SETS))
def test_power_sums(name):
    """sum lambda^p = trace G^p, p = 1..9, which hold to rounding also where the
    eigenvalues themselves are ill conditioned: the solver's lambda are those
    of G + E with ||E|| <= 100 eps ||G|| (some 30 sweeps of 8 rotations on a
    matrix of order 9), and 9 p ||G||^(p-1) ||E|| bounds what E moves the trace by."""
    kx, ky = waves()
    lam, G = lbm.vn_amplification(SETS[name], kx, ky, want_G=True)
    assert np.isfinite(lam).all()
    norm = np.linalg.norm(G, axis=(1, 2))
    P = np.eye(9, dtype=complex)[None]
    for p in range(1, 10):
        P = P @ G
        err = abs((lam ** p).sum(1) - np.trace(P, axis1=1, axis2=2))
        assert (err <= 9 * p * 100 * 2.3e-16 * np.maximum(norm, 1e-300) ** p).all(), (name, p)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("at", [0, 31, 63, 64, 100])
def test_a_lane_without_a_spectrum_leaves_the_others(bad, at):
    kx, ky = waves()
    want = lbm.vn_amplification(SETS["mrt flow"], kx, ky)
    kb = kx.copy()
    kb[at] = bad
    got = lbm.vn_amplification(SETS["mrt flow"], kb, ky)
    keep = np.arange(len(kx)) != at
    assert np.isnan(got[at]).all()
    assert np.array_equal(got[keep], want[keep])
