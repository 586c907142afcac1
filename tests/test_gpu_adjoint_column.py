"""Column sweeps of the adjoint against its other forms, at the edges of their windows.

A window is 64 columns by 24 or 32 rows, less a halo of one column or row per step and
side. The gradient, dJ/dE^0 and J have the same bits with the one-cell-per-thread reverse
kernels and with every checkpoint interval (K sets which sweeps of four, two and one step
make up a pass). More than 64 probes take the slab sweeps: J is a sum over probes, so the
J of a list of 65 is the J of its halves to the rounding of a float64 sum, and the gradient,
which is linear in the probe terms, to the FP32 bar of 1e-5.
"""

import numpy as np
import pytest

import cavity_inputs as ci
from tests.test_gpu_adjoint import _pkg, rel

pytestmark = pytest.mark.gpu


def gradient(shape, src, probes, nsteps, k, mu=False):
    nx, ny, nz = shape
    P, A = _pkg()
    eps = ci.uniform_cell_eps(nx, ny, nz, seed=8, lo=1.0, hi=4.0)
    kw = {"mu_r": ci.uniform_cell_eps(nx, ny, nz, seed=9, lo=1.0, hi=2.0)} if mu else {}
    wave = ci.gaussian_pulse(nsteps, center=4.0, width=3.0)
    with P.Solver(nx, ny, nz, eps_r=eps, **kw) as s:
        s.set_fields(ci.random_e(nx, ny, nz, seed=7))
        with A.Adjoint(s, src, wave, probes, nsteps, checkpoint_every=k) as a:
            J = a.forward()
            g, lam = a.backward(lam0=True)
    return J, g, lam


# columns about one and two windows of 64, 60 and 56 own ones; rows about the edges of 24, 28 and 32
CASES = [
    ((7, 5, 3), 9, False), ((60, 20, 5), 8, False), ((61, 28, 6), 7, False), ((64, 32, 9), 10, True),
    ((65, 33, 8), 6, False), ((120, 23, 17), 11, False), ((125, 49, 4), 5, True), ((9, 25, 70), 12, False),
]


@pytest.mark.parametrize("shape,nsteps,mu", CASES, ids=["x".join(map(str, c[0])) for c in CASES])
@pytest.mark.parametrize("nprobes", [0, 1, 40])
def test_column_sweeps_same_bits(shape, nsteps, mu, nprobes, monkeypatch):
    nx, ny, nz = shape
    # a source and a probe in the halo of two windows, the others anywhere
    src = (2, min(nx - 1, 61), min(ny - 1, 21), nz - 1)
    nodes = [(min(nx - 1, 59), min(ny - 1, 27), nz // 2)] + ci.distinct_nodes(3, 39, (1, 1, 0), (nx, ny, nz))
    probes = [(2,) + tuple(p) for p in nodes[:nprobes]]
    J, g, lam = gradient(shape, src, probes, nsteps, 0, mu)
    assert np.isfinite(g).all() and (nprobes == 0 or np.any(g))
    runs = [gradient(shape, src, probes, nsteps, k, mu) for k in (1, 2, 3, 4)]
    monkeypatch.setenv("FDTD_ADJ_FUSED", "0")
    runs.append(gradient(shape, src, probes, nsteps, 0, mu))
    for J2, g2, lam2 in runs:
        assert J2 == J
        assert np.array_equal(g2, g)
        assert all(np.array_equal(a, b) for a, b in zip(lam2, lam))


@pytest.mark.parametrize("shape", [(66, 30, 6), (40, 33, 13)], ids=["66x30x6", "40x33x13"])
def test_slab_sweeps_agree(shape):
    nx, ny, nz = shape
    src, nsteps = (2, nx // 2, ny // 2, nz // 2), 10
    probes = [(2,) + tuple(p) for p in ci.distinct_nodes(4, 65, (1, 1, 0), shape)]
    J, g, lam = gradient(shape, src, probes, nsteps, 0)
    half = [gradient(shape, src, p, nsteps, 0) for p in (probes[:32], probes[32:])]
    assert abs(half[0][0] + half[1][0] - J) <= 65 * nsteps * 2.0**-53 * J
    assert rel(half[0][1] + half[1][1], g) <= 1e-5
    for q in range(3):
        assert rel(half[0][2][q].astype(np.float64) + half[1][2][q], lam[q]) <= 1e-5
