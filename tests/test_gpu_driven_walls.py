"""The adjoint's forward on states that are not finite: the walls stay as they are.

A wall-tangential E node never changes, whatever the field beside it, so the state after a driven
forward is the plain schedule's, NaN for NaN and bit for bit elsewhere. Seeds beside the walls and
the windows' edges (64 columns; 16, 24 and 32 rows), sweeps of 4, 2 and 1 steps.
"""

import numpy as np
import pytest

import cavity_inputs as ci
from tests.test_gpu_adjoint import _pkg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [np.nan, np.inf, -3e38])
@pytest.mark.parametrize("shape", [(20, 18, 16), (66, 34, 9), (130, 20, 12)], ids=lambda s: "x".join(map(str, s)))
def test_walls_of_a_state_that_is_not_finite(shape, value):
    P, A = _pkg()
    nx, ny, nz = shape
    eps = ci.uniform_cell_eps(nx, ny, nz, seed=8, lo=1.0, hi=4.0)
    mu = ci.uniform_cell_eps(nx, ny, nz, seed=9, lo=1.0, hi=2.0)
    nsteps = 11
    for mu_r in (None, mu):
        for k, j, i in ((nz // 2, ny // 2, nx - 2), (1, 1, 1), (nz - 2, ny - 2, nx // 2)):
            e = [a.copy() for a in ci.random_e(nx, ny, nz, seed=9, dtype=np.float32)]
            e[1][k, j, i] = value
            with P.Solver(nx, ny, nz, eps_r=eps, mu_r=mu_r, kernel="plain") as s:
                s.set_fields(e)
                s.step(nsteps)
                want = s.get_fields(np.float32)
            for every in (0, 3):
                with P.Solver(nx, ny, nz, eps_r=eps, mu_r=mu_r) as s:
                    s.set_fields(e)
                    with A.Adjoint(s, None, None, [(2, nx // 2, ny // 2, nz // 2)], nsteps,
                                   checkpoint_every=every) as a:
                        a.forward()
                        got = s.get_fields(np.float32)
                for x, y in zip(got, want):
                    assert np.array_equal(x, y, equal_nan=True)
