"""The adjoint's forms give the same bits: column sweeps, single steps in slabs, slab sweeps throughout.

More than 64 probes take slab sweeps for every pass of FP32 fields; the state after a forward does not
depend on the probes, so it is the state of a run with few of them, in column sweeps, bit for bit.
FDTD_NT_STORES = 1 makes a small state take the single steps that a large one takes. Sources of each component
on the edges of the windows (64, 60 and 56 columns, 32, 28 and 24 rows).
"""

import numpy as np
import pytest

import cavity_inputs as ci
from tests.test_gpu_adjoint import _pkg

pytestmark = pytest.mark.gpu

S = 0.5 / 3 ** 0.5
SOURCES = [(0, 59, 27, 5), (0, 63, 31, 1), (1, 60, 28, 4), (1, 55, 23, 7), (2, 61, 21, 8), (2, 64, 32, 0), None]


def nodes(shape, count, seed):
    """Interior nodes of every component."""
    out = []
    for q, (i, j, k) in enumerate(ci.distinct_nodes(seed, count, (1, 1, 1), shape)):
        out.append((q % 3, i, j, k))
    return out


def run(shape, src, probes, steps, every, mu=False, backward=True):
    P, A = _pkg()
    eps = ci.uniform_cell_eps(*shape, seed=8, lo=1.0, hi=4.0)
    kw = {"mu_r": ci.uniform_cell_eps(*shape, seed=9, lo=1.0, hi=2.0)} if mu else {}
    wave = ci.gaussian_pulse(steps, center=4.0, width=3.0) if src else None
    with P.Solver(*shape, 1.0, S, eps_r=eps, **kw) as s:
        s.set_fields(ci.random_e(*shape, seed=7))
        with A.Adjoint(s, src, wave, probes, steps, checkpoint_every=every) as a:
            J = a.forward()
            state = s.get_fields(np.float32)
            g, lam = a.backward(lam0=True) if backward else (None, ())
    return J, state, g, lam


def same(a, b):
    return all(np.array_equal(x, y) and np.array_equal(np.signbit(x), np.signbit(y)) for x, y in zip(a, b))


@pytest.mark.parametrize("mu", [False, True])
@pytest.mark.parametrize("src", SOURCES, ids=str)
def test_column_forward_equals_the_slab_forward(src, mu):
    shape, steps = (121, 50, 9), 11
    many = nodes(shape, 65, 3)
    slab = run(shape, src, many, steps, 0, mu, backward=False)[1]
    for every in (0, 1, 3):
        for probes in ([], many[:64]):
            assert same(run(shape, src, probes, steps, every, mu, backward=False)[1], slab), (every, len(probes))


@pytest.mark.parametrize("mu", [False, True])
@pytest.mark.parametrize("nprobes", [0, 5, 40])
def test_single_steps_in_slabs_same_bits(nprobes, mu, monkeypatch):
    shape, steps = (66, 34, 13), 10
    probes = nodes(shape, nprobes, 4)
    for every in (1, 3, 5, 0):
        outs = []
        for nt in ("0", "1"):
            monkeypatch.setenv("FDTD_NT_STORES", nt)
            outs.append(run(shape, (1, 60, 28, 4), probes, steps, every, mu))
        (ja, sa, ga, la), (jb, sb, gb, lb) = outs
        assert ja == jb and same(sa, sb) and np.array_equal(ga, gb) and same(la, lb), every
        assert nprobes == 0 or np.any(ga)


@pytest.mark.parametrize("every", [0, 7])
def test_slab_reverse_equals_the_plain_kernels(every, monkeypatch):
    """FP32 with one Ch and more probes than any sweep carries: slab sweeps and probe kernels, both passes."""
    shape, steps = (150, 37, 41), 20
    probes = nodes(shape, 70, 5)
    outs = []
    for fused in ("1", "0"):
        monkeypatch.setenv("FDTD_ADJ_FUSED", fused)
        outs.append(run(shape, (1, 70, 18, 20), probes + probes[:3], steps, every))
    (ja, sa, ga, la), (jb, sb, gb, lb) = outs
    assert ja == jb and same(sa, sb) and np.array_equal(ga, gb) and same(la, lb)
    assert np.abs(ga).max() > 0
