"""Single steps of the temporal schedule, which a cavity that fills the chip takes in slabs: same bits.

Cavities on both sides of the rule, step by step, as remainders and as a schedule of their own, with
scalar and per-cell coefficients; a chosen z-split keeps the column form.
"""

import numpy as np
import pytest

import cavity_inputs as ci

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("medium", ["vacuum", "eps", "mu", "both"])
@pytest.mark.parametrize("shape", [(128, 128, 128), (127, 66, 140), (129, 65, 139), (96, 96, 96), (250, 41, 63)],
                         ids=lambda s: "x".join(map(str, s)))
def test_single_steps_same_bits(shape, medium):
    import paper_2504_09118_amd as P

    eps = ci.uniform_cell_eps(*shape, seed=4, lo=1.0, hi=4.0) if medium in ("eps", "both") else None
    mu = ci.uniform_cell_eps(*shape, seed=5, lo=1.0, hi=2.0) if medium in ("mu", "both") else None
    e, h = ci.random_e(*shape, seed=63, dtype=np.float32), ci.random_h(*shape, seed=64, dtype=np.float32)
    with P.Solver(*shape, eps_r=eps, mu_r=mu, kernel="plain") as s:
        s.set_fields(e, h)
        s.step(7)
        want = s.get_fields(dtype=np.float32)

    def same(s):
        got = s.get_fields(dtype=np.float32)
        return s.steps_done == 7 and all(
            np.array_equal(a, b) and np.array_equal(np.signbit(a), np.signbit(b)) for a, b in zip(got, want))

    with P.Solver(*shape, eps_r=eps, mu_r=mu) as s:
        s.set_fields(e, h)
        for n in (1, 1, s.schedule["tb_steps"] + 1, 4 - s.schedule["tb_steps"]):
            s.step(n)
        assert same(s)
    with P.Solver(*shape, eps_r=eps, mu_r=mu, tb_steps=1) as s:
        s.set_fields(e, h)
        s.step(3)
        s.set_schedule("temporal", 1, 0, 5)
        s.step(2)
        s.set_schedule("temporal", 2, 1, 3)
        s.step(1)
        s.set_schedule("temporal", 2, 0, 4)
        s.step(1)
        assert same(s)
