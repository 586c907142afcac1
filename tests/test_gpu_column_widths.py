"""16-bit column sweeps with both coefficient arrays: full workgroups of 16, 12 and 8 waves.

The cavities are large enough for the full width at each number of steps (and, at 8 waves, for more
tiles than CUs); a sweep rounds once, so the form that large states take gives the same bits.
"""

import numpy as np
import pytest

import cavity_inputs as ci

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f16", "bf16", "f16c", "bf16c"])
@pytest.mark.parametrize("shape", [(130, 120, 40), (121, 57, 66), (65, 140, 33)], ids=lambda s: "x".join(map(str, s)))
def test_full_workgroups_equal_the_streaming_form(shape, storage, monkeypatch):
    import paper_2504_09118_amd as P

    eps = ci.uniform_cell_eps(*shape, seed=4, lo=1.0, hi=4.0)
    mu = ci.uniform_cell_eps(*shape, seed=5, lo=1.0, hi=2.0)
    for tb in (1, 2, 3, 4):
        outs = []
        for pol, splits in (("1", [None]), ("0", [None, 1, 7, shape[2]])):
            monkeypatch.setenv("FDTD_NT_STORES", pol)
            with P.Solver(*shape, eps_r=eps, mu_r=mu, storage=storage, tb_steps=tb) as s:
                for zc in splits:
                    if zc:
                        s.set_schedule("temporal", tb, 0, zc)
                    s.init_random(12)
                    s.step(2 * tb + 1)
                    outs.append(s.get_fields(dtype=np.float32))
        for got in outs[1:]:
            assert all(np.array_equal(a, b) for a, b in zip(got, outs[0])), f"tb {tb}"
