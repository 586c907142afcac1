"""Sweeps of plain 16-bit fields on both sides of the rule that chooses their form.

The state rounds once a sweep whatever the form, so the default form, the column form
(FDTD_NT_STORES = 0) and the one that large states take (1) give the same bits, remainders included.
"""

import numpy as np
import pytest

import cavity_inputs as ci

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f16", "bf16"])
@pytest.mark.parametrize("shape", [(128, 64, 374), (126, 60, 300), (65, 64, 90), (192, 101, 186)],
                         ids=lambda s: "x".join(map(str, s)))
def test_every_form_same_bits(shape, storage, monkeypatch):
    import paper_2504_09118_amd as P

    eps = ci.uniform_cell_eps(*shape, seed=4, lo=1.0, hi=4.0)
    mu = ci.uniform_cell_eps(*shape, seed=5, lo=1.0, hi=2.0)
    for ce, ch in ((None, None), (eps, None), (None, mu), (eps, mu)):
        for tb, n in ((3, 6), (2, 5), (4, 7)):
            outs = []
            for form in (None, "0", "1"):
                if form is None:
                    monkeypatch.delenv("FDTD_NT_STORES", raising=False)
                else:
                    monkeypatch.setenv("FDTD_NT_STORES", form)
                with P.Solver(*shape, eps_r=ce, mu_r=ch, storage=storage, tb_steps=tb) as s:
                    s.init_random(12)
                    s.step(n)
                    outs.append(s.get_fields(dtype=np.float32))
            for got in outs[1:]:
                assert all(np.array_equal(a, b) for a, b in zip(got, outs[0])), (tb, n)
