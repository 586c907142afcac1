"""z-splits of the temporal schedule: what the search tries, and what a remainder sweep takes.

The default split of a sweep depends on its steps (the windows differ), so the search tries each one's own
beside the powers of two; every split gives the same bits.
"""

import numpy as np
import pytest

import cavity_inputs as ci

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(64, 64, 64), (30, 41, 50)], ids=lambda s: "x".join(map(str, s)))
def test_the_search_tries_the_default_split_of_every_sweep_length(shape):
    import paper_2504_09118_amd as P

    eps = ci.uniform_cell_eps(*shape, seed=4, lo=1.0, hi=4.0)
    with P.Solver(*shape, eps_r=eps) as s:
        s.init_random(1)
        _, tried = s.autotune(trial_steps=2)
    for tb in (1, 2, 3, 4):
        with P.Solver(*shape, eps_r=eps, tb_steps=tb) as s:
            own = s.schedule["zchunks"]
        assert any(t["kernel"] == "temporal" and t["tb_steps"] == tb and t["variant"] == 0 and t["zchunks"] == own
                   for t in tried), (tb, own)


@pytest.mark.parametrize("nt", ["0", "1"])
@pytest.mark.parametrize("fixed", [None, "3"])
def test_remainder_sweeps_after_a_schedule_same_bits(nt, fixed, monkeypatch):
    import paper_2504_09118_amd as P

    shape = (70, 40, 37)
    monkeypatch.setenv("FDTD_NT_STORES", nt)
    if fixed:
        monkeypatch.setenv("FDTD_TZCHUNKS", fixed)
    eps = ci.uniform_cell_eps(*shape, seed=4, lo=1.0, hi=4.0)
    with P.Solver(*shape, eps_r=eps, kernel="plain") as s:
        s.init_random(2)
        s.step(13)
        want = s.get_fields(dtype=np.float32)
    with P.Solver(*shape, eps_r=eps) as s:
        for tb, variant, zc in ((4, 0, None), (4, 0, 1), (3, 0, 37), (3, 1, 2), (2, 0, 5), (4, 0, 2)):
            s.set_schedule("temporal", tb, variant, zc or s.schedule["zchunks"])
            s.init_random(2)
            for n in (tb, 1, tb + 1, 13 - 2 * tb - 2):
                s.step(n)
            for a, b in zip(s.get_fields(dtype=np.float32), want):
                assert np.array_equal(a, b), (tb, variant, zc)
