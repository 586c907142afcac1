"""Column sweeps in workgroups of 8 waves (small FP32 cavities): 16-row windows, at their edges.

Every FP32 schedule gives the same bits, so the plain one-cell-per-thread kernel is the oracle.
ny about one window (16 rows), and two and three at 8 to 14 own rows; nx about one and two
windows; nz below, at and above one plane per tile; sweeps of 1 to 4 steps and their remainder;
scalar and per-cell coefficients; z-splits that make it one workgroup a CU, two and more.
"""

import numpy as np
import pytest

import cavity_inputs as ci

pytestmark = pytest.mark.gpu

CASES = [(5, 16, 3), (64, 17, 7), (65, 24, 9), (12, 25, 33), (60, 30, 16), (57, 31, 5), (121, 15, 20), (30, 41, 64),
         (70, 70, 2), (2, 2, 2)]


@pytest.mark.parametrize("medium", ["vacuum", "eps", "mu", "both"])
@pytest.mark.parametrize("shape", CASES, ids=lambda s: "x".join(map(str, s)))
def test_narrow_windows_same_bits(shape, medium):
    import paper_2504_09118_amd as P

    nx, ny, nz = shape
    eps = ci.uniform_cell_eps(nx, ny, nz, seed=4, lo=1.0, hi=4.0) if medium in ("eps", "both") else None
    mu = ci.uniform_cell_eps(nx, ny, nz, seed=5, lo=1.0, hi=2.0) if medium in ("mu", "both") else None
    for tb in (1, 2, 3, 4):
        n = 2 * tb + (tb - 1)
        with P.Solver(nx, ny, nz, eps_r=eps, mu_r=mu, kernel="plain") as s:
            s.init_random(11)
            s.step(n)
            want = s.get_fields(dtype=np.float32)
        with P.Solver(nx, ny, nz, eps_r=eps, mu_r=mu, tb_steps=tb) as s:
            own = s.schedule["zchunks"]
            for zc in sorted({own, 1, nz}):
                if zc != own:
                    s.set_schedule("temporal", tb, 0, zc)
                s.init_random(11)
                s.step(n)
                got = s.get_fields(dtype=np.float32)
                for name, a, b in zip(("Ex", "Ey", "Ez", "Hx", "Hy", "Hz"), got, want):
                    assert np.array_equal(a, b), f"tb {tb} zchunks {zc}: {name}"


@pytest.mark.parametrize("storage", ["f16", "bf16", "f16c", "bf16c"])
@pytest.mark.parametrize("shape", [(64, 17, 7), (12, 25, 33), (121, 15, 20), (2, 2, 2)],
                         ids=lambda s: "x".join(map(str, s)))
def test_narrow_windows_16bit_equal_the_streaming_form(shape, storage, monkeypatch):
    """16-bit storage rounds once a sweep, as the form that large states take (FDTD_NT_STORES = 1): equal."""
    import paper_2504_09118_amd as P

    nx, ny, nz = shape
    eps = ci.uniform_cell_eps(nx, ny, nz, seed=4, lo=1.0, hi=4.0)
    mu = ci.uniform_cell_eps(nx, ny, nz, seed=5, lo=1.0, hi=2.0)
    for e, m in ((None, None), (eps, None), (eps, mu)):
        for tb in (1, 2, 3, 4):
            outs = []
            for pol, splits in (("1", [None]), ("0", [None, 1, nz])):
                monkeypatch.setenv("FDTD_NT_STORES", pol)
                with P.Solver(nx, ny, nz, eps_r=e, mu_r=m, storage=storage, tb_steps=tb) as s:
                    for zc in splits:
                        if zc:
                            s.set_schedule("temporal", tb, 0, zc)
                        s.init_random(12)
                        s.step(2 * tb + 1)
                        outs.append(s.get_fields(dtype=np.float32))
            for got in outs[1:]:
                assert all(np.array_equal(a, b) for a, b in zip(got, outs[0])), f"tb {tb}"
