"""Long thin cavities, whose planes share a workgroup: layout, seeded state, coefficients, diagnostics.

Planes of 9 to 342 nodes about the powers of two at which the workgroup's shape changes, numbers of
planes that its planes do not divide, and cavities just too short for it (511 cells). Copies are exact; the sums differ from the oracle's by the order of
their N terms only: 8 N 2^-53.
"""

import numpy as np
import pytest

import cavity_inputs as ci
import oracle
from tests.test_gpu_layout import close_walls

pytestmark = pytest.mark.gpu

DIMS = [(2, 2, 700), (3, 3, 565), (4, 2, 627), (7, 7, 2001), (7, 8, 530), (10, 11, 563), (15, 15, 550), (16, 15, 631),
        (17, 16, 512), (18, 17, 517), (17, 16, 511), (2, 2, 511)]


@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("dims", DIMS, ids=lambda s: "x".join(map(str, s)))
def test_thin_planes(dims, storage):
    import torch

    import paper_2504_09118_amd as P

    dt, n = 0.5 / 3 ** 0.5, 6 * (dims[0] + 1) * (dims[1] + 1) * (dims[2] + 1)
    real = np.float32 if storage == "f32" else np.float64
    e, h = ci.random_e(*dims, seed=71, dtype=np.float32), ci.random_h(*dims, seed=72, dtype=np.float32)
    eps = ci.uniform_cell_eps(*dims, seed=74, lo=1.0, hi=4.0)
    mu = ci.uniform_cell_eps(*dims, seed=75, lo=1.0, hi=1.5)
    want = close_walls([a.copy() for a in e]) + list(h)
    ce = oracle.round_to(oracle.coef_e(*dims, 1.0, dt, eps), real)
    ch = oracle.round_to(oracle.coef_h(*dims, 1.0, dt, mu), real)
    with P.Solver(*dims, 1.0, dt, eps_r=eps, mu_r=mu, storage=storage) as s:
        assert all(np.array_equal(a, b) for a, b in zip(s.get_coefs(np.float64), list(ce) + list(ch)))
        s.set_fields(e, h)
        for dtype in (torch.float32, torch.float64):
            out = [torch.full(sh, np.nan, dtype=dtype, device="cuda") for sh in s.shapes]
            torch.cuda.synchronize()
            s.get_fields_device(out)
            s.sync()
            assert all(np.array_equal(a.cpu().numpy(), b) for a, b in zip(out, want))
        s.set_fields_device(out)
        d, state = s.diag(), s.get_fields(np.float64)
        assert all(np.array_equal(a, b) for a, b in zip(state, want))
        w, se, sh = oracle.energy(state, ce, ch)
        for got, ref in ((d["energy"], w), (d["sum_e2"], se), (d["sum_h2"], sh)):
            assert abs(got - ref) <= 8 * n * 2.0**-53 * (se / ce[0].max() + sh / ch[0].max() + ref)
        assert d["nonfinite"] == 0 and d["max_e_tan"] == 0.0
        s.init_random(73)
        seeded = close_walls([a.copy() for a in ci.random_e(*dims, seed=73, dtype=real)])
        got = s.get_fields(np.float64)
        assert all(np.array_equal(a, b.astype(np.float64)) for a, b in zip(got[:3], seeded))
        assert all(not f.any() for f in got[3:])
