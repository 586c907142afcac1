"""Layout kernels (pack, unpack, seeded state, coefficients) where their launches end: planes of less and
more than one workgroup's run, more planes than a launch's y extent."""

import numpy as np
import pytest

import cavity_inputs as ci

pytestmark = pytest.mark.gpu

# (31, 32, 3): 1024 and 1056 elements a plane against runs of 1024; 66000 planes against 65535
DIMS = [(2, 2, 66000), (31, 32, 3), (2, 513, 4), (1030, 2, 2)]


def close_walls(e):
    for f, axes in zip(e, ((0, 1), (0, 2), (1, 2))):
        for a in axes:
            view = np.moveaxis(f, a, 0)
            view[0] = 0
            view[-1] = 0
    return e


@pytest.mark.parametrize("dims", DIMS)
def test_set_get_and_seeded_state(dims):
    import torch

    from paper_2504_09118_amd import Solver

    e = [a.copy() for a in ci.random_e(*dims, seed=71, dtype=np.float32)]
    h = ci.random_h(*dims, seed=72, dtype=np.float32)
    want = close_walls([a.copy() for a in e]) + list(h)
    for storage in ("f32", "f64"):
        with Solver(*dims, storage=storage, kernel="plain") as s:
            s.set_fields(e, h)
            for a, b in zip(s.get_fields(np.float32), want):
                assert np.array_equal(a, b)
            dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in list(e) + list(h)]
            out = [torch.full_like(t, np.nan, dtype=torch.float64) for t in dev]
            torch.cuda.synchronize()
            s.set_fields_device(dev)
            s.get_fields_device(out)
            s.sync()
            for a, b in zip(out, want):
                assert np.array_equal(a.cpu().numpy(), b.astype(np.float64))
            s.init_random(73)
            seeded = close_walls([a.copy() for a in ci.random_e(*dims, seed=73, dtype=np.float32 if storage == "f32" else np.float64)])
            got = s.get_fields(np.float64)
            for a, b in zip(got[:3], seeded):
                assert np.array_equal(a, b.astype(np.float64))
            assert all(not f.any() for f in got[3:])


@pytest.mark.parametrize("dims", DIMS[:3])
def test_coefficients(dims, oracle_mod):
    """Bit for bit the FP64 oracle's coefficients rounded to FP32."""
    from paper_2504_09118_amd import Solver

    eps = ci.uniform_cell_eps(*dims, seed=74, lo=1.0, hi=4.0)
    mu = ci.uniform_cell_eps(*dims, seed=75, lo=1.0, hi=1.5)
    dt = 0.5 / 3 ** 0.5
    with Solver(*dims, 1.0, dt, eps_r=eps, mu_r=mu, kernel="plain") as s:
        got = s.get_coefs(np.float32)
    want = list(oracle_mod.coef_e(*dims, 1.0, dt, eps)) + list(oracle_mod.coef_h(*dims, 1.0, dt, mu))
    for a, b in zip(got, want):
        assert np.array_equal(a, np.asarray(b).astype(np.float32))
