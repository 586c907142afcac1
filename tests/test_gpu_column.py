"""The column form of the temporal sweep (states that the last-level cache holds) at the sizes where
its windows end: 64 columns, 32 or 24 rows, one z-plane per workgroup, more tiles than CUs."""

import numpy as np
import pytest

import cavity_inputs as ci

pytestmark = pytest.mark.gpu

DT = 0.5 / 3 ** 0.5
# (nx, ny, nz): one window exactly, one cell more or less, two windows exactly (64 + 56 columns, 32 + 24
# rows at 4 steps), a third one of a single column, thin in z
DIMS = [(63, 31, 5), (64, 32, 9), (65, 33, 3), (120, 56, 8), (121, 57, 2), (66, 24, 7), (177, 25, 6)]


def media(nx, ny, nz):
    eps = ci.uniform_cell_eps(nx, ny, nz, seed=61, lo=1.0, hi=4.0)
    mu = ci.uniform_cell_eps(nx, ny, nz, seed=62, lo=1.0, hi=1.5)
    return [(None, None), (eps, None), (None, mu), (eps, mu)]


def solve(dims, eps, mu, e, h, steps, zchunks=None, **kw):
    from paper_2504_09118_amd import Solver

    with Solver(*dims, 1.0, DT, eps_r=eps, mu_r=mu, **kw) as s:
        if zchunks:
            s.set_schedule("temporal", kw["tb_steps"], 0, min(zchunks, dims[2]))
        s.set_fields(e, h)
        s.step(steps)
        return s.get_fields(np.float32)


@pytest.mark.parametrize("dims", DIMS)
def test_fp32_equals_the_plain_schedule(dims):
    """Same bits as one-cell-per-thread steps for every steps per sweep and coefficient kind, with the
    default z-split, one chunk and one plane per chunk; the last sweep is a remainder."""
    e = ci.random_e(*dims, seed=63, dtype=np.float32)
    h = ci.random_h(*dims, seed=64, dtype=np.float32)
    for eps, mu in media(*dims):
        for tb in (1, 2, 3, 4):
            steps = 2 * tb + 1
            want = solve(dims, eps, mu, e, h, steps, kernel="plain")
            for zc in (None, 1, dims[2]):
                got = solve(dims, eps, mu, e, h, steps, zc, kernel="temporal", tb_steps=tb)
                for a, b in zip(got, want):
                    assert np.array_equal(a, b) and np.array_equal(np.signbit(a), np.signbit(b)), (tb, zc)


@pytest.mark.parametrize("storage", ["f16", "bf16", "f16c", "bf16c"])
@pytest.mark.parametrize("dims", [(64, 32, 9), (121, 57, 2), (66, 24, 7)])
def test_16bit_storage_equals_the_streaming_form(monkeypatch, dims, storage):
    """16-bit storage: same bits as the form that large states take."""
    e = ci.random_e(*dims, seed=65, dtype=np.float32)
    h = ci.random_h(*dims, seed=66, dtype=np.float32)
    for eps, mu in media(*dims):
        for tb in (1, 3, 4):
            outs = []
            for pol in ("1", "0"):
                monkeypatch.setenv("FDTD_NT_STORES", pol)
                outs.append(solve(dims, eps, mu, e, h, 2 * tb + 1, storage=storage, tb_steps=tb))
            for a, b in zip(*outs):
                assert np.array_equal(a, b), tb


def test_more_tiles_than_compute_units_take_the_queue():
    """18 windows x 40 chunks: tiles come from the queue, over several sweeps (the counters return to 0)."""
    dims = (130, 130, 40)
    e = ci.random_e(*dims, seed=67, dtype=np.float32)
    h = ci.random_h(*dims, seed=68, dtype=np.float32)
    eps, mu = media(*dims)[3]
    want = solve(dims, eps, mu, e, h, 14, kernel="plain")
    got = solve(dims, eps, mu, e, h, 14, 40, kernel="temporal", tb_steps=4)
    for a, b in zip(got, want):
        assert np.array_equal(a, b)
