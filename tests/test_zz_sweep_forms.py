"""Both forms of the temporal sweep on the cavities that the other files run with the default one.

States that the last-level cache holds take the column form, so small cavities no longer reach the form
that every larger state runs; FDTD_NT_STORES = 1 gives it to them. Its sweeps always take tiles from
the queue; a column sweep does with full workgroups and more tiles than CUs, which the last tests see to:
counters that are not reset, or that two solvers share, leave tiles out.
"""

import numpy as np
import pytest

import cavity_inputs as ci
from tests import test_gpu_parity as parity
from tests import test_zz_no_alloc as noalloc

pytestmark = pytest.mark.gpu


@pytest.fixture(params=["0", "1"], ids=["column", "streaming"])
def form(request, monkeypatch):
    monkeypatch.setenv("FDTD_NT_STORES", request.param)
    return request.param


@pytest.mark.parametrize("tb", [1, 2, 3, 4])
def test_ragged(form, tb):
    parity.test_temporal_parity_ragged(tb)
    parity.test_temporal_per_node_ch_with_scalar_ce(tb)


@pytest.mark.parametrize("dims", parity.DEGENERATE_DIMS)
def test_degenerate_grids(form, dims):
    parity.test_degenerate_grids_every_schedule(dims)


def test_bits(form, monkeypatch):
    parity.test_wall_normal_h_and_walls_keep_their_bits()
    parity.test_kernels_bitwise_equal(monkeypatch)


def test_counters(form):
    parity.test_two_solvers_on_two_streams_keep_their_bits()
    parity.test_schedule_changes_between_sweeps_keep_the_bits()


@pytest.mark.parametrize("tb", [3, 4])
def test_noalloc(form, tb):
    noalloc.test_noalloc_steps_equal_fdtd_step_on_two_calls_second_smaller(tb)
    for storage in ("f16", "bf16", "f16c", "bf16c"):
        noalloc.test_noalloc_16bit_storage(storage, tb)


# with both arrays and 4 steps full workgroups have 12 waves: windows of 64 x 24, 16 of their rows own
QUEUED = [((130, 130, 40), 40), ((125, 75, 66), 33)]


def queued(dims, seed, **kw):
    from paper_2504_09118_amd import Solver

    eps = ci.uniform_cell_eps(*dims, seed=seed, lo=1.0, hi=4.0)
    mu = ci.uniform_cell_eps(*dims, seed=seed + 1, lo=1.0, hi=1.5)
    s = Solver(*dims, eps_r=eps, mu_r=mu, **kw)
    s.set_fields(ci.random_e(*dims, seed=seed + 2, dtype=np.float32), ci.random_h(*dims, seed=seed + 3, dtype=np.float32))
    return s


def test_queues_of_two_solvers_at_once():
    import torch

    want = []
    for q, (dims, _) in enumerate(QUEUED):
        with queued(dims, 80 + 10 * q, kernel="plain") as s:
            s.step(14)
            want.append(s.get_fields(np.float32))
    solvers = [queued(dims, 80 + 10 * q, tb_steps=4, stream=torch.cuda.Stream()) for q, (dims, _) in enumerate(QUEUED)]
    try:
        for s, (_, zc) in zip(solvers, QUEUED):
            s.set_schedule("temporal", 4, 0, zc)
        for n in (4, 4, 4, 2):
            for s in solvers:
                s.step(n)
        for s, w in zip(solvers, want):
            assert all(np.array_equal(a, b) for a, b in zip(s.get_fields(np.float32), w))
    finally:
        for s in solvers:
            s.close()


def test_queue_of_the_calls_without_allocation():
    for q, (dims, zc) in enumerate(QUEUED):
        with queued(dims, 80 + 10 * q, kernel="plain") as s:
            s.step(14)
            want = s.get_fields(np.float32)
        with queued(dims, 80 + 10 * q, tb_steps=4) as s:
            s.set_schedule("temporal", 4, 0, zc)
            for n in (4, 4, 4, 2):
                noalloc._noalloc(s, n)
            assert all(np.array_equal(a, b) for a, b in zip(s.get_fields(np.float32), want))
