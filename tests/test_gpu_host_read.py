"""Reads into host memory at the edges of the pinned slots (2 MiB, 8 of them), against a device copy.

Fresh, warm and unaligned pageable memory, pinned memory, one array given for two fields
(the later one's values stay), FP32 and FP64 buffers, with work still queued on the stream:
whole numbers of bytes, so they are equal.
"""

import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _pkg():
    import paper_2504_09118_amd as P

    return P


# (n+1)-node arrays of less than a slot, about one, a few, and more than the ring holds
@pytest.mark.parametrize("shape", [(2, 2, 2), (16, 16, 16), (50, 50, 50), (63, 63, 127), (64, 64, 128), (131, 97, 64),
                                   (240, 200, 120)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("dtype", [np.float32, np.float64], ids=["f32", "f64"])
def test_fields_equal_device_copy(shape, dtype):
    import torch

    P = _pkg()
    td = torch.float32 if dtype == np.float32 else torch.float64
    with P.Solver(*shape) as s:
        s.init_random(3)
        s.step(23)  # still running when the read begins
        got = [s.get_fields(dtype=dtype)]
        got.append(s.get_fields(dtype=dtype))
        dev = [torch.empty(q, dtype=td, device="cuda") for q in s.shapes]
        s.get_fields_device(dev)
        s.sync()
        want = [d.cpu().numpy() for d in dev]
        raw = [np.empty(a.nbytes + 3, np.uint8) for a in want]
        odd = [r[3:].view() for r in raw]
        pin = [torch.empty(q, dtype=td, pin_memory=True) for q in s.shapes]
        for ptr in ([r.ctypes.data for r in odd], [p.data_ptr() for p in pin]):
            assert s._lib.fdtd_get_fields(s._h, (ctypes.c_void_p * 6)(*ptr), 0 if dtype == np.float64 else 1) == 0
        got.append([np.frombuffer(o.tobytes(), dtype).reshape(w.shape) for o, w in zip(odd, want)])
        got.append([p.numpy() for p in pin])
        same = [np.empty(max(a.size for a in want), dtype)] * 6
        ptr = (ctypes.c_void_p * 6)(*[a.ctypes.data for a in same])
        assert s._lib.fdtd_get_fields(s._h, ptr, 0 if dtype == np.float64 else 1) == 0
        assert np.array_equal(same[0][:want[5].size], want[5].ravel())
    for g in got:
        assert all(np.array_equal(a, b) for a, b in zip(g, want))


def test_pool_fetch_from_threads():
    import threading

    P = _pkg()
    shapes = [(48, 40, 56), (96, 64, 80), (130, 66, 70)]
    with P.Pool(2 << 30) as pool:
        ids = [pool.submit(*q, 7, seed=5 + i, keep=True) for i, q in enumerate(shapes)]
        pool.wait(-1)
        want = []
        for i, q in enumerate(shapes):
            with P.Solver(*q) as s:
                s.init_random(5 + i)
                s.step(7)
                want.append(s.get_fields(dtype=np.float32))
        out = {}
        ts = [threading.Thread(target=lambda i=i, t=t: out.__setitem__((i, t), pool.fetch(ids[i], *shapes[i],
                                                                                          dtype=np.float32)))
              for i in range(3) for t in range(2)]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
    for (i, _), got in out.items():
        assert all(np.array_equal(a, b) for a, b in zip(got, want[i]))
    assert len(out) == 6
