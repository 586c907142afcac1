"""get_fields_device into tensors that share memory: the last component written stays, as with one at a time."""

import numpy as np
import pytest

import cavity_inputs as ci

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(70, 70, 70), (130, 40, 33)], ids=lambda s: "x".join(map(str, s)))
def test_tensors_that_share_memory(dims):
    import torch

    import paper_2504_09118_amd as P

    with P.Solver(*dims) as s:
        s.set_fields(ci.random_e(*dims, seed=1, dtype=np.float32), ci.random_h(*dims, seed=2, dtype=np.float32))
        s.step(3)
        want = s.get_fields(np.float32)
        sizes = [int(np.prod(sh)) for sh in s.shapes]
        for dtype in (torch.float32, torch.float64):
            for _ in range(4):
                one = torch.full((max(sizes) + 8,), np.nan, dtype=dtype, device="cuda")
                # all six from element 0; E in memory of its own, H one element after the other
                apart = [torch.empty(sh, dtype=dtype, device="cuda") for sh in s.shapes[:3]]
                for views in ([one[:n].view(sh) for n, sh in zip(sizes, s.shapes)],
                              apart + [one[q:q + n].view(sh) for q, (n, sh) in enumerate(zip(sizes[3:], s.shapes[3:]))]):
                    torch.cuda.synchronize()
                    s.get_fields_device(views)
                    s.sync()
                    assert np.array_equal(views[5].cpu().numpy(), want[5])
                assert all(np.array_equal(a.cpu().numpy(), b) for a, b in zip(apart, want))
