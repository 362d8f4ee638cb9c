"""Constraint norms of a plan with more blocks than a launch can have workgroups of
1,024 threads (2^32 threads), on the GPU.  The plan lists one block of one point
over and over, so that the state stays small: every block has the norms of the
single block's plan."""
import ctypes

import numpy as np
import pytest

from paper_2311_04989_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_norms_of_more_blocks_than_a_grid():
    from paper_2311_04989_amd import z4c as Z
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 2 ** 32 // 1024 + 5
    rng = np.random.default_rng(W.SEED_BASE + 7000)
    bt = W.Batch([W.Block(1, 1, 1, 3, 0.1, 0.1, 0.1, 0.0, 0.0, 0.0)], with_matter=False)
    bt.u[:] = rng.uniform(-1e-2, 1e-2, size=bt.u.size)
    for f in ("chi", "gxx", "gyy", "gzz", "alpha"):
        bt.view(bt.u, 0, W.FIELDS.index(f))[...] += 1.0
    bt.params = W.Params(fd_order=4)
    prm = Z.make_params(bt.params, Z.ARITH_FP64)
    one = Z.make_blocks(bt.block_table())
    many = (type(one)._type_ * n).from_buffer_copy(bytes(one) * n)
    u = torch.from_numpy(bt.u).to("cuda:0")
    got = []
    for blocks, count in ((one, 1), (many, n)):
        print(f"norms of {count} blocks", flush=True)
        h = ctypes.c_void_p()
        assert Z.lib().z4c_plan_create(ctypes.byref(prm), blocks, count, 0, ctypes.byref(h)) == 0
        norms = torch.full((count, 16), -7.0, dtype=torch.float64, device="cuda:0")
        assert Z.lib().z4c_constraints(h, u.data_ptr(), None, None, norms.data_ptr(), None) == 0
        torch.cuda.synchronize()
        Z.lib().z4c_plan_destroy(h)
        got.append(norms)
    assert (got[0] > 0.0).any()
    assert bool((got[1] == got[0]).all())
