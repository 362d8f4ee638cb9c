"""The VC <-> CC interpolations of a plan with more columns times fields than a
launch can have workgroups of 256 threads (2^32 threads), on the GPU.  The plan
lists one small block over and over, so that the arrays stay small: every copy
writes the same values to the same place, those of the single block's plan."""
import ctypes

import numpy as np
import pytest

from paper_2311_04989_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_more_columns_than_a_grid_of_columns_and_fields():
    from paper_2311_04989_amd import z4c as Z
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 2_400_000
    assert 7 * n * 256 >= 2 ** 32 > 256 * n
    rng = np.random.default_rng(W.SEED_BASE + 6000)
    mb = W.MatterBatch([W.MBlock(2, 1, 3, 2, 1, 0.5)])
    mb.u[:] = rng.uniform(0.5, 1.5, size=mb.u.size)
    mb.adm[:] = rng.uniform(0.5, 1.5, size=mb.adm.size)
    one = Z.make_mblocks(mb.table())
    many = (Z.MBlock * n).from_buffer_copy(bytes(one) * n)
    dev = lambda a: torch.from_numpy(a).to("cuda:0")  # noqa: E731
    got = []
    for blocks, count in ((one, 1), (many, n)):
        print(f"interp of {count} blocks", flush=True)
        h = ctypes.c_void_p()
        assert Z.lib().z4c_mplan_create(blocks, count, 0, ctypes.byref(h)) == 0
        geom, matter = dev(np.full(mb.geom.size, -7.0)), dev(np.full(mb.matter.size, -7.0))
        u, adm = dev(mb.u), dev(mb.adm)
        for call, src, dst in ((Z.lib().z4c_metric_to_cc, u, geom),
                               (Z.lib().z4c_sources_to_vc, adm, matter)):
            ext = (0,) if dst is geom else ()
            st = call(h, 2, *ext, src.data_ptr(), dst.data_ptr(), None)
            assert st == 0, Z.lib().z4c_last_error()
        torch.cuda.synchronize()
        Z.lib().z4c_mplan_destroy(h)
        got.append((geom.cpu().numpy(), matter.cpu().numpy()))
    for a, b in zip(*got):
        assert (a != -7.0).any()
        assert np.array_equal(a, b)
