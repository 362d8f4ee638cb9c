"""z4c_plan_autotune on a stream that is being captured: refused, and neither the
capture, the plan's launch shapes and tile count nor the tuning cache change."""
import numpy as np
import pytest

from paper_2311_04989_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_autotune_under_capture_changes_nothing(tmp_path):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2311_04989_amd import z4c as Z
    print("autotune on a captured stream", flush=True)
    one = W.random_batch(3, nblocks=1, nmax=12, fd_order=6)
    two = W.random_batch(3, nblocks=2, nmax=12, fd_order=6)
    size = lambda b: (b.nx, b.ny, b.nz)  # noqa: E731
    assert size(one.blocks[0]) == size(two.blocks[0]) != size(two.blocks[1])
    bufs = lambda bt: [torch.from_numpy(bt.u.copy()).to("cuda:0") for _ in range(3)]  # noqa: E731
    path = tmp_path / "tune.txt"
    Z.set_tune_cache(path)
    try:
        p1 = Z.plan_for(one)   # the first size into the cache
        p1.autotune(*bufs(one), None, reps=1)
        p1.close()
        text = path.read_text()
        plan, b = Z.plan_for(two), bufs(two)
        before = [plan.get_launch(*size(x)) for x in two.blocks], plan.tiles
        x = torch.zeros(8, device="cuda:0")
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            x.add_(1.0)
            with pytest.raises(Z.Z4cError):
                plan.autotune(*b, None, reps=1, stream=torch.cuda.current_stream())
        assert ([plan.get_launch(*size(y)) for y in two.blocks], plan.tiles) == before
        assert path.read_text() == text
        for n in range(3):
            g.replay()
            torch.cuda.synchronize()
            assert np.array_equal(x.cpu().numpy(), np.full(8, n + 1.0, dtype=np.float32))
        plan.autotune(*b, None, reps=1)   # and outside of it works
        assert len(path.read_text().strip().splitlines()) == 2
        torch.cuda.synchronize()
        plan.close()
    finally:
        Z.set_tune_cache(None)
