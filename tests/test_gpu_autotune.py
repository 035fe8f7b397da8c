"""With GBS_AUTOTUNE=1 the lane-grid tuner runs for calls that have a lane grid
to choose, and for no call on the subset tree."""
import pytest

import paper_2010_15595_amd as gbs
from paper_2010_15595_amd import workloads

pytestmark = pytest.mark.gpu


def test_only_calls_on_lane_grids_are_tuned(tmp_path, monkeypatch):
    import torch

    cache = tmp_path / "grids"
    monkeypatch.setenv("GBS_AUTOTUNE", "1")
    monkeypatch.setenv("GBS_AUTOTUNE_CACHE", str(cache))
    gbs.finalize()  # a fresh context: nothing tuned
    gbs.init(0)
    try:
        A = workloads.random_normal_symmetric(14, seed=3, scale=0.5)
        At = torch.from_numpy(A).cuda()
        out = torch.zeros(1, dtype=torch.complex128, device="cuda")
        v = gbs.lhaf(A)
        gbs.lhaf_device(At, out)
        plan = gbs.BatchPlan([14, 13])
        torch.cuda.synchronize()
        plan.close()
        assert not cache.exists()
        gbs.lhaf_device(At, out, prec=gbs.GBS_FP32_COMP)
        torch.cuda.synchronize()
        orders = {int(line.split()[1]) for line in cache.read_text().splitlines()}
        assert orders == {7}
        # the tuned grids are not forced ones: FP64 stays on the tree, bit for bit
        assert gbs.lhaf(A) == v
        assert abs(complex(out.cpu()[0]) - v) <= 5e-6 * gbs.lhaf(A, with_diag=True)[1]["abs_sum"]
    finally:
        gbs.finalize()
        gbs.init(0)
