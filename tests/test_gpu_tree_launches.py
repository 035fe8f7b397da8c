"""Launches of the subset tree: the names under which they are timed, the number
of launches a plan captures, and stream capture of orders whose kernels need more
than 64 KB of LDS (N >= 43)."""
import numpy as np
import pytest

import paper_2010_15595_amd as gbs
from paper_2010_15595_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _init():
    gbs.init(0)


def _matrix(N):
    return workloads.random_normal_symmetric(N, seed=3100 + N, scale=0.5 / max(1.0, N / 24.0))


@pytest.mark.parametrize("N, prec, kernels", [
    # one level, of one parent
    (12, gbs.GBS_FP64, {"tree_sub_kernel<6>", "tree_top_elim_kernel<6>"}),
    (40, gbs.GBS_FP64, {"tree_sub_kernel<20>"}),
    # eight levels of at most 256 parents
    (16, gbs.GBS_DD, {"tree_top_elim_kernel<dd>", "tree_dd_leaf_kernel"}),
    (36, gbs.GBS_DD, {"tree_lane_elim_kernel<dd>"}),
])
def test_launches_are_timed_under_their_kernels_name(N, prec, kernels):
    A = _matrix(N)
    gbs.lhaf(A, prec=prec)
    gbs.profile_enable(True)
    try:
        gbs.lhaf(A, prec=prec)
        prof = gbs.profile_read()
    finally:
        gbs.profile_enable(False)
    assert prof["dominant_kernel"] in kernels


def test_captured_orders_above_64_kb_of_lds():
    """Captured before any eager call of that order here, so that the kernels' LDS
    limit is raised under capture; replays, with eager work between them, equal the
    eager call."""
    import torch

    A = torch.from_numpy(_matrix(44)).cuda()
    other = torch.from_numpy(_matrix(23)).cuda()
    out = torch.zeros(1, dtype=torch.complex128, device="cuda")
    ab = torch.zeros(1, dtype=torch.float64, device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        gbs.lhaf_device_noalloc(A, out, ab)
    ref = torch.zeros(1, dtype=torch.complex128, device="cuda")
    ref_ab = torch.zeros(1, dtype=torch.float64, device="cuda")
    gbs.lhaf_device_noalloc(A, ref, ref_ab)
    torch.cuda.synchronize()
    tmp = torch.zeros(1, dtype=torch.complex128, device="cuda")
    for _ in range(3):
        out.fill_(complex(np.nan, np.nan))
        ab.fill_(np.nan)
        gbs.lhaf_device_noalloc(other, tmp)
        g.replay()
        torch.cuda.synchronize()
        assert complex(out.cpu()[0]) == complex(ref.cpu()[0]) and float(ab.cpu()[0]) == float(ref_ab.cpu()[0])


def test_plans_of_large_orders():
    """A plan's graph holds a bounded number of launches per item: an item of
    N = 50 takes 20 levels above its subtrees, in pieces that fit the entry store."""
    import torch

    dims = [44, 50, 43, 20]
    mats = [_matrix(N) for N in dims]
    plan = gbs.BatchPlan(dims)
    assert plan.info()["kernel_nodes"] <= 600
    pk = torch.from_numpy(gbs.pack(mats)).cuda()
    for _ in range(2):
        out = torch.full((len(dims),), complex(np.nan, np.nan), dtype=torch.complex128, device="cuda")
        plan.run(pk, out, None)
        torch.cuda.synchronize()
        for A, v in zip(mats, out.cpu().numpy()):
            w, d = gbs.lhaf(A, with_diag=True)
            assert abs(v - w) <= 2e-14 * d["abs_sum"]
    plan.close()


def test_small_orders_keep_no_entry_store():
    """Up to five pairs a subtree kernel reads the matrices themselves: a plan holds
    their copy, three doubles and a record of five per item, and its tables."""
    plan = gbs.BatchPlan([10] * 4000)
    bytes_ = plan.info()["workspace_bytes"]
    plan.close()
    assert bytes_ <= 4000 * (16 * 100 + 100) + (1 << 20)
