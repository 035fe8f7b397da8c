"""The register-tile and small-item paths in FP64, which run when gbs_set_layout
selects a lane grid: full sums on mixed tuned grids, size classes on concurrent
streams, and plans that mix tree, tile, small and empty items.

Tolerances as for the other FP64 parity tests, |a - b| <= 2e-14 sum_S |t_S|, and
sum_S |t_S| to 1e-12; FP32-compensated 5e-6 sum_S |t_S|."""
import contextlib
import os
import sys

import numpy as np
import pytest

import oracle
import paper_2010_15595_amd as gbs
from paper_2010_15595_amd import workloads
from paper_2010_15595_amd._lib import LAYOUTS

sys.path.insert(0, os.path.join(os.path.dirname(__file__), "golden"))
import make_lhaf_refs  # noqa: E402

pytestmark = pytest.mark.gpu

NORMWISE = 2e-14


@pytest.fixture(scope="module", autouse=True)
def _init():
    gbs.init(0)


@contextlib.contextmanager
def _grids(n, layouts):
    """Lane grid `layouts[s]` for subsets of size s of n-pair loop hafnians."""
    try:
        for s, lay in layouts.items():
            gbs.set_layout(n, s, lay)
        yield
    finally:
        gbs.set_layout(n, 0, -1)


def _device(A, prec=gbs.GBS_FP64):
    import torch

    At = torch.from_numpy(A).cuda()
    out = torch.zeros(1, dtype=torch.complex128, device="cuda")
    ab = torch.zeros(1, dtype=torch.float64, device="cuda")
    gbs.lhaf_device(At, out, ab, prec=prec)
    torch.cuda.synchronize()
    return complex(out.cpu()[0]), float(ab.cpu()[0])


@pytest.mark.parametrize("N", [40, 44, 50])
def test_full_sums_on_tuned_grids(N):
    """The grids the tuner picks, one per subset size, against the stored
    long-double sums; the tree's value differs from it in the last bits."""
    Nr, re, im, ab_ref = make_lhaf_refs.load()[f"c3_{N}"]
    ref, ab_ref = complex(float(re), float(im)), float(ab_ref)
    st = workloads.config3(N)
    A = oracle.expand(st["B"], st["gamma"], st["pattern"])
    tree = _device(A)
    rep, lays = gbs.autotune(N // 2), list(LAYOUTS.values())
    with _grids(N // 2, {s: lays.index(lay) for s, (lay, _) in rep.items()}):
        v, ab = _device(A)
    assert Nr == N and (v, ab) != tree
    assert abs(v - ref) <= NORMWISE * ab_ref
    assert ab == pytest.approx(ab_ref, rel=1e-12)


@pytest.mark.parametrize("prec", [gbs.GBS_FP64, gbs.GBS_FP32_COMP])
@pytest.mark.parametrize("N", [10, 24, 32, 40, 44])
def test_concurrent_size_classes_on_tiles(N, prec):
    """Up to N = 44 the size classes run concurrently on auxiliary streams, with
    profiling on they run on one: the same partial records, bit for bit."""
    A = workloads.random_normal_symmetric(N, seed=N + 7, scale=0.4)
    with _grids(N // 2, {0: 2} if prec == gbs.GBS_FP64 else {}):
        res = [_device(A, prec)]
        gbs.profile_enable(True)
        try:
            res.append(_device(A, prec))
            prof = gbs.profile_read()
        finally:
            gbs.profile_enable(False)
    assert "charpoly_kernel" in prof["dominant_kernel"]
    assert res[0] == res[1]
    tree, ab = _device(A)
    assert abs(res[0][0] - tree) <= (NORMWISE if prec == gbs.GBS_FP64 else 5e-6) * ab


def test_plan_of_tree_tile_small_and_empty_items():
    """n = 3 and 8 on the small-item kernel, n = 9 and 13 on tiles, the others on
    the tree, with empty items between them; replayed, then the same plan
    rebuilt with no grid set."""
    import torch

    dims = [0, 5, 6, 18, 11, 0, 25, 26, 16, 15, 17, 2, 22, 1, 0, 6, 26, 18, 20]
    mats = [workloads.random_normal_symmetric(N, seed=2100 + i, scale=0.5) for i, N in enumerate(dims)]
    refs = []
    for A in mats:
        if len(A) == 0:
            refs.append((1.0 + 0.0j, 1.0))
            continue
        r, ab = oracle.lhaf_pt(A, prec="ld", with_abs=True)
        refs.append((oracle.to_complex(r), float(ab)))
    pk = torch.from_numpy(gbs.pack(mats)).cuda()

    def check():
        plan = gbs.BatchPlan(dims)
        for _ in range(3):
            out = torch.full((len(dims),), complex(np.nan, np.nan), dtype=torch.complex128, device="cuda")
            ab = torch.full((len(dims),), np.nan, dtype=torch.float64, device="cuda")
            plan.run(pk, out, ab)
            torch.cuda.synchronize()
            for v, a, (r, abr), N in zip(out.cpu().numpy(), ab.cpu().numpy(), refs, dims):
                assert abs(v - r) <= NORMWISE * abr, N
                assert a == pytest.approx(abr, rel=1e-12), N
        tiles = plan.info()["tiles"]
        plan.close()
        return tiles

    with contextlib.ExitStack() as grids:
        for n in (3, 8, 9, 13):
            grids.enter_context(_grids(n, {0: 2}))
        assert check() > 0
    assert check() == 0
