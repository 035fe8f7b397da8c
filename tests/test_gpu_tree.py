"""The subset tree (FP64 sums without a forced lane grid) against the oracle
and against the register-tile kernels, which gbs_set_layout selects, for every
order n it has an instance of.

Both sides sum the same subset terms; tolerance as for the other FP64 parity
tests, |a - b| <= 2e-14 sum_S |t_S|, and sum_S |t_S| to 1e-12 (both sides'
terms are good to a few 1e-13 relative)."""
import numpy as np
import pytest

import oracle
import paper_2010_15595_amd as gbs
from paper_2010_15595_amd import workloads

pytestmark = pytest.mark.gpu

NORMWISE = 2e-14


@pytest.fixture(scope="module", autouse=True)
def _init():
    gbs.init(0)


def _matrix(N):
    return workloads.random_normal_symmetric(N, seed=1200 + N, scale=0.5 / max(1.0, N / 24.0))


@pytest.mark.parametrize("N", list(range(1, 21)) + [25, 26])
def test_against_the_oracle(N):
    A = _matrix(N)
    ref, ab = oracle.lhaf_pt(A, prec="ld", with_abs=True)
    ref, ab = oracle.to_complex(ref), float(ab)
    val, d = gbs.lhaf(A, with_diag=True)
    assert abs(val - ref) <= NORMWISE * ab
    assert d["abs_sum"] == pytest.approx(ab, rel=1e-12)


@pytest.mark.parametrize("N", [2, 7, 10, 12, 14] + list(range(22, 51, 2)) + [52, 54])
def test_against_the_register_tiles(N):
    import torch

    At = torch.from_numpy(_matrix(N)).cuda()
    got = []
    for layout in (-1, 2):
        gbs.set_layout((N + 1) // 2, 0, layout)
        try:
            o = torch.zeros(1, dtype=torch.complex128, device=At.device)
            a = torch.zeros(1, dtype=torch.float64, device=At.device)
            gbs.lhaf_device(At, o, a)
            torch.cuda.synchronize()
            got.append((complex(o.cpu()[0]), float(a.cpu()[0])))
        finally:
            gbs.set_layout((N + 1) // 2, 0, -1)
    (v, ab), (w, ab_w) = got
    assert abs(v - w) <= NORMWISE * ab_w
    assert ab == pytest.approx(ab_w, rel=1e-12)


def test_batch_of_every_order():
    """Items of every dimension 0..30 with two of each, one plan, against
    single evaluations; replayed."""
    import torch

    dims = [N for N in range(31) for _ in range(2)]
    mats = [workloads.random_normal_symmetric(N, seed=1300 + i, scale=0.5) for i, N in enumerate(dims)]
    plan = gbs.BatchPlan(dims)
    pk = torch.from_numpy(gbs.pack(mats)).cuda()
    for _ in range(2):
        out = torch.zeros(len(dims), dtype=torch.complex128, device="cuda")
        ab = torch.zeros(len(dims), dtype=torch.float64, device="cuda")
        plan.run(pk, out, ab)
        torch.cuda.synchronize()
        for i, A in enumerate(mats):
            v, d = gbs.lhaf(A, with_diag=True)
            assert abs(complex(out[i].cpu()) - v) <= NORMWISE * d["abs_sum"], dims[i]
            assert float(ab[i].cpu()) == pytest.approx(d["abs_sum"], rel=1e-12)
    plan.close()


def test_nan_entries_reach_the_result():
    """A device matrix is not checked: a NaN in it must not vanish."""
    import torch

    for N in (6, 17):
        A = _matrix(N)
        A[1, 0] = A[0, 1] = np.nan
        o = torch.zeros(1, dtype=torch.complex128, device="cuda")
        gbs.lhaf_device(torch.from_numpy(A).cuda(), o)
        torch.cuda.synchronize()
        assert np.isnan(complex(o.cpu()[0]).real)


@pytest.mark.parametrize("N", [1, 2, 3, 4, 9, 30, 32, 33, 35, 43, 49])
def test_double_double(N):
    """Orders on both sides of the switch from 16 to 32 lanes per solve (n = 16 /
    17), of the row kept in LDS or in memory and of one or several parents per
    workgroup: a permuted matrix (other subsets, other rounding) gives the same
    value to double-double accuracy, and the FP64 sum agrees to its own."""
    A = _matrix(N)
    p = np.random.default_rng(N).permutation(N)
    v, d = gbs.lhaf(A, prec=gbs.GBS_DD, with_diag=True)
    w, e = gbs.lhaf(np.ascontiguousarray(A[np.ix_(p, p)]), prec=gbs.GBS_DD, with_diag=True)
    f, g = gbs.lhaf(A, with_diag=True)
    # the two splits have different sum_S |t_S|; each value is good to 2e-30 of its own
    assert abs((v - w) + (d["lhaf_lo"] - e["lhaf_lo"])) <= 2e-30 * (d["abs_sum"] + e["abs_sum"])
    assert abs(f - v) <= NORMWISE * d["abs_sum"]
    assert d["abs_sum"] == pytest.approx(g["abs_sum"], rel=1e-12)
