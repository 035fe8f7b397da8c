"""Matrices whose rows differ in scale.  Scaling vertex i of a pair by r and its
partner by 1 / r changes no subset term, so the error of a sum may not depend on
such a grading: FP64 and double-double sums of graded matrices against the
long-double oracle, through every entry point that runs on the subset tree.

Tolerance as for the other FP64 parity tests, |a - b| <= 2e-14 sum_S |t_S|; the
oracle's own error on these matrices is below 1e-15 sum_S |t_S| (against a
binary128 evaluation)."""
import numpy as np
import pytest

import paper_2010_15595_amd as gbs

oracle = pytest.importorskip("oracle")

pytestmark = pytest.mark.gpu

NORMWISE = 2e-14


@pytest.fixture(scope="module", autouse=True)
def _init():
    gbs.init(0)


def _graded(N, kind):
    """Row and column j scaled by r_j, a loop weight (on the diagonal) by r_j."""
    rng = np.random.default_rng(9000 + N)
    A = 0.5 * (rng.standard_normal((N, N)) + 1j * rng.standard_normal((N, N)))
    A = (A + A.T) / 2
    n, d = (N + 1) // 2, np.diagonal(A).copy()
    if kind == "loops":  # loop weights of the second half, where the matrix is zero
        A[n:, n:] = 0.0
        d[n:] *= 1e5
        r = np.ones(N)
    elif kind == "vertices":
        r = 10.0 ** rng.uniform(-1.5, 1.5, N)
    elif kind == "entry":
        r = np.ones(N)
        A[0, 1] = A[1, 0] = 1e4
    else:
        r = np.r_[np.ones(n), np.full(N - n, 1.0 / kind)]
    A = A * np.outer(r, r)
    A[np.arange(N), np.arange(N)] = d * r
    return np.ascontiguousarray(A)


KINDS = [30, 100, 1000, "loops", "vertices", "entry"]


def _oracle(A):
    ref, ab = oracle.lhaf_pt(A, prec="ld", with_abs=True)
    return oracle.to_complex(ref), float(ab)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("N", [6, 9, 12, 17, 20])
def test_single_evaluations(N, kind):
    import torch

    A = _graded(N, kind)
    ref, ab = _oracle(A)
    At = torch.from_numpy(A).cuda()
    o = torch.zeros(2, dtype=torch.complex128, device="cuda")
    gbs.lhaf_device(At, o[:1])
    gbs.lhaf_device_noalloc(At, o[1:])
    torch.cuda.synchronize()
    hi, d = gbs.lhaf(A, prec=gbs.GBS_DD, with_diag=True)
    got = [complex(o[0].cpu()), complex(o[1].cpu()), gbs.lhaf(A), hi + d["lhaf_lo"]]
    print(f"[graded N={N} {kind}] " + " ".join(f"{abs(v - ref) / ab:.1e}" for v in got), flush=True)
    for v in got:
        assert abs(v - ref) <= NORMWISE * ab


def test_larger_orders_against_double_double():
    """The many-parent elimination kernel and every depth of the subtrees."""
    for N in (27, 34, 40):
        for kind in (1000, "vertices"):
            A = _graded(N, kind)
            ref, d = gbs.lhaf(A, prec=gbs.GBS_DD, with_diag=True)
            v = gbs.lhaf(A)
            print(f"[graded N={N} {kind}] {abs(v - ref) / d['abs_sum']:.1e}", flush=True)
            assert abs(v - ref) <= NORMWISE * d["abs_sum"]


def test_exact_gradings_change_nothing():
    """A power of two on one vertex of each pair and its inverse on the partner is
    exact, and the terms stay as they are: every intermediate is scaled as a whole, so
FP64 and double-double values are the same bit for bit."""
    for N in (10, 20, 33):
        A = _graded(N, 1)
        n = (N + 1) // 2
        s = 2.0 ** np.random.default_rng(N).integers(-12, 13, n)
        r = np.r_[s, 1.0 / s[: N - n]]  # (an odd N: the partner that is added has loop weight 1)
        if N & 1:
            r[n - 1] = 1.0
        B = np.ascontiguousarray(A * np.outer(r, r))
        B[np.arange(N), np.arange(N)] = np.diagonal(A) * r
        v, d = gbs.lhaf(A, prec=gbs.GBS_DD, with_diag=True)
        w, e = gbs.lhaf(B, prec=gbs.GBS_DD, with_diag=True)
        assert v == w and d["lhaf_lo"] == e["lhaf_lo"]
        assert gbs.lhaf(A) == gbs.lhaf(B)


def test_batch():
    import torch

    mats = [_graded(N, k) for N in (2, 5, 8, 11, 14, 16, 18) for k in KINDS]
    plan = gbs.BatchPlan([len(A) for A in mats])
    out = torch.zeros(len(mats), dtype=torch.complex128, device="cuda")
    plan.run(torch.from_numpy(gbs.pack(mats)).cuda(), out, None)
    torch.cuda.synchronize()
    for A, v in zip(mats, out.cpu().numpy()):
        ref, ab = _oracle(A)
        assert abs(v - ref) <= NORMWISE * ab, len(A)
    plan.close()
