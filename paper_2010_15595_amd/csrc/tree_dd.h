#pragma once
// Subset tree in double-double (see tree_device.h for the method).  A complex
// dd multiply-add takes 48 FP64 instructions, so series products are spread over
// lanes by output coefficient instead of unrolled per lane: the loops stay rolled,
// a lane holds one accumulator, and every level down to the leaves goes through
// device memory, which costs little next to the arithmetic.  Bound by the issue
// of FP64 instructions at the deep levels (a lane's product has as many terms as
// its coefficient's index, so about half of the lanes work, and a solve is a chain
// of n steps), by the latency of those chains at the first ten.  Against the
// LDS-resident characteristic polynomial of each subset: N = 28 5.61 -> 0.53 ms,
// N = 36 94 -> 6.9 ms, N = 44 2250 -> 135 ms, N = 50 25.3 -> 1.25 s.
// Included by lhaf_lds.hip alone (floating-point contraction is off there).
#include "dd.h"
#include "tree_lane.h"

namespace gbs {

namespace treedd {

// Unnormalised accumulator: hi carries the sum rounded at every step, lo the
// exact rounding errors and the products' low parts (a compensated dot product
// of dd operands); its error is a few n 2^-106 of the summed magnitudes, at 12
// instead of 27 instructions per real product.  (A permuted matrix gives the same
// sum to 1e-33 of sum |t_S| at N = 40.)
struct Acc {
    double rh, rl, ih, il;
};
__device__ __forceinline__ Acc acc_of(cdd a) { return Acc{a.re.hi, a.re.lo, a.im.hi, a.im.lo}; }
__device__ __forceinline__ cdd value(const Acc& a) { return cdd{two_sum_dd(a.rh, a.rl), two_sum_dd(a.ih, a.il)}; }
__device__ __forceinline__ void term(double& h, double& l, double ah, double al, double bh, double bl) {
    const double p = ah * bh;
    double e = fma(ah, bh, -p);
    e = fma(ah, bl, fma(al, bh, e));
    const dd s = two_sum_dd(h, p);
    h = s.hi;
    l += s.lo + e;
}
__device__ __forceinline__ void mac(Acc& c, const cdd& a, const cdd& b) {
    term(c.rh, c.rl, a.re.hi, a.re.lo, b.re.hi, b.re.lo);
    term(c.rh, c.rl, -a.im.hi, -a.im.lo, b.im.hi, b.im.lo);
    term(c.ih, c.il, a.re.hi, a.re.lo, b.im.hi, b.im.lo);
    term(c.ih, c.il, a.im.hi, a.im.lo, b.re.hi, b.re.lo);
}

constexpr int kThreads = treelane::kThreads;

struct Arith {
    using V = cdd;
    using Acc = treedd::Acc;
    static constexpr int kUnroll = 1;
    static __device__ __forceinline__ Acc acc_of(const V& a) { return treedd::acc_of(a); }
    static __device__ __forceinline__ V value(const Acc& a) { return treedd::value(a); }
    static __device__ __forceinline__ void mac(Acc& c, const V& a, const V& b) { treedd::mac(c, a, b); }
    static __device__ __forceinline__ V scale(const V& a, double x) { return cdd_mul_d(a, x); }
    static __device__ __forceinline__ V add(const V& a, const V& b) { return cdd_add(a, b); }
    template <int I>
    static __device__ __forceinline__ V bcast(const V& a) {
        return cdd{dd{treelane::row_bcast<I>(a.re.hi), treelane::row_bcast<I>(a.re.lo)},
                   dd{treelane::row_bcast<I>(a.im.hi), treelane::row_bcast<I>(a.im.lo)}};
    }
};

}  // namespace treedd

// Signed terms of the leaves g0 .. g0 + count - 1 (subset masks), one on as many
// lanes as a solve: k e_k = sum_j (p_j + j q_j) / 2 e_(k-j), lane k - 1 holding e_k.
__global__ void __launch_bounds__(treedd::kThreads) tree_dd_leaf_kernel(TreeMap mp, uint64_t g0, uint64_t count,
                                                                        cdd* __restrict__ terms) {
    using namespace treedd;
    __shared__ cdd f[2 * kThreads], e[2 * kThreads];  // kThreads / P groups of P + 1
    const int n = mp.n, P = treelane::solve_lanes(n), grp = threadIdx.x / P, k = (threadIdx.x & (P - 1)) + 1;
    const uint64_t i0 = (uint64_t)blockIdx.x * (kThreads / P) + grp;
    if (i0 >= count) return;
    const uint64_t g = g0 + i0;
    const treelane::Block<cdd> b = treelane::node_block<cdd>(mp, n, g);
    cdd *fs = f + grp * (P + 1), *es = e + grp * (P + 1);
    const bool mine = k <= n;
    if (mine) {
        const cdd p = b.base[k * b.stride], q = b.base[k * b.stride + 1];
        fs[k] = cdd_mul_d(cdd_add(p, cdd_mul_d(q, (double)k)), 0.5);
    }
    if (k == 1) es[0] = cdd_make(1.0, 0.0);
    tree::order_wave();
    Acc a{0.0, 0.0, 0.0, 0.0};
    for (int i = 0; i < n; ++i) {
        if (mine && k > i) treedd::mac(a, fs[k - i], es[i]);
        if (k == i + 1) {
            const cdd v = value(a);
            const dd d = dd_make((double)k);
            es[k] = cdd{dd_div(v.re, d), dd_div(v.im, d)};
        }
        tree::order_wave();
    }
    if (k == n) {
        const cdd t = es[n];
        terms[i0] = ((n - __popcll(g)) & 1) ? cdd{dd_neg(t.re), dd_neg(t.im)} : t;
    }
}

// The root of one matrix (N x N, leading dimension N): see tree_root_kernel.
__global__ void __launch_bounds__(64) tree_dd_root_kernel(TreeMap mp, const double2* __restrict__ A, int N) {
    const int n = mp.n, E = tree_entries(n);
    const int e = blockIdx.x * 64 + threadIdx.x;
    if (e >= E) return;
    auto at = [&](int r, int c) -> cdd {
        if (r == c || r >= N || c >= N) return cdd_zero();
        const double2 x = A[r * N + c], y = A[c * N + r];
        return cdd{dd_mul_d(two_sum_dd(x.x, y.x), 0.5), dd_mul_d(two_sum_dd(x.y, y.y), 0.5)};
    };
    auto loop = [&](int r) -> cdd {
        return r < N ? cdd_make(A[r * N + r].x, A[r * N + r].y) : cdd_make(1.0, 0.0);
    };
    cdd v = cdd_zero();
    if (e > 0) {
        const int x = e - 1;
        int j = (int)((__builtin_sqrtf(8.0f * (float)x + 1.0f) - 1.0f) * 0.5f);
        if (tree_tri(j + 1, 0) <= x) ++j;
        if (tree_tri(j, 0) > x) --j;
        const int k = x - tree_tri(j, 0);
        if (j > 0) v = k == 0 ? loop(tree::root_row(j, n)) : at(tree::root_row(j, n), tree::root_row(k, n));
    }
    cdd* p = reinterpret_cast<cdd*>(mp.arena) + mp.off[0] + e;
    p[0] = v;
    for (int k = 1; k <= n; ++k) p[k * E] = cdd_zero();
}

hipError_t launch_tree_dd_root(const TreeMap& mp, const double2* A, int N, hipStream_t st) {
    hipLaunchKernelGGL(tree_dd_root_kernel, dim3((unsigned)((tree_entries(mp.n) + 63) / 64)), dim3(64), 0, st, mp, A, N);
    return hipGetLastError();
}

// Up to here a parent's row of lanes per series is faster than several parents
// packed into a workgroup: N = 28, with one row update less than now, for a limit
// of 32, 128, 256, 512, 1024: 531, 520, 521, 540, 565 us.
constexpr uint64_t kTopParentsDd = 256;

bool tree_dd_elim_top(uint64_t count) { return count <= kTopParentsDd; }

hipError_t launch_tree_dd_elim(const TreeMap& mp, int level, uint64_t g0, uint64_t count, hipStream_t st) {
    if (tree_dd_elim_top(count)) return launch_tree_top_elim<treedd::Arith>(mp, level, g0, count, st);
    return launch_tree_lane_elim<treedd::Arith>(mp, level, g0, count, st);
}

hipError_t launch_tree_dd_leaf(const TreeMap& mp, uint64_t g0, uint64_t count, void* terms, hipStream_t st) {
    if (count == 0) return hipSuccess;
    const unsigned per = (unsigned)(treedd::kThreads / treelane::solve_lanes(mp.n));
    hipLaunchKernelGGL(tree_dd_leaf_kernel, dim3((unsigned)((count + per - 1) / per)), dim3(treedd::kThreads), 0, st, mp,
                       g0, count, static_cast<cdd*>(terms));
    return hipGetLastError();
}

}  // namespace gbs
