#pragma once
// Subset tree in double-double (see tree_device.h for the method).  A complex
// dd multiply-add takes 48 FP64 instructions, so series products are spread over
// lanes by output coefficient instead of unrolled per lane: the loops stay rolled,
// a lane holds one accumulator, and every level down to the leaves goes through
// device memory, which costs little next to the arithmetic.  Bound by the issue
// of FP64 instructions at the deep levels (a lane's product has as many terms as
// its coefficient's index, so about half of the lanes work, and a solve is a chain
// of n steps), by the latency of those chains at the first ten.  Against the
// LDS-resident characteristic polynomial of each subset: N = 20 1.43 -> 0.27 ms,
// N = 28 5.67 -> 0.55 ms, N = 36 94 -> 6.7 ms, N = 41 1030 -> 60 ms.
// Included by lhaf_lds.hip alone (floating-point contraction is off there).
#include "dd.h"
#include "tree_device.h"

namespace gbs {

namespace treedd {

// Unnormalised accumulator: hi carries the sum rounded at every step, lo the
// exact rounding errors and the products' low parts (a compensated dot product
// of dd operands); its error is a few n 2^-106 of the summed magnitudes, as that
// of n dd additions, at 12 instead of 27 instructions per real product.
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

// Block of a node (coefficient k of entry e at base[k stride + e]).
struct Block {
    cdd* base;
    int stride;
};
__device__ __forceinline__ Block node_block(const TreeMap& mp, int level, uint64_t g) {
    const uint64_t b = g & ((1ull << level) - 1ull);
    const int z = b ? __builtin_ctzll(b) : level;
    const int lv = level - z;
    const uint64_t slot = b ? (g >> z) >> 1 : g >> level;
    const int E = tree_entries(mp.n - lv);
    return Block{reinterpret_cast<cdd*>(mp.arena) + mp.off[lv] + (slot - mp.win[lv]) * (uint64_t)(E * (mp.n + 1)), E};
}

constexpr int kThreads = 256;      // 16 or 8 solves at a time
constexpr int kWideThreads = 512;   // a node on several workgroups: what each repeats should be short

// A solve runs on 16 or 32 lanes, one per coefficient (n <= 31).
__host__ __device__ constexpr int solve_lanes(int n) { return n <= 16 ? 16 : 32; }
__host__ __device__ constexpr int lds_stride(int n) { return n | 1; }  // odd: spreads the series over the banks
// LDS series per node: y (W + 1, the last y_v), z (W), the power sums of the two
// vertices, the updated row of v (W + 2), and with `rows` the row of u (W + 1)
__host__ __device__ constexpr int lds_series(int T, bool rows) {
    return 3 * (2 * T + 1) + 5 + (rows ? 2 * T + 2 : 0);
}

}  // namespace treedd

// Include children of parents g0 .. g0 + count - 1 of `level`, `per` parents per
// workgroup; gridDim.y workgroups share the couplings of the same parents and
// each repeat the solves.  ROWS: the row of u is copied to LDS; otherwise it is
// read from the parent's block (the row of v, which changes, always moves to LDS).
template <bool ROWS>
__global__ void __launch_bounds__(treedd::kWideThreads) tree_dd_elim_kernel(TreeMap mp, int level, uint64_t g0,
                                                                            uint64_t count, int per) {
    using namespace treedd;
    extern __shared__ double4 lds_dd[];
    cdd* lds = reinterpret_cast<cdd*>(lds_dd);
    const int n = mp.n, T = n - level - 1, W = 2 * T + 1, E = tree_entries(T), R = 2 * W + 3;
    const int ns = lds_stride(n), sl = lds_series(T, ROWS), P = solve_lanes(n);
    const int tid = threadIdx.x, NT = blockDim.x, kl = tid & (P - 1);
    const uint64_t first = (uint64_t)blockIdx.x * per;
    const int nodes = (int)min((uint64_t)per, count - first);
    auto parent = [&](int c) { return treedd::node_block(mp, level, g0 + first + c); };
    auto child = [&](int c) {
        return Block{reinterpret_cast<cdd*>(mp.arena) + mp.off[level + 1] +
                         (g0 + first + c - mp.win[level + 1]) * (uint64_t)(E * (n + 1)),
                     E};
    };
    auto y_at = [&](int c, int j, int k) -> cdd& { return lds[((c * sl) + j) * ns + k]; };              // j <= W
    auto z_at = [&](int c, int j, int k) -> cdd& { return lds[((c * sl) + W + 1 + j) * ns + k]; };      // j < W
    auto p_at = [&](int c, int q, int k) -> cdd& { return lds[((c * sl) + 2 * W + 1 + q) * ns + k]; };  // q < 2
    // row of u: u_j (j <= W, the last m_uu); row of v: v_j (j <= W + 1: m_uv, m_vv)
    auto v_at = [&](int c, int j, int k) -> cdd& { return lds[((c * sl) + 2 * W + 3 + j) * ns + k]; };
    auto u_at = [&](int c, const Block& pb, int j, int k) -> const cdd& {
        return ROWS ? lds[((c * sl) + 3 * W + 5 + j) * ns + k] : pb.base[k * pb.stride + E + j];
    };
    {
        const int r0 = ROWS ? 0 : W + 1, Q = R - r0;
        for (int q = tid; q < nodes * Q * n; q += NT) {
            const int c = q / (Q * n), x = q - c * (Q * n), k = x / Q, r = r0 + x - k * Q;
            const Block pb = parent(c);
            lds[((c * sl) + (r <= W ? 3 * W + 5 + r : W + 2 + r)) * ns + k] = pb.base[k * pb.stride + E + r];
        }
        __syncthreads();
    }
    for (int ph = 0; ph < 2; ++ph) {
        // y_j = m_uj / (1 - x m_uu), j < W and j = W (v), then z_j with the updated row
        // of v; j = -1: the power sums.  Lane k accumulates coefficient k; coefficient i
        // is complete at step i and handed to the others through LDS.
        const int solves = ph == 0 ? W + 2 : W + 1;
        for (int t0 = 0; t0 < nodes * solves; t0 += NT / P) {
            const int t = t0 + tid / P;
            const bool on = t < nodes * solves;
            const int c = on ? t / solves : 0, j = on ? t - c * solves - 1 : 0;
            const Block pb = parent(c);
            auto pivot = [&](int k) -> const cdd& { return ph == 0 ? u_at(c, pb, W, k) : v_at(c, W + 1, k); };
            cdd* out = j < 0 ? &p_at(c, ph, 0) : (ph == 0 ? &y_at(c, j, 0) : &z_at(c, j, 0));
            const bool mine = on && kl < n;
            Acc a{0.0, 0.0, 0.0, 0.0};
            if (mine) {
                if (j < 0) a = acc_of(cdd_mul_d(pivot(kl), (double)(kl + 1)));
                else if (ph == 0 && j < W) a = acc_of(u_at(c, pb, j, kl));
                else a = acc_of(v_at(c, j, kl));
            }
            for (int i = 0; i < n; ++i) {
                if (mine && kl == i) out[i] = value(a);
                tree::order_wave();
                if (mine && kl > i) treedd::mac(a, out[i], pivot(kl - 1 - i));
            }
        }
        __syncthreads();
        if (ph == 0) {
            // row of v: m_vj + x y_v m_uj (j < W), m_vv + x y_v m_uv; lanes of one
            // coefficient together.  m_uv itself stays.
            const int rows = nodes * (W + 1);
            for (int t = tid; t < rows * n; t += NT) {
                const int k = t / rows, q = t - k * rows, c = q / (W + 1), x = q - c * (W + 1);
                const Block pb = parent(c);
                const int j = x < W ? x : W + 1;
                Acc a = acc_of(v_at(c, j, k));
                for (int i = 0; i < k; ++i)
                    treedd::mac(a, y_at(c, W, i), x < W ? u_at(c, pb, x, k - 1 - i) : v_at(c, W, k - 1 - i));
                v_at(c, j, k) = value(a);
            }
            __syncthreads();
        }
    }
    if (blockIdx.y == 0)
        for (int t = tid; t < nodes * n; t += NT) {
        const int c = t / n, k = t - c * n;
        const Block pb = parent(c), cb = child(c);
        cb.base[k * cb.stride] = cdd_add(pb.base[k * pb.stride], cdd_add(p_at(c, 0, k), p_at(c, 1, k)));
    }
    // the children's couplings m_jk + x y_j m_uk + x z_j m_vk (the border's own held
    // times x, n + 1 coefficients)
    const int D = E - 1, all = nodes * D;
    for (int t = blockIdx.y * NT + tid; t < all * n + nodes; t += NT * gridDim.y) {
        int k, c, x;
        if (t < all * n) {
            k = t / all;
            const int q = t - k * all;
            c = q / D;
            x = q - c * D;
        } else {
            k = n;
            c = t - all * n;
            x = 0;
        }
        const Block pb = parent(c), cb = child(c);
        int j = (int)((__builtin_sqrtf(8.0f * (float)x + 1.0f) - 1.0f) * 0.5f);
        if (tree_tri(j + 1, 0) <= x) ++j;
        if (tree_tri(j, 0) > x) --j;
        const int k0 = x - tree_tri(j, 0);
        Acc a = acc_of(pb.base[k * pb.stride + 1 + x]);
        for (int i = 0; i < k; ++i) {
            treedd::mac(a, y_at(c, j, i), u_at(c, pb, k0, k - 1 - i));
            treedd::mac(a, z_at(c, j, i), v_at(c, k0, k - 1 - i));
        }
        cb.base[k * cb.stride + 1 + x] = value(a);
    }
}

// Signed terms of the leaves g0 .. g0 + count - 1 (subset masks), one on as many
// lanes as a solve: k e_k = sum_j (p_j + j q_j) / 2 e_(k-j), lane k - 1 holding e_k.
__global__ void __launch_bounds__(treedd::kThreads) tree_dd_leaf_kernel(TreeMap mp, uint64_t g0, uint64_t count,
                                                                        cdd* __restrict__ terms) {
    using namespace treedd;
    __shared__ cdd f[2 * kThreads], e[2 * kThreads];  // kThreads / P groups of P + 1
    const int n = mp.n, P = solve_lanes(n), grp = threadIdx.x / P, k = (threadIdx.x & (P - 1)) + 1;
    const uint64_t i0 = (uint64_t)blockIdx.x * (kThreads / P) + grp;
    if (i0 >= count) return;
    const uint64_t g = g0 + i0;
    const Block b = treedd::node_block(mp, n, g);
    cdd *fs = f + grp * (P + 1), *es = e + grp * (P + 1);
    const bool mine = k <= n;
    if (mine) {
        const cdd p = b.base[(k - 1) * b.stride], q = b.base[k * b.stride + 1];
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
    auto minus_i = [](cdd a) { return cdd{a.im, dd_neg(a.re)}; };
    auto neg = [](cdd a) { return cdd{dd_neg(a.re), dd_neg(a.im)}; };
    cdd v = cdd_zero();
    if (e > 0) {
        const int x = e - 1;
        int j = (int)((__builtin_sqrtf(8.0f * (float)x + 1.0f) - 1.0f) * 0.5f);
        if (tree_tri(j + 1, 0) <= x) ++j;
        if (tree_tri(j, 0) > x) --j;
        const int k = x - tree_tri(j, 0);
        const int pj = (j - 1) >> 1, pk = (k - 1) >> 1;
        const bool vj = ((j - 1) & 1) != 0, vk = ((k - 1) & 1) != 0;
        if (k == 0 && j > 0) {
            const dd h{0.70710678118654757, -4.8336466567264567e-17};  // 1 / sqrt 2
            const cdd a = loop(pj), b = loop(pj + n);
            v = cdd_mul_dd(vj ? minus_i(cdd_sub(a, b)) : cdd_add(a, b), h);
        } else if (k > 0) {
            const cdd a = at(pj, pk), b = at(pj, pk + n), c = at(pj + n, pk), d = at(pj + n, pk + n);
            cdd s = cdd_add(cdd_add(a, vk ? neg(b) : b), cdd_add(vj ? neg(c) : c, vj != vk ? neg(d) : d));
            s = cdd_mul_d(s, 0.5);
            v = (vj && vk) ? neg(s) : ((vj || vk) ? minus_i(s) : s);
        }
    }
    cdd* p = reinterpret_cast<cdd*>(mp.arena) + mp.off[0] + e;
    p[0] = v;
    for (int k = 1; k <= n; ++k) p[k * E] = cdd_zero();
}

hipError_t launch_tree_dd_root(const TreeMap& mp, const double2* A, int N, hipStream_t st) {
    hipLaunchKernelGGL(tree_dd_root_kernel, dim3((unsigned)((tree_entries(mp.n) + 63) / 64)), dim3(64), 0, st, mp, A, N);
    return hipGetLastError();
}

hipError_t launch_tree_dd_elim(const TreeMap& mp, int level, uint64_t g0, uint64_t count, hipStream_t st) {
    const int n = mp.n, T = n - level - 1;
    if (count == 0) return hipSuccess;
    if (n < 1 || n > kMaxDdPairs || T < 0) return hipErrorInvalidValue;
    static_assert(kMaxDdPairs <= 31, "a coefficient per lane of a half wavefront");
    const size_t series = sizeof(cdd) * (size_t)treedd::lds_stride(n);
    // Several wide workgroups per parent while there are fewer parents than two per
    // CU (N = 28: 0.55 ms with them, 0.90 ms with one workgroup each); the row of u in
    // LDS while a node's series take at most 64 KB; then as many nodes per
    // workgroup as fit 32 KB (five workgroups per CU).  N = 41: 60.9 ms; with 16, 24
    // or 40 KB 65.7, 62.6, 64.2 ms; with 128 threads 73.3, with 512 67.4 ms; with the
    // row of u always in memory 66.2 ms.
    const uint64_t units = (uint64_t)(tree_entries(T) - 1) * n;
    const unsigned slices =
        (unsigned)std::max<uint64_t>(1, std::min<uint64_t>((units + treedd::kWideThreads - 1) / treedd::kWideThreads, 512 / count));
    const bool rows = series * treedd::lds_series(T, true) <= 64 * 1024;
    const size_t node = series * treedd::lds_series(T, rows);
    const bool wide = count <= 512 && units > treedd::kThreads;
    const int per = wide ? 1 : (int)std::min<uint64_t>(count, std::max<size_t>(1, std::min<size_t>(16, 32 * 1024 / node)));
    const size_t lds = node * per;
    static_assert(sizeof(cdd) * treedd::lds_stride(kMaxDdPairs) * treedd::lds_series(kMaxDdPairs - 1, false) <= 160 * 1024,
                  "LDS of the largest elimination");
    const auto k = rows ? tree_dd_elim_kernel<true> : tree_dd_elim_kernel<false>;
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k, dim3((unsigned)((count + per - 1) / per), wide ? slices : 1),
                       dim3(wide ? treedd::kWideThreads : treedd::kThreads), lds, st, mp, level, g0, count, per);
    return hipGetLastError();
}

hipError_t launch_tree_dd_leaf(const TreeMap& mp, uint64_t g0, uint64_t count, void* terms, hipStream_t st) {
    if (count == 0) return hipSuccess;
    const unsigned per = (unsigned)(treedd::kThreads / treedd::solve_lanes(mp.n));
    hipLaunchKernelGGL(tree_dd_leaf_kernel, dim3((unsigned)((count + per - 1) / per)), dim3(treedd::kThreads), 0, st, mp,
                       g0, count, static_cast<cdd*>(terms));
    return hipGetLastError();
}

}  // namespace gbs
