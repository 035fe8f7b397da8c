#pragma once
// Subset tree: the signed terms t_S of all 2^n pair subsets by Schur
// complements over power series (gfx950 / CDNA4).
//
// With X the pair swap and C_S = X_S A0_S,
//     sum_k tr(C_S^k) x^k / k           = -log det(X - x A0)_S (up to the sign of det X),
//     sum_k (d^T C_S^(k-1) X d)_S x^k   = x d_S^T (X - x A0)_S^-1 d_S,
// and both follow from eliminating the pairs (u, v) of S one by one from the
// bordered matrix [[., d^T], [d, A0]] over power series in x.  With a = m_uu,
// b = m_uv and c = m_vv the pivot block of a pair is [[-x a, 1 - x b],
// [1 - x b, -x c]], and 1 - x b is pivoted on:
//     y_j  = m_uj / (1 - x b),  h = a / (1 - x b)   (triangular Toeplitz solves)
//     v_j' = m_vj + x c y_j,    u_j' = m_uj + x h m_vj,    b' = b + x c h,
//     z_j  = v_j' / (1 - x b'),
//     m_jk <- m_jk + x y_j m_vk + x z_j u_k'        (symmetric, j >= k is kept),
//     sum_k p_k x^k gains x (x b)' / (1 - x b) and the same of b'  (the same solves).
// No division by a small number occurs (pivots start with 1).  Scaling vertex u by
// s and v by 1 / s leaves every term as it is and scales each quantity above as a
// whole, by powers of two exactly: a matrix with large u and small v rows, or
// loop weights, loses nothing.  (A rotation of each pair to a symmetric M with
// M_S ~ C_S needs one row update less, but mixes the two scales, and powers of M
// then cancel: with the second halves' vertices scaled by 1/30, 1/100, 1/1000 the
// error over sum |t_S| was 2e-14, 2e-11, 9e-7 at N = 16; this way it is 1e-16 at
// any scale.)  Eliminating a pair serves every subset that shares it: the subsets
// form a binary tree whose root has eliminated nothing, where a node with T pairs
// left has an exclude child (the entries without that pair, not copied) and an
// include child (the updated entries).  Levels close to the root are shared by
// many subsets; a level of T remaining pairs costs a subset about 2^-T (2T)^2
// series products, in all about 40 products of n^2 / 2 complex multiply-adds
// against the about 47000 multiply-adds a Hessenberg reduction and characteristic
// polynomial of the same subset take on average at n = 25.
//
// Entry list of a node with T pairs left (E_T = 1 + (2T+1)(T+1) series of n
// coefficients): 0: the power sums p_1..p_n so far; 1 + tri(j, k), j >= k, the
// coupling of vertices j and k, vertex 0 being the border, vertices 2i+1 and
// 2i+2 pair i.  Entry 1, the border with itself, is held times x (n + 1
// coefficients, the first zero): it alone takes its products without the
// factor x of the others, and so all entries are updated alike.  Entry 0 is held
// in coefficients 1..n.  The last pair is eliminated first, so an exclude
// child's list is a prefix of its parent's.
//
// Work split: one lane per series product, all coefficients of the operands in
// registers (n^2 / 2 complex multiply-adds from one 16 n byte load of one
// operand; the other operand is streamed from LDS, one coefficient per n
// multiply-adds), so the kernels are bound by FP64 FMA issue and not by LDS or
// cross-lane traffic.

#include <type_traits>

#include "tree_kernels.h"

namespace gbs {

// Subset-tree geometry -------------------------------------------------------
__host__ __device__ constexpr int tree_tri(int j, int k) { return j * (j + 1) / 2 + k; }
// LDS series of tree_elim_kernel, T pairs left after the elimination.
__host__ __device__ constexpr int tree_temps(int T) { return 8 * T + 9; }
constexpr int kTreeDepth = 5;  // pairs of the subtrees that one wavefront finishes

namespace tree {

__device__ __forceinline__ void order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// The same for LDS only (LDS accesses of one wavefront execute in order, so this
// only keeps the compiler from reordering them).
__device__ __forceinline__ void order_wave() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Keeps reads and multiply-adds where they stand in the source, through all
// compiler passes: a and b are computed before, later reads come after.
__device__ __forceinline__ void keep_order(double2& a, double2& b) {
    asm volatile("" : "+v"(a.x), "+v"(a.y), "+v"(b.x), "+v"(b.y)::"memory");
    __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ double2 mac(double2 a, double2 b, double2 c) {
    return make_double2(fma(-a.y, b.y, fma(a.x, b.x, c.x)), fma(a.y, b.x, fma(a.x, b.y, c.y)));
}

// A node's block in device memory: coefficient k of entry e at base[k stride + e],
// so lanes with consecutive entries access consecutive 16-byte values.  Both
// members are wave-uniform.
typedef double Raw __attribute__((ext_vector_type(2)));
struct Block {
    double2* base;
    int stride;
};
// Reads or writes one entry's coefficients in order.  The address steps in scalar
// registers (kept opaque: the addresses of many coefficients held at once would
// spill), so an access costs no vector address arithmetic.
struct Cursor {
    using Byte = __attribute__((address_space(1))) char;
    using Vec = __attribute__((address_space(1))) Raw;
    Byte* p;
    int step;
    uint32_t o;
    __device__ __forceinline__ Cursor(const Block& a, int e) : p((Byte*)(a.base)), step(a.stride * 16), o(e * 16u) {}
    __device__ __forceinline__ void next() {
        p += step;
        asm volatile("" : "+s"(p));
    }
    __device__ __forceinline__ double2 get(int) {
        const Raw v = *(Vec*)(p + o);
        next();
        return make_double2(v.x, v.y);
    }
    __device__ __forceinline__ void put(int, double2 v) {
        *(Vec*)(p + o) = Raw{v.x, v.y};
        next();
    }
};
// One series in LDS, PLANE (or `plane`) entries per coefficient.
template <int PLANE>
struct LdsSeries {
    double2* p;
    __device__ __forceinline__ double2 get(int k) const { return p[k * PLANE]; }
    __device__ __forceinline__ void put(int k, double2 v) const { p[k * PLANE] = v; }
};
// Series products in order of the larger index: step d multiplies y_d and m_d
// with the lower coefficients, so the first products start as soon as the first
// coefficients arrive, coefficient d > n / 2 is needed in its own step only
// (half of each operand stays in registers), output k is first touched in step
// k / 2 and complete after step k - 1.  Operands are read kAhead steps ahead, in
// source order (left to itself the compiler moves all reads to the front and
// spills).
template <int NN>
constexpr int kAhead = NN < 28 ? 4 : 3;  // n = 28 spills with 4

// acc_k += sum_(i + j = k - 1) y_i m_j for k <= K (K <= NN); Y, M: get(k), called in order.
template <int NN, int K, class Y, class M>
__device__ __forceinline__ void conv(double2 (&acc)[NN + 1], Y ys, M ms) {
    double2 y[NN], m[NN];
#pragma unroll
    for (int d = 0; d < kAhead<NN> && d < K; ++d) {
        y[d] = ys.get(d);
        m[d] = ms.get(d);
    }
#pragma unroll
    for (int d = 0; d < K; ++d) {
        if (d + kAhead<NN> < K) {
            y[d + kAhead<NN>] = ys.get(d + kAhead<NN>);
            m[d + kAhead<NN>] = ms.get(d + kAhead<NN>);
        }
#pragma unroll
        for (int i = 0; i <= d; ++i) {
            if (i + d + 1 <= K) {
                if (i < d) acc[i + d + 1] = mac(y[i], m[d], acc[i + d + 1]);
                acc[i + d + 1] = mac(y[d], m[i], acc[i + d + 1]);
            }
        }
        keep_order(acc[d + 1], acc[2 * d + 1 < K ? 2 * d + 1 : K]);
    }
}

// out_k = in_k + sum_(i + j = k - 1) y_i m_j, k < NN: inputs read when first
// touched, outputs written when complete (In and Out may be the same series).
template <int NN, class Y, class M, class In, class Out>
__device__ __forceinline__ void conv_stream(Y ys, M ms, In in, Out out) {
    double2 y[NN], m[NN], acc[NN + 1];
    acc[0] = in.get(0);
    constexpr int K = NN - 1;
#pragma unroll
    for (int d = 0; d < kAhead<NN> && d < K; ++d) {
        y[d] = ys.get(d);
        m[d] = ms.get(d);
        if (d > 0) acc[2 * d] = 2 * d < NN ? in.get(2 * d) : acc[0];
        if (2 * d + 1 < NN) acc[2 * d + 1] = in.get(2 * d + 1);
    }
    out.put(0, acc[0]);
#pragma unroll
    for (int d = 0; d < K; ++d) {
        const int q = d + kAhead<NN>;
        if (q < K) {
            y[q] = ys.get(q);
            m[q] = ms.get(q);
        }
        if (2 * q < NN) acc[2 * q] = in.get(2 * q);
        if (2 * q + 1 < NN) acc[2 * q + 1] = in.get(2 * q + 1);
#pragma unroll
        for (int i = 0; i <= d; ++i) {
            if (i + d + 1 < NN) {
                if (i < d) acc[i + d + 1] = mac(y[i], m[d], acc[i + d + 1]);
                acc[i + d + 1] = mac(y[d], m[i], acc[i + d + 1]);
            }
        }
        out.put(d + 1, acc[d + 1]);
        keep_order(acc[d + 1], acc[2 * d + 1 < NN ? 2 * d + 1 : NN - 1]);
    }
}

// y = r / (1 - x u), r_k scaled by 1 + scale k: y_d is complete before step d,
// handed to done(d, y_d), and multiplies u_0..u_d; u_d multiplies y_0..y_(d-1).
template <int NN, class U, class R, class F>
__device__ __forceinline__ void solve(U us, R rs, double scale, F done) {
    double2 y[NN], u[NN];
    auto rhs = [&](int k) {
        const double2 r = rs.get(k);
        const double f = fma(scale, (double)k, 1.0);
        y[k] = make_double2(r.x * f, r.y * f);
    };
    y[0] = rs.get(0);
#pragma unroll
    for (int d = 0; d < kAhead<NN>; ++d) {
        if (d + 1 < NN) u[d] = us.get(d);
        if (d > 0 && 2 * d < NN) rhs(2 * d);
        if (2 * d + 1 < NN) rhs(2 * d + 1);
    }
#pragma unroll
    for (int d = 0; d < NN; ++d) {
        const int q = d + kAhead<NN>;
        if (q + 1 < NN) u[q] = us.get(q);
        if (2 * q < NN) rhs(2 * q);
        if (2 * q + 1 < NN) rhs(2 * q + 1);
        done(d, y[d]);
#pragma unroll
        for (int i = 0; i <= d; ++i) {
            if (i + d + 1 < NN) {
                y[i + d + 1] = mac(y[d], u[i], y[i + d + 1]);
                if (i < d) y[i + d + 1] = mac(y[i], u[d], y[i + d + 1]);
            }
        }
        if (d + 1 < NN) keep_order(y[d + 1], y[2 * d + 1 < NN ? 2 * d + 1 : NN - 1]);
    }
}

// Value of the even (P = 0) or odd (P = 1) lane of the caller's pair of lanes.
template <int P>
__device__ __forceinline__ double pair_bcast(double x) {
    const long long b = __double_as_longlong(x);
    constexpr int ctrl = P ? 0xF5 : 0xA0;  // quad_perm 1 1 3 3, 0 0 2 2
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, ctrl, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), ctrl, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// The same products on a pair of lanes, each with the outputs of its parity p
// (half of the multiply-adds): out_k = in_k + sum_(i + j = k - 1) y_i m_j for k =
// 2t + p.  With m'_j = m_(j-1+p), m'_0 = 0 for p = 0, output t takes the products
// with i + j = 2t on either lane.  SOLVE: y is the output itself (out = in / (1 -
// x m)), handed over between the lanes.  Every in_k is read before out_k is
// written, and m_k, too.  in_k is scaled by 1 + scale k.  For odd NN the odd lane
// also reads and writes coefficient NN, with no meaning.  In tree_sub_kernel<25> a
// solve takes 5400 cycles this way and 7900 on single lanes, a round of row updates
// 4300 and 6650 (5200 are the multiply-adds of a whole product).
template <int NN, bool SOLVE, class Y, class M, class In, class Out>
__device__ __forceinline__ void half_products(int p, double scale, Y ys, M ms, In in, Out out) {
    constexpr int H = (NN + 1) / 2, D = 2 * H - 1, A = kAhead<NN>;
    double2 y[D], m[D], acc[H];
    auto load_m = [&](int d) { m[d] = ms.get(d == 0 ? 0 : d - 1 + p); };
    auto load_in = [&](int t) {
        const double2 r = in.get(2 * t + p);
        if (SOLVE) {
            const double f = fma(scale, (double)(2 * t + p), 1.0);
            acc[t] = make_double2(r.x * f, r.y * f);
        } else {
            acc[t] = r;
        }
    };
    load_m(0);
    m[0] = make_double2(p ? m[0].x : 0.0, p ? m[0].y : 0.0);
#pragma unroll
    for (int d = 0; d < A; ++d) {
        if (d + 1 < D) load_m(d + 1);
        if (!SOLVE && d < D) y[d] = ys.get(d);
        if (d < H) load_in(d);
    }
    // step d: y_d with m'_0..m'_(d+1) and m'_(d+1) with the lower y, so that out_(d+1)
    // is complete after it on either lane
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const int q = d + A;
        if (q + 1 < D) load_m(q + 1);
        if (!SOLVE && q < D) y[q] = ys.get(q);
        if (q < H) load_in(q);
        if (SOLVE)
            y[d] = (d & 1) ? make_double2(pair_bcast<1>(acc[d / 2].x), pair_bcast<1>(acc[d / 2].y))
                           : make_double2(pair_bcast<0>(acc[d / 2].x), pair_bcast<0>(acc[d / 2].y));
#pragma unroll
        for (int i = 0; i <= d; i += 2) {
            const int j = i + (d & 1), l = i + ((d + 1) & 1);
            if (l < d && l + d + 1 < D) acc[(l + d + 1) / 2] = mac(y[l], m[d + 1], acc[(l + d + 1) / 2]);
            if (d + j < D) acc[(d + j) / 2] = mac(y[d], m[j], acc[(d + j) / 2]);
        }
        if (!(d & 1)) out.put(d + p, acc[d / 2]);
        keep_order(acc[(d + 1) / 2 < H ? (d + 1) / 2 : H - 1], acc[d < H ? d : H - 1]);
    }
}

// Eliminates the last pair of a parent (block pb, T pairs left afterwards) and
// writes its include child (block cb): the couplings d0 <= d < d1 of its
// (2T+1)(T+1), and with d0 = 0 the power sums.  LDS (PLANE >= tree_temps(T)
// series): row u (W + 1, updated in place, h over a), row v (W + 2, b' over b) of
// the pair's vertices, y (W), v' and then z (W) and the two power sums, W = 2T + 1.
// The rows are read in one go: taken from device memory coefficient by coefficient,
// the solves waited for it (84 us instead of 50 for 2048 nodes at n = 25).
template <int NN, int PLANE>
__device__ __forceinline__ void elim_pair(Block pb, Block cb, double2* lds, int T, int d0, int d1) {
    const int lane = threadIdx.x;
    const int W = 2 * T + 1;
    auto tmp = [&](int slot) { return LdsSeries<PLANE>{lds + slot}; };
    {
        const int R = 2 * W + 3, E = tree_entries(T);
        for (int q = lane; q < R * NN; q += 64) {
            const int k = q / R, e = q - k * R;
            lds[k * PLANE + e] = pb.base[k * pb.stride + E + e];
        }
    }
    order();
    const int j = lane - 1;
#pragma unroll 1
    for (int ph = 0; ph < 2; ++ph) {
        // phase 0: y_j for every other vertex j < W and h (j = W); phase 1: z_j;
        // j = -1: the power sums
        if (j <= (ph == 0 ? W : W - 1)) {
            const int su = 2 * W + 1;
            const int sz = 2 * W + 3 + ph * W + j;
            const LdsSeries<PLANE> to = tmp(j < 0 ? PLANE - 2 + ph : (j < W ? sz : W));
            solve<NN>(tmp(su), tmp(j < 0 ? su : (ph == 0 ? j : sz)), j < 0 ? 1.0 : 0.0,
                      [&](int k, double2 v) { to.put(k, v); });
        }
        order_wave();
        // v_j' to the place of z_j (t < W), b' (t = W) and u_j' (t > W)
        for (int t = lane; ph == 0 && t <= 2 * W; t += 64) {
            const int su = t <= W ? W + 1 + t : t - W - 1;
            conv_stream<NN>(tmp(t < W ? 2 * W + 3 + t : W), tmp(t <= W ? 2 * W + 2 : t), tmp(su),
                            tmp(t < W ? 3 * W + 3 + t : su));
        }
        order_wave();
    }
    if (d0 == 0 && lane < NN) {
        const double2 p = pb.base[(lane + 1) * pb.stride], u = tmp(PLANE - 2).get(lane), v = tmp(PLANE - 1).get(lane);
        cb.base[(lane + 1) * cb.stride] = make_double2(p.x + u.x + v.x, p.y + u.y + v.y);
    }
    // the child's couplings m_jk + x y_j m_vk + x z_j u_k'; the border's own is
    // held times x, so that it takes the same products
    for (int x = d0 + lane; x < d1; x += 64) {
        int i = (int)((__builtin_sqrtf(8.0f * (float)x + 1.0f) - 1.0f) * 0.5f);
        if (tree_tri(i + 1, 0) <= x) ++i;
        if (tree_tri(i, 0) > x) --i;
        const int k0 = x - tree_tri(i, 0);
        double2 acc[NN + 1];
        Cursor in(pb, 1 + x), out(cb, 1 + x);
#pragma unroll
        for (int k = 0; k <= NN; ++k) acc[k] = in.get(k);
#pragma unroll 1
        for (int ph = 0; ph < 2; ++ph)
            conv<NN, NN>(acc, tmp(2 * W + 3 + ph * W + i), tmp(k0 + (1 - ph) * (W + 1)));
#pragma unroll
        for (int k = 0; k <= NN; ++k) out.put(k, acc[k]);
    }
}

// e_n of exp(sum_k (p_k / 2k + q_k / 2) x^k): k e_k = sum_j (p_j + j q_j) / 2 e_(k-j),
template <int NN, class S>
__device__ __forceinline__ double2 leaf_term(S ps, S qs) {
    double2 f[NN], acc[NN + 1];
#pragma unroll
    for (int k = 0; k < NN; ++k) {
        const double2 p = ps.get(k), q = qs.get(k);
        f[k] = make_double2(0.5 * fma((double)(k + 1), q.x, p.x), 0.5 * fma((double)(k + 1), q.y, p.y));
        acc[k + 1] = make_double2(0.0, 0.0);
    }
    acc[0] = make_double2(1.0, 0.0);
#pragma unroll
    for (int i = 0; i < NN; ++i) {
        if (i > 0) acc[i] = make_double2(acc[i].x * (1.0 / i), acc[i].y * (1.0 / i));
#pragma unroll
        for (int k = i + 1; k <= NN; ++k) acc[k] = mac(acc[i], f[k - 1 - i], acc[k]);
        keep_order(acc[i + 1], acc[NN]);
    }
    return make_double2(acc[NN].x * (1.0 / NN), acc[NN].y * (1.0 / NN));
}

// Level-0 entries of one root: with a = A with zero diagonal, symmetrised, and d its
// diagonal, vertices 2i + 1 and 2i + 2 being rows i + n and i: entry (j, k) = a_jk,
// entry (j, border) = d_j, constant series.  An odd N gets one more vertex with
// loop weight 1 and no edges.  (Which row of a pair comes first is free: the
// terms' errors are of one size.  At N = 40 of the benchmark family the sum's is
// 2.6e-18 of sum |t_S| this way and 6e-19 with i first, 1e-19 to 2.5e-18 over
// permutations of the pairs; the comparison with long doubles in the tests asks
// that it be more than 20 times theirs, 8e-20.)
__device__ __forceinline__ int root_row(int j, int n) { return ((j - 1) >> 1) + (((j - 1) & 1) ? 0 : n); }
__device__ __forceinline__ double2 root_at(const double2* A, int N, int r, int c) {
    if (r == c || r >= N || c >= N) return make_double2(0.0, 0.0);
    const double2 x = A[r * N + c], y = A[c * N + r];
    return make_double2(0.5 * (x.x + y.x), 0.5 * (x.y + y.y));
}
__device__ __forceinline__ double2 root_loop(const double2* A, int N, int r) {
    return r < N ? A[r * N + r] : make_double2(1.0, 0.0);
}

// Coefficient 0 of entry e, the only one that is not zero.
__device__ __forceinline__ double2 root_entry(const double2* A, int N, int n, int e) {
    double2 v = make_double2(0.0, 0.0);
    if (e > 0) {
        const int x = e - 1;
        int j = (int)((__builtin_sqrtf(8.0f * (float)x + 1.0f) - 1.0f) * 0.5f);
        if (tree_tri(j + 1, 0) <= x) ++j;
        if (tree_tri(j, 0) > x) --j;
        const int k = x - tree_tri(j, 0);
        if (j > 0) v = k == 0 ? root_loop(A, N, root_row(j, n)) : root_at(A, N, root_row(j, n), root_row(k, n));
    }
    return v;
}
// Matrix and dimension of root r of a forest.
__device__ __forceinline__ const double2* root_matrix(const TreeSource& src, uint64_t r, int& N) {
    N = src.N;
    if (!src.list) return src.mats;
    const int i = src.list[r];
    N = src.dims[i];
    return src.mats + src.in_off[i];
}

// Block of node g (level `level` of its item's tree; the item's root is level 0):
// that of the include child nearest above it, or the root's.
__device__ __forceinline__ Block node_block(const TreeMap& mp, int level, uint64_t g) {
    const uint64_t b = g & ((1ull << level) - 1ull);
    const int z = b ? __builtin_ctzll(b) : level;
    const int lv = level - z;
    const uint64_t slot = b ? (g >> z) >> 1 : g >> level;
    const int E = tree_entries(mp.n - lv);
    return Block{mp.arena + mp.off[lv] + (slot - mp.win[lv]) * (uint64_t)(E * (mp.n + 1)), E};
}

__device__ __forceinline__ bool node_active(const TreeShard& sh, int n, int level, uint64_t b) {
    if (!sh.on) return true;
    const int T = n - level;
    const int pc = __popcll(b);
    const uint64_t lo = b << T, hi = (b + 1) << T;  // masks lo..hi-1
    for (int s = pc; s <= pc + T; ++s)
        if (sh.lo[s] < hi && sh.hi[s] > lo) return true;
    return false;
}

// Node order of a shard's launch: workgroups go round robin to the 8 XCDs and a
// node's low bits decide, through their number, whether it is active, so the low
// three bits are scrambled by the others (a permutation of each aligned 8).
__device__ __forceinline__ uint32_t shard_order(const TreeShard& sh, uint32_t i, uint32_t count) {
    return (sh.on && (count & 7u) == 0) ? i ^ (((i >> 3) * 0x9E3779B1u) >> 29) : i;
}

}  // namespace tree

// One include child per `slices` wavefronts: parents g0 .. g0 + count - 1 of
// `level`.  The couplings of large nodes are split over the slices (each does
// the short solves itself), so that the few nodes near the root fill the device.
template <int NN, int PLANE>
__global__ void __launch_bounds__(64, (NN <= 25 ? 2 : 1)) tree_elim_kernel(TreeMap mp, TreeShard sh, int level, uint64_t g0, int slices) {
    extern __shared__ double2 lds[];
    const int T = mp.n - level - 1;
    const uint64_t g = g0 + tree::shard_order(sh, blockIdx.x / slices, gridDim.x / slices);
    const int sl = blockIdx.x % slices;
    if (!tree::node_active(sh, mp.n, level + 1, 2 * (g & ((1ull << level) - 1ull)) + 1)) return;
    const int E = tree_entries(T) - 1;
    const int per = (((E + slices - 1) / slices) + 63) & ~63;
    const int d0 = sl * per, d1 = min(E, d0 + per);
    if (d0 >= d1) return;
    const tree::Block pb = tree::node_block(mp, level, g);
    const tree::Block cb{mp.arena + mp.off[level + 1] + (g - mp.win[level + 1]) * (uint64_t)((E + 1) * (NN + 1)), E + 1};
    tree::elim_pair<NN, PLANE>(pb, cb, lds, T, d0, d1);
}

// LDS series per parent while a pair is eliminated, T pairs left after it, in
// tree_sub_kernel: row u (W + 1, updated in place, h over a) and row v (W + 2, b'
// over b) of the pair's vertices and y (W, then v', then z), W = 2T + 1, and where a
// solve runs on pairs of lanes in both phases the first power sums.
__host__ __device__ constexpr int tree_slots(int T) { return T >= 2 ? 6 * T + 7 : 6 * T + 6; }
constexpr int kTreeOne = 96;  // 2^(4-T) parents, T = 0..4; the series 1 after them
constexpr int kTreeSlots = 97;
__host__ __device__ constexpr int tree_lanes(int T) { return T == 0 ? 4 : tree_entries(T); }

// Row updates of T <= 2 (44 to 56 rows) as one round of whole products, 6650 cycles
// at n = 25, not two on pairs of lanes, 8600; n = 12 at two waves per SIMD, 27 and 28
// would need scratch for it.
template <int NN>
constexpr bool kTreeWholeRows = NN <= 26 && NN != 12;

// The subtree of up to kTreeDepth pairs below nodes g0 + blockIdx.x of `level`:
// one wavefront per node, all its subset terms summed in a fixed order
// into one record (sum re, compensation, sum im, compensation, sum |t|).
//
// The subtree runs breadth first with its entries in registers: at each level
// lane c L + e holds entry e of parent c's exclude child (sa) and include child
// (sb), 2^(4-T) parents of at most 64 entries in all, and only the eliminated
// pair's rows and the y and z series, which other lanes read, go through LDS.
// (With the entries of each level in device memory instead, 134 KB a wavefront
// at n = 25, the kernel moved 150 GB at N = 44 and kept the VALU 33% busy.)
// Between levels the entries change lanes through one 2 KB LDS line per
// coefficient.  Bound by FP64 issue: 65536 nodes at n = 25 take 5.37 ms (85 us
// per 1024), in which the SIMDs issue a VALU instruction in 65% of the cycles, 84%
// of them FP64 FMAs.  Of a wavefront's time the couplings take 32%, on 45 to 60 of
// 64 lanes, the first solves 19%, the second ones 13%, the row updates 15%, the
// changes of lanes 13%, the leaves 5%.  (With all products on single lanes, and one
// row update less, it was 112 us per 1024 nodes, then 95 on pairs of lanes, in
// launches of 1024.)
template <int NN>
__global__ void __launch_bounds__(64, (NN <= 12 ? 2 : 1))
    tree_sub_kernel(TreeMap mp, TreeShard sh, int level, uint64_t g0, double* __restrict__ records, TreeSource src,
                    uint64_t r0) {
    extern __shared__ double2 lds[];
    constexpr int PL = kTreeSlots;
    double2* line = lds + NN * PL;
    const int lane = threadIdx.x;
    auto row = [&](int slot) { return tree::LdsSeries<PL>{lds + slot}; };
    const int T0 = mp.n - level;  // pairs left, 1..kTreeDepth
    const uint32_t i = tree::shard_order(sh, blockIdx.x, gridDim.x);
    const uint64_t g = g0 + i;
    const uint64_t b = g & ((1ull << level) - 1ull);
    double* rec = records + 5 * (int64_t)i;
    if (!tree::node_active(sh, mp.n, level, b)) {
        if (lane < 5) rec[lane] = 0.0;
        return;
    }
    double2 sa[NN + 1], sb[NN + 1];
    if (lane < NN) row(kTreeOne).put(lane, make_double2(lane == 0 ? 1.0 : 0.0, 0.0));
    // the node's prefix to sa, its last pair's rows to LDS
    if constexpr (NN <= kTreeDepth) {
        // a whole tree: from its matrix (with a kernel before this one that writes the
        // root's entries to memory N = 10 took 22.9 us, now 20.2)
        int N;
        const double2* A = tree::root_matrix(src, r0 + g, N);
        const int Ec = tree_entries(NN - 1), nr = tree_entries(NN) - Ec;
        const double2 va = tree::root_entry(A, N, NN, lane < Ec ? lane : 0);
        const double2 vr = tree::root_entry(A, N, NN, Ec + (lane < nr ? lane : 0));
#pragma unroll
        for (int k = 0; k <= NN; ++k) sa[k] = make_double2(k ? 0.0 : va.x, k ? 0.0 : va.y);
        if (lane < nr) {
#pragma unroll
            for (int k = 0; k < NN; ++k) row(lane).put(k, sa[1]);
            row(lane).put(0, vr);
        }
    } else {
        const tree::Block root = tree::node_block(mp, level, g);
        const int Ec = tree_entries(T0 - 1), nr = tree_entries(T0) - Ec;
        tree::Cursor pre(root, lane < Ec ? lane : 0), rows(root, Ec + (lane < nr ? lane : 0));
        double2 r[NN];
#pragma unroll
        for (int k = 0; k <= NN; ++k) sa[k] = pre.get(k);
#pragma unroll
        for (int k = 0; k < NN; ++k) r[k] = rows.get(k);
        if (lane < nr) {
#pragma unroll
            for (int k = 0; k < NN; ++k) row(lane).put(k, r[k]);
        }
    }
    for (int T = T0 - 1; T >= 0; --T) {
        const int P = 1 << (T0 - 1 - T), W = 2 * T + 1, E = tree_entries(T), L = tree_lanes(T);
        const int c = lane / L, x = lane - c * L;
        const bool on = c < P;
        if (T < T0 - 1) {
            // from the previous level: parent c is the exclude (c even) or include
            // child of its parent c / 2
            const int Lp = tree_lanes(T + 1), Ep = tree_entries(T + 1);
            const int cp = lane / Lp, ep = lane - cp * Lp;
            const bool rowp = cp < P / 2 && ep >= E && ep < Ep;
            const int slot = 2 * cp * tree_slots(T) + ep - E;
            if (rowp) {
#pragma unroll
                for (int k = 0; k < NN; ++k) {
                    row(slot).put(k, sa[k]);
                    row(slot + tree_slots(T)).put(k, sb[k]);
                }
            }
            const int from = on && x < E ? ((c >> 1) * Lp + x + 64 * (c & 1)) : lane;
#pragma unroll
            for (int k = 0; k <= NN; ++k) {
                line[lane] = sa[k];
                line[64 + lane] = sb[k];
                tree::order_wave();
                sa[k] = line[from];
                tree::order_wave();
            }
        }
#pragma unroll
        for (int k = 0; k <= NN; ++k) sb[k] = sa[k];
        tree::order_wave();
        const int tb = c * tree_slots(T);
        const int xc = max(x - 1, 0);  // coupling (j, k0)
        int j = (int)((__builtin_sqrtf(8.0f * (float)xc + 1.0f) - 1.0f) * 0.5f);
        if (tree_tri(j + 1, 0) <= xc) ++j;
        if (tree_tri(j, 0) > xc) --j;
        const int k0 = xc - tree_tri(j, 0);
#pragma unroll 1
        for (int ph = 0; ph < 2; ++ph) {
            // phase 0: y_j for every other vertex j < W and h (row W + 1); phase 1:
            // z_j; row 0: the power sums.  On pairs of lanes where 32 rows do.
            const int pl = lane & 1, rows = W + 2 - ph;
            if (ph == 0 && T < 2) {
                if (on && x <= W + 1) {
                    const int su = tb + 2 * W + 1;
                    double2 y[NN];
                    tree::solve<NN>(row(su), row(x == 0 ? su : tb + x - 1), x == 0 ? 1.0 : 0.0,
                                    [&](int k, double2 v) { y[k] = v; });
                    tree::order_wave();
                    if (x == 0) {
#pragma unroll
                        for (int k = 0; k < NN; ++k) sb[k + 1] = make_double2(sb[k + 1].x + y[k].x, sb[k + 1].y + y[k].y);
                    } else {
                        const int so = x == W + 1 ? W : 2 * W + 2 + x;
#pragma unroll
                        for (int k = 0; k < NN; ++k) row(tb + so).put(k, y[k]);
                    }
                }
            } else {
                const int cr = (lane >> 1) / rows, xr = (lane >> 1) - cr * rows, tr = cr * tree_slots(T);
                if (cr < P) {
                    const int su = tr + 2 * W + 1, sz = tr + 2 * W + 2 + xr;
                    const int sr = xr == 0 ? su : (ph == 0 ? tr + xr - 1 : sz);
                    const int so = xr == 0 ? tr + (ph == 0 ? 3 * W + 3 : W) : (xr == W + 1 ? tr + W : sz);
                    tree::half_products<NN, true>(pl, xr == 0 ? 1.0 : 0.0, row(su), row(su), row(sr), row(so));
                }
            }
            tree::order_wave();
            // the include child's couplings: m_jk + x y_j m_vk, then + x z_j u_k'; its
            // power sums (x = 0) are those of b and b' times 1
            if (on && x < E && (x > 0 || T >= 2 || ph == 1)) {
                const int sy = x == 0 ? (ph == 0 ? 3 * W + 3 : W) : 2 * W + 3 + j;
                tree::conv<NN, NN>(sb, row(tb + sy), row(x == 0 ? kTreeOne : tb + k0 + (ph == 0 ? W + 1 : 0)));
            }
            if (ph == 0) {
                // v_j' over y_j (xr < W), b' (xr = W) and u_j' (xr > W)
                auto update = [&](int t, auto&& products) {
                    const int cr = t / (2 * W + 1), xr = t - cr * (2 * W + 1), tr = cr * tree_slots(T);
                    if (cr < P) {
                        const int sr = xr <= W ? W + 1 + xr : xr - W - 1, sy = xr < W ? 2 * W + 3 + xr : W;
                        products(row(tr + sy), row(tr + (xr <= W ? 2 * W + 2 : xr)), row(tr + sr),
                                 row(tr + (xr < W ? sy : sr)));
                    }
                };
                if (T > 2 || !kTreeWholeRows<NN>) {
                    // (one round for T > 2)
#pragma unroll 1
                    for (int t = lane >> 1; t < P * (2 * W + 1); t += 32)
                        update(t, [&](auto y, auto m, auto in, auto out) {
                            tree::half_products<NN, false>(pl, 0.0, y, m, in, out);
                        });
                } else if constexpr (kTreeWholeRows<NN>) {
                    update(lane, [&](auto y, auto m, auto in, auto out) { tree::conv_stream<NN>(y, m, in, out); });
                }
                tree::order_wave();
            }
        }
    }
    // the 2^T0 leaves, one per lane: leaf 2c + s has its power sums and border
    // series in lanes 4c and 4c + 1 of sa (s = 0) or sb (s = 1)
    {
        const int x = lane & 3, sl = (lane >> 2) * 4 + x;
        tree::order_wave();
        if (x < 2) {
#pragma unroll
            for (int k = 0; k < NN; ++k) {
                lds[k * PL + sl] = sa[k + 1];
                lds[k * PL + sl + 2] = sb[k + 1];
            }
        }
        tree::order_wave();
    }
    double2 t = make_double2(0.0, 0.0);
    if (lane < (1 << T0)) {
        const uint64_t mask = (b << T0) | (uint64_t)lane;
        const int s = __popcll(mask);
        if (!sh.on || (mask >= sh.lo[s] && mask < sh.hi[s])) {
            t = tree::leaf_term<NN>(row(2 * lane), row(2 * lane + 1));
            if ((mp.n - s) & 1) t = make_double2(-t.x, -t.y);
        }
    }
    tree::order_wave();
    double sr = t.x, cr = 0.0, si = t.y, ci = 0.0, ab = sqrt(fma(t.x, t.x, t.y * t.y));
#pragma unroll
    for (int off = 1; off < (1 << kTreeDepth); off <<= 1) {
        // TwoSum of lanes l and l ^ off
        auto sh2 = [&](double v) {
            const int lo = __shfl_xor(__double2loint(v), off), hi = __shfl_xor(__double2hiint(v), off);
            return __hiloint2double(hi, lo);
        };
        const double br = sh2(sr), bcr = sh2(cr), bi = sh2(si), bci = sh2(ci), bab = sh2(ab);
        const double s1 = sr + br, v1 = s1 - sr;
        cr = (cr + bcr) + ((sr - (s1 - v1)) + (br - v1));
        sr = s1;
        const double s2 = si + bi, v2 = s2 - si;
        ci = (ci + bci) + ((si - (s2 - v2)) + (bi - v2));
        si = s2;
        ab += bab;
    }
    if (lane == 0) {
        rec[0] = sr;
        rec[1] = cr;
        rec[2] = si;
        rec[3] = ci;
        rec[4] = ab;
    }
}

}  // namespace gbs
