#pragma once
// Elimination of a pair with one series coefficient per lane (see tree_device.h
// for the method): a lane holds one accumulator, and several lanes share a
// parent.  AR is the arithmetic: V a coefficient, Acc an accumulator.
#include <algorithm>

#include "lhaf_kernels.h"
#include "tree_device.h"

namespace gbs {

namespace treelane {

// Block of a node (coefficient k of entry e at base[k stride + e]).
template <class V>
struct Block {
    V* base;
    int stride;
};
template <class V>
__device__ __forceinline__ Block<V> node_block(const TreeMap& mp, int level, uint64_t g) {
    const uint64_t b = g & ((1ull << level) - 1ull);
    const int z = b ? __builtin_ctzll(b) : level;
    const int lv = level - z;
    const uint64_t slot = b ? (g >> z) >> 1 : g >> level;
    const int E = tree_entries(mp.n - lv);
    return Block<V>{reinterpret_cast<V*>(mp.arena) + mp.off[lv] + (slot - mp.win[lv]) * (uint64_t)(E * (mp.n + 1)), E};
}

// A value of lane I of the caller's row of 16 lanes.
template <int I>
__device__ __forceinline__ double row_bcast(double x) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x150 + I, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x150 + I, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <int A, int B, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (A < B) {
        f(std::integral_constant<int, A>{});
        static_for<A + 1, B>(f);
    }
}

constexpr int kThreads = 256;      // 16 or 8 solves at a time

// A solve runs on 16 or 32 lanes, one per coefficient (n <= 31).
__host__ __device__ constexpr int solve_lanes(int n) { return n <= 16 ? 16 : 32; }
__host__ __device__ constexpr int lds_stride(int n) { return n | 1; }  // odd: spreads the series over the banks
// LDS series per node: y (W + 1, the last h), v' and then z (W), the two power
// sums, the updated row of u (W + 2: u_j', a, b'), and with `rows` the row of v
// (W + 1: m_vj, c)
__host__ __device__ constexpr int lds_series(int T, bool rows) {
    return 3 * (2 * T + 1) + 5 + (rows ? 2 * T + 2 : 0);
}


}  // namespace treelane

// Include children of parents g0 .. g0 + count - 1 of `level`, `per` parents per
// workgroup.  ROWS: the row of v is copied to LDS; otherwise it is read from the
// parent's block (the row of u, which changes, always moves to LDS).
template <class AR, bool ROWS>
__global__ void __launch_bounds__(treelane::kThreads) tree_lane_elim_kernel(TreeMap mp, int level, uint64_t g0,
                                                                            uint64_t count, int per) {
    using namespace treelane;
    using V = typename AR::V;
    using Acc = typename AR::Acc;
    extern __shared__ double4 lds_lane[];
    V* lds = reinterpret_cast<V*>(lds_lane);
    const int n = mp.n, T = n - level - 1, W = 2 * T + 1, E = tree_entries(T), R = 2 * W + 3;
    const int ns = lds_stride(n), sl = lds_series(T, ROWS), P = solve_lanes(n);
    const int tid = threadIdx.x, NT = blockDim.x, kl = tid & (P - 1);
    const uint64_t first = (uint64_t)blockIdx.x * per;
    const int nodes = (int)min((uint64_t)per, count - first);
    auto parent = [&](int c) { return treelane::node_block<V>(mp, level, g0 + first + c); };
    auto child = [&](int c) {
        return Block<V>{reinterpret_cast<V*>(mp.arena) + mp.off[level + 1] +
                         (g0 + first + c - mp.win[level + 1]) * (uint64_t)(E * (n + 1)),
                     E};
    };
    auto y_at = [&](int c, int j, int k) -> V& { return lds[((c * sl) + j) * ns + k]; };              // j <= W
    auto z_at = [&](int c, int j, int k) -> V& { return lds[((c * sl) + W + 1 + j) * ns + k]; };      // j < W
    auto p_at = [&](int c, int q, int k) -> V& { return lds[((c * sl) + 2 * W + 1 + q) * ns + k]; };  // q < 2
    // row of u: u_j (j < W), a (W), b (W + 1); row of v: m_vj (j < W), c (W)
    auto u_at = [&](int c, int j, int k) -> V& { return lds[((c * sl) + 2 * W + 3 + j) * ns + k]; };
    auto v_at = [&](int c, const Block<V>& pb, int j, int k) -> const V& {
        return ROWS ? lds[((c * sl) + 3 * W + 5 + j) * ns + k]
                    : pb.base[k * pb.stride + E + W + 1 + (j < W ? j : W + 1)];
    };
    {
        const int Q = ROWS ? R : W + 2;
        for (int q = tid; q < nodes * Q * n; q += NT) {
            const int c = q / (Q * n), x = q - c * (Q * n), k = x / Q, i = x - k * Q;
            const int r = ROWS || i <= W ? i : 2 * W + 1;  // of the parent's entries E ..: u (W + 1), m_vj (W), b, c
            const Block<V> pb = parent(c);
            const int to = r <= W ? 2 * W + 3 + r : (r <= 2 * W ? 2 * W + 4 + r : (r == 2 * W + 1 ? 3 * W + 4 : 4 * W + 5));
            lds[((c * sl) + to) * ns + k] = pb.base[k * pb.stride + E + r];
        }
        __syncthreads();
    }
    // unit t of the couplings: coefficient k of entry 1 + x of node c; a thread's
    // first one is read ahead of the solves
    const int D = E - 1, all = nodes * D, units = all * n + nodes, t1 = tid;
    auto unit = [&](int t, int& c, int& k, int& x) {
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
    };
    V m1{};
    if (t1 < units) {
        int c, k, x;
        unit(t1, c, k, x);
        const Block<V> pb = parent(c);
        m1 = pb.base[k * pb.stride + 1 + x];
    }
    for (int ph = 0; ph < 2; ++ph) {
        // y_j, j < W, and h (j = W), then z_j from the v_j' in its place; j = -1: the
        // power sums.  Lane k accumulates coefficient k; coefficient i is complete at
        // step i and handed to the others through LDS.
        const int solves = ph == 0 ? W + 2 : W + 1;
        for (int t0 = 0; t0 < nodes * solves; t0 += NT / P) {
            const int t = t0 + tid / P;
            const bool on = t < nodes * solves;
            const int c = on ? t / solves : 0, j = on ? t - c * solves - 1 : 0;
            auto pivot = [&](int k) -> const V& { return u_at(c, W + 1, k); };
            V* out = j < 0 ? &p_at(c, ph, 0) : (ph == 0 ? &y_at(c, j, 0) : &z_at(c, j, 0));
            const bool mine = on && kl < n;
            Acc a{};
            if (mine) {
                if (j < 0) a = AR::acc_of(AR::scale(pivot(kl), (double)(kl + 1)));
                else a = AR::acc_of(ph == 0 ? u_at(c, j, kl) : out[kl]);
            }
            for (int i = 0; i < n; ++i) {
                if (mine && kl == i) out[i] = AR::value(a);
                tree::order_wave();
                if (mine && kl > i) AR::mac(a, out[i], pivot(kl - 1 - i));
            }
        }
        __syncthreads();
        if (ph == 0) {
            // v_j' = m_vj + x y_j c (x < W), b' = b + x h c (x = W), u_j' = m_uj + x h m_vj;
            // lanes of one coefficient together
            const int rows = nodes * (2 * W + 1);
            for (int t = tid; t < rows * n; t += NT) {
                const int k = t / rows, q = t - k * rows, c = q / (2 * W + 1), x = q - c * (2 * W + 1);
                const Block<V> pb = parent(c);
                const int y = min(x, W), v = x <= W ? W : x - W - 1;
                V& io = x < W ? z_at(c, x, k) : u_at(c, x == W ? W + 1 : v, k);
                Acc a = AR::acc_of(x < W ? v_at(c, pb, x, k) : io);
                for (int i = 0; i < k; ++i) AR::mac(a, y_at(c, y, i), v_at(c, pb, v, k - 1 - i));
                io = AR::value(a);
            }
            __syncthreads();
        }
    }
    for (int t = tid; t < nodes * n; t += NT) {
        const int c = t / n, k = t - c * n;
        const Block<V> pb = parent(c), cb = child(c);
        cb.base[(k + 1) * cb.stride] = AR::add(pb.base[(k + 1) * pb.stride], AR::add(p_at(c, 0, k), p_at(c, 1, k)));
    }
    // the children's couplings m_jk + x y_j m_vk + x z_j u_k' (the border's own held
    // times x, n + 1 coefficients)
    for (int t = t1; t < units; t += NT) {
        int c, k, x;
        unit(t, c, k, x);
        int j = (int)((__builtin_sqrtf(8.0f * (float)x + 1.0f) - 1.0f) * 0.5f);
        if (tree_tri(j + 1, 0) <= x) ++j;
        if (tree_tri(j, 0) > x) --j;
        const int k0 = x - tree_tri(j, 0);
        const Block<V> pb = parent(c), cb = child(c);
        V m = m1;
        if (t != t1) m = pb.base[k * pb.stride + 1 + x];
        Acc a = AR::acc_of(m);
#pragma unroll AR::kUnroll
        for (int i = 0; i < k; ++i) {
            AR::mac(a, y_at(c, j, i), v_at(c, pb, k0, k - 1 - i));
            AR::mac(a, z_at(c, j, i), u_at(c, k0, k - 1 - i));
        }
        cb.base[k * cb.stride + 1 + x] = AR::value(a);
    }
}

// Launches it for parents g0 .. g0 + count - 1.
template <class AR>
hipError_t launch_tree_lane_elim(const TreeMap& mp, int level, uint64_t g0, uint64_t count, hipStream_t st) {
    using namespace treelane;
    static_assert(kMaxDdPairs <= 31 && kTreeMaxPairs <= kMaxDdPairs, "a coefficient per lane of a half wavefront");
    const int n = mp.n, T = n - level - 1;
    if (count == 0) return hipSuccess;
    if (n < 1 || n > kMaxDdPairs || T < 0) return hipErrorInvalidValue;
    const size_t series = sizeof(typename AR::V) * (size_t)lds_stride(n);
    // The row of v in LDS while a node's series take at most 64 KB; then as many
    // nodes per workgroup as fit 32 KB (five workgroups per CU).  N = 41 in
    // double-double, with one row update less than now: 60.9 ms; with 16, 24 or 40
    // KB 65.7, 62.6, 64.2 ms; with 128 threads 73.3, with 512 67.4 ms; with the row
    // that stays always in memory 66.2 ms.
    const bool rows = series * lds_series(T, true) <= 64 * 1024;
    const size_t node = series * lds_series(T, rows);
    const int per = (int)std::min<uint64_t>(count, std::max<size_t>(1, std::min<size_t>(16, 32 * 1024 / node)));
    const size_t lds = node * per;
    static_assert(sizeof(typename AR::V) * lds_stride(kMaxDdPairs) * lds_series(kMaxDdPairs - 1, false) <= 160 * 1024,
                  "LDS of the largest elimination");
    const auto k = rows ? tree_lane_elim_kernel<AR, true> : tree_lane_elim_kernel<AR, false>;
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k, dim3((unsigned)((count + per - 1) / per)), dim3(kThreads), lds, st, mp, level, g0, count, per);
    return hipGetLastError();
}

// The same for few parents, where a launch lasts as long as its longest chain of
// dependent steps.  One parent per gridDim.y workgroups, which each repeat the
// solves and share the couplings.  A series takes 16 lanes (coefficients k and,
// WIDE, k + 16): a solve's next coefficient reaches them as a row broadcast (DPP),
// and the series it multiplies is read from LDS ahead of the chain.  With the
// coefficient handed on through LDS a step took 156 ns, and of the 12 us of a
// level at n = 16 (36 at n = 25) the two solves took 5 (26), loads 2, the row update
// 1.2, the couplings 1, launch and kernel end 2.7; now, with two row updates, 8 (12
// to 15) in all up to 32 (16) parents, 24 (114) for 1024.  ROWS as above.
template <class AR, bool WIDE, bool ROWS>
__global__ void __launch_bounds__(1024) tree_top_elim_kernel(TreeMap mp, int level, uint64_t g0) {
    using namespace treelane;
    using V = typename AR::V;
    using Acc = typename AR::Acc;
    constexpr int kSteps = WIDE ? 32 : 16;
    extern __shared__ double4 lds_lane[];
    V* lds = reinterpret_cast<V*>(lds_lane);
    const int n = mp.n, T = n - level - 1, W = 2 * T + 1, E = tree_entries(T);
    const int ns = lds_stride(n);
    const int tid = threadIdx.x, NT = blockDim.x, kl = tid & 15, r = tid >> 4;
    const Block<V> pb = treelane::node_block<V>(mp, level, g0 + blockIdx.x);
    const Block<V> cb{reinterpret_cast<V*>(mp.arena) + mp.off[level + 1] +
                          (g0 + blockIdx.x - mp.win[level + 1]) * (uint64_t)(E * (n + 1)),
                      E};
    // series whose shifts x^(i+1) are read: b (then b'), c, h, each after 32 zeros
    auto shifted = [&](int q) { return lds + 64 * q; };
    V* rows = lds + 3 * 64;
    auto y_at = [&](int j, int k) -> V& { return rows[j * ns + k]; };
    auto z_at = [&](int j, int k) -> V& { return rows[(W + j) * ns + k]; };
    auto u_at = [&](int j, int k) -> V& { return rows[(2 * W + j) * ns + k]; };
    auto v_at = [&](int j, int k) -> const V& {
        return ROWS ? rows[(3 * W + j) * ns + k] : pb.base[k * pb.stride + E + W + 1 + j];
    };

    // row r: j < W the others, u0: m_uj, v0: m_vj; W: h and b', u0: a, v0: b; W + 1:
    // the power sums, u0: b, v0: c (1: coefficients 16 on)
    const bool lo = kl < n, hi = WIDE && kl + 16 < n;
    V u0{}, u1{}, v0{}, v1{};
    const int ue = E + (r <= W ? r : 2 * W + 1), ve = E + W + 1 + r;
    if (r <= W + 1 && lo) {
        u0 = pb.base[kl * pb.stride + ue];
        v0 = pb.base[kl * pb.stride + ve];
        if (hi) {
            u1 = pb.base[(kl + 16) * pb.stride + ue];
            v1 = pb.base[(kl + 16) * pb.stride + ve];
        }
    }
    // a thread's first coupling: coefficient k of entry 1 + x (that of the border
    // with itself, held times x, has n + 1)
    const int D = E - 1, units = D * n + 1, step = NT * gridDim.y, t1 = blockIdx.y * NT + tid;
    V m1{};
    if (t1 < units) {
        const int k = t1 / D;
        m1 = pb.base[k * pb.stride + 1 + t1 - k * D];
    }
    for (int q = tid; q < 3 * 64; q += NT) lds[q] = V{};
    __syncthreads();
    if (r == W + 1) {
        if (lo) shifted(0)[32 + kl] = u0;
        if (hi) shifted(0)[48 + kl] = u1;
        if (lo) shifted(1)[32 + kl] = v0;
        if (hi) shifted(1)[48 + kl] = v1;
    }
    if (ROWS && r < W) {
        if (lo) rows[(3 * W + r) * ns + kl] = v0;
        if (hi) rows[(3 * W + r) * ns + kl + 16] = v1;
    }
    __syncthreads();
    V p0{}, p1{};  // power sums of b
    for (int ph = 0; ph < 2; ++ph) {
        const V* s = shifted(0) + 31 + kl;
        V a0 = ph == 0 ? u0 : v0, a1 = ph == 0 ? u1 : v1;
        if (r == W + 1) {  // b, then b'
            a0 = AR::scale(s[1], (double)(kl + 1));
            if (WIDE) a1 = AR::scale(s[17], (double)(kl + 17));
        }
        Acc c0 = AR::acc_of(a0), c1 = AR::acc_of(a1);
        // y = rhs / (1 - x pivot): coefficient i is final at step i
        static_for<0, kSteps>([&](auto I) {
            constexpr int i = decltype(I)::value;
            if (i < n - 1) {
                const V y = AR::template bcast<(i & 15)>(AR::value(i < 16 ? c0 : c1));
                if (i < 15) AR::mac(c0, s[-i], y);
                if (WIDE) AR::mac(c1, s[16 - i], y);
            }
        });
        a0 = AR::value(c0);
        a1 = AR::value(c1);
        if (r < W) {
            V* out = ph == 0 ? &y_at(r, kl) : &z_at(r, kl);
            if (lo) out[0] = a0;
            if (hi) out[16] = a1;
        } else if (ph == 0 && r == W) {
            if (lo) shifted(2)[32 + kl] = a0;
            if (hi) shifted(2)[48 + kl] = a1;
        } else if (ph == 0) {
            p0 = a0;
            p1 = a1;
        } else if (r == W + 1 && blockIdx.y == 0) {
            if (lo) cb.base[(kl + 1) * E] = AR::add(pb.base[(kl + 1) * pb.stride], AR::add(p0, a0));
            if (hi) cb.base[(kl + 17) * E] = AR::add(pb.base[(kl + 17) * pb.stride], AR::add(p1, a1));
        }
        __syncthreads();
        if (ph == 0) {
            // v_j' = m_vj + x c y_j (row W: b' = b + x c h), then u_j' = m_uj + x h m_vj
            auto update = [&](int q0, V& x0, V& x1, const V& y0, const V& y1) {
                const V* q = shifted(q0) + 31 + kl;
                Acc d0 = AR::acc_of(x0), d1 = AR::acc_of(x1);
                static_for<0, kSteps>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    if (i < n - 1) {
                        const V y = AR::template bcast<(i & 15)>(i < 16 ? y0 : y1);
                        if (i < 15) AR::mac(d0, q[-i], y);
                        if (WIDE) AR::mac(d1, q[16 - i], y);
                    }
                });
                x0 = AR::value(d0);
                x1 = AR::value(d1);
            };
            update(2, u0, u1, v0, v1);
            update(1, v0, v1, a0, a1);
            if (r < W) {
                if (lo) u_at(r, kl) = u0;
                if (hi) u_at(r, kl + 16) = u1;
            } else if (r == W) {
                if (lo) shifted(0)[32 + kl] = v0;
                if (hi) shifted(0)[48 + kl] = v1;
            }
            __syncthreads();
        }
    }
    // the child's couplings m_jk + x y_j m_vk + x z_j u_k'
    for (int t = t1; t < units; t += step) {
        const int k = t / D, x = t - k * D;
        int j = (int)((__builtin_sqrtf(8.0f * (float)x + 1.0f) - 1.0f) * 0.5f);
        if (tree_tri(j + 1, 0) <= x) ++j;
        if (tree_tri(j, 0) > x) --j;
        const int k0 = x - tree_tri(j, 0);
        V m = m1;
        if (t != t1) m = pb.base[k * pb.stride + 1 + x];
        Acc a = AR::acc_of(m);
#pragma unroll AR::kUnroll
        for (int i = 0; i < k; ++i) {
            AR::mac(a, y_at(j, i), v_at(k0, k - 1 - i));
            AR::mac(a, z_at(j, i), u_at(k0, k - 1 - i));
        }
        cb.base[k * cb.stride + 1 + x] = AR::value(a);
    }
}

template <class AR>
hipError_t launch_tree_top_elim(const TreeMap& mp, int level, uint64_t g0, uint64_t count, hipStream_t st) {
    using namespace treelane;
    const int n = mp.n, T = n - level - 1, W = 2 * T + 1;
    if (count == 0) return hipSuccess;
    if (n < 1 || n > kMaxDdPairs || T < 0 || count > (uint64_t)INT32_MAX) return hipErrorInvalidValue;
    const int NT = std::max(512, (16 * (W + 2) + 63) / 64 * 64);
    static_assert(16 * (2 * (kMaxDdPairs - 1) + 3) <= 960, "a row per 16 threads");
    constexpr size_t kLds = 160 * 1024;
    auto bytes = [&](int per) { return sizeof(typename AR::V) * (size_t)(3 * 64 + per * W * lds_stride(n)); };
    static_assert(sizeof(typename AR::V) * (3 * 64 + 3 * (2 * kMaxDdPairs - 1) * lds_stride(kMaxDdPairs)) <= kLds,
                  "LDS of the largest elimination");
    const bool rows = bytes(4) <= kLds;
    const size_t lds = bytes(rows ? 4 : 3);
    const uint64_t units = (uint64_t)(tree_entries(T) - 1) * n + 1;
    const unsigned slices = (unsigned)std::max<uint64_t>(1, std::min<uint64_t>((units + NT - 1) / NT, 256 / count));
    const auto k = n <= 16 ? tree_top_elim_kernel<AR, false, true>
                           : (rows ? tree_top_elim_kernel<AR, true, true> : tree_top_elim_kernel<AR, true, false>);
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k, dim3((unsigned)count, slices), dim3(NT), lds, st, mp, level, g0);
    return hipGetLastError();
}

}  // namespace gbs
