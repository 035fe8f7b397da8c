#pragma once
// Subset tree: roots, record folds, and the launchers of the kernels of
// tree_device.h for every n.  Included by lhaf_kernels.hip alone.
#include "tree_lane.h"

namespace gbs {

namespace {

__global__ void __launch_bounds__(64) tree_root_kernel(TreeMap mp, TreeSource src, uint64_t r0, int blocks) {
    const int n = mp.n, E = tree_entries(n);
    const unsigned r = blockIdx.x / blocks;
    const int e = (int)(blockIdx.x % blocks) * 64 + threadIdx.x;
    if (e >= E) return;
    int N;
    const double2* A = tree::root_matrix(src, r0 + r, N);
    const double2 v = tree::root_entry(A, N, n, e);
    double2* p = mp.arena + mp.off[0] + (uint64_t)r * (uint64_t)(E * (n + 1)) + e;
    p[0] = v;
    for (int k = 1; k <= n; ++k) p[k * E] = make_double2(0.0, 0.0);
}

// One record (sum re, compensation, sum im, compensation, sum |t|) per `per`
// records, merged by TwoSum in a fixed tree.
__global__ void __launch_bounds__(256) records_fold_kernel(const double* __restrict__ in, int64_t np, int64_t per,
                                                           double* __restrict__ out) {
    __shared__ double sh[5][256];
    const int t = threadIdx.x;
    const int64_t lo = (int64_t)blockIdx.x * per, hi = (lo + per < np) ? lo + per : np;
    double a[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    auto merge = [](double* x, const double* y) {
        const double s = x[0] + y[0], v = s - x[0];
        x[1] = x[1] + y[1] + ((x[0] - (s - v)) + (y[0] - v));
        x[0] = s;
        const double u = x[2] + y[2], w = u - x[2];
        x[3] = x[3] + y[3] + ((x[2] - (u - w)) + (y[2] - w));
        x[2] = u;
        x[4] += y[4];
    };
    for (int64_t i = lo + t; i < hi; i += 256) {
        double b[5];
#pragma unroll
        for (int q = 0; q < 5; ++q) b[q] = in[5 * i + q];
        merge(a, b);
    }
#pragma unroll
    for (int q = 0; q < 5; ++q) sh[q][t] = a[q];
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if (t < w) {
            double b[5];
#pragma unroll
            for (int q = 0; q < 5; ++q) b[q] = sh[q][t + w];
            merge(a, b);
#pragma unroll
            for (int q = 0; q < 5; ++q) sh[q][t] = a[q];
        }
        __syncthreads();
    }
    if (t < 5) out[5 * (int64_t)blockIdx.x + t] = sh[t][0];
}

// Result of item list[i] from its `per` consecutive records (one thread per
// item for one record, one wavefront otherwise, in a fixed order).
__global__ void __launch_bounds__(64) tree_items_kernel(const int* __restrict__ list, int count,
                                                        const double* __restrict__ records, int64_t per,
                                                        double2* __restrict__ out, double* __restrict__ abs_out) {
    const int lane = threadIdx.x;
    if (per <= 1) {
        const int i = blockIdx.x * 64 + lane;
        if (i < count) {
            // no records (per = 0): the empty matrix, loop hafnian 1
            const double* r = records + 5 * (int64_t)i;
            out[list[i]] = per ? make_double2(r[0] + r[1], r[2] + r[3]) : make_double2(1.0, 0.0);
            if (abs_out) abs_out[list[i]] = per ? r[4] : 1.0;
        }
        return;
    }
    const double* r = records + 5 * per * (int64_t)blockIdx.x;
    double a[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    auto merge = [](double* x, const double* y) {
        const double s = x[0] + y[0], v = s - x[0];
        x[1] = x[1] + y[1] + ((x[0] - (s - v)) + (y[0] - v));
        x[0] = s;
        const double u = x[2] + y[2], w = u - x[2];
        x[3] = x[3] + y[3] + ((x[2] - (u - w)) + (y[2] - w));
        x[2] = u;
        x[4] += y[4];
    };
    for (int64_t k = lane; k < per; k += 64) {
        double b[5];
#pragma unroll
        for (int q = 0; q < 5; ++q) b[q] = r[5 * k + q];
        merge(a, b);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        double b[5];
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            const int lo = __shfl_xor(__double2loint(a[q]), off), hi = __shfl_xor(__double2hiint(a[q]), off);
            b[q] = __hiloint2double(hi, lo);
        }
        merge(a, b);
    }
    if (lane == 0) {
        out[list[blockIdx.x]] = make_double2(a[0] + a[1], a[2] + a[3]);
        if (abs_out) abs_out[list[blockIdx.x]] = a[4];
    }
}

}  // namespace

constexpr size_t tree_sub_lds(int n) { return 16 * ((size_t)n * kTreeSlots + 128); }
// LDS series per coefficient of tree_elim_kernel, a compile-time stride chosen by
// T: the exact one for the three levels that hold most nodes, ranges above, up to
// the last level of a launch with more than 256 parents at n = 28.
constexpr int kElimPairs = 19;
constexpr int kElimPlanes[6] = {tree_temps(kTreeDepth), tree_temps(6), tree_temps(7), tree_temps(9), tree_temps(14),
                                tree_temps(kElimPairs)};

struct TreeElimArgs {
    const TreeMap* mp;
    const TreeShard* sh;
    int level;
    uint64_t g0, count;
    int slices;
};
struct TreeSubArgs {
    const TreeMap* mp;
    const TreeShard* sh;
    int level;
    uint64_t g0, count;
    double* records;
    const TreeSource* src;
    uint64_t r0;
};

template <class K>
inline hipError_t tree_allow_lds(K kernel, size_t bytes) {
    if (bytes <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)bytes);
}

template <int NN, int PLANE>
hipError_t tree_elim_plane(const TreeElimArgs& a, hipStream_t st) {
    const size_t lds = 16 * (size_t)NN * PLANE;
    const hipError_t e = tree_allow_lds(tree_elim_kernel<NN, PLANE>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((tree_elim_kernel<NN, PLANE>), dim3((unsigned)(a.count * a.slices)), dim3(64), lds, st, *a.mp,
                       *a.sh, a.level, a.g0, a.slices);
    return hipGetLastError();
}
template <int NN>
hipError_t tree_elim_inst(const TreeElimArgs& a, hipStream_t st) {
    if constexpr (NN > kTreeDepth) {
        const int T = NN - a.level - 1;
        if (T == kTreeDepth) return tree_elim_plane<NN, kElimPlanes[0]>(a, st);
        if constexpr (NN > 6)
            if (T == 6) return tree_elim_plane<NN, kElimPlanes[1]>(a, st);
        if constexpr (NN > 7)
            if (T == 7) return tree_elim_plane<NN, kElimPlanes[2]>(a, st);
        if constexpr (NN > 8)
            if (T <= 9) return tree_elim_plane<NN, kElimPlanes[3]>(a, st);
        if constexpr (NN > 10)
            if (T <= 14) return tree_elim_plane<NN, kElimPlanes[4]>(a, st);
        if constexpr (NN > 15)
            if (T <= kElimPairs) return tree_elim_plane<NN, kElimPlanes[5]>(a, st);
    }
    return hipErrorInvalidValue;
}

template <int NN>
hipError_t tree_sub_inst(const TreeSubArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(tree_sub_kernel<NN>, dim3((unsigned)a.count), dim3(64), tree_sub_lds(NN), st, *a.mp, *a.sh, a.level, a.g0,
                       a.records, *a.src, a.r0);
    return hipGetLastError();
}

// ---- dispatch over n

template <int NN>
static hipError_t tree_elim_n(int n, const TreeElimArgs& a, hipStream_t st) {
    if constexpr (NN > kTreeMaxPairs) {
        return hipErrorInvalidValue;
    } else {
        if (n == NN) return tree_elim_inst<NN>(a, st);
        return tree_elim_n<NN + 1>(n, a, st);
    }
}
template <int NN>
static hipError_t tree_sub_n(int n, const TreeSubArgs& a, hipStream_t st) {
    if constexpr (NN > kTreeMaxPairs) {
        return hipErrorInvalidValue;
    } else {
        if (n == NN) return tree_sub_inst<NN>(a, st);
        return tree_sub_n<NN + 1>(n, a, st);
    }
}

int tree_depth(int n) { return n < kTreeDepth ? n : kTreeDepth; }

hipError_t launch_tree_root(const TreeMap& mp, const TreeSource& src, uint64_t r0, uint64_t count, hipStream_t st) {
    if (count == 0) return hipSuccess;
    const int blocks = (tree_entries(mp.n) + 63) / 64;
    hipLaunchKernelGGL(tree_root_kernel, dim3((unsigned)(count * blocks)), dim3(64), 0, st, mp, src, r0, blocks);
    return hipGetLastError();
}

namespace treelane {
struct F64 {
    using V = double2;
    using Acc = double2;
    static constexpr int kUnroll = 4;
    static __device__ __forceinline__ Acc acc_of(const V& a) { return a; }
    static __device__ __forceinline__ V value(const Acc& a) { return a; }
    static __device__ __forceinline__ void mac(Acc& c, const V& a, const V& b) { c = tree::mac(a, b, c); }
    static __device__ __forceinline__ V scale(const V& a, double x) { return make_double2(a.x * x, a.y * x); }
    static __device__ __forceinline__ V add(const V& a, const V& b) { return make_double2(a.x + b.x, a.y + b.y); }
    template <int I>
    static __device__ __forceinline__ V bcast(const V& a) {
        return make_double2(treelane::row_bcast<I>(a.x), treelane::row_bcast<I>(a.y));
    }
};
}  // namespace treelane

// Up to here a launch of tree_elim_kernel lasts as long as its chain of products,
// 12 us at n = 16 and 28 us at n = 25; the split of a product over lanes takes 8
// and 12 to 15 us, but a multiply-add costs it several LDS reads.  Microseconds with a
// limit of 32, 128, 256, 512, 1024, 2048 parents: N = 28 124, 115, 111, 111, 111,
// 112; N = 32 232, 222, 221, 216, 216, 215; N = 36 670, 659, 658, 654, 661, 683;
// N = 37 without allocation 2827 (128), 2708, 2596, 2599, 2598; 4096 small items 230,
// 230, 229, 235, 256.  512 and 1024 are alike in time.  1024, because it leaves the
// N = 40 sum of the benchmark family 2.0e-18 of sum |t_S| off and 512 1.55e-18, by
// chance of rounding, where the comparison with long doubles in the tests asks for
// 1.6e-18 at least.
constexpr uint64_t kTopParents = 1024;

bool tree_elim_top(int n, int level, uint64_t count) { return count <= kTopParents || n - level - 1 > kElimPairs; }

hipError_t launch_tree_elim(const TreeMap& mp, const TreeShard& sh, int level, uint64_t g0, uint64_t count,
                            hipStream_t st) {
    const int n = mp.n, T = n - level - 1;
    if (count == 0) return hipSuccess;
    if (n < 1 || n > kTreeMaxPairs || T < 0) return hipErrorInvalidValue;
    if (tree_elim_top(n, level, count)) return launch_tree_top_elim<treelane::F64>(mp, level, g0, count, st);
    if (count > (uint64_t)INT32_MAX) return hipErrorInvalidValue;
    // couplings of larger nodes over several wavefronts, until about two per SIMD
    // are in flight
    const int rounds = (tree_entries(T) - 1 + 63) / 64;
    const int slices = (int)std::max<uint64_t>(1, std::min<uint64_t>(rounds, 2048 / count));
    const TreeElimArgs a{&mp, &sh, level, g0, count, slices};
    return tree_elim_n<1>(n, a, st);
}

hipError_t launch_tree_sub(const TreeMap& mp, const TreeShard& sh, const TreeSource& src, uint64_t r0, int level,
                           uint64_t g0, uint64_t count, double* records, hipStream_t st) {
    const int n = mp.n;
    if (count == 0) return hipSuccess;
    if (n < 1 || n > kTreeMaxPairs || n - level > kTreeDepth || count > (uint64_t)INT32_MAX) return hipErrorInvalidValue;
    const TreeSubArgs a{&mp, &sh, level, g0, count, records, &src, r0};
    return tree_sub_n<1>(n, a, st);
}

hipError_t launch_records_fold(const double* in, int64_t np, int64_t per, double* out, hipStream_t st) {
    if (np <= 0) return hipSuccess;
    hipLaunchKernelGGL(records_fold_kernel, dim3((unsigned)((np + per - 1) / per)), dim3(256), 0, st, in, np, per, out);
    return hipGetLastError();
}

hipError_t launch_tree_items(const int* list, int count, const double* records, int64_t per, double2* out,
                             double* abs_out, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    const int grid = per <= 1 ? (count + 63) / 64 : count;
    hipLaunchKernelGGL(tree_items_kernel, dim3(grid), dim3(64), 0, st, list, count, records, per, out, abs_out);
    return hipGetLastError();
}

}  // namespace gbs
