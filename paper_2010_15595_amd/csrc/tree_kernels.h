// Launch interface of the subset-tree kernels (FP64; see tree_device.h).
#pragma once

#include "lhaf_kernels.h"

namespace gbs {

// Largest n on the subset tree: the entries one lane of tree_sub_kernel holds
// (8 (n + 1) doubles) and its operands fit the registers without scratch; n = 29
// and above would need it, and keep the register-tile kernels.  (Instances with
// scratch gave wrong sums; why was not found.  The build refuses them.)
constexpr int kTreeMaxPairs = 28;

// Entry store of a forest of equal trees (n pairs each).  A node with T pairs
// left is one block of (n + 1) x tree_entries(T) values, coefficient-major; level
// lv's blocks (level 0: the roots; lv > 0: the include children of slots win[lv]
// ..) start at arena + off[lv].  An exclude child is the first entries of its
// parent's block.
struct TreeMap {
    double2* arena;
    int n;
    uint32_t off[kTreeMaxPairs + 1];
    uint32_t win[kTreeMaxPairs + 1];
};
// Subsets of size s that are summed: masks lo[s] <= mask < hi[s] (all when !on).
struct TreeShard {
    int on;
    uint32_t lo[kTreeMaxPairs + 1], hi[kTreeMaxPairs + 1];
};
// A captured graph holds a copy per launch, and the no-allocation entry point
// takes 15000 launches at N = 50: 32 bits are enough for stores of 4 GiB and masks
// of kTreeMaxPairs bits.
static_assert(kTreeMaxPairs < 32 && sizeof(TreeMap) + sizeof(TreeShard) <= 512, "kernel arguments");
// Matrices of a forest: root r is item i = list[r] of packed matrices, dims[i] x
// dims[i] row-major at mats + in_off[i], or (list null) the one N x N matrix
// mats.  2n - 1 <= dimension <= 2n.
struct TreeSource {
    const double2* mats;
    const int64_t* in_off;
    const int* dims;
    const int* list;
    int N;
};
// Pairs of the subtrees one wavefront finishes.
int tree_depth(int n);
// Entries (series) of a node with T pairs left.
__host__ __device__ constexpr int tree_entries(int T) { return 1 + (2 * T + 1) * (T + 1); }
// Level-0 entries of roots r0 .. r0 + count - 1 of `src`.
hipError_t launch_tree_root(const TreeMap& mp, const TreeSource& src, uint64_t r0, uint64_t count, hipStream_t st);
hipError_t launch_tree_elim(const TreeMap& mp, const TreeShard& sh, int level, uint64_t g0, uint64_t count,
                            hipStream_t st);
// Whether that runs tree_top_elim_kernel (few parents) or tree_elim_kernel.
bool tree_elim_top(int n, int level, uint64_t count);
hipError_t launch_tree_sub(const TreeMap& mp, const TreeShard& sh, const TreeSource& src, uint64_t r0, int level,
                           uint64_t g0, uint64_t count, double* records, hipStream_t st);
// Fixed-order fold of np records into ceil(np / per) records.
hipError_t launch_records_fold(const double* in, int64_t np, int64_t per, double* out, hipStream_t st);
// Results of items list[0 .. count-1] (device) from `per` consecutive records
// each; per = 0: items of dimension 0.
hipError_t launch_tree_items(const int* list, int count, const double* records, int64_t per, double2* out,
                             double* abs_out, hipStream_t st);

// ---- double-double (tree_dd.h): blocks of cdd values, one matrix, down to the
// leaves (level n)
hipError_t launch_tree_dd_root(const TreeMap& mp, const double2* A, int N, hipStream_t st);
hipError_t launch_tree_dd_elim(const TreeMap& mp, int level, uint64_t g0, uint64_t count, hipStream_t st);
// Whether that runs tree_top_elim_kernel or tree_lane_elim_kernel.
bool tree_dd_elim_top(uint64_t count);
// Signed terms (double-double) of subset masks g0 .. g0 + count - 1.
hipError_t launch_tree_dd_leaf(const TreeMap& mp, uint64_t g0, uint64_t count, void* terms, hipStream_t st);

}  // namespace gbs
