// Internal declarations shared by the host translation units of libgbs_lhaf.
#pragma once

#include <hip/hip_runtime.h>

#include <complex>
#include <cstdint>
#include <functional>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/gbs_lhaf.h"
#include "tree_kernels.h"

namespace gbs_host {

// Sets the thread-local error text and returns st.
gbs_status fail(gbs_status st, const char* fmt, ...);

#define HIP_TRY(call)                                                                                         \
    do {                                                                                                      \
        hipError_t e_ = (call);                                                                               \
        if (e_ != hipSuccess)                                                                                 \
            return gbs_host::fail(e_ == hipErrorOutOfMemory ? GBS_E_NOMEM : GBS_E_DEVICE, "%s: %s (%s:%d)", \
                                  #call, hipGetErrorString(e_), __FILE__, __LINE__);                          \
    } while (0)

uint64_t binom_host(int a, int b);
// Cholesky factorisation Q = L L^H of a Hermitian matrix (row-major n x n, in
// place, lower triangle); false when not positive definite.
bool cholesky(std::vector<std::complex<double>>& L, int n);
// Flop yardstick of one subset of size s of an n-pair loop hafnian.
double subset_flops(int n, int s);

struct BatchRunner;

// Per-device workspace.  All library calls take g_mutex, so one context is
// used by one call at a time; `done` orders reuse across caller streams.
constexpr int kAuxStreams = 4;  // streams that run the size classes of a small loop hafnian concurrently

struct DevCtx {
    int device = -1;
    hipStream_t stream = nullptr;
    hipEvent_t done = nullptr, t0 = nullptr, t1 = nullptr;
    hipStream_t aux[kAuxStreams] = {};     // default priority, created with the context
    hipEvent_t fork = nullptr, join[kAuxStreams] = {};
    uint64_t* binom = nullptr;
    int4* lbmap = nullptr;      // La Budde lane maps (gbs::lb_fill_table)
    double2* A0 = nullptr;      // 64 x 64
    double2* dvec = nullptr;    // 64
    double2* Ain = nullptr;     // host-call staging, 64 x 64
    double2* res = nullptr;     // [0] lhaf, [1] (abs_sum, -)
    void* E = nullptr;
    size_t E_cap = 0;           // bytes
    double* partials = nullptr;
    size_t partials_cap = 0;    // partial records
    uint64_t* masks = nullptr;
    double2* terms = nullptr;
    size_t masks_cap = 0, terms_cap = 0;
    BatchRunner* runner = nullptr;  // eager batch runner of the sampling chain, created on first use
    void* smats = nullptr;          // packed loop-hafnian matrices of one sampling step
    size_t smats_cap = 0;           // bytes
    void* na_scratch = nullptr;     // device address of this device's no-allocation scratch array
    // lane grid per (n, s); -1 = heuristic default.  layout_multi is the
    // choice for batch plans, where many launches share the device: the
    // tuner's best among the grids with one La Budde team per subset group
    int layout[gbs::kMaxPairs + 1][gbs::kMaxPairs + 1];
    int layout_multi[gbs::kMaxPairs + 1][gbs::kMaxPairs + 1];
    bool tuned[gbs::kMaxPairs + 1];
    bool cache_read[gbs::kMaxPairs + 1] = {};
    bool forced[gbs::kMaxPairs + 1][gbs::kMaxPairs + 1] = {};  // lane grid chosen by gbs_set_layout
    char name[64] = {0};
    DevCtx() {
        for (auto& row : layout)
            for (int& v : row) v = -1;
        for (auto& row : layout_multi)
            for (int& v : row) v = -1;
        for (bool& t : tuned) t = false;
    }
};

extern std::mutex g_mutex;  // serialises every library call

gbs_status current_ctx(DevCtx** out);
// Context of device `dev` if gbs_init (or an earlier call) created it, else
// nullptr; never creates one (caller holds g_mutex).
DevCtx* existing_ctx(int dev);
// Looks up this device's no-allocation scratch array (gbs_noalloc.cpp).
gbs_status noalloc_setup(DevCtx* c);
// Lane grid of subsets of size s of an n-pair loop hafnian; batch = true
// gives the batch-plan choice.
int layout_for(const DevCtx* c, int n, int s, bool batch = false, bool fp32 = false);
// Tile offset of C for size-s subsets on `lay` (charpoly_front_offset of m = 2s).
int layout_front_offset(int lay, int s);
// Consults the autotune cache / runs the tuner once per n (uses the workspace,
// so it is called before the caller's matrix is prepared).  tree: the call runs on
// the subset tree and has no lane grid to choose; the tuner is left to one that has.
gbs_status maybe_tune(DevCtx* c, int n, bool tree = false);
gbs_status ensure_buffer(void** p, size_t* cap, size_t need, size_t elem);
// Every device allocation of the library goes through here.  Test hook for the
// out-of-memory paths: while the environment variable GBS_TEST_FAIL_ALLOC is
// "1", it fails (nullptr, hipErrorOutOfMemory) without allocating.
hipError_t dev_malloc(void** p, size_t bytes);
// Times each valid lane grid per subset size of an n-pair loop hafnian.
gbs_status autotune_impl(DevCtx* c, int n, gbs_tune_report* rep);

// ---- subset tree (gbs_host.cpp): FP64 sums without a forced lane grid ----

// How a forest of `items` trees of n pairs is expanded within a memory budget.
struct TreeSched {
    int n = 0, levels = 0;       // levels above the nodes that one wavefront finishes
    uint64_t items = 0, roots = 0;   // trees, and trees expanded at a time
    uint64_t sub = 0;                // most subtree nodes of one launch
    uint64_t fold = 1;               // node records folded into one
    uint64_t records_per_item = 1;   // records per tree
    uint64_t mid = 0;                // folded records that are folded once more into one (0: they are the result)
    uint64_t entries = 0;            // series of the entry store
    uint64_t piece[gbs::kMaxPairs + 1] = {}, off[gbs::kMaxPairs + 2] = {};
    size_t arena_bytes = 0;
};
// Device memory of a schedule: the entry store, with fold > 1 the node records
// of one launch (S.sub), with mid > 0 that many folded records.
struct TreeBufs {
    void* arena = nullptr;
    double* nodes = nullptr;
    double* mid = nullptr;
};
// False when even one path of the tree does not fit the budget.  Levels down to
// the nodes with `depth` pairs left, `value` bytes per coefficient.
bool tree_sched(int n, uint64_t items, size_t budget, TreeSched& S, uint64_t mid_records, int depth, size_t value);
inline bool tree_sched(int n, uint64_t items, size_t budget, TreeSched& S, uint64_t mid_records = 1ull << 20) {
    return tree_sched(n, items, budget, S, mid_records, gbs::tree_depth(n), sizeof(double2));
}
// Enqueues the sums of all trees: items * records_per_item records, in item
// order.  `shard` (nullable) restricts the subsets.  No allocation, no
// synchronisation.  With `prof`, launches are timed when gbs_profile_enable is
// on (never under stream capture).
gbs_status tree_enqueue(const TreeSched& S, const TreeBufs& b, const gbs::TreeSource& src, const gbs::TreeShard* shard,
                        double* records, hipStream_t st, int* launches, bool prof);
// Subsets of shard g of G: colex ranks [C_s g / G, C_s (g + 1) / G) of every size s.
gbs::TreeShard tree_shard(int n, int shard, int nshards);
// Share of the subtree nodes that hold one of its subsets.
double tree_shard_share(const gbs::TreeShard& sh, int n);
// Whether FP64 sums of n pairs run on the subset tree (gbs_set_layout selects
// the register-tile kernels instead).
inline bool tree_route(const DevCtx* c, int n, bool fp32) {
    if (fp32 || n < 1 || n > gbs::kTreeMaxPairs) return false;
    for (bool f : c->forced[n])
        if (f) return false;
    return true;
}

// ---- batches of loop hafnians (gbs_batch.cpp) ----

// One persistent per-subset launch of a batch schedule.
struct CharpolyLaunch {
    int round, layout, s_rep, inst, variant, offset;
    int tile_begin, ntiles;  // range in the device tile array
    int counter;
    double flops = 0.0, subsets = 0.0;  // yardstick flops and subsets of its tiles
    std::string kernel;                 // kernel instance name (as the profiler prints it)
};
// One series launch (all blocks of one round and one n).
struct SeriesLaunch {
    int round, n;
    int block_begin, nblocks;
};

// Items of a batch that run on the subset tree and have the same n.
constexpr int kBatchBranches = 4;  // parallel streams of a batch's launches
struct TreeGroup {
    TreeSched S;
    int begin, count;  // range of BatchSchedule::tlist
    int branch;        // stream, entry store and node records it uses
    int64_t rec;       // first record
};

// Host-side schedule of a batch of loop hafnians of dimensions `dims`:
// tiles, rounds over two coefficient buffers, launches, and the sizes of the
// device arrays they need.  Built without touching the device.
struct BatchSchedule {
    int count = 0;
    bool fp32 = false;
    int64_t tile_subsets = 0;
    int series_per_thread = 8;  // subsets per lane of a series block (64 lanes; a block never spans tiles)
    int rounds = 0;
    int max_n = 0;
    int64_t subset_terms = 0;
    double flops = 0.0;
    int64_t in_elems = 0, a0_elems = 0, d_elems = 0;  // packed input, padded A0 blocks, loop weights
    int64_t ebuf_bytes = 16;                          // per coefficient buffer
    std::vector<int> dims, npair;
    std::vector<int64_t> in_off, a0_off, d_off;
    std::vector<gbs::BatchTile> tiles;  // device order: (round, instance), largest first
    std::vector<gbs::SeriesBlock> sblocks;
    std::vector<int64_t> pbeg;          // partial records of item i: [pbeg[i], pbeg[i+1])
    std::vector<CharpolyLaunch> cp;
    std::vector<SeriesLaunch> se;
    std::vector<TreeGroup> tree;        // items on the subset tree, most work first
    std::vector<int> tlist;             // their indices, grouped
    size_t tree_arena[kBatchBranches] = {};
    uint64_t tree_nodes[kBatchBranches] = {};
    int64_t tree_records = 0;
    int empty = 0;                      // matrices of dimension 0, last in tlist
    bool tiled = false;                 // some item runs on tiles or as a small item: only then npair, a0_off, d_off
                                        // and pbeg are filled
    std::vector<int> small;             // FP64 items with 1 <= n <= kSmallPairs, largest n first: one wavefront each
    int64_t partials() const { return pbeg.empty() ? 0 : pbeg.back(); }
    // As new, with the per-item arrays' memory kept: a sampling chain schedules
    // tens of thousands of items per step, and pages of fresh arrays cost it more
    // than filling them.
    void reset() {
        BatchSchedule n;
        std::vector<int>*kept[] = {&dims, &npair, &tlist, &small}, *to[] = {&n.dims, &n.npair, &n.tlist, &n.small};
        std::vector<int64_t>*kept8[] = {&in_off, &a0_off, &d_off, &pbeg}, *to8[] = {&n.in_off, &n.a0_off, &n.d_off, &n.pbeg};
        for (int i = 0; i < 4; ++i) {
            kept[i]->clear();
            to[i]->swap(*kept[i]);
            kept8[i]->clear();
            to8[i]->swap(*kept8[i]);
        }
        *this = std::move(n);
    }
};
// tile_offsets: FP64 tiles keep C at the front tile offset of their m (one
// persistent launch per offset); captured plans use it, the sampler's eagerly
// run steps do not (the extra launches cost it more than the offset saves).
void batch_schedule(const DevCtx* c, const std::vector<int>& dims, bool fp32, int64_t tile_subsets,
                    int64_t round_bytes, bool tile_offsets, BatchSchedule& S);

// Device arrays a schedule runs on.  `mats` is the packed input.
struct BatchDev {
    const double2* mats = nullptr;
    double2 *a0 = nullptr, *dv = nullptr;
    gbs::BatchItem* items = nullptr;
    int64_t* in_off = nullptr;
    int* dims = nullptr;
    gbs::BatchTile* tiles = nullptr;
    gbs::SeriesBlock* sblocks = nullptr;
    int64_t* pbeg = nullptr;
    double* partials = nullptr;
    unsigned* counters = nullptr;
    void* ebuf[2] = {nullptr, nullptr};
    double2* out = nullptr;
    double* abs = nullptr;
    int* small = nullptr;
    int* tlist = nullptr;
    void* tarena[kBatchBranches] = {};
    double* tnodes[kBatchBranches] = {};
    double* trec = nullptr;
    const uint64_t* binom = nullptr;  // binomial table (kBinomStride^2)
    const int4* lbmap = nullptr;      // La Budde lane maps (gbs::lb_fill_table)
};
// Issues the whole schedule: counter fill, prep, rounds of per-subset launches
// on the branch streams (joined into `cs` through events from `new_event`),
// series launches and the per-item reduction, all ordered after prior work on
// `cs`.  Works eagerly and under stream capture alike.
// With `prof`, per-subset launches are timed when gbs_profile_enable is on
// (never under stream capture).
gbs_status batch_enqueue(DevCtx* c, const BatchSchedule& S, const BatchDev& d, hipStream_t cs, hipStream_t* br,
                         const std::function<hipError_t(hipEvent_t*)>& new_event, bool prof, int* tree_launches = nullptr);

// Per-launch timing (gbs_profile_*): true while profiling is on.
bool profiling_on();
// Runs `launch`; while profiling is on, brackets it with a HIP event pair on
// `st`, recorded as a per-subset kernel launch of instance `kernel`.
hipError_t prof_charpoly_launch(double flops, double subsets, hipStream_t st,
                                const std::function<hipError_t()>& launch, const std::string& kernel);

// Eager runner of batch schedules on reusable, growing device buffers, for
// callers whose batches change from one run to the next.
struct BatchRunner;
gbs_status runner_create(DevCtx* c, BatchRunner** out);
void runner_free(BatchRunner* r);
// Runs the batch of dimensions S.dims on packed matrices mats_dev (device).
// The meta arrays (items, offsets, tiles) are uploaded first; `before_sum`
// (optional) is then enqueued on `st` so that it can fill mats_dev from them
// (it receives the device in_off and dims arrays).  Results: out[i] and
// abs[i] in the runner's device buffers (runner_out / runner_abs), valid
// after `st` completes.
gbs_status runner_run(BatchRunner* r, const BatchSchedule& S, const double2* mats_dev, hipStream_t st,
                      const std::function<gbs_status(const int64_t* in_off_dev, const int* dims_dev)>& before_sum);
double2* runner_out(BatchRunner* r);

}  // namespace gbs_host
