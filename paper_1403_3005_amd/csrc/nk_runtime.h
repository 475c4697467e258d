// Host runtime shared by the C ABI (nk_api.hip) and the serving loop
// (nk_server.hip): error reporting, device properties, the pooled scratch
// allocator, tuning state and the persistent-kernel runner.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "../../include/nk_bc.h"
#include "nk_kernels.h"

namespace nk {

nk_status fail(nk_status code, const char *fmt, ...);
void clear_error();

#define NK_HIP(expr)                                                                              \
    do {                                                                                          \
        hipError_t e_ = (expr);                                                                   \
        if (e_ != hipSuccess) return ::nk::fail(NK_E_HIP, "%s failed: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

struct DevInfo {
    int device;
    int cus;
    size_t lds_per_block;
};
nk_status dev_info(DevInfo *out);

// Pooled device scratch.  Blocks return to the pool when the holder is
// destroyed; the pool keeps them for later calls until nk_shutdown.
// Scratch block tags (contents that stay meaningful across calls).
// Pair-mode record blocks: every record unreached (whatever graph or stride
// the next launch brings).
constexpr uint64_t kTagPairRecords = 1;
// Pair-mode hash tables: every entry free and unreached.
constexpr uint64_t kTagPairTables = 2;

class Scratch {
public:
    Scratch() = default;
    ~Scratch();
    Scratch(const Scratch &) = delete;
    Scratch &operator=(const Scratch &) = delete;
    // Returns NK_OK and a device pointer of at least `bytes` bytes (256-byte aligned).
    nk_status get(size_t bytes, void **out);
    template <typename T>
    nk_status get(long long count, T **out) {
        return get((size_t)(count > 0 ? count : 1) * sizeof(T), (void **)out);
    }
    void release_all();
    // A block that keeps a meaning across calls: `tag` != 0 asks for a free
    // block last marked with that tag (*clean = true if one was found; its
    // contents are as the marking call left them).  *block_bytes is the
    // whole block's size, which may exceed `bytes`: a caller that marks the
    // block must have prepared all of it.  Any block handed out loses its
    // tag until mark() sets it again.
    nk_status get_tagged(size_t bytes, uint64_t tag, void **out, bool *clean, size_t *block_bytes);
    void mark(void *p, uint64_t tag);

private:
    std::vector<void *> held_;
};
void pool_clear();
void pool_trim();           // frees the current device's idle blocks
size_t pool_bytes_in_use();
size_t pool_bytes_idle();   // idle pooled bytes on the current device

nk_tuning tuning_get();
void tuning_set(const nk_tuning &t);

// While alive, tuning_get() on this thread returns *t (nothing changes when
// t is NULL); scopes nest.
class TuningOverride {
public:
    explicit TuningOverride(const nk_tuning *t);
    ~TuningOverride();
    TuningOverride(const TuningOverride &) = delete;
    TuningOverride &operator=(const TuningOverride &) = delete;

private:
    const nk_tuning *prev_;
};

// Autotuner cache (nk_tune.hip): the tuning registered for graphs shaped
// like (n, m, max degree), merged into the global tuning (flags and
// scratch cap stay global); false when no cache is registered or it has no
// entry for the shape.  *in_lds: the entry was timed on a kernel of
// nk_lds.hip, and its block and ratios say nothing of the others.
bool cached_tuning(int32_t n, int64_t m, int64_t max_deg, nk_tuning *out, bool *in_lds);
bool tuning_cache_active();
// Maximum degree of a CSR (one reduction kernel; synchronises s).
nk_status graph_max_degree(const int32_t *rowptr, int32_t n, hipStream_t s, int64_t *out);

// Per-thread statistics of the last call (nk_last_stats).
// lds: 0 global bitmap, 1 bitmap in LDS, 2 whole graph in LDS
void stats_record(const DevStatus &st, int grid, int block, int lds, float kernel_ms);
void stats_clear();

// Launch configuration chosen for a persistent Brandes launch.
struct LaunchPlan {
    int mode;
    int block;
    bool lds;
    int grid;
    size_t dyn_lds;
    long long stride;
    long long bm_words;
    KernelRef kernel;
    void *pair_rec;   // pair mode: the record block the launch used (set by the caller after the launch)
    long long dag_words;   // weighted mode: per-slot words of the DAG-arc bitmap
    bool narrow;           // a thin graph ends the launch (Params::narrow): plan again with thin = true
};
// The tag a pair-mode record block of `plan` carries after a successful
// launch (records or hash tables, by the plan's mode).
inline uint64_t pair_block_tag(const LaunchPlan &plan) {
    return plan.mode == kModePairHash ? kTagPairTables : kTagPairRecords;
}

// Picks block size, bitmap placement and grid for graphs of at most n_max
// vertices and `ntasks` tasks.  max_slots > 0 caps the grid.  m_arcs: the
// arcs of the graph (weighted mode sizes its DAG-arc bitmap by them; 0 = not
// known).  The block size goes by the vertices alone where m_arcs is 0 or thin
// is set (a graph of many narrow levels).
nk_status plan_launch(int mode, int32_t n_max, long long ntasks, int max_slots, LaunchPlan *plan,
                      int64_t m_arcs = 0, bool thin = false);
// Block size of a persistent launch over graphs of at most n_max vertices
// when the tuning leaves it open.
int auto_block(int32_t n_max);

// Multi-source launch (nk_multi.hip): b sources per task.
struct MsPlan {
    LaunchPlan lp;
    int b;
    int32_t nl;            // vertices whose visited masks sit in LDS
    long long stride;      // per-slot vertex capacity
    long long cap;         // per-slot union-list capacity (stride * b)
    long long visg_words;  // per-slot words of global masks
    long long ntasks;      // tasks of the launch (set by plan_ms for a single graph)
};
// Sources per task for a graph of at most n_max vertices (the tuning's
// batch, or the automatic choice); 1 means the one-source kernels.
int ms_batch_for(int32_t n_max, long long nsources);
// Plan for graphs of at most n_max vertices and `nsources` sources in all
// (tasks = ceil(nsources / b)).
nk_status plan_ms(int b, int32_t n_max, long long nsources, MsPlan *mp);
nk_status ms_alloc(const MsPlan &mp, Params &p, Scratch &scr);
// Clears the path counts, new-source masks and global visited masks, then
// launches (p.ntasks is replaced by the plan's task count).
nk_status ms_enqueue(const MsPlan &mp, const Params &p, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1);
void stats_set_batch(int b);

// Group launch (nk_group.hip): one source per group of workgroups sharing
// an XCD's L2.
struct GroupPlan {
    LaunchPlan lp;
    int gpx;               // groups per XCD
    int groups;            // groups allocated (XCDs x gpx)
    int nxcc;              // XCDs of the device
    long long stride;      // per-group vertex capacity
    long long timeout;     // wall-clock ticks a wait may last
    long long reg_wait;    // ... and the wait for the whole grid to be resident
    bool narrow;           // a thin graph ends the launch (Params::narrow)
};
// Whether the group kernel takes a graph of n_max vertices and m_arcs arcs:
// automatically for sparse graphs of 10^5 to 3 * 10^5 vertices, for every
// graph under tuning flag bit 3, never under bit 4 or an explicit
// multi-source batch; and only if its visited bitmap fits LDS.
// nsources: the sources of the run (a batch, whose graphs share one launch,
// gives kManySources).
constexpr long long kManySources = 1LL << 40;
bool group_wanted(int32_t n_max, int64_t m_arcs, long long nsources);
nk_status plan_group(int32_t n_max, long long nsources, GroupPlan *gp);
nk_status group_alloc(const GroupPlan &gp, Params &p, Scratch &scr);
// Clears the path counts, control blocks and registration counters, then
// launches (cooperatively unless the stream is being captured).
nk_status group_enqueue(const GroupPlan &gp, const Params &p, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1);

// Grid-wide direction-optimising breadth-first search (nk_bfs.hip).
struct BfsWork {
    int32_t *d;        // n distances from the source (-1 unreached)
    int32_t *f0, *f1;  // frontier lists, n entries each
    int32_t *f2;       // n + 1: deferred vertices, or a frontier's degrees
    int32_t *off;      // n + 1 arc offsets of a top-down frontier
    long long *cnt;    // 9 words: two level counter sets and one spare
    void *tmp;         // prefix-sum temporary storage
    size_t tmp_bytes;
};
nk_status bfs_work_get(Scratch &scr, int32_t n, hipStream_t s, BfsWork *w);
// Distances from src into w.d; out = {eccentricity of src, lowest id at
// that distance (-1 unless want_lowest), vertices reached}.  src_deg: the
// source's degree if the caller knows it (else -1: read from rowptr).
// Synchronises s.
nk_status grid_bfs(const int32_t *rowptr, const int32_t *colidx, int32_t n, int64_t m, int32_t src,
                   const BfsWork &w, hipStream_t s, int32_t out[3], int32_t src_deg = -1, bool want_lowest = true);
// Size of the largest connected component among the vertices with
// skip[v] < 0 (label, size: n ints of scratch; flag: one int).
nk_status largest_unreached_component(const int32_t *rowptr, const int32_t *colidx, int32_t n, const int32_t *skip,
                                      int32_t *label, int32_t *size, int32_t *flag, hipStream_t s, int32_t *out);

// Closeness by bit-parallel searches, up to 1024 sources a pass
// (nk_close.hip): exact (sources NULL, k = n) or sampled scores into out.
// *done = false (nothing written but scratch and, for a source out of
// range, the status; scr empty again) for small calls, where the bits do not
// fit the scratch, and where the graph has too many levels (*deep).  The
// counters go to the status.
nk_status close_bits(const int32_t *rowptr, const int32_t *colidx, int32_t n, int64_t m, const int32_t *sources,
                     int32_t k, bool sampled, double *out, DevStatus *dst, Scratch &scr, hipStream_t s, bool *done,
                     bool *deep);

// All-in-LDS betweenness plan for graphs needing at most `dyn_bytes` of
// dynamic LDS; returns false (and plans nothing) when they do not fit or
// tuning flag bit 2 turns the path off.
bool plan_lds(size_t dyn_bytes, int32_t n_max, long long ntasks, LaunchPlan *plan);

// State-in-LDS launch (nk_lds.hip): one source per workgroup, its path
// counts and levels in LDS, the graph in global memory.
struct StatePlan {
    LaunchPlan lp;
    bool cold;             // path counts from vertex `hot` on, and the lists, in global scratch
    int32_t hot;
};
// Plans it for graphs of at most n_max vertices; false (nothing planned)
// for larger ones than it takes and where the tuning asks for another
// kernel (flag bits 0, 2 and 3, or a multi-source batch).
bool plan_state(int32_t n_max, long long ntasks, StatePlan *sp);
// Whether so many sources of a graph of n vertices go to the one-source kernel
// if the graph is thin: up to 2 * 10^4 vertices a compute unit runs four
// sources there and one or two here, and a chain's level costs a barrier or two
// on either (ms here / there: a cycle of 9,000 vertices, 512 sources 32 / 38,
// 1024 63 / 41; 2,000 cliques of 8, 1024 sources 57 / 37; a ring lattice of
// 12,000, 1024 21 / 16; a chain of 400 cliques of 32, 4096 40 / 36 and not thin).
bool state_asks_thin(const StatePlan &sp, int32_t n, long long ntasks);
// Whether most of the probed searches of a graph stay thin (nk_lds.hip), from
// the sources (k of them, or NULL) or vertices spread over it.  Synchronises s;
// host: the thread's pinned status, whose info it uses.
nk_status thin_graph(const int32_t *rowptr, const int32_t *colidx, int32_t n, int64_t m, const int32_t *sources,
                     long long k, DevStatus *host, hipStream_t s, bool *thin);
// The same for several graphs, four entries of tab each: the first in rowptr,
// the vertices, the first in colidx, the arcs.
nk_status thin_graphs(const int32_t *rowptr, const int32_t *colidx, const std::vector<long long> &tab, hipStream_t s,
                      std::vector<int32_t> *thin);
// Scratch of the launch, and the launch.
nk_status state_alloc(const StatePlan &sp, Params &p, Scratch &scr);
nk_status state_enqueue(const StatePlan &sp, const Params &p, hipStream_t s);

// Allocates per-slot scratch for `plan`, clears the path counts, fills the
// scratch fields of `p` and launches the persistent kernel on `s`,
// recording HIP events around it when ev0/ev1 are non-null.
nk_status launch_persistent(const LaunchPlan &plan, Params &p, Scratch &scr, hipStream_t s, hipEvent_t ev0,
                            hipEvent_t ev1);
// The two halves of launch_persistent: persistent_alloc takes the scratch
// and fills the scratch fields of `p` (it enqueues nothing, except in pair
// mode the fill of a record block that is not clean); persistent_enqueue
// clears what the kernel expects clear and launches it -- kernels only, so
// a non-pair launch can be captured into a HIP graph and replayed.
nk_status persistent_alloc(const LaunchPlan &plan, Params &p, Scratch &scr, hipStream_t s);
nk_status persistent_enqueue(const LaunchPlan &plan, const Params &p, hipStream_t s, hipEvent_t ev0,
                             hipEvent_t ev1);

// Copies the status block to the host, synchronises `s` and maps error bits
// to a status code.
nk_status finish(DevStatus *dst, DevStatus *host, hipStream_t s);

nk_status map_err(int32_t err);

// Per-thread pinned status buffer and timing events.
DevStatus *host_status();
nk_status thread_events(hipEvent_t *ev0, hipEvent_t *ev1);

// Graph argument checks shared by every entry point.
nk_status check_graph_args(const int32_t *rowptr, const int32_t *colidx, int32_t n, int64_t m);

// Degree-order relabelling (nk_relabel.hip).  Kernels skip their work when
// the structural check already failed.
// Directed graphs (nk_directed.hip): the in-arc CSR of out-arcs (rows
// sorted by tail), and a check that trowptr's row lengths are the
// in-degrees of colidx (sets kErrGraph in dst otherwise).
nk_status transpose_graph(const int32_t *rowptr, const int32_t *colidx, int32_t n, int64_t m, int32_t *trowptr,
                          int32_t *tcolidx, Scratch &scr, hipStream_t s);
nk_status check_transpose(const int32_t *colidx, int32_t n, int64_t m, const int32_t *trowptr, DevStatus *dst,
                          Scratch &scr, hipStream_t s);

nk_status relabel_graph(const int32_t *rowptr, const int32_t *colidx, int32_t n, int64_t m, const DevStatus *st,
                        Scratch &scr, hipStream_t s, Relabeled *out);
// The same renaming applied to per-arc int32 values (arc weights), and to a
// second CSR over the same vertices (the in-arcs of a directed graph; its
// rows get the renamed in-neighbours, in their original order).
nk_status relabel_weights(const int32_t *wts, const int32_t *rowptr, int32_t n, int64_t m, const Relabeled &g,
                          const DevStatus *st, Scratch &scr, hipStream_t s, int32_t **out);
nk_status relabel_second_csr(const int32_t *rowptr2, const int32_t *colidx2, int32_t n, int64_t m, const Relabeled &g,
                             const DevStatus *st, Scratch &scr, hipStream_t s, int32_t **rp_out, int32_t **ci_out);
hipError_t launch_map_sources(const int32_t *src, int32_t k, const int32_t *perm, int32_t n, int32_t *out,
                              hipStream_t s);
hipError_t launch_arcs_back(const double *in, const int32_t *rp_new, const int32_t *inv, const int32_t *rowptr,
                            int32_t n, double *out, hipStream_t s);
// Score accumulators of a run over n vertices (all graphs of a batch
// together): one copy per XCD up to 2^25 vertices (8 x 8 bytes a vertex),
// a single shared one above, and where the copies of more than half a million
// vertices (kScoreCopiesFree bytes) pass the tuning's scratch cap or, with
// none set, an eighth of the device memory that is free or idle in the pool:
// the slots' scratch matters more than the copies.
constexpr int kScoreCopies = 8;
constexpr long long kScoreCopiesMax = 1LL << 25;
constexpr long long kScoreCopiesFree = 32LL << 20;
struct ScoreAcc {
    double *acc;
    long long n, x;        // vertices; doubles from one copy to the next
    int copies;
};
nk_status score_acc(long long n, Scratch &scr, ScoreAcc *a);
void score_params(const ScoreAcc &a, Params *p);
hipError_t score_clear(const ScoreAcc &a, hipStream_t s);
// out[v] = scale * sum of the copies at perm[v] (v where perm is NULL); with
// host, also *host = *st (pinned memory; read it after the stream is done).
hipError_t launch_gather_scores(const ScoreAcc &a, const int32_t *perm, double scale, double *out, hipStream_t s,
                                const DevStatus *st = nullptr, DevStatus *host = nullptr);
hipError_t launch_gather_u32(const uint32_t *in, const int32_t *perm, int32_t n, uint32_t *out, hipStream_t s);

// Vertex-diameter bound (see nk_vd_bound); runs synchronously on `s`.
// lower = false skips the second sweep, which gives only the lower bound
// (info[3] is then -1 and info[5] 0): the upper bound info[4] is the same.
nk_status vd_bound_impl(const int32_t *rowptr, const int32_t *colidx, int32_t n, int64_t m, int32_t *info,
                        hipStream_t s, bool lower = true);

}  // namespace nk
