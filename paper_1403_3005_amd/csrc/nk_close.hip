// Closeness by bit-parallel breadth-first search.
//
// Closeness needs distances only (Table 1, "closeness" and "ap. closeness":
// one search from each node, or from a sample of them), so up to 1024
// searches run at once: every vertex holds one bit per source for "reached"
// and for "reached on the last level", and one level of all the searches is
// one pass over the arcs -- a vertex that some source has not reached yet
// ORs its neighbours' last-level bits.  (Searches as bits side by side are the
// idea of Then et al., "The More the Merrier: Efficient Multi-Source Graph
// Traversal", PVLDB 8(4), 2014.)  New bits times the level are added
// to the vertex's distance sum.  On an undirected graph the distances from
// the sources to v summed over all sources are the distances from v, so the
// exact form takes the same sums, with every vertex as a source.
//
// What bounds it: each active arc of a level reads one neighbour's bits, at
// 1024 sources one 128-byte line; the whole array (128 n bytes) stays in the
// Infinity Cache up to about 2 * 10^6 vertices.  A bitmap of the vertices
// with any last-level bit (n / 8 bytes, in L2) is tested first, so sparse
// levels read little; a vertex stops scanning once all its missing bits are
// found, and one that every live search has reached is skipped.  R-MAT-18
// (8 * 10^6 arcs), 1024 sources: 0.83 ms a call, of which the two dense levels
// are 0.21 and 0.29; 12.9 ms with one workgroup per search, which reads every arc
// once per source.
//
// A level is a launch, so graphs of many levels go to the one-workgroup-per-
// source kernel instead, whose levels cost it less (CloseGrowth, kCloseDeep).
#include <string.h>

#include <algorithm>

#include "nk_runtime.h"

namespace nk {

namespace {

constexpr int kCloseBlock = 256;
constexpr int kLanes = 16;                       // lanes of a group
constexpr int kGroups = kCloseBlock / kLanes;    // groups of a block
constexpr int kVerts = 64;                       // vertices of a block
// Rows of more arcs than these go to a wave, or a block, each, from lists:
// hubs sit next to each other in many graphs, and a wave that met several
// of them among its own vertices took 5 of a level's 6 ms.
constexpr int kWaveRow = 64;
constexpr int kBlockRow = 512;
constexpr int kCloseDeep = 96;                   // levels the first pass may take
constexpr int kCloseFirst = 6;                   // levels before the first look at them
constexpr int kCloseRows = 128;                  // levels whose masks and counters are kept
constexpr int kCloseXcd = 8;                     // counter lines a level
constexpr int kCloseTotals = 64;                 // lines of the call's totals: eight an XCD, as adds to a line queue up
constexpr int kCloseRow = 16 * (1 + kCloseXcd);  // words a level: masks, counters
// (source, vertex) pairs found, arcs of their vertices, arcs looked at (a
// level's line holds the first, the call's totals all), levels run
enum CloseCount { kCcPairs = 0, kCcArcs, kCcScanned, kCcLevels, kCloseCount };
constexpr int kListBlocks = 2048;                // blocks that take each list, at most
// A launch holds less than 2^32 threads (a larger one runs nothing and
// reports nothing), and a level takes four threads a vertex.
constexpr int32_t kCloseMax = 1 << 29;
static_assert((kCloseMax / kVerts + 2LL * kListBlocks) * kCloseBlock < 1LL << 32, "threads of a level");

struct CloseArgs {
    const int32_t *rp;
    const int32_t *ci;
    int32_t n;
    unsigned long long *seen;
    const unsigned long long *front; // bits set on the last level, valid where act has the vertex's bit
    unsigned long long *next;
    const uint32_t *act;
    uint32_t *act_next;              // clear
    uint32_t *act_clear;             // to clear for the level after
    unsigned long long *acc;         // distance sums
    const unsigned long long *alive_prev;   // 16 words: the sources that reached something on the last level
    unsigned long long *alive;       // ... on this one (clear)
    unsigned long long *counts;      // this level's counter, a line per XCD
    unsigned long long *totals;      // the call's (kCloseTotals lines)
    const int32_t *list[2];          // rows for a wave, for a block
    const int32_t *nlist;            // their counts
    int32_t level;
    int32_t big_blocks, wave_blocks; // first blocks: the block rows, then the wave rows
    const DevStatus *st;
};

template <int W>
__device__ __forceinline__ unsigned long long or_slots(unsigned long long x) {
#pragma unroll
    for (int o = W; o < kLanes; o <<= 1) x |= __shfl_xor(x, o, kWave);
    return x;
}

// The OR, word by word, of the last-level bits of the wave's heads: every
// lane brings one head (u, or -1) and learns whether it has any such bits;
// then each W lanes together read their heads' W words, four heads at a
// time, skipping the heads without.  Lane's share: word lane % W.
template <int W>
__device__ __forceinline__ unsigned long long or_heads(const CloseArgs &a, int32_t u) {
    const int lane = lane_id();
    const int base = lane & ~(W - 1), word = lane & (W - 1);
    const bool on = u >= 0 && ((a.act[u >> 5] >> (u & 31)) & 1u);
    if (W == 1) return on ? a.front[u] : 0ULL;
    uint32_t m = (uint32_t)(__ballot(on) >> base) & ((1u << W) - 1u);
    unsigned long long r = 0ULL;
    while (m) {
        unsigned long long x[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            x[j] = 0ULL;
            if (m) {
                const int32_t h = __shfl(u, base + __builtin_ctz(m), kWave);
                m &= m - 1u;
                x[j] = a.front[(long long)h * W + word];
            }
        }
        r |= (x[0] | x[1]) | (x[2] | x[3]);
    }
    return r;
}

// What a block adds up in LDS before it goes to the level's words.
template <int W>
struct CloseSums {
    unsigned long long alive[W];
    unsigned long long count[kCloseCount];
};

// New bits of vertex v of `deg` arcs (word `word` of them in this lane, slot 0
// counts): stored, added to the distance sum; true if there are any.
template <int W>
__device__ __forceinline__ bool settle(const CloseArgs &a, CloseSums<W> &sums, int32_t v, int32_t deg, int gl,
                                       unsigned long long seen, unsigned long long fresh) {
    const int word = gl % W;
    const bool mine = gl < W;
    int32_t c = mine ? (int32_t)__popcll(fresh) : 0;
#pragma unroll
    for (int o = 1; o < kLanes; o <<= 1) c += __shfl_xor(c, o, kWave);
    if (c == 0) return false;
    if (mine) {
        a.next[(long long)v * W + word] = fresh;
        a.seen[(long long)v * W + word] = seen | fresh;
        if (fresh) atomicOr(&sums.alive[word], fresh);
    }
    if (gl == 0) {
        a.acc[v] += (unsigned long long)a.level * (unsigned long long)c;
        atomicAdd(&sums.count[kCcPairs], (unsigned long long)c);
        atomicAdd(&sums.count[kCcArcs], (unsigned long long)c * (unsigned long long)deg);
    }
    return true;
}

// The block's searches that reached something, added to the level's mask
// (read first: most blocks bring nothing new, and adds to the one line by all
// XCDs are slow), and its counts, to its XCD's lines.  scanned: arcs this
// thread looked at.
template <int W>
__device__ __forceinline__ void sums_out(const CloseArgs &a, CloseSums<W> &sums, uint32_t scanned) {
    scanned = wave_sum<uint32_t>(scanned);
    if (lane_id() == 0 && scanned) atomicAdd(&sums.count[kCcScanned], (unsigned long long)scanned);
    __syncthreads();
    if (threadIdx.x < W) {
        unsigned long long *al = a.alive + threadIdx.x;
        const unsigned long long x = sums.alive[threadIdx.x];
        if (x & ~__hip_atomic_load(al, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicOr(al, x);
    } else if (threadIdx.x >= kWave && threadIdx.x < kWave + kCcLevels) {
        const int i = threadIdx.x - kWave, xcd = xcc_id() & (kCloseXcd - 1);
        if (sums.count[i]) {
            atomicAdd(a.totals + (xcd * 8 + (blockIdx.x & 7)) * 16 + i, sums.count[i]);
            if (i == kCcPairs) atomicAdd(a.counts + xcd * 16, sums.count[i]);
        }
    }
}

template <int W>
__global__ __launch_bounds__(kCloseBlock) void k_close_level(CloseArgs a) {
    __shared__ CloseSums<W> sums;
    __shared__ uint32_t bits[kVerts / 32];
    __shared__ unsigned long long part[W];
    __shared__ int32_t stop;
    if (a.st->err & kErrGraph) return;
    {
        // no search left: nothing to do
        unsigned long long left = 0ULL;
        for (int w = 0; w < W; ++w) left |= a.alive_prev[w];
        if (left == 0ULL) return;
    }
    const int tid = threadIdx.x, lane = lane_id();
    const int gl = tid % kLanes, word = gl % W;
    // the searches still going: those that reached something on the last
    // level (the bits of the others are not looked for)
    const unsigned long long full = a.alive_prev[word];
    int32_t blk = (int32_t)blockIdx.x;
    uint32_t scanned = 0;
    if (tid == 0 && blockIdx.x == 0) atomicAdd(a.totals + kCcLevels, 1ULL);
    if (tid < W) sums.alive[tid] = 0ULL;
    if (tid < kCloseCount) sums.count[tid] = 0ULL;
    __syncthreads();

    if (blk < a.big_blocks) {
        // a block per row; every group holds all words
        const int32_t nb = a.nlist[1];
        for (int32_t t = blk; t < nb; t += a.big_blocks) {
            const int32_t v = a.list[1][t];
            const int32_t a0 = a.rp[v], deg = a.rp[v + 1] - a0;
            const unsigned long long seen = a.seen[(long long)v * W + word];
            if (tid < W) part[tid] = 0ULL;
            if (tid == 0) stop = 0;
            __syncthreads();
            unsigned long long got = 0ULL;
            const bool go = __ballot((full & ~seen) != 0ULL) != 0ULL;
            int32_t u = go && tid < deg ? a.ci[a0 + tid] : -1;
            for (int32_t i = tid; go && i - tid < deg; i += 2 * kCloseBlock) {
                const int32_t u1 = i + kCloseBlock < deg ? a.ci[a0 + i + kCloseBlock] : -1;
                const int32_t u2 = i + 2 * kCloseBlock < deg ? a.ci[a0 + i + 2 * kCloseBlock] : -1;
                scanned += (u >= 0 ? 1u : 0u) + (u1 >= 0 ? 1u : 0u);
                const unsigned long long c = or_slots<W>(or_heads<W>(a, u) | or_heads<W>(a, u1));
                if (gl < W && c) atomicOr(&part[word], c);
                __syncthreads();
                got = part[word];
                const bool lack = __ballot((full & ~(seen | got)) != 0ULL) != 0ULL;
                if (tid == 0 && !lack) stop = 1;
                __syncthreads();
                if (stop) break;
                u = u2;
            }
            if (tid < kWave) {
                // the first group settles
                const bool fresh = settle<W>(a, sums, v, deg, lane < kLanes ? gl : kLanes, seen,
                                             lane < kLanes ? got & full & ~seen : 0ULL);
                if (lane == 0 && fresh) atomicOr(&a.act_next[v >> 5], 1u << (v & 31));
            }
            __syncthreads();
        }
        sums_out<W>(a, sums, scanned);
        return;
    }
    blk -= a.big_blocks;
    if (blk < a.wave_blocks) {
        // a wave per row
        constexpr int NW = kCloseBlock / kWave;
        const int32_t nb = a.nlist[0];
        for (int32_t t = blk * NW + wave_id(); t < nb; t += a.wave_blocks * NW) {
            const int32_t v = a.list[0][t];
            const int32_t a0 = a.rp[v], deg = a.rp[v + 1] - a0;
            const unsigned long long seen = a.seen[(long long)v * W + word];
            if (__ballot((full & ~seen) != 0ULL) == 0ULL) continue;
            unsigned long long got = 0ULL;
            int32_t u = lane < deg ? a.ci[a0 + lane] : -1;
            for (int32_t i = lane; i - lane < deg; i += kWave) {
                const int32_t u1 = i + kWave < deg ? a.ci[a0 + i + kWave] : -1;
                scanned += u >= 0 ? 1u : 0u;
                unsigned long long c = or_slots<W>(or_heads<W>(a, u));
                c |= __shfl_xor(c, 16, kWave);
                c |= __shfl_xor(c, 32, kWave);
                got |= c;
                if (__ballot((full & ~(seen | got)) != 0ULL) == 0ULL) break;
                u = u1;
            }
            const bool fresh = settle<W>(a, sums, v, deg, lane < kLanes ? gl : kLanes, seen,
                                         lane < kLanes ? got & full & ~seen : 0ULL);
            if (lane == 0 && fresh) atomicOr(&a.act_next[v >> 5], 1u << (v & 31));
        }
        sums_out<W>(a, sums, scanned);
        return;
    }
    blk -= a.wave_blocks;

    // the other rows, a group each
    const int32_t base = blk * kVerts;
    if (tid < kVerts / 32) bits[tid] = 0u;
    __syncthreads();
    for (int k = tid / kLanes; k < kVerts; k += kGroups) {
        const int32_t v = base + k;
        int32_t a0 = 0, deg = 0;
        unsigned long long seen = full, got = 0ULL;
        if (v < a.n) {
            a0 = a.rp[v];
            deg = a.rp[v + 1] - a0;
            if (deg > 0 && deg <= kWaveRow) seen = a.seen[(long long)v * W + word];
        }
        // missing in any word of the group?
        const unsigned long long miss = __ballot((full & ~seen) != 0ULL);
        const int32_t end = ((miss >> (lane & ~(kLanes - 1))) & 0xFFFFULL) != 0ULL ? deg : 0;
        bool done = false;
        int32_t u = gl < end ? a.ci[a0 + gl] : -1;
        for (int32_t i = gl;; i += kLanes) {
            const bool go = i - gl < end && !done;
            if (!__any(go)) break;
            const int32_t u1 = go && i + kLanes < end ? a.ci[a0 + i + kLanes] : -1;
            scanned += u >= 0 ? 1u : 0u;
            got |= or_heads<W>(a, u);
            const unsigned long long lack = __ballot((full & ~(seen | got)) != 0ULL);
            done = W == kLanes && ((lack >> (lane & ~(kLanes - 1))) & 0xFFFFULL) == 0ULL;
            u = done ? -1 : u1;
        }
        got = or_slots<W>(got);
        if (settle<W>(a, sums, v, deg, gl, seen, got & full & ~seen)) {
            if (gl == 0) atomicOr(&bits[k >> 5], 1u << (k & 31));
        }
    }
    sums_out<W>(a, sums, scanned);
    if (tid < kVerts / 32) {
        const int32_t w = base / 32 + tid;
        if (w < (a.n + 31) / 32) {
            a.act_clear[w] = 0u;
            if (bits[tid]) atomicOr(&a.act_next[w], bits[tid]);
        }
    }
}

// Clears the bits of one pass and its levels' search masks (level 0: the
// count sources of the pass) and counters.
__global__ void k_close_clear(unsigned long long *seen, long long words, uint32_t *act, long long act_words,
                              unsigned long long *rows, int32_t count) {
    const long long stride = (long long)gridDim.x * blockDim.x;
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    for (long long i = t; i < words; i += stride) seen[i] = 0ULL;
    for (long long i = t; i < act_words; i += stride) act[i] = 0u;
    for (long long i = t; i < kCloseRows * kCloseRow; i += stride) {
        const int32_t w = (int32_t)i - kCloseRow;   // (level 0 is row 1)
        const int32_t left = count - 64 * w;
        rows[i] = w < 0 || w >= 16 || left <= 0 ? 0ULL : left >= 64 ? ~0ULL : (1ULL << left) - 1ULL;
    }
}

// The sources' own bits: `front` rows of the sources zeroed by the first
// launch (set = 0), then source i's bit set in both arrays (and the sources
// themselves added to the totals).
__global__ void k_close_sources(const int32_t *rp, const int32_t *src, int32_t s0, int32_t count, int32_t n, int W,
                                unsigned long long *seen, unsigned long long *front, uint32_t *act,
                                unsigned long long *totals, int32_t set, DevStatus *st) {
    if (st->err & kErrGraph) return;
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t v = i < count ? (src ? src[s0 + i] : s0 + i) : 0;
    if (set) {
        const bool ok = i < count && v >= 0 && v < n;
        const unsigned long long arcs = wave_sum<unsigned long long>(ok ? (unsigned long long)(rp[v + 1] - rp[v]) : 0ULL);
        const unsigned long long pairs = (unsigned long long)__popcll(__ballot(ok));
        if (lane_id() == 0) {
            atomicAdd(totals + kCcPairs, pairs);
            atomicAdd(totals + kCcArcs, arcs);
        }
    }
    if (i >= count) return;
    if (v < 0 || v >= n) {
        atomicOr(&st->err, kErrArg);
        return;
    }
    if (!set) {
        for (int w = 0; w < W; ++w) front[(long long)v * W + w] = 0ULL;
        return;
    }
    const unsigned long long bit = 1ULL << (i & 63);
    atomicOr(&seen[(long long)v * W + (i >> 6)], bit);
    atomicOr(&front[(long long)v * W + (i >> 6)], bit);
    atomicOr(&act[v >> 5], 1u << (v & 31));
}

// The rows for a wave and for a block each (one add to a count per block).
__global__ void k_close_lists(const int32_t *rp, int32_t n, int32_t *list0, int32_t *list1, int32_t *nlist,
                              const DevStatus *st) {
    __shared__ int32_t cnt[2], at[2];
    if (st->err & kErrGraph) return;
    if (threadIdx.x < 2) cnt[threadIdx.x] = 0;
    __syncthreads();
    const int32_t v = blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t deg = v < n ? rp[v + 1] - rp[v] : 0;
    const int q = deg > kBlockRow ? 1 : 0;
    int32_t pos = 0;
    if (deg > kWaveRow) pos = atomicAdd(&cnt[q], 1);
    __syncthreads();
    if (threadIdx.x < 2 && cnt[threadIdx.x] > 0) at[threadIdx.x] = atomicAdd(&nlist[threadIdx.x], cnt[threadIdx.x]);
    __syncthreads();
    if (deg > kWaveRow) (q ? list1 : list0)[at[q] + pos] = v;
}

// Exact form: sources that reached v in this pass.
__global__ void k_close_reach(const unsigned long long *seen, int W, int32_t n, int32_t *reach, const DevStatus *st) {
    if (st->err & kErrGraph) return;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        int32_t c = 0;
        for (int w = 0; w < W; ++w) c += (int32_t)__popcll(seen[v * W + w]);
        reach[v] += c;
    }
}

// The call's totals into the status block (by one wave of the last kernel).
__device__ __forceinline__ void totals_out(const unsigned long long *totals, DevStatus *st) {
    static_assert(kCloseTotals == kWave, "a line a lane");
    if (blockIdx.x != 0 || threadIdx.x >= kWave || (st->err & kErrGraph)) return;
    constexpr int where[kCloseCount] = {kStReached, kStArcsReached, kStArcsFwd, kStBu};
#pragma unroll
    for (int i = 0; i < kCloseCount; ++i) {
        const unsigned long long x = wave_sum<unsigned long long>(totals[16 * threadIdx.x + i]);
        if (threadIdx.x == 0) st->stat[where[i]] = x;
    }
}

// Exact form, generalised to disconnected graphs: reach counts v itself.
__global__ void k_close_exact(const unsigned long long *acc, const int32_t *reach, int32_t n, double *out,
                              const unsigned long long *totals, DevStatus *st) {
    totals_out(totals, st);
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        const int32_t r = reach[v];
        const double share = n > 1 ? (double)(r - 1) / (double)(n - 1) : 0.0;
        out[v] = (r <= 1 || n <= 1) ? 0.0 : share * ((double)(r - 1) / (double)(long long)acc[v]);
    }
}

// Sampled form (k_close_finish, under the caller's ids).
__global__ void k_close_sampled(const unsigned long long *acc, int32_t n, int32_t k, double *out,
                                const unsigned long long *totals, DevStatus *st) {
    totals_out(totals, st);
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        const double F = (double)n / (double)k * (double)acc[v];
        out[v] = F > 0.0 ? (double)(n - 1) / F : 0.0;
    }
}

template <int W>
hipError_t launch_level(const CloseArgs &a, hipStream_t s) {
    hipLaunchKernelGGL(k_close_level<W>, dim3(a.big_blocks + a.wave_blocks + (a.n + kVerts - 1) / kVerts), dim3(kCloseBlock), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_level(int W, const CloseArgs &a, hipStream_t s) {
    switch (W) {
        case 1: return launch_level<1>(a, s);
        case 2: return launch_level<2>(a, s);
        case 4: return launch_level<4>(a, s);
        case 8: return launch_level<8>(a, s);
        default: return launch_level<16>(a, s);
    }
}

// The vertices that the searches of a pass found level by level.
struct CloseGrowth {
    unsigned long long all, peak, found[4];   // in all; most on two levels; the last four levels, the latest first
    void add(unsigned long long pairs) {
        for (int i = 3; i > 0; --i) found[i] = found[i - 1];
        found[0] = pairs;
        all += pairs;
        peak = std::max(peak, pairs + found[1]);
    }
    // Whether they will end soon, of the `most` there could be: they have seen
    // a good part of the graph, or are well past their peak, or still multiply
    // -- two levels gain over the two before, and at the first look by more
    // than on a plane, where level l holds some l vertices.  Searches that do
    // none of these are those of chains, rings and planar lattices.
    bool ends_soon(bool first, unsigned long long most) const {
        const double now = (double)(found[0] + found[1]), before = (double)(found[2] + found[3]);
        const double plane = (2.0 * kCloseFirst - 1.0) / (2.0 * kCloseFirst - 5.0);
        return all >= most / 8 || 4.0 * now <= (double)peak || now >= (first ? 1.05 * plane : 1.0) * before;
    }
};

}  // namespace

nk_status close_bits(const int32_t *rowptr, const int32_t *colidx, int32_t n, int64_t m, const int32_t *sources,
                     int32_t k, bool sampled, double *out, DevStatus *dst, Scratch &scr, hipStream_t s, bool *done,
                     bool *deep) {
    *done = false;
    *deep = false;
    // A level costs a launch (about 12 us with its latencies, ten levels a
    // pass), the other kernel about k m / 200 G arcs/s and 100 us of
    // preparation: small calls stay there (G(300, 900), 100 sources: 142 us
    // there, 196 here; G(5000, 5000) exact: 1.8 and 3.3 ms; BA-9973, 64
    // sources: 513 and 190 us; exact: 3.7 and 2.2 ms).
    // A graph of many levels is left after its first look (CloseGrowth), about
    // 0.1 ms gone; lattices and trees have less than 5 arcs a vertex, and there
    // the calls that this would lengthen by more than a twelfth stay away (a
    // 60 x 60 grid, 256 sources: 0.83 ms there, 0.96 with the look; 1024: 1.16
    // and 1.25; a 300 x 300 grid, 64: 4.3 and 4.3).  Levels run to their end
    // here against there: 60 x 60 grid, 256 sources 2.3 / 0.8 ms, 20^3 grid
    // 1.0 / 1.45, small world of 10^5 vertices and 64 sources 0.9 / 6.2.
    if (n > kCloseMax) return NK_OK;
    const bool one_pass = k <= 1024;
    const double least = m < 5LL * n && m < 150000 ? 1e7 : 2e6;
    if (one_pass ? (double)k * (double)m < least : m < 20000) return NK_OK;
    int W = 1;
    while (W < 16 && 64 * W < k) W *= 2;
    // three bit arrays within the scratch allowed (fewer sources a pass
    // where they do not fit; below 64 a pass the other kernel runs)
    const int32_t cap_mib = tuning_get().scratch_mib;
    size_t avail = (size_t)cap_mib << 20;
    if (cap_mib <= 0) {
        size_t fr = 0, tot = 0;
        NK_HIP(hipMemGetInfo(&fr, &tot));
        avail = (size_t)((double)(fr + pool_bytes_idle()) * 0.85);
    }
    const auto need = [&](int w) { return (size_t)n * ((size_t)w * 24 + 16) + 4096; };
    while (W > 1 && need(W) > avail) W /= 2;
    if (need(W) > avail) return NK_OK;
    nk_status st;
    const long long words = (long long)n * W, aw = ((long long)n + 31) / 32;
    unsigned long long *seen, *f[2], *acc;
    uint32_t *act;
    int32_t *list0, *list1, *nlist, *reach = nullptr;
    unsigned long long *rows, *totals;
    // (no more such rows than this)
    const long long max0 = std::min<long long>(n, m / kWaveRow + 1), max1 = std::min<long long>(n, m / kBlockRow + 1);
    const auto take = [&]() -> nk_status {
        if ((st = scr.get(words, &seen)) != NK_OK) return st;
        if ((st = scr.get(words, &f[0])) != NK_OK) return st;
        if ((st = scr.get(words, &f[1])) != NK_OK) return st;
        if ((st = scr.get(n, &acc)) != NK_OK) return st;
        if ((st = scr.get(3 * aw, &act)) != NK_OK) return st;
        if ((st = scr.get(max0, &list0)) != NK_OK) return st;
        if ((st = scr.get(max1, &list1)) != NK_OK) return st;
        if ((st = scr.get(kCloseRows * kCloseRow, &rows)) != NK_OK) return st;
        if ((st = scr.get(kCloseTotals * 16 + 1, &totals)) != NK_OK) return st;
        nlist = reinterpret_cast<int32_t *>(totals + kCloseTotals * 16);
        return sampled ? NK_OK : scr.get(n, &reach);
    };
    if ((st = take()) != NK_OK) {
        scr.release_all();
        if (st != NK_E_NO_MEMORY) return st;
        clear_error();
        return NK_OK;
    }
    NK_HIP(launch_fill_u64(acc, 0ULL, n, s));
    NK_HIP(launch_fill_u64(totals, 0ULL, kCloseTotals * 16 + 1, s));
    if (!sampled) NK_HIP(launch_fill_i32(reach, 0, n, s));
    hipLaunchKernelGGL(k_close_lists, dim3((n + 255) / 256), dim3(256), 0, s, rowptr, n, list0, list1, nlist, dst);
    NK_HIP(hipGetLastError());
    CloseArgs a;
    memset(&a, 0, sizeof(a));
    a.rp = rowptr;
    a.ci = colidx;
    a.n = n;
    a.seen = seen;
    a.acc = acc;
    a.totals = totals;
    a.list[0] = list0;
    a.list[1] = list1;
    a.nlist = nlist;
    a.big_blocks = (int32_t)std::min<long long>(kListBlocks, m / kBlockRow);
    a.wave_blocks = (int32_t)std::min<long long>(kListBlocks, (m / kWaveRow + 3) / 4);
    a.st = dst;
    int guess = kCloseFirst;    // levels launched before the searches left are read
    // levels the first pass may take: what the other kernel's arcs cost it
    // (at most 170 arcs/us and source), at 15 us a level
    const int most_levels = (int)std::max<int64_t>(kCloseDeep, m / (170 * 15));
    unsigned long long look[kCloseFirst][kCloseRow];
    // (looks come after kCloseFirst levels and then every fourth, so the rows of
    // the levels between two looks are neighbours)
    static_assert((kCloseFirst + 2) % 4 == 0 && kCloseRows % 4 == 0, "rows of a look");
    const auto row_of = [&](int l) { return rows + (l + 1) % kCloseRows * kCloseRow; };
    for (long long s0 = 0; s0 < k; s0 += 64 * W) {
        const int32_t count = (int32_t)std::min<long long>(64 * W, k - s0);
        const long long grid = std::min<long long>((words + 255) / 256, 16384);
        hipLaunchKernelGGL(k_close_clear, dim3(std::max<long long>(grid, 8)), dim3(256), 0, s, seen, words, act, 3 * aw,
                           rows, count);
        NK_HIP(hipGetLastError());
        for (int set = 0; set < 2; ++set) {
            hipLaunchKernelGGL(k_close_sources, dim3((count + 255) / 256), dim3(256), 0, s, rowptr, sources, (int32_t)s0,
                               count, n, W, seen, f[0], act, totals, set, dst);
            NK_HIP(hipGetLastError());
        }
        int launched = 0;
        CloseGrowth growth = {};
        growth.add((unsigned long long)count);
        for (;;) {
            const int from = launched, upto = launched == 0 ? guess : launched + 4;
            while (launched < upto) {
                const int l = ++launched;
                unsigned long long *row = row_of(l);
                if (l + 1 >= kCloseRows) NK_HIP(launch_fill_u64(row, 0ULL, kCloseRow, s));
                a.level = l;
                a.front = f[(l - 1) & 1];
                a.next = f[l & 1];
                a.act = act + ((l - 1) % 3) * aw;
                a.act_next = act + (l % 3) * aw;
                a.act_clear = act + ((l + 1) % 3) * aw;
                a.alive_prev = row_of(l - 1);
                a.alive = row;
                a.counts = row + 16;
                NK_HIP(launch_level(W, a, s));
            }
            // the last level's masks; in the first pass every level's counters
            // too (a later pass goes on to its end, the ones before it are done)
            unsigned long long any = 0ULL;
            const int got = s0 == 0 ? launched - from : 1;
            NK_HIP(hipMemcpyAsync(look, row_of(launched - got + 1), s0 == 0 ? got * sizeof(look[0]) : 16 * sizeof(any),
                                  hipMemcpyDeviceToHost, s));
            NK_HIP(hipStreamSynchronize(s));
            for (int w = 0; w < 16; ++w) any |= look[got - 1][w];
            if (!any) break;
            if (s0 == 0) {
                for (int i = 0; i < got; ++i) {
                    unsigned long long pairs = 0;
                    for (int x = 0; x < kCloseXcd; ++x) pairs += look[i][16 + 16 * x + kCcPairs];
                    growth.add(pairs);
                }
                *deep = launched >= most_levels ||
                        !growth.ends_soon(from == 0, (unsigned long long)n * (unsigned long long)count);
            }
            if (*deep) {
                // the caller's other kernel.  The stream is done with the
                // bits; where they are much of the memory at hand, the pool
                // does not keep them in their sizes either
                scr.release_all();
                if (need(W) > avail / 8) pool_trim();
                return NK_OK;
            }
        }
        guess = launched;
        if (!sampled) {
            hipLaunchKernelGGL(k_close_reach, dim3(std::min<long long>((n + 255LL) / 256, 65536)), dim3(256), 0, s, seen,
                               W, n, reach, dst);
            NK_HIP(hipGetLastError());
        }
    }
    const unsigned last = (unsigned)std::min<long long>((n + 255LL) / 256, 65536);
    if (sampled)
        hipLaunchKernelGGL(k_close_sampled, dim3(last), dim3(256), 0, s, acc, n, k, out, totals, dst);
    else
        hipLaunchKernelGGL(k_close_exact, dim3(last), dim3(256), 0, s, acc, reach, n, out, totals, dst);
    NK_HIP(hipGetLastError());
    *done = true;
    return NK_OK;
}

}  // namespace nk
