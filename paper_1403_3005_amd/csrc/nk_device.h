// Device-side building blocks for the Brandes kernels (gfx950, wave64).
//
// Everything here runs inside one workgroup: wave-level scans and ballot
// compaction, a block-wide exclusive scan, the counter-based SplitMix64
// draw used by pair sampling, and the LDS tile that stages a slice of a
// vertex list (ids, adjacency starts, degree prefix sums, one 8-byte value
// per vertex) for load-balanced arc processing.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nk {

constexpr int kWave = 64;

// Error bits raised by kernels; the host maps them to nk_status codes.
enum : int32_t {
    kErrGraph = 1,      // CSR structure check failed
    kErrArg = 2,        // a source id or pair index out of range
    kErrOverflow = 4,   // a path count wrapped past 2^64 - 1
    kErrInternal = 8,   // list capacity exceeded (only after a wrap)
    kErrBusy = 16,      // a group launch's workgroups were not all resident in time: nothing was run
    kErrNarrow = 32     // a launch planned for wide levels met a thin graph and left: nothing counts
};

// Per-call device status block: error bits, the dynamic task counter and
// work counters (see nk_last_stats).
struct DevStatus {
    int32_t err;
    int32_t pad;
    unsigned long long head;
    unsigned long long stat[12];
    int32_t info[8];   // reserved
    unsigned long long cycles[8];  // shader clock cycles per phase, summed over workgroups
    unsigned long long sub[8];     // shader clock cycles per sub-phase
};

enum PhaseIdx { kPhInit = 0, kPhTd, kPhBu, kPhMark, kPhPull, kPhPush, kPhReset, kPhOther, kNumPhases };
// sub-phases of the bottom-up and pull levels (staging + scans, arc loop, finalize)
enum SubIdx { kSbBuStage = 0, kSbBuArcs, kSbBuFin, kSbPlStage, kSbPlArcs, kSbPlFin, kNumSub };
// pair mode reuses the first four slots: search, meeting-vertex choice, walks, clearing
enum PairSubIdx { kSbPairSearch = 0, kSbPairSelect, kSbPairWalk, kSbPairClear };

enum StatIdx {
    kStSources = 0, kStReached, kStArcsFwd, kStArcsBwd, kStDag, kStTd, kStBu, kStArcsReached, kStBwPush,
    kStDone,   // sources (or samples) finished so far, added as each task ends (progress of a long run)
    kStDeferred,   // pair samples left by the hashed-record launch to one with a record per vertex
    kNumStats = 12
};

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }
__device__ __forceinline__ int wave_id() { return threadIdx.x / kWave; }

// XCC (XCD) index of the executing compute unit.
__device__ __forceinline__ int32_t xcc_id() {
    return (int32_t)(__builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20) & 15u);
}

// SplitMix64 output function (Steele, Lea, Flood 2014).
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    return z ^ (z >> 31);
}

// Counter-based draw: output t+1 of a SplitMix64 stream whose seed is
// output j+1 of a stream whose seed is output stream+1 of the stream
// seeded with `seed` (k-th output of a stream seeded x = mix64(x + k*gamma)).
__device__ __forceinline__ uint64_t draw(uint64_t seed, uint64_t stream, uint64_t j, uint64_t t) {
    const uint64_t g = 0x9E3779B97F4A7C15ULL;
    uint64_t a = mix64(seed + (stream + 1) * g);
    uint64_t b = mix64(a + (j + 1) * g);
    return mix64(b + (t + 1) * g);
}

// floor(x * N / 2^64) (multiply-shift range reduction).
__device__ __forceinline__ uint64_t bounded(uint64_t x, uint64_t N) { return __umul64hi(x, N); }

template <typename T>
__device__ __forceinline__ T wave_incl_scan(T v) {
    const int lane = lane_id();
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        T y = __shfl_up(v, off, kWave);
        if (lane >= off) v += y;
    }
    return v;
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

__device__ __forceinline__ int32_t wave_min(int32_t v) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        int32_t y = __shfl_xor(v, off, kWave);
        v = y < v ? y : v;
    }
    return v;
}

// Shared-memory tile for BLOCK vertices plus block-level scalars.
template <int BLOCK>
struct Tile {
    // tile_rows: each wave's row marks, four bytes a thread (zero between
    // uses; tile_init clears them)
    uint32_t mark[BLOCK];
    int32_t a0[BLOCK];         // rowptr[v]
    int32_t pre[BLOCK + 1];    // exclusive prefix of degrees, pre[cnt] = total arcs
    union {
        unsigned long long u[BLOCK];  // sigma of a frontier vertex / bottom-up path-count sum
        double f[BLOCK];              // backward: sum of (1 + delta_w) / sigma_w
    } val;
    int32_t wsum[BLOCK / kWave + 1];
    // block scalars
    long long task;
    long long mf;              // arcs leaving the current frontier
    long long mu;              // arcs of vertices not yet visited
    long long acc_mf;          // reduction target while marking a new level
    int32_t count;             // append counter (next level / candidates)
    int32_t redmin;
    int32_t flag;
    int32_t levels;
    int32_t lvl_lo[2];
    // timing (thread 0 only)
    unsigned long long cyc[8];
    unsigned long long sub[8];
    long long t0, ts;
};

// Block-wide exclusive scan of one int per thread; returns the thread's
// exclusive prefix and the block total.  Contains barriers: every thread of
// the block must call it.
template <int BLOCK>
__device__ __forceinline__ int32_t block_excl_scan(int32_t x, Tile<BLOCK> &sm, int32_t &total) {
    constexpr int NW = BLOCK / kWave;
    const int lane = lane_id(), wid = wave_id();
    int32_t incl = wave_incl_scan<int32_t>(x);
    if (lane == kWave - 1) sm.wsum[wid] = incl;
    __syncthreads();
    if (wid == 0) {
        int32_t s = lane < NW ? sm.wsum[lane] : 0;
        int32_t si = wave_incl_scan<int32_t>(s);
        if (lane < NW) sm.wsum[lane] = si - s;
        if (lane == NW - 1) sm.wsum[NW] = si;
    }
    __syncthreads();
    total = sm.wsum[NW];
    int32_t r = incl - x + sm.wsum[wid];
    __syncthreads();
    return r;
}

// Ballot compaction: every active lane of the wave calls this; lanes with
// pred write `value` to out[base + rank], where base comes from one LDS
// atomic per wave.  Positions >= cap are dropped and flagged.
__device__ __forceinline__ void wave_append(bool pred, int32_t value, int32_t *out, int32_t *counter,
                                            int32_t cap, int32_t *err) {
    unsigned long long mask = __ballot(pred);
    if (mask == 0ULL) return;
    const int lane = lane_id();
    const int leader = __ffsll((long long)mask) - 1;
    int32_t base = 0;
    if (lane == leader) base = atomicAdd(counter, (int32_t)__popcll(mask));
    base = __shfl(base, leader, kWave);
    if (pred) {
        int32_t pos = base + (int32_t)__popcll(mask & ((1ULL << lane) - 1ULL));
        if (pos < cap)
            out[pos] = value;
        else
            atomicOr(err, kErrInternal);
    }
}

// As wave_append for N values a lane, at one LDS atomic a wave.
template <int N>
__device__ __forceinline__ void wave_append_all(const bool (&pred)[N], const int32_t (&value)[N], int32_t *out,
                                                int32_t *counter, int32_t cap, int32_t *err) {
    int32_t before[N], tot = 0;
    const unsigned long long below = (1ULL << lane_id()) - 1ULL;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const unsigned long long mask = __ballot(pred[j]);
        before[j] = tot + (int32_t)__popcll(mask & below);
        tot += (int32_t)__popcll(mask);
    }
    if (tot == 0) return;
    int32_t base = 0;
    if (lane_id() == 0) base = atomicAdd(counter, tot);
    base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
    for (int j = 0; j < N; ++j)
        if (pred[j]) {
            if (base + before[j] < cap)
                out[base + before[j]] = value[j];
            else
                atomicOr(err, kErrInternal);
        }
}

// As wave_append, and returns the lane's position in `out` (or -1 when
// pred is false or the position is past cap).
__device__ __forceinline__ int32_t wave_append_pos(bool pred, int32_t value, int32_t *out, int32_t *counter,
                                                   int32_t cap, int32_t *err) {
    unsigned long long mask = __ballot(pred);
    if (mask == 0ULL) return -1;
    const int lane = lane_id();
    const int leader = __ffsll((long long)mask) - 1;
    int32_t base = 0;
    if (lane == leader) base = atomicAdd(counter, (int32_t)__popcll(mask));
    base = __shfl(base, leader, kWave);
    if (!pred) return -1;
    const int32_t pos = base + (int32_t)__popcll(mask & ((1ULL << lane) - 1ULL));
    if (pos < cap) {
        out[pos] = value;
        return pos;
    }
    atomicOr(err, kErrInternal);
    return -1;
}

template <int BLOCK>
__device__ __forceinline__ void tile_init(Tile<BLOCK> &sm) {
    sm.mark[threadIdx.x] = 0u;
}

// Inclusive prefix maximum over the wave (row shifts, then the row
// broadcasts), values >= 0.
__device__ __forceinline__ int32_t wave_prefix_max(int32_t x) {
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));
    return x;
}

// Tile rows and CSR positions of the thread's kTileArcs consecutive arcs of
// the tile, base + kTileArcs * threadIdx.x ...: kk[j] = row, or -1 past the
// tile's end.  Every thread of the wave calls it.
//
// A wave's 256 arcs are consecutive, so the wave finds the row of its first
// arc once (two ballots over the prefix array), every later row that starts
// among them leaves its number at its start position, and a prefix maximum
// over the lanes hands each thread its row.  (A search per thread is ten
// dependent LDS reads and a walk over the row starts, together half of the
// arc loops' instructions.)  With the wave's rows, the heads' 16-byte loads
// and add_to_rows: R-MAT scale 20, 4096 sources 460 ms to 417, scale 18,
// 64 sources 8.4 ms to 7.1.  Where a tile has a few rows of a few arcs the
// search was the shorter chain: edge scores of a path of 3,000 vertices 18 ms
// to 21, path counts of a 500 x 500 grid 34 to 38, bisection on sparse graphs of
// 2.5 * 10^5 vertices 5 to 10% (two forms in one kernel cost it registers).
constexpr int kTileArcs = 4;
template <int BLOCK>
__device__ __forceinline__ void tile_rows(Tile<BLOCK> &sm, int32_t cnt, int32_t total, int32_t base,
                                          int32_t (&kk)[kTileArcs], int32_t (&arc)[kTileArcs]) {
    constexpr int SPAN = kWave * kTileArcs, STEP = BLOCK / kWave;
    const int lane = lane_id();
    const int wid = __builtin_amdgcn_readfirstlane(wave_id());
    const int32_t b0 = base + wid * SPAN;
#pragma unroll
    for (int j = 0; j < kTileArcs; ++j) {
        kk[j] = -1;
        arc[j] = 0;
    }
    if (b0 >= total) return;
    // the last row that starts at or before b0
    int32_t q = lane * STEP < cnt ? sm.pre[lane * STEP] : 0x7fffffff;
    const int32_t blk = (int32_t)__popcll(__ballot(q <= b0)) - 1;
    q = lane < STEP && blk * STEP + lane < cnt ? sm.pre[blk * STEP + lane] : 0x7fffffff;
    const int32_t k0 = blk * STEP + (int32_t)__popcll(__ballot(q <= b0)) - 1;
    const int32_t i = b0 + kTileArcs * lane;
    // all of the wave's arcs in one long row: nothing to mark
    if (sm.pre[k0 + 1] - b0 >= SPAN) {
        const int32_t off = sm.a0[k0] - sm.pre[k0];
#pragma unroll
        for (int j = 0; j < kTileArcs; ++j) {
            kk[j] = k0;
            arc[j] = off + i + j;
        }
        return;
    }
    // (rows without arcs share their start with the row after them, and can
    // put a row's number past a mark's 255)
    asm volatile("" ::: "memory");
    uint8_t *mark = reinterpret_cast<uint8_t *>(sm.mark) + wid * SPAN;
    bool far = false;
    for (int32_t k1 = k0 + 1; k1 < cnt; k1 += kWave) {
        const int32_t k = k1 + lane;
        const int32_t s = k < cnt ? sm.pre[k] - b0 : SPAN;
        if (s < SPAN && sm.pre[k + 1] - b0 > s) {
            mark[s] = (uint8_t)(k - k0);
            far = far || k - k0 > 255;
        }
        if (__ballot(s < SPAN) != ~0ULL) break;
    }
    asm volatile("" ::: "memory");
    const uint32_t f = sm.mark[threadIdx.x];
    sm.mark[threadIdx.x] = 0u;
    asm volatile("" ::: "memory");
    if (__ballot(far)) {
        if (i >= total) return;
        int32_t k = k0, hi = cnt - 1;
        while (k < hi) {
            const int32_t mid = (k + hi + 1) >> 1;
            if (sm.pre[mid] <= i)
                k = mid;
            else
                hi = mid - 1;
        }
#pragma unroll
        for (int j = 0; j < kTileArcs; ++j)
            if (i + j < total) {
                while (sm.pre[k + 1] <= i + j) ++k;
                kk[j] = k;
                arc[j] = sm.a0[k] - sm.pre[k] + i + j;
            }
        return;
    }
    int32_t m[kTileArcs];
    m[0] = (int32_t)(f & 0xFFu);
    m[1] = max(m[0], (int32_t)(f >> 8 & 0xFFu));
    m[2] = max(m[1], (int32_t)(f >> 16 & 0xFFu));
    m[3] = max(m[2], (int32_t)(f >> 24));
    const int32_t before = __builtin_amdgcn_update_dpp(0, wave_prefix_max(m[3]), 0x138, 0xf, 0xf, false);
    int32_t off = 0;
#pragma unroll
    for (int j = 0; j < kTileArcs; ++j) {
        const int32_t k = k0 + max(before, m[j]);
        if (i + j < total) {
            if (j == 0 || k != kk[j > 0 ? j - 1 : 0]) off = sm.a0[k] - sm.pre[k];
            kk[j] = k;
            arc[j] = off + i + j;
        }
    }
}

// Heads of the thread's tile arcs (ci[0] or 0 where there is none).  Four
// arcs of one row are one 16-byte load: the vector cache takes a line per
// cycle, and four 4-byte loads each touch every line of the wave's kilobyte.
// SHORT (mean degrees near 8, where few threads have one row): 16-byte loads
// only where the whole wave can, and no branch per thread otherwise -- 200k
// vertices of mean degree 8, 1024 sources: 26.1 ms against 26.8; R-MAT scale
// 20 the other way round, 426 ms against 416.
template <bool SHORT>
__device__ __forceinline__ void tile_heads(const int32_t *ci, const int32_t (&kk)[kTileArcs],
                                           const int32_t (&arc)[kTileArcs], int32_t (&w)[kTileArcs]) {
    static_assert(kTileArcs == 4, "four arcs a thread");
    struct __attribute__((packed, aligned(4))) Four { int32_t x[4]; };
    const bool whole = kk[0] >= 0 && kk[0] == kk[3];
    if (SHORT && __ballot(whole) != ~0ULL) {
#pragma unroll
        for (int j = 0; j < kTileArcs; ++j) w[j] = ci[(uint32_t)arc[j]];
        return;
    }
#pragma unroll
    for (int j = 0; j < kTileArcs; ++j) w[j] = 0;
    if (whole) {
        const Four f = *reinterpret_cast<const Four *>(ci + (uint32_t)arc[0]);
#pragma unroll
        for (int j = 0; j < kTileArcs; ++j) w[j] = f.x[j];
    } else {
#pragma unroll
        for (int j = 0; j < kTileArcs; ++j)
            if (kk[j] >= 0) w[j] = ci[(uint32_t)arc[j]];
    }
}

template <int CTRL>
__device__ __forceinline__ unsigned long long dpp_u64(unsigned long long x) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int32_t)(uint32_t)x, CTRL, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int32_t)(uint32_t)(x >> 32), CTRL, 0xf, 0xf, true);
    return ((unsigned long long)hi << 32) | lo;
}
// Addends of the tile's row sums: path counts (a wrap past 2^64 raises *ovf)
// or FP64 terms.
struct RowU64 {
    using T = unsigned long long;
    static __device__ __forceinline__ T add(T a, T b, bool &ovf) {
        const T s = a + b;
        ovf |= s < a;
        return s;
    }
    template <int CTRL>
    static __device__ __forceinline__ T step(T x, bool &ovf) { return add(x, dpp_u64<CTRL>(x), ovf); }
    static __device__ __forceinline__ void to_row(T *p, T x, bool &ovf) {
        const T o = atomicAdd(p, x);
        ovf |= o + x < o;
    }
};
struct RowF64 {
    using T = double;
    static __device__ __forceinline__ T add(T a, T b, bool &) { return a + b; }
    template <int CTRL>
    static __device__ __forceinline__ T step(T x, bool &) {
        return x + __longlong_as_double((long long)dpp_u64<CTRL>((unsigned long long)__double_as_longlong(x)));
    }
    static __device__ __forceinline__ void to_row(T *p, T x, bool &) { atomicAdd(p, x); }
};

// Adds the thread's terms x[j] (zero: none) of its tile arcs, rows kk[j], to
// the row sums in LDS.  Where sixteen threads in a row hold arcs of one row
// only, their sum is formed first and added once: adds to one LDS address
// are taken one after the other, and in a tile of hubs every thread of the
// workgroup adds to the same few.  Every thread of the wave calls it.
template <class R>
__device__ __forceinline__ void add_to_rows(typename R::T *rows, const int32_t (&kk)[kTileArcs],
                                            const typename R::T (&x)[kTileArcs], bool &ovf) {
    using T = typename R::T;
    static_assert(kTileArcs == 4, "four arcs a thread");
    // the wave's arcs all in one row (in order, so the ends tell)
    const int32_t first = __builtin_amdgcn_readlane(kk[0], 0), last = __builtin_amdgcn_readlane(kk[3], kWave - 1);
    if (first == last) {
        if (first < 0) return;
        T s = R::add(R::add(x[0], x[1], ovf), R::add(x[2], x[3], ovf), ovf);
        s = R::template step<0xB1>(s, ovf);
        s = R::template step<0x4E>(s, ovf);
        s = R::template step<0x141>(s, ovf);
        s = R::template step<0x140>(s, ovf);
        if ((lane_id() & 15) == 0 && s != (T)0) R::to_row(rows + first, s, ovf);
        return;
    }
    int32_t k = kk[0];
    T acc = x[0];
#pragma unroll
    for (int j = 1; j < kTileArcs; ++j) {
        if (kk[j] >= 0 && kk[j] != k) {
            if (acc != (T)0) R::to_row(rows + k, acc, ovf);
            k = kk[j];
            acc = (T)0;
        }
        if (kk[j] >= 0) acc = R::add(acc, x[j], ovf);
    }
    const int lane = lane_id();
    // one row here, and the same as the lane before (in the 16)
    const int32_t mine = kk[0] == k ? k : -2;
    const int32_t prev = __builtin_amdgcn_update_dpp(0, mine, 0x111, 0xf, 0xf, false);
    const bool same = mine >= 0 && ((lane & 15) == 0 || mine == prev);
    const bool one = ((__ballot(same) >> (lane & 48)) & 0xFFFFULL) == 0xFFFFULL;
    bool o16 = false;
    T s = R::template step<0xB1>(acc, o16);    // lane ^ 1
    s = R::template step<0x4E>(s, o16);        // lane ^ 2
    s = R::template step<0x141>(s, o16);       // the other four of eight
    s = R::template step<0x140>(s, o16);       // the other eight
    if (one) {
        ovf |= o16;
        if ((lane & 15) == 0 && s != (T)0) R::to_row(rows + k, s, ovf);
    } else if (acc != (T)0) {
        R::to_row(rows + k, acc, ovf);
    }
}

// Largest k in [0, cnt) with pre[k] <= i (pre[0] = 0 <= i).
__device__ __forceinline__ int32_t tile_search(const int32_t *pre, int32_t cnt, int32_t i) {
    int32_t lo = 0, hi = cnt - 1;
    while (lo < hi) {
        int32_t mid = (lo + hi + 1) >> 1;
        if (pre[mid] <= i) lo = mid; else hi = mid - 1;
    }
    return lo;
}

}  // namespace nk
