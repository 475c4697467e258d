// Brandes kernels whose per-source state lives in LDS.
//
// When a source's state fits a workgroup's 160 KB of LDS, the forward
// path-counting search and the backward dependency sweep of Brandes'
// algorithm (the betweenness method the paper relies on, "Heuristics and
// Approximation Algorithms" and Table 1) make their random accesses there,
// and global memory sees only sequential reads of the graph and one add per
// vertex and source into bc.  Two forms share the code:
//
//   graph in LDS (CSR = true)   small graphs; the workgroup copies the CSR
//       into LDS once, column indices as 16-bit values, and keeps it while
//       its tasks stay on one graph.  Always top-down and pull.
//   state in LDS (CSR = false)  graphs of up to 65,534 vertices; the CSR is
//       read from global memory (it stays in L2: every workgroup reads the
//       same one) and levels run bottom-up where that scans fewer arcs.
//       Path counts of the vertices past `hot` (0 when all fit) live in a
//       per-workgroup global array: a single graph runs in degree order, so
//       those are the vertices with the fewest arcs, and its isolated ones are
//       left out; a batch's graphs run under their own ids, where they are
//       whatever comes last (25,000 vertices of preferential attachment, exact:
//       40 ms with the hubs first, 54 with shuffled ids, 58 either way on the
//       one-source kernel).
//
// Tasks are (graph, source) pairs, drawn from one dynamic counter, for a
// single graph or for a batch of concatenated graphs.
//
// LDS layout (dynamic part, n vertices, m arcs):
//   sig  u64[hot]   sigma during the forward phase, coef = (1 + delta) /
//                   sigma (FP64 bits) once a vertex's level is swept
//   rp   i32[n+1]   row pointers      (graph in LDS)
//   d    u16[n]     level of each vertex, 0xFFFF = unreached, padded to 16 B
//   lv   u16[n]     concatenated level lists (visit order)
//   ci   u16[m]     column indices    (graph in LDS)
//
// What bounds it and why it is laid out so: every access is an LDS access
// or an L2 round trip, so the rates that matter are LDS instructions per
// arc and the length of the dependent chain per row.  Rows are given to
// groups of G lanes (4, 8 or 16 by mean degree), a row's arcs two per lane at a
// time; consecutive rows of a level go to different waves, and a row of
// more than 16 G arcs is taken by its whole wave.  That needs no prefix sum
// over the level, no search for an arc's row and no barrier inside a level
// -- the scan-and-search tiles this replaces spent about 40 LDS
// instructions per four arcs and a dozen barriers per level.  A level is
// one (top-down, pull) or two (bottom-up) barriers, which wait for LDS only,
// so the adds into bc drain behind the following levels.  The level
// of a vertex is a 16-bit value rather than a visited bit, so no pass marks
// or unmarks levels.
#include "nk_runtime.h"

namespace nk {

namespace {

constexpr int kThinProbes = 8;           // searches that judge whether a graph is thin
constexpr uint32_t kUnseen = 0xFFFFu;   // level of an unreached vertex
constexpr int kLvlCache = 256;          // level offsets kept; deeper ones are searched

// ------------------------------------------------------------ wave pieces --

template <int CTRL>
__device__ __forceinline__ int32_t dpp_mov(int32_t x) {
    return __builtin_amdgcn_mov_dpp(x, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ unsigned long long dpp_mov64(unsigned long long x) {
    const uint32_t lo = (uint32_t)dpp_mov<CTRL>((int32_t)(uint32_t)x);
    const uint32_t hi = (uint32_t)dpp_mov<CTRL>((int32_t)(uint32_t)(x >> 32));
    return ((unsigned long long)hi << 32) | lo;
}
// exchange within a quad (lane ^ 1, lane ^ 2), then the mirrors of 8 and 16
// lanes, whose halves hold equal values by then
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kHalfMirror = 0x141, kMirror = 0x140;

__device__ __forceinline__ double lf64(unsigned long long x) { return __longlong_as_double((long long)x); }
__device__ __forceinline__ unsigned long long lu64(double x) { return (unsigned long long)__double_as_longlong(x); }

// Sums that every lane of its group of W lanes receives.  The integer form
// reports a wrap past 2^64 in *ovf.
struct SumF64 {
    using T = double;
    template <int CTRL>
    static __device__ __forceinline__ double step(double x, bool &) {
        return x + lf64(dpp_mov64<CTRL>(lu64(x)));
    }
    static __device__ __forceinline__ double add(double a, double b, bool &) { return a + b; }
    static __device__ __forceinline__ unsigned long long bits(double x) { return lu64(x); }
    static __device__ __forceinline__ double val(unsigned long long x) { return lf64(x); }
};
template <bool CHECK>
struct SumU64 {
    using T = unsigned long long;
    template <int CTRL>
    static __device__ __forceinline__ unsigned long long step(unsigned long long x, bool &ovf) {
        return add(x, dpp_mov64<CTRL>(x), ovf);
    }
    static __device__ __forceinline__ unsigned long long add(unsigned long long a, unsigned long long b, bool &ovf) {
        const unsigned long long s = a + b;
        if (CHECK) ovf |= s < a;
        return s;
    }
    static __device__ __forceinline__ unsigned long long bits(unsigned long long x) { return x; }
    static __device__ __forceinline__ unsigned long long val(unsigned long long x) { return x; }
};
template <class S, int W>
__device__ __forceinline__ typename S::T group_sum(typename S::T x, bool &ovf) {
    x = S::template step<kXor1>(x, ovf);
    x = S::template step<kXor2>(x, ovf);
    if (W >= 8) x = S::template step<kHalfMirror>(x, ovf);
    if (W >= 16) x = S::template step<kMirror>(x, ovf);
    return x;
}
__device__ __forceinline__ unsigned long long lane_u64(unsigned long long x, int lane) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)x, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int32_t)(uint32_t)(x >> 32), lane);
    return ((unsigned long long)hi << 32) | lo;
}
template <class S>
__device__ __forceinline__ typename S::T wave_total(typename S::T x, bool &ovf) {
    const unsigned long long b = S::bits(group_sum<S, 16>(x, ovf));
    typename S::T t = S::add(S::val(lane_u64(b, 0)), S::val(lane_u64(b, 16)), ovf);
    t = S::add(t, S::val(lane_u64(b, 32)), ovf);
    return S::add(t, S::val(lane_u64(b, 48)), ovf);
}
// Inclusive prefix sum over the wave (row shifts, then the row broadcasts).
__device__ __forceinline__ int32_t wave_prefix(int32_t x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    return x;
}

// ----------------------------------------------------------------- state --

struct LdsShared {
    long long task;
    int32_t flag;
    int32_t loaded;                  // graph whose CSR is in LDS, -1 = none
    int32_t maxdeg;                  // largest degree of the graphs loaded so far
    int32_t nnew[3], ncand[3];       // per level, slot = level % 3
    unsigned long long dsum[3];      // degree sum of the level's new vertices
    unsigned long long stat[8];
    uint16_t lvl[kLvlCache];         // first list entry of each level
};

template <bool CSR>
struct ArcId { using T = int32_t; };
template <>
struct ArcId<true> { using T = uint16_t; };

template <bool CSR, bool COLD>
struct LdsGraph {
    unsigned long long *sig;         // LDS, vertices below hot
    unsigned long long *cold;        // global, indexed by vertex; only [hot, n) is used
    uint16_t *d;
    uint16_t *lv;                    // LDS, or global with COLD
    const int32_t *rp;
    const typename ArcId<CSR>::T *ci;
    int32_t hot;

    // (the empty statements keep the LDS and the global access apart: merged
    // into one generic access they wait for both memories)
    __device__ __forceinline__ unsigned long long get(int32_t v) const {
        unsigned long long x = sig[!COLD || v < hot ? v : 0];
        if (COLD && v >= hot) {
            x = cold[v];
            asm volatile("");
        }
        return x;
    }
    __device__ __forceinline__ void put(int32_t v, unsigned long long x) const {
        if (COLD && v >= hot) {
            cold[v] = x;
            asm volatile("");
        } else {
            sig[v] = x;
        }
    }
    __device__ __forceinline__ unsigned long long add(int32_t v, unsigned long long x) const {
        if (COLD && v >= hot) {
            const unsigned long long o = atomicAdd(&cold[v], x);
            asm volatile("");
            return o;
        }
        return atomicAdd(&sig[v], x);
    }
};

struct LdsCounters {
    unsigned long long arcs_fwd, arcs_bwd, dag, reached, tasks, td, bu, arcs_reached;
};

// 1 / s for a path count s (1 <= s < 2^64): the hardware's estimate and two
// Newton steps (to within an ulp), a third of a correctly rounded divide's
// instructions.
__device__ __forceinline__ double count_inverse(double s) {
    double r = __builtin_amdgcn_rcp(s);
    r = __builtin_fma(__builtin_fma(-s, r, 1.0), r, r);
    return __builtin_fma(__builtin_fma(-s, r, 1.0), r, r);
}

// Set bits of a wave mask below this lane.
__device__ __forceinline__ uint32_t lanes_below(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Rows row(0) .. row(cnt - 1) of the graph, a group of G lanes each.  Per row:
// begin(v) gives a lane-uniform value, arcs(w0, ok0, w1, ok1, value, acc)
// handles two of its heads, and done(v, degree, value, acc) runs in the
// group's first lane with the group's sum of acc.  A row of more than 16 G
// arcs is scanned by its whole wave.  Four neighbouring rows go to a wave,
// the next four to the next wave: neighbours in a list are often neighbours
// in memory, so their adds into bc share lines, and the waves share the hubs
// that a list in degree order starts with.  The loads are pipelined over
// rows: while a row is worked on, the next row's first heads and the range
// of the one after it are on their way.
template <int BLOCK, int G, class S, class Gr, class Row, class Begin, class Arcs, class Done>
__device__ __forceinline__ void for_rows(const Gr &L, int32_t cnt, bool &ovf, Row row, Begin begin, Arcs arcs,
                                         Done done) {
    constexpr int NW = BLOCK / kWave, ROWS = BLOCK / G, BIG = 16 * G;
    const int lane = lane_id();
    const int gl = lane % G, gw = lane / G;
    int32_t r = (gw / 4) * (4 * NW) + wave_id() * 4 + gw % 4;
    int32_t v = 0, a0 = 0, dg = 0, v2 = 0, a2 = 0, dg2 = 0;
    if (r < cnt) {
        v = row(r);
        a0 = L.rp[v];
        dg = L.rp[v + 1] - a0;
    }
    if (r + ROWS < cnt) {
        v2 = row(r + ROWS);
        a2 = L.rp[v2];
        dg2 = L.rp[v2 + 1] - a2;
    }
    int32_t w0 = 0, w1 = 0;
    if (gl < dg && dg <= BIG) {
        const auto *q = L.ci + (uint32_t)(a0 + gl);
        w0 = q[0];
        w1 = q[gl + G < dg ? G : 0];
    }
    for (int32_t r0 = 0; r0 < cnt; r0 += ROWS, r += ROWS) {
        const bool ok = r < cnt;
        int32_t n0 = 0, n1 = 0, v3 = 0, a3 = 0, b3 = 0;
        if (gl < dg2 && dg2 <= BIG) {
            const auto *q = L.ci + (uint32_t)(a2 + gl);
            n0 = q[0];
            n1 = q[gl + G < dg2 ? G : 0];
        }
        if (r + 2 * ROWS < cnt) {
            v3 = row(r + 2 * ROWS);
            a3 = L.rp[v3];
            b3 = L.rp[v3 + 1];
        }
        const unsigned long long val = ok ? begin(v) : 0ULL;
        typename S::T acc = 0;
        const bool big = dg > BIG;
        const int32_t end = big ? 0 : dg;
        arcs(w0, gl < end, w1, gl + G < end, val, acc);
        for (int32_t i = gl + 2 * G; i < end; i += 2 * G) {
            const auto *q = L.ci + (uint32_t)(a0 + i);
            const bool two = i + G < end;
            arcs((int32_t)q[0], true, (int32_t)q[two ? G : 0], two, val, acc);
        }
        acc = group_sum<S, G>(acc, ovf);
        unsigned long long mb = __ballot(big && gl == 0);
        while (mb) {
            const int b = __ffsll((long long)mb) - 1;
            mb &= mb - 1ULL;
            const int32_t ab = __builtin_amdgcn_readlane(a0, b), db = __builtin_amdgcn_readlane(dg, b);
            const unsigned long long vb = lane_u64(val, b);
            typename S::T part = 0;
            for (int32_t i = lane; i < db; i += 2 * kWave) {
                const auto *q = L.ci + (uint32_t)(ab + i);
                const bool two = i + kWave < db;
                arcs((int32_t)q[0], true, (int32_t)q[two ? kWave : 0], two, vb, part);
            }
            part = wave_total<S>(part, ovf);
            if (lane == b) acc = part;
        }
        if (ok && gl == 0) done(v, dg, val, acc);
        v = v2;
        a0 = a2;
        dg = dg2;
        v2 = v3;
        a2 = a3;
        dg2 = b3 - a3;
        w0 = n0;
        w1 = n1;
    }
}

// One pass over the levels d: the vertices at level lv1 are listed at
// lv[f1 ...] (when want_new) and the unreached ones at lv[n-1], lv[n-2], ...
// (the list's unused end), with their counts added to *nnew and *ncand.
template <int BLOCK, class Gr>
__device__ __forceinline__ void list_levels(const Gr &L, int32_t n, int32_t f1, uint32_t lv1, bool want_new,
                                            int32_t *nnew, int32_t *ncand) {
    const uint4 *d4 = reinterpret_cast<const uint4 *>(L.d);
    const int32_t n4 = (n + 7) >> 3;
    const int lane = lane_id();
    for (int32_t i0 = 0; i0 < n4; i0 += BLOCK) {
        const int32_t i = i0 + threadIdx.x;
        // (entries past n hold 0xFFFE, which is neither)
        const uint4 q = i < n4 ? d4[i] : make_uint4(0xFFFEFFFEu, 0xFFFEFFFEu, 0xFFFEFFFEu, 0xFFFEFFFEu);
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
        uint32_t mn = 0u, mc = 0u;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t x = (w[j >> 1] >> (16 * (j & 1))) & 0xFFFFu;
            mc |= x == kUnseen ? 1u << j : 0u;
            mn |= want_new && x == lv1 ? 1u << j : 0u;
        }
        const int32_t cn = __popc(mn), cc = __popc(mc);
        const int32_t incl = wave_prefix(cn | (cc << 16));
        const int32_t tot = __builtin_amdgcn_readlane(incl, kWave - 1);
        if (tot == 0) continue;
        int32_t bn = 0, bc = 0;
        if (lane == 0) {
            if (tot & 0xFFFF) bn = atomicAdd(nnew, tot & 0xFFFF);
            if (tot >> 16) bc = atomicAdd(ncand, tot >> 16);
        }
        int32_t pn = f1 + __builtin_amdgcn_readlane(bn, 0) + (incl & 0xFFFF) - cn;
        int32_t pc = n - 1 - (__builtin_amdgcn_readlane(bc, 0) + (incl >> 16) - cc);
        while (mn) {
            const int b = __builtin_ctz(mn);
            mn &= mn - 1u;
            // (the list can run over only after a path count has wrapped)
            if (pn < n) L.lv[pn++] = (uint16_t)(8 * i + b);
        }
        while (mc) {
            const int b = __builtin_ctz(mc);
            mc &= mc - 1u;
            L.lv[pc--] = (uint16_t)(8 * i + b);
        }
    }
}

// First list entry of level l, whose vertices end at list entry hi.
template <class Gr>
__device__ __forceinline__ int32_t level_start(const LdsShared &S, const Gr &L, int32_t l, int32_t hi) {
    if (l < kLvlCache) return S.lvl[l];
    int32_t a = 0, b = hi;                       // lowest entry at level >= l
    while (a < b) {
        const int32_t mid = (a + b) >> 1;
        if ((int32_t)L.d[L.lv[mid]] < l) a = mid + 1; else b = mid;
    }
    return a;
}

// A bottom-up level: every candidate (lv[n-1-r], r < nc) sums the path counts
// of its neighbours on level lvl; one with any joins level lvl + 1.
// CHECK: watch for sums past 2^64.  Returns the lane's share of the new
// level's degree sum.
template <int BLOCK, int G, bool CHECK, class Gr>
__device__ __forceinline__ uint32_t up_level(const Gr &L, int32_t n, int32_t nc, uint32_t lvl, bool &ovf,
                                             uint32_t &arcs, uint32_t &dag) {
    using Sum = SumU64<CHECK>;
    uint32_t ds = 0;
    for_rows<BLOCK, G, Sum>(
        L, nc, ovf, [&](int32_t r) { return (int32_t)L.lv[n - 1 - r]; }, [](int32_t) { return 0ULL; },
        [&](int32_t u0, bool ok0, int32_t u1, bool ok1, unsigned long long, unsigned long long &acc) {
            const bool t0 = ok0 && L.d[u0] == lvl, t1 = ok1 && L.d[u1] == lvl;
            const unsigned long long x0 = t0 ? L.get(u0) : 0ULL, x1 = t1 ? L.get(u1) : 0ULL;
            acc = Sum::add(Sum::add(acc, x0, ovf), x1, ovf);
            dag += (t0 ? 1u : 0u) + (t1 ? 1u : 0u);
        },
        [&](int32_t v, int32_t dg, unsigned long long, unsigned long long sum) {
            arcs += (uint32_t)dg;
            if (sum != 0ULL) {
                L.put(v, sum);
                L.d[v] = (uint16_t)(lvl + 1u);
                ds += (uint32_t)dg;
            }
        });
    return ds;
}

// A top-down level: the vertices lv[f0, f1) of level lvl add their path
// counts to their neighbours that are unreached, or reached on this very
// level; the first adder lists the neighbour at lv[f1 ...] (*nnew counts).
template <int BLOCK, int G, bool CHECK, class Gr>
__device__ __forceinline__ void down_level(const Gr &L, int32_t n, int32_t f0, int32_t f1, uint32_t lvl, int32_t *nnew,
                                           bool &ovf, uint32_t &arcs, uint32_t &dag) {
    const uint32_t lv1 = lvl + 1u;
    for_rows<BLOCK, G, SumU64<false>>(
        L, f1 - f0, ovf, [&](int32_t r) { return (int32_t)L.lv[f0 + r]; }, [&](int32_t v) { return L.get(v); },
        [&](int32_t w0, bool ok0, int32_t w1, bool ok1, unsigned long long sv, unsigned long long &) {
            const uint32_t d0 = L.d[w0], d1 = L.d[w1];
            const bool t0 = ok0 && (d0 == kUnseen || d0 == lv1), t1 = ok1 && (d1 == kUnseen || d1 == lv1);
            const unsigned long long o0 = t0 ? L.add(w0, sv) : 1ULL, o1 = t1 ? L.add(w1, sv) : 1ULL;
            if (CHECK) ovf |= (t0 && o0 + sv < o0) || (t1 && o1 + sv < o1);
            dag += (t0 ? 1u : 0u) + (t1 ? 1u : 0u);
            const bool n0 = o0 == 0ULL, n1 = o1 == 0ULL;
            const unsigned long long m0 = __ballot(n0), m1 = __ballot(n1);
            if (m0 | m1) {
                const int lead = __ffsll((long long)(m0 | m1)) - 1;
                const int32_t k0 = (int32_t)__popcll(m0);
                int32_t base = 0;
                if (lane_id() == lead) base = atomicAdd(nnew, k0 + (int32_t)__popcll(m1));
                base = f1 + __builtin_amdgcn_readlane(base, lead);
                // (the list can run over only after a path count has wrapped)
                if (n0) {
                    L.d[w0] = (uint16_t)lv1;
                    const int32_t p = base + (int32_t)lanes_below(m0);
                    if (p < n) L.lv[p] = (uint16_t)w0;
                }
                if (n1) {
                    L.d[w1] = (uint16_t)lv1;
                    const int32_t p = base + k0 + (int32_t)lanes_below(m1);
                    if (p < n) L.lv[p] = (uint16_t)w1;
                }
            }
        },
        [&](int32_t, int32_t dg, unsigned long long, unsigned long long) { arcs += (uint32_t)dg; });
}

// One source.  Thread 0 returns the next task in *next (fetched while the
// last sweep level runs).
template <int BLOCK, int G, bool CSR, bool COLD>
__device__ __forceinline__ void lds_source(const Params &p, LdsShared &S, const LdsGraph<CSR, COLD> &L, int32_t n,
                                           int64_t m, int32_t src, double *bcg, LdsCounters &c, long long *next) {
    const int tid = threadIdx.x;
    bool ovf = false;
    uint32_t afw = 0, abw = 0, dag = 0;   // of this source (below 2^31 arcs)
    {
        const int32_t h = COLD ? min(n, L.hot) : n;
        for (int32_t v = tid; v < h; v += BLOCK) L.sig[v] = v == src ? 1ULL : 0ULL;
        if (COLD)
            for (int32_t v = h + tid; v < n; v += BLOCK) L.cold[v] = v == src ? 1ULL : 0ULL;
        uint32_t *d2 = reinterpret_cast<uint32_t *>(L.d);
        const int32_t n2 = ((n + 7) >> 3) * 4;
        for (int32_t i = tid; i < n2; i += BLOCK) {
            uint32_t lo = 2 * i < n ? kUnseen : 0xFFFEu, hi = 2 * i + 1 < n ? kUnseen : 0xFFFEu;
            if (2 * i == src) lo = 0u;
            if (2 * i + 1 == src) hi = 0u;
            d2[i] = lo | (hi << 16);
        }
        if (tid < 3) {
            S.nnew[tid] = 0;
            S.ncand[tid] = 0;
            S.dsum[tid] = 0ULL;
        }
        if (tid == 0) {
            L.lv[0] = (uint16_t)src;
            S.lvl[0] = 0;
            S.lvl[1] = 1;
        }
    }
    const int32_t dsrc = L.rp[src + 1] - L.rp[src];
    __syncthreads();

    // ---- forward
    int32_t lvl = 0, f0 = 0, f1 = 1;
    double mf = (double)dsrc, mu = (double)(m - dsrc);
    // No path count of the next level exceeds the largest of this one times
    // a vertex's arcs, or times the arcs of this level (parallel arcs add
    // once each, so the level's size would not do), so levels whose product
    // of these stays below 2^63 need no overflow checks (checked throughout:
    // G(2000, 10000) 228 us against 224, 16 graphs of up to 25,000 vertices
    // 104 ms against 100).
    double most = 1.0;
    bool cand_ok = false;
    const bool td_only = CSR || !(p.bu_ratio > 0.0f);
    for (;;) {
        // Counters of this level (sl) and the next one's, cleared while no
        // thread can still read or add to them: slot (lvl + 1) % 3 was last
        // read two levels ago.
        const int sl = lvl % 3, sl1 = (lvl + 1) % 3, sl2 = (lvl + 2) % 3;
        const uint32_t lv1 = (uint32_t)lvl + 1u;
        const bool bu = !td_only && mu < (double)p.bu_ratio * mf;
        most *= CSR ? (double)S.maxdeg : td_only ? (double)m : mf;
        const bool check = most >= 9.2e18;
        if (bu) {
            // the candidates: listed by the previous bottom-up level, or now
            if (!cand_ok) {
                list_levels<BLOCK>(L, n, f1, lv1, false, &S.nnew[sl2], &S.ncand[sl2]);
                __syncthreads();
            }
            const int32_t nc = S.ncand[sl2];
            const uint32_t part = check ? up_level<BLOCK, G, true>(L, n, nc, (uint32_t)lvl, ovf, afw, dag)
                                        : up_level<BLOCK, G, false>(L, n, nc, (uint32_t)lvl, ovf, afw, dag);
            const uint32_t ds = wave_sum<uint32_t>(part);
            if (lane_id() == 0 && ds) atomicAdd(&S.dsum[sl], (unsigned long long)ds);
            __syncthreads();
            if (tid == 0) {
                S.nnew[sl1] = 0;
                S.ncand[sl1] = 0;
                S.dsum[sl1] = 0ULL;
                c.bu++;
            }
            list_levels<BLOCK>(L, n, f1, lv1, true, &S.nnew[sl], &S.ncand[sl]);
            __syncthreads();
            cand_ok = true;
        } else {
            if (check)
                down_level<BLOCK, G, true>(L, n, f0, f1, (uint32_t)lvl, &S.nnew[sl], ovf, afw, dag);
            else
                down_level<BLOCK, G, false>(L, n, f0, f1, (uint32_t)lvl, &S.nnew[sl], ovf, afw, dag);
            if (tid == 0) {
                S.nnew[sl1] = 0;
                S.ncand[sl1] = 0;
                S.dsum[sl1] = 0ULL;
                c.td++;
            }
            __syncthreads();
            if (!td_only) {
                // the new level's arcs decide the next direction
                const int32_t top = min(n, f1 + S.nnew[sl]);
                uint32_t ds = 0;
                for (int32_t i = f1 + tid; i < top; i += BLOCK) {
                    const int32_t v = L.lv[i];
                    ds += (uint32_t)(L.rp[v + 1] - L.rp[v]);
                }
                ds = wave_sum<uint32_t>(ds);
                if (lane_id() == 0 && ds) atomicAdd(&S.dsum[sl], (unsigned long long)ds);
                __syncthreads();
            }
            cand_ok = false;
        }
        const int32_t nnew = min(S.nnew[sl], n - f1);
        if (!td_only) {
            mf = (double)S.dsum[sl];
            mu -= mf;
        }
        if (nnew == 0) break;
        f0 = f1;
        f1 += nnew;
        ++lvl;
        if (tid == 0 && lvl + 1 < kLvlCache) S.lvl[lvl + 1] = (uint16_t)f1;
    }
    const int32_t Ld = lvl;
    c.arcs_fwd += afw;
    c.dag += dag;
    if (td_only) c.arcs_reached += afw;   // every reached vertex was expanded
    if (tid == 0) {
        if (!td_only) c.arcs_reached += (unsigned long long)((double)m - mu);
        c.reached += (unsigned long long)f1;
        c.tasks++;
        atomicAdd(&p.st->stat[kStDone], 1ULL);
    }
    if (ovf) atomicOr(&p.st->err, kErrOverflow);

    // ---- backward: level l pulls (1 + delta) / sigma from level l + 1
    long long nx = -1;
    if (Ld > 1) {
        for (int32_t i = f0 + tid; i < f1; i += BLOCK) {
            const int32_t v = L.lv[i];
            L.put(v, lu64(count_inverse((double)L.get(v))));
        }
        __syncthreads();
        int32_t hi = f0;
        for (int32_t l = Ld - 1; l >= 1; --l) {
            const int32_t lo = level_start(S, L, l, hi);
            if (l == 1 && tid == 0) nx = (long long)atomicAdd(&p.st->head, 1ULL);
            // linear scaling: pair weights d(s,v)/d(s,t) factor as l/(l+1) per DAG step
            const double wfac = p.linear ? (double)l / (double)(l + 1) : 1.0;
            const uint32_t lw = (uint32_t)l + 1u;
            bool none = false;
            for_rows<BLOCK, G, SumF64>(
                L, hi - lo, none, [&](int32_t r) { return (int32_t)L.lv[lo + r]; },
                [&](int32_t v) { return L.get(v); },
                [&](int32_t w0, bool ok0, int32_t w1, bool ok1, unsigned long long, double &acc) {
                    const bool t0 = ok0 && L.d[w0] == lw, t1 = ok1 && L.d[w1] == lw;
                    const double x0 = t0 ? lf64(L.get(w0)) : 0.0, x1 = t1 ? lf64(L.get(w1)) : 0.0;
                    acc += x0;
                    acc += x1;
                },
                [&](int32_t v, int32_t dg, unsigned long long sg, double sum) {
                    abw += (uint32_t)dg;
                    // (1 + delta) / sigma = 1 / sigma + sum * wfac
                    const double s = (double)sg, x = sum * wfac;
                    L.put(v, lu64(count_inverse(s) + x));
                    if (x != 0.0) atomicAdd(bcg + v, s * x);
                });
            __syncthreads();
            hi = lo;
        }
    }
    c.arcs_bwd += abw;
    if (tid == 0) *next = nx >= 0 ? nx : (long long)atomicAdd(&p.st->head, 1ULL);
}

// Vertices of the graph but for the isolated ones at its end (where the
// degree order puts all of them): the first v with rp[v] = m.  Clearing,
// listing and scanning them cost every source (6 * 10^4 vertices of which 300
// have arcs, 1024 sources: 3.8 ms to 0.85; 2 * 10^4 of mean degree 4 and as many
// isolated, 4096 sources: 4.9 to 2.5).
template <int BLOCK>
__device__ __forceinline__ int32_t without_isolated(const int32_t *rp, int32_t n, int32_t m, int32_t *count) {
    int32_t lo = 0, step = n;
    while (step > 1) {
        // the last of the pieces that start before it
        const int32_t len = (step + BLOCK - 1) / BLOCK;
        if (threadIdx.x == 0) *count = 0;
        __syncthreads();
        const int32_t v = lo + (int32_t)threadIdx.x * len;
        const int32_t c = (int32_t)__popcll(__ballot(v < min(n, lo + step) && rp[v] < m));
        if (lane_id() == 0 && c) atomicAdd(count, c);
        __syncthreads();
        lo += max(*count - 1, 0) * len;
        step = len;
        __syncthreads();
    }
    return min(n, lo + 1);
}

template <int BLOCK, bool CSR, bool COLD>
__global__ __launch_bounds__(BLOCK) void k_brandes_lds(Params p) {
    extern __shared__ __attribute__((aligned(16))) unsigned long long lds_dyn[];
    __shared__ LdsShared S;
    const int tid = threadIdx.x;
    if (tid == 0) {
        S.flag = p.st->err & kErrGraph;
        S.loaded = -1;
        S.maxdeg = 0;
        S.task = (long long)atomicAdd(&p.st->head, 1ULL);
    }
    __syncthreads();
    if (S.flag) return;
    LdsCounters c = {0, 0, 0, 0, 0, 0, 0, 0};
    // (a batch's graphs are not in degree order)
    const int32_t live = CSR || p.G > 0 ? p.n : without_isolated<BLOCK>(p.rowptr, p.n, p.m, &S.nnew[0]);
    // The vertices left out keep a level that is none, so that an arc into one
    // (the graph need not be symmetric to be safe) passes for an arc to a
    // visited vertex, as in the one-source kernel.
    if (!CSR && live < p.n) {
        const size_t at = (8 * (size_t)(COLD ? min(live, p.lds_hot) : live) + 15) / 16 * 16;
        uint16_t *d = reinterpret_cast<uint16_t *>(reinterpret_cast<char *>(lds_dyn) + at);
        for (int32_t i = live + tid; i < p.n; i += BLOCK) d[i] = 0xFFFEu;
    }
    for (;;) {
        const long long task = S.task;
        if (task >= p.ntasks) break;

        int32_t gid = 0, src = 0, n = p.n;
        long long m = p.m;
        const int32_t *rpg = p.rowptr, *cig = p.colidx;
        long long vbase = 0;
        if (p.G > 0) {
            int32_t lo = 0, hi = p.G - 1;
            while (lo < hi) {
                const int32_t mid = (lo + hi + 1) >> 1;
                if (p.g_task[mid] <= task) lo = mid; else hi = mid - 1;
            }
            gid = p.g_order[lo];
            vbase = p.g_vtx[gid];
            rpg = p.rowptr + vbase + gid;
            cig = p.colidx + p.g_arc[gid];
            n = (int32_t)(p.g_vtx[gid + 1] - vbase);
            m = p.g_arc[gid + 1] - p.g_arc[gid];
            src = (int32_t)(task - p.g_task[lo]);
        } else {
            src = p.sources ? p.sources[task] : (int32_t)task;
            if (!CSR && src >= 0 && src < n) n = max(live, 1);
        }
        long long next = 0;
        if (src < 0 || src >= n) {
            if (tid == 0) {
                if (src >= 0 && src < p.n && p.G == 0) {
                    // isolated: it reaches itself, on the level that finds nothing
                    c.reached++;
                    c.tasks++;
                    c.td++;
                    atomicAdd(&p.st->stat[kStDone], 1ULL);
                } else {
                    atomicOr(&p.st->err, kErrArg);
                }
                next = (long long)atomicAdd(&p.st->head, 1ULL);
            }
        } else {
            LdsGraph<CSR, COLD> L;
            char *q = reinterpret_cast<char *>(lds_dyn);
            L.hot = COLD ? p.lds_hot : n;
            L.sig = reinterpret_cast<unsigned long long *>(q);
            q += 8 * (size_t)(COLD ? min(n, L.hot) : n);
            L.cold = COLD ? p.sigma + (long long)blockIdx.x * p.stride : nullptr;
            // (16-byte alignment of the levels)
            q += (16 - ((size_t)(q - reinterpret_cast<char *>(lds_dyn)) & 15)) & 15;
            L.d = reinterpret_cast<uint16_t *>(q);
            q += 2 * (size_t)((((CSR || p.G > 0 ? n : p.n) + 7) >> 3) << 3);
            if (COLD) {
                L.lv = reinterpret_cast<uint16_t *>(p.lv + (long long)blockIdx.x * p.stride);
            } else {
                L.lv = reinterpret_cast<uint16_t *>(q);
                q += 2 * (size_t)(((n + 1) >> 1) << 1);
            }
            if constexpr (CSR) {
                int32_t *rp = reinterpret_cast<int32_t *>(q);
                uint16_t *ci = reinterpret_cast<uint16_t *>(q + 4 * ((size_t)n + 1));
                if (gid != S.loaded) {
                    int32_t md = 0;
                    for (int32_t i = tid; i <= n; i += BLOCK) {
                        const int32_t r = rpg[i];
                        rp[i] = r;
                        if (i < n) md = max(md, rpg[i + 1] - r);
                    }
                    md = wave_prefix_max(md);
                    if (lane_id() == kWave - 1) atomicMax(&S.maxdeg, md);
                    for (int32_t i0 = 0; i0 < (int32_t)m; i0 += 4 * BLOCK) {
                        int32_t x[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const int32_t i = i0 + j * BLOCK + tid;
                            x[j] = i < (int32_t)m ? cig[i] : 0;
                        }
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const int32_t i = i0 + j * BLOCK + tid;
                            if (i < (int32_t)m) ci[i] = (uint16_t)x[j];
                        }
                    }
                    __syncthreads();
                    if (tid == 0) S.loaded = gid;
                }
                L.rp = rp;
                L.ci = ci;
            } else {
                L.rp = rpg;
                L.ci = cig;
            }
            // lanes per row by the mean degree
            const long long avg2 = 2 * m / (n > 0 ? n : 1);
            double *bcg = score_copy(p) + vbase;
            if (avg2 < 24)
                lds_source<BLOCK, 4, CSR, COLD>(p, S, L, n, m, src, bcg, c, &next);
            else if (avg2 < 80)
                lds_source<BLOCK, 8, CSR, COLD>(p, S, L, n, m, src, bcg, c, &next);
            else
                lds_source<BLOCK, 16, CSR, COLD>(p, S, L, n, m, src, bcg, c, &next);
        }
        // every thread has read the task; it is replaced between two barriers
        __syncthreads();
        if (tid == 0) S.task = next;
        __syncthreads();
    }
    // counters: summed over the workgroup first (one add per workgroup and
    // counter on the status block's shared lines)
    if (tid < 8) S.stat[tid] = 0ULL;
    __syncthreads();
    const unsigned long long per_lane[4] = {c.dag, c.arcs_fwd, c.arcs_bwd, c.arcs_reached};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const unsigned long long x = wave_sum<unsigned long long>(per_lane[i]);
        if (lane_id() == 0 && x) atomicAdd(&S.stat[i], x);
    }
    if (tid == 0) {
        S.stat[4] = c.tasks;
        S.stat[5] = c.reached;
        S.stat[6] = c.td;
        S.stat[7] = c.bu;
    }
    __syncthreads();
    constexpr int where[8] = {kStDag, kStArcsFwd, kStArcsBwd, kStArcsReached, kStSources, kStReached, kStTd, kStBu};
    if (tid < 8 && S.stat[tid]) atomicAdd(&p.st->stat[where[tid]], S.stat[tid]);
}

template <int BLOCK, bool CSR, bool COLD>
void launch_lds(dim3 grid, dim3 block, size_t lds, hipStream_t s, const Params &p) {
    hipLaunchKernelGGL((k_brandes_lds<BLOCK, CSR, COLD>), grid, block, lds, s, p);
}

template <bool CSR, bool COLD>
KernelRef lds_ref(int block) {
    switch (block) {
        case 256: return KernelRef{(const void *)&k_brandes_lds<256, CSR, COLD>, &launch_lds<256, CSR, COLD>};
        case 512: return KernelRef{(const void *)&k_brandes_lds<512, CSR, COLD>, &launch_lds<512, CSR, COLD>};
        default: return KernelRef{(const void *)&k_brandes_lds<1024, CSR, COLD>, &launch_lds<1024, CSR, COLD>};
    }
}

// One workgroup column per graph: the structural CSR checks of k_validate
// for every graph of a batch in one launch.
__global__ void k_validate_batched(const int32_t *rowptr_cat, const int32_t *colidx_cat, const long long *g_vtx,
                                   const long long *g_arc, DevStatus *st) {
    const int32_t g = blockIdx.x;
    const long long v0 = g_vtx[g];
    const int32_t n = (int32_t)(g_vtx[g + 1] - v0);
    const long long m = g_arc[g + 1] - g_arc[g];
    if (n == 0) return;
    const int32_t *rowptr = rowptr_cat + v0 + g;
    const int32_t *colidx = colidx_cat + g_arc[g];
    const long long tid = (long long)blockIdx.y * blockDim.x + threadIdx.x;
    const long long stride = (long long)gridDim.y * blockDim.x;
    int bad = 0;
    if (tid == 0 && (rowptr[0] != 0 || (long long)rowptr[n] != m)) bad = 1;
    for (long long i = tid; i < n; i += stride)
        if (rowptr[i + 1] < rowptr[i]) bad = 1;
    for (long long e = tid; e < m; e += stride) {
        const int32_t x = colidx[e];
        if (x < 0 || x >= n) bad = 1;
    }
    if (bad) atomicOr(&st->err, kErrGraph);
}

// One thread per arc e = u -> v with u < v: finds the reverse arc by binary
// search in v's ascending adjacency and writes the scaled sum to both.
__global__ void k_edge_symmetrize(const int32_t *rowptr, const int32_t *colidx, int32_t n, double *ebc, double scale,
                                  DevStatus *st) {
    if (st->err & kErrGraph) return;
    const long long stride = (long long)gridDim.x * blockDim.x;
    const long long m = rowptr[n];
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += stride) {
        // tail u of arc e: the last u with rowptr[u] <= e
        int32_t lo = 0, hi = n - 1;
        while (lo < hi) {
            const int32_t mid = (lo + hi + 1) >> 1;
            if (rowptr[mid] <= e) lo = mid; else hi = mid - 1;
        }
        const int32_t u = lo, v = colidx[e];
        if (v <= u) continue;
        int32_t a = rowptr[v], b = rowptr[v + 1] - 1;
        int32_t r = -1;
        while (a <= b) {
            const int32_t mid = (a + b) >> 1;
            const int32_t x = colidx[mid];
            if (x == u) { r = mid; break; }
            if (x < u) a = mid + 1; else b = mid - 1;
        }
        if (r < 0) {
            atomicOr(&st->err, kErrGraph);
            continue;
        }
        const double tot = (ebc[e] + ebc[r]) * scale;
        ebc[e] = tot;
        ebc[r] = tot;
    }
}

// Whether searches of a graph stay thin: a workgroup a search (kThinProbes a
// graph, from vertices, or listed sources, spread over it) sets its entry of
// `thin` to 1 if kThinProbeLevels levels hold fewer than kThinProbeFound vertices,
// else to 0.
// The visited set is a hash table in LDS, which the limit keeps sparse.  The
// graph need not be valid: every index is checked.
constexpr int32_t kThinProbeLevels = 16, kThinProbeFound = 256;
constexpr int kThinTable = 2048;
__device__ bool thin_search(const int32_t *rp, const int32_t *ci, int32_t n, long long m, int32_t src) {
    __shared__ int32_t table[kThinTable], list[kThinTable];
    __shared__ int32_t count;
    for (int h = threadIdx.x; h < kThinTable; h += blockDim.x) table[h] = -1;
    if (src < 0 || src >= n) return false;
    if (threadIdx.x == 0) {
        list[0] = src;
        count = 1;
    }
    __syncthreads();
    if (threadIdx.x == 0) table[((uint32_t)src * 2654435761u) >> 21] = src;
    __syncthreads();
    int32_t f0 = 0, f1 = 1;
    for (int l = 0; l < kThinProbeLevels; ++l) {
        for (int32_t r = f0 + wave_id(); r < f1; r += 256 / kWave) {
            const int32_t v = list[r];
            const long long a = rp[v], b = rp[v + 1];
            if (a < 0 || b > m) continue;
            for (long long e = a + lane_id(); e < b; e += kWave) {
                if (__hip_atomic_load(&count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >= kThinProbeFound) break;
                const int32_t u = ci[e];
                if (u < 0 || u >= n) continue;
                // (at most 256 vertices and one of each thread come in: a free
                // place is found)
                uint32_t h = ((uint32_t)u * 2654435761u) >> 21;
                for (;; h = (h + 1) & (kThinTable - 1)) {
                    const int32_t old = atomicCAS(&table[h], -1, u);
                    if (old == u) break;
                    if (old == -1) {
                        list[atomicAdd(&count, 1)] = u;
                        break;
                    }
                }
            }
        }
        __syncthreads();
        const int32_t c = count;
        __syncthreads();
        if (c >= kThinProbeFound || c == f1) return false;
        f0 = f1;
        f1 = c;
    }
    return true;
}

// One graph of n vertices and m arcs, or (tab) several: four entries each, the
// first in rowptr, the vertices, the first in colidx, the arcs.
__global__ __launch_bounds__(256) void k_thin_probe(const int32_t *rowptr, const int32_t *colidx, int32_t n, long long m,
                                                    const long long *tab, const int32_t *sources, long long k,
                                                    int32_t *thin) {
    const int32_t g = blockIdx.x, i = blockIdx.y;
    if (tab) {
        rowptr += tab[4 * g];
        n = (int32_t)tab[4 * g + 1];
        colidx += tab[4 * g + 2];
        m = tab[4 * g + 3];
    }
    const long long at = (sources ? k : n) * (2 * i + 1) / (2 * kThinProbes);
    const bool is = thin_search(rowptr, colidx, n, m, sources ? sources[at] : (int32_t)at);
    if (threadIdx.x == 0) thin[g * kThinProbes + i] = is ? 1 : 0;
}

__global__ void k_reset_head(DevStatus *st) {
    if (threadIdx.x == 0) st->head = 0ULL;
}

}  // namespace

static size_t up16(size_t x) { return (x + 15) & ~(size_t)15; }

size_t lds_graph_bytes(int32_t n, int64_t m) {
    if (n > 65534) return (size_t)1 << 40;   // 16-bit vertex ids
    return lds_state_bytes(n) + 4 * ((size_t)n + 1) + 2 * (size_t)m;
}

size_t lds_state_bytes(int32_t n) {
    if (n > 65534) return (size_t)1 << 40;
    return up16(8 * (size_t)n) + 2 * (((size_t)n + 7) / 8 * 8) + 2 * (((size_t)n + 1) / 2 * 2);
}

size_t lds_hot_bytes(int32_t n, int32_t hot) { return up16(8 * (size_t)hot) + 2 * (((size_t)n + 7) / 8 * 8); }

KernelRef brandes_lds_kernel(int block) { return lds_ref<true, false>(block); }

KernelRef brandes_state_kernel(int block, bool cold) {
    return cold ? lds_ref<false, true>(block) : lds_ref<false, false>(block);
}

hipError_t launch_validate_batched(const int32_t *rowptr_cat, const int32_t *colidx_cat, const long long *g_vtx,
                                   const long long *g_arc, int32_t G, DevStatus *st, hipStream_t s) {
    if (G <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_validate_batched, dim3(G, 16), dim3(256), 0, s, rowptr_cat, colidx_cat, g_vtx, g_arc, st);
    return hipGetLastError();
}

hipError_t launch_edge_symmetrize(const int32_t *rowptr, const int32_t *colidx, int32_t n, double *ebc,
                                  double scale, DevStatus *st, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_edge_symmetrize, dim3(1024), dim3(256), 0, s, rowptr, colidx, n, ebc, scale, st);
    return hipGetLastError();
}

nk_status thin_graph(const int32_t *rowptr, const int32_t *colidx, int32_t n, int64_t m, const int32_t *sources,
                     long long k, DevStatus *host, hipStream_t s, bool *thin) {
    static_assert(sizeof(host->info) == sizeof(int32_t) * kThinProbes, "an entry a probe");
    hipLaunchKernelGGL(k_thin_probe, dim3(1, kThinProbes), dim3(256), 0, s, rowptr, colidx, n, (long long)m,
                       (const long long *)nullptr, sources, k, host->info);
    NK_HIP(hipGetLastError());
    NK_HIP(hipStreamSynchronize(s));
    int c = 0;
    for (int32_t x : host->info) c += x;
    *thin = c > kThinProbes / 2;
    return NK_OK;
}

nk_status thin_graphs(const int32_t *rowptr, const int32_t *colidx, const std::vector<long long> &tab, hipStream_t s,
                      std::vector<int32_t> *thin) {
    Scratch scr;
    long long *d;
    int32_t *out;
    nk_status st;
    const size_t count = tab.size() / 4;
    std::vector<int32_t> h(count * kThinProbes);
    if ((st = scr.get((long long)tab.size(), &d)) != NK_OK) return st;
    if ((st = scr.get((long long)h.size(), &out)) != NK_OK) return st;
    NK_HIP(hipMemcpyAsync(d, tab.data(), sizeof(long long) * tab.size(), hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_thin_probe, dim3((unsigned)count, kThinProbes), dim3(256), 0, s, rowptr, colidx, 0, 0LL, d,
                       (const int32_t *)nullptr, 0LL, out);
    NK_HIP(hipGetLastError());
    NK_HIP(hipMemcpyAsync(h.data(), out, sizeof(int32_t) * h.size(), hipMemcpyDeviceToHost, s));
    NK_HIP(hipStreamSynchronize(s));
    thin->assign(count, 0);
    for (size_t g = 0; g < count; ++g) {
        int c = 0;
        for (int i = 0; i < kThinProbes; ++i) c += h[g * kThinProbes + i];
        (*thin)[g] = c > kThinProbes / 2;
    }
    return NK_OK;
}

hipError_t launch_reset_head(DevStatus *st, hipStream_t s) {
    hipLaunchKernelGGL(k_reset_head, dim3(1), dim3(64), 0, s, st);
    return hipGetLastError();
}

}  // namespace nk
