// watch.h -- AC-6 trimming of one graph by one workgroup or one wavefront
// (Section 6.2, Alg. par-ac-6-trim), for graphs whose vertex statuses fit LDS.
//
// The supporting sets (Section 6.1) tell a removed vertex whom to hand back.
// Within one compute unit they are not needed as lists: every vertex keeps its
// support, and passes over the vertices read the status bit of each one's
// support in LDS and list those whose support was removed (the vertices handed
// back); each of them then resumes its DoPost after its old support.  The
// support searches, and so the successor checks counted, are those of the list
// form: every position is passed at most once, only when its target is
// removed, and removals are final, so the totals are the same for every
// schedule.
//
// Why: a hand-back through lists in device memory is a chain of dependent
// accesses (exchange, one link per member, record, heads, CAS; 0.3 to 1 us
// each), which bounded every phase of a small graph at 10 to 26 us.  A pass
// over the supports stays in LDS for graphs of up to 65,536 vertices (statuses
// one bit, supports 16 bits per vertex: 136 KB of the 160 KB).  What bounds it
// is instructions: a wavefront's instruction takes four cycles, so a pass over
// 65,536 vertices with 25 instructions per vertex took 12.8 us.  Hence two
// supports per 32-bit read, no test of the vertex's own status (a removed
// vertex's support becomes the null vertex, below) and no bounds tests (the
// supports are padded with the null vertex to whole batches).
//
// The null vertex is one that was removed before the sweep: nobody's support,
// so its 16-bit id is free to stand for "never handed back".  During the
// passes its status bit is clear; scans recognise it by its id.  Without such
// a vertex nothing is removed at all and there are no passes.
//
// Steps of one graph (a group = a workgroup or a wavefront; group barriers in
// between):
//   init    status bits: set for vertices without successors, preset ones and
//           the positions past n;
//   sweep   DoPost of every vertex against those bits; the vertices that find
//           no live successor go to a second bitmap;
//   forest  (optional) the collapse of the last-successor forest: the links
//           sit in the supports' LDS array and are jumped in place until a
//           round settles nothing more;
//   passes  watch the supports and resume the scans of the vertices handed
//           back, until a pass hands none back, or many have handed back few:
//   lists   every vertex left joins its support's list, and phases over the
//           lists finish (group_lists.h).
#pragma once
#include <climits>

#include "trim_device.h"
#include "layout.h"
#include "group_lists.h"

namespace trim {

namespace {

constexpr int kWatchMaxN = 1 << 19;     // status bits in LDS up to this many
constexpr int kWatchUnroll = 8;         // vertices per lane in flight in the sweep
constexpr int kWatchScan = 4;           // successors per step of a resumed scan
constexpr int kWatchHops = 4;           // links followed per forest round
constexpr int kWatchSlots = 2 * kWatchReads;   // vertices per lane and step of a pass
constexpr int kWatchSteps = 8;          // steps whose finds are listed in one go
constexpr int kWatchList = 512;         // list entries of one wavefront
static_assert(kWatchSlots * kWatchSteps == 64, "the finds of a lane are the bits of one word");
constexpr int kWatchCnt = 4;            // LDS words of a group: flags, null vertex
// A pass costs the same however few vertices it hands back: 3.4 us at 56,000
// vertices, 2.1 at 20,000, 2.6 by one wavefront at 4,000, and 8 and 17 with the
// supports of 100,000 and 300,000 in device memory; a phase over lists
// (group_lists.h) takes about 1.8, after the vertices left were registered (0.2
// ms at 56,000).  So a graph that had more than so many passes in which no
// wavefront handed back more than kNarrowLanes vertices goes on with lists.
// Paths v -> v + 1 with every edge twice, us: one of 56,000 vertices 188,700 ->
// 101,800 (device-wide lists 175,900), of 66 levels among them 387 -> 386 (341); in
// a batch one of 3,000 among 100,000 vertices 23,800 -> 6,130 (lists
// from the start 5,680), of 1,000 among 500,000 27,200 -> 4,780 (4,890).
constexpr int kNarrowLanes = 8;
constexpr int kNarrowLds = 64, kNarrowMem = 24;   // supports in LDS, in device memory
// The limit for a workgroup with supports in LDS; below 16,384 vertices its
// passes cost no more than phases.
__device__ __forceinline__ int narrow_limit(int n) { return n < 16384 ? INT_MAX : kNarrowLds; }

// Graph views with plain loads: a small graph is read again from the caches.
struct CachedView {
    const int* row_off;
    const int* col;
    int m;
    __device__ __forceinline__ int vctx(int) const { return 0; }
    __device__ __forceinline__ int begin(int v) const { return row_off[v]; }
    __device__ __forceinline__ int end(int v) const { return row_off[v + 1]; }
    __device__ __forceinline__ int target(int, int p, int) const { return col[p]; }
};

// The targets at p .. p + kWatchScan - 1, clamped to e - 1.  One lane's scan is
// contiguous and every lane's is elsewhere, and a compute unit takes one
// address a cycle, so where the array allows it they come in 16-byte loads:
// eight 4-byte loads a step made the scans of core+tail 65,536 cost 90 us.
template <class View>
__device__ __forceinline__ void wt_targets(const View& g, int u, uint32_t p, int e, int ctx,
                                           int (&w)[kWatchScan]) {
#pragma unroll
    for (int j = 0; j < kWatchScan; ++j) w[j] = g.target(u, (int)step_index(p, j, e), ctx);
}
__device__ __forceinline__ void wt_targets(const CachedView& g, int, uint32_t p, int e, int,
                                           int (&w)[kWatchScan]) {
    typedef int v4 __attribute__((ext_vector_type(4), aligned(4)));
    if (p + kWatchScan <= (uint32_t)g.m) {   // the entries past e belong to other lists
#pragma unroll
        for (int j = 0; j < kWatchScan; j += 4) {
            const v4 x = *reinterpret_cast<const v4*>(g.col + p + j);
            w[j] = x.x;
            w[j + 1] = x.y;
            w[j + 2] = x.z;
            w[j + 3] = x.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < kWatchScan; ++j) w[j] = g.col[step_index(p, j, e)];
    }
}

constexpr int kWatchWG = __HIP_MEMORY_SCOPE_WORKGROUP;
// Supports and positions in device memory (int): every word is touched by the
// group that owns the graph only.
__device__ __forceinline__ int wt_get(const int* t, int v) { return ld_s<kWatchWG>(t + v); }
__device__ __forceinline__ void wt_set(int* t, int v, int x) {
    __hip_atomic_store(t + v, x, __ATOMIC_RELAXED, kWatchWG);
}
// LDS is read with plain loads (several stay in flight; an atomic load is
// waited for on the spot when it sits under a condition).  Between two reads
// of a word that matters lies a barrier or an atomic, which keep the compiler
// from reusing the first; a status read late only delays a removal's effect.
__device__ __forceinline__ int wt_get(const uint16_t* t, int v) { return t[v]; }
__device__ __forceinline__ void wt_set(uint16_t* t, int v, int x) { t[v] = (uint16_t)x; }
__device__ __forceinline__ bool wt_bit(const uint32_t* bits, int v) {
    return __builtin_amdgcn_ubfe(bits[v >> 5], (unsigned)v, 1) != 0;   // the low five bits of v
}

// Keeps the compiler from moving an LDS access across it (the LDS itself serves
// a wavefront's accesses in order).
__device__ __forceinline__ void wt_order() { asm volatile("" ::: "memory"); }

enum WatchEnd { kStalled, kDone, kNarrow };

// One graph: vertices 0 .. n - 1 of the view g, targets in the same numbering.
//   Sup   uint16_t: supports in LDS; int: in device memory
//   Cur   the supports' positions, likewise
//   Item  the list's entries (LDS)
template <class View, class Sup, class Cur, class Item, bool kWaveGroup>
struct Watch {
    const View& g;
    const int n;
    uint32_t* bits;   // LDS: statuses, whole 64-bit pairs of words
    Sup* sup;         // watch_padded(n, lanes) entries when 16-bit, else n
    Cur* cur;
    Item* list;       // LDS: kWatchList entries per wavefront; before the
                      // passes, room for a second bitmap
    int* cnt;         // LDS: kWatchCnt words of the group
    const int sched;
    WatchTotals& t;
    int steps = 0, jumps = 0;   // passes and forest rounds run

    __device__ __forceinline__ int rank() const {
        return kWaveGroup ? lane_id() : (int)threadIdx.x;
    }
    __device__ __forceinline__ int size() const { return kWaveGroup ? kWave : (int)blockDim.x; }
    __device__ __forceinline__ void sync() const {
        complete_mem();
        if (kWaveGroup) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else {
            __syncthreads();
        }
    }
    // Between passes only LDS passes from one wavefront to another (a vertex's
    // position and a support in device memory are its own wavefront's), so the
    // stores to device memory are not waited for.
    __device__ __forceinline__ void sync_lds() const {
        if (kWaveGroup) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            wt_order();
        }
    }
    // the null vertex (after init), or -1
    __device__ __forceinline__ int null_vertex() const { return cnt[3] - 1; }

    __device__ __forceinline__ void init(const uint32_t* preset) {
        constexpr int U = kWatchUnroll;
        if (rank() < kWatchCnt) cnt[rank()] = 0;
        sync();
        const int rounds = (n + size() - 1) / size();
        for (int i = 0; i < rounds; i += U) {
            int b[U], e[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int v = min((i + k) * size() + rank(), n - 1);
                b[k] = g.begin(v);
                e[k] = g.end(v);
            }
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int v = (i + k) * size() + rank();
                const bool in = v < n;
                if (in) t.deg += (uint64_t)(e[k] - b[k]);
                const bool gone =
                    in && (b[k] == e[k] || (preset && ((preset[v >> 5] >> (v & 31)) & 1u)));
                const uint64_t m = ballot(gone), past = ballot(!in);
                if (lane_id() == 0 && in) {
                    bits[v >> 5] = (uint32_t)(m | past);
                    bits[(v >> 5) + 1] = (uint32_t)((m | past) >> 32);
                    if (m) cnt[3] = v + __ffsll((unsigned long long)m);   // any of them
                }
            }
        }
        sync();
    }

    // The support search of every vertex; only the vertices of `bits` are
    // removed while it runs.  sup gets the supports, or, with kForest, the
    // links (v's support when that is its last successor, else v), and `keep`
    // the supports.
    template <bool kForest, class Keep>
    __device__ __forceinline__ void sweep(Keep* keep) {
        constexpr int U = kWatchUnroll;
        const int null = null_vertex();
        uint32_t* none = reinterpret_cast<uint32_t*>(list);
        const int rounds = (n + size() - 1) / size();
        uint64_t edges = 0;
        for (int i0 = 0; i0 < rounds; i0 += U) {
            int v[U], b[U], e[U], p[U], w[U], ctx[U];
            bool in[U], gone[U], ok[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                int i = i0 + k;
                if (sched & TRIM_SCHED_REVERSE) i = rounds - 1 - i;
                v[k] = i * size() + rank();
                in[k] = i >= 0 && v[k] < n;
                const int x = in[k] ? v[k] : 0;
                b[k] = g.begin(x);
                e[k] = g.end(x);
                gone[k] = wt_bit(bits, x);
            }
#pragma unroll
            for (int k = 0; k < U; ++k) {
                if (!in[k] || gone[k]) e[k] = b[k];
                ctx[k] = b[k] < e[k] ? g.vctx(v[k]) : 0;
                w[k] = b[k] < e[k] ? g.target(v[k], b[k], ctx[k]) : 0;
                p[k] = b[k];
            }
#pragma unroll
            for (int k = 0; k < U; ++k) ok[k] = !wt_bit(bits, w[k]) && b[k] < e[k];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                if (b[k] < e[k] && !ok[k]) {   // the rare scan past removed vertices
                    for (++p[k]; p[k] < e[k]; ++p[k]) {
                        w[k] = g.target(v[k], p[k], ctx[k]);
                        if (!wt_bit(bits, w[k])) break;
                    }
                    ok[k] = p[k] < e[k];
                }
                if (ok[k]) {
                    edges += (uint64_t)(p[k] - b[k] + 1);
                    wt_set(cur, v[k], p[k]);
                } else {
                    edges += (uint64_t)(e[k] - b[k]);
                }
                if (in[k]) {
                    const int s = ok[k] ? w[k] : null;
                    wt_set(sup, v[k], !kForest ? s : ok[k] && p[k] + 1 == e[k] ? s : v[k]);
                    if (kForest) wt_set(keep, v[k], s);
                }
                const uint64_t m = ballot(b[k] < e[k] && !ok[k]);
                if (lane_id() == 0 && in[k]) {
                    none[v[k] >> 5] = (uint32_t)m;
                    none[(v[k] >> 5) + 1] = (uint32_t)(m >> 32);
                }
            }
        }
        t.sweep += edges;
        t.edges += edges;
        sync();
        const int nwords = (n + 31) >> 5;
        for (int i = rank(); i < nwords; i += size()) {
            const uint32_t m = none[i];
            bits[i] |= m;
            if (kForest) t.forest += __popc(m);
            else t.closes += __popc(m);
        }
        sync();
    }

    // The collapse of the last-successor forest over the links in sup.  A
    // member with a removed vertex up its links is removed; one whose links
    // end at an open root becomes one itself.  A round that settles no member
    // leaves only links into cycles.  Then sup gets the supports (`keep`) of
    // the vertices left.  False when `budget` rounds did not do.
    template <class Keep>
    __device__ __forceinline__ bool forest(const Keep* keep, int budget) {
        constexpr int U = kWatchSlots;
        const int rounds = (n + size() - 1) / size();
        if (rank() < 3) cnt[rank()] = 0;
        sync();
        const int wave = __builtin_amdgcn_readfirstlane(kWaveGroup ? 0 : rank() / kWave);
        Item* mine = list + wave * kWatchList;
        for (;; ++jumps) {
            bool settled = false, left = false;
            auto jump = [&](int v) {
                int x = wt_get(sup, v);
                bool open = false, dead = wt_bit(bits, x);
                for (int h = 0; h < kWatchHops && !dead && !open; ++h) {
                    const int y = wt_get(sup, x);
                    wt_order();   // a removal sets the bit, then the link
                    open = y == x;
                    x = y;
                    dead = wt_bit(bits, x);
                }
                if (dead) {
                    atomicOr(bits + (v >> 5), 1u << (v & 31));
                    t.forest += 1;
                    settled = true;
                    wt_order();
                    wt_set(sup, v, v);
                } else if (open) {
                    settled = true;
                    wt_set(sup, v, v);
                } else {
                    left = true;
                    wt_set(sup, v, x);
                }
            };
            for (int i0 = 0; i0 < rounds; i0 += U * kWatchSteps) {
                uint64_t found = 0;   // members not settled yet
#pragma unroll 1
                for (int b = 0; b < kWatchSteps; ++b) {
                    const int i = i0 + b * U;
                    if (i >= rounds) break;
                    int a[U];
                    uint32_t f = 0;
#pragma unroll
                    for (int k = 0; k < U; ++k)
                        a[k] = wt_get(sup, min((i + k) * size() + rank(), n - 1));
#pragma unroll
                    for (int k = 0; k < U; ++k) {
                        const int v = (i + k) * size() + rank();
                        f |= (uint32_t)(v < n && a[k] != v) << k;
                    }
                    found |= (uint64_t)f << (U * b);
                }
                take(found, [&](int s) { return (i0 + s) * size() + rank(); }, mine, jump);
            }
            // flags rotate over three words: the one cleared was last read
            // before this barrier and is next written after the next one
            int* flag = cnt + jumps % 3;
            const int f0 = (ballot(settled) ? 1 : 0) | (ballot(left) ? 2 : 0);
            if (f0 && lane_id() == 0) atomicOr(flag, f0);
            sync_lds();
            const int f = __hip_atomic_load(flag, __ATOMIC_RELAXED, kWatchWG);
            if (rank() == 0) cnt[(jumps + 2) % 3] = 0;
            if (jumps >= budget) return false;
            if (f != 3) break;   // nothing settled, or nothing left
        }
        ++jumps;
        sync();
        const int null = null_vertex();
        for (int i = 0; i < rounds; i += U) {
            int s[U];
#pragma unroll
            for (int k = 0; k < U; ++k)
                s[k] = wt_get(keep, min((i + k) * size() + rank(), n - 1));
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int v = (i + k) * size() + rank();
                if (v < n) wt_set(sup, v, wt_bit(bits, v) ? null : s[k]);
            }
        }
        sync();
        return true;
    }

    // Lists the vertices vertex(s) of every lane's finds (the set bits s of f)
    // and has run() take them, 64 at a time.  The lanes' places come from the
    // bits of their counts, one ballot each; listing every step's finds by
    // themselves, a ballot for each of eight slots, took 6 of 11 us a pass at
    // 65,536 vertices, and an LDS counter that the lanes add to is turned into
    // a loop over the lanes by the compiler and took more.
    template <class Vertex, class Run>
    __device__ __forceinline__ void take(uint64_t f, Vertex vertex, Item* mine, Run run) {
        while (ballot(f != 0)) {   // once, unless there are more than kWatchList
            const int c = __popcll(f);
            int at = 0, total = 0;
#pragma unroll 1
            for (int b = 0; ballot((c >> b) != 0); ++b) {
                const uint64_t m = ballot((c >> b) & 1);
                at += (int)__builtin_amdgcn_mbcnt_hi(
                          (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0)) << b;
                total += __builtin_popcountll(m) << b;
            }
            for (; f && at < kWatchList; f &= f - 1)
                mine[at++] = (Item)vertex(__ffsll((unsigned long long)f) - 1);
            wt_order();
            if (total > kWatchList) total = kWatchList;
#pragma unroll 1
            for (int i = lane_id(); i < total; i += kWave) run((int)mine[i]);
            wt_order();
        }
    }

    // Resume DoPost of u after its old support.
    __device__ __forceinline__ void resume_scan(int u, int null) {
        constexpr int K = kWatchScan;
        const int p0 = wt_get(cur, u) + 1;
        const int e = g.end(u), ctx = g.vctx(u);
        if (sched & TRIM_SCHED_JITTER) jitter_nap((uint64_t)u);
        t.visited += 1;
        int at = -1, to = 0;
        for (uint32_t p = p0; p < (uint32_t)e && at < 0; p += K) {
            int w[K];
            bool live[K];
            wt_targets(g, u, p, e, ctx, w);
#pragma unroll
            for (int j = 0; j < K; ++j) live[j] = !wt_bit(bits, w[j]) && w[j] != null;
#pragma unroll
            for (int j = 0; j < K; ++j)
                if (at < 0 && p + j < (uint32_t)e && live[j]) {
                    at = (int)(p + j);
                    to = w[j];
                }
        }
        if (at >= 0) {
            t.edges += (uint64_t)(at - p0 + 1);
            wt_set(cur, u, at);
            wt_set(sup, u, to);
            t.joins += 1;
        } else {
            t.edges += (uint64_t)(e - p0);
            atomicOr(bits + (u >> 5), 1u << (u & 31));
            wt_set(sup, u, null);
            t.closes += 1;
        }
    }

    // One wavefront's share of a pass; true when it handed a vertex back.  It
    // goes from its last vertex down and resumes scans every kWatchSteps steps,
    // so removals take effect within the pass.
    __device__ __forceinline__ bool watch(Item* mine, int wave, int waves, int null) {
        bool any = false;
        auto run = [&](int u) { resume_scan(u, null); };
        if constexpr (sizeof(Sup) == 2) {
            constexpr int R = kWatchReads;
            const uint32_t* pair = reinterpret_cast<const uint32_t*>(sup);
            const int per = watch_padded(n, waves * kWave) / 2 / waves;   // pairs per wavefront
            for (int top = (wave + 1) * per - R * kWave; top >= wave * per;
                 top -= kWatchSteps * R * kWave) {
                uint64_t found = 0;
#pragma unroll 1
                for (int b = 0; b < kWatchSteps; ++b) {
                    const int j0 = top - b * R * kWave;
                    if (j0 < wave * per) break;
                    const uint32_t* q = pair + j0 + lane_id();
                    uint32_t x[R], lo[R], hi[R], f = 0;
#pragma unroll
                    for (int k = 0; k < R; ++k) x[k] = q[k * kWave];
#pragma unroll
                    for (int k = 0; k < R; ++k) {
                        lo[k] = *reinterpret_cast<const uint32_t*>(
                            reinterpret_cast<const char*>(bits) + ((x[k] >> 3) & 0x1FFCu));
                        hi[k] = *reinterpret_cast<const uint32_t*>(
                            reinterpret_cast<const char*>(bits) + ((x[k] >> 19) & 0x1FFCu));
                    }
#pragma unroll
                    for (int k = 0; k < R; ++k) {
                        f |= __builtin_amdgcn_ubfe(lo[k], x[k], 1) << (2 * k);
                        f |= __builtin_amdgcn_ubfe(hi[k], x[k] >> 16, 1) << (2 * k + 1);
                    }
                    found |= (uint64_t)f << (kWatchSlots * b);
                }
                if (ballot(found != 0) == 0) continue;
                any = true;
                take(found, [&](int s) {
                    return 2 * (top + ((s % kWatchSlots >> 1) - s / kWatchSlots * R) * kWave +
                                lane_id()) + (s & 1);
                }, mine, run);
            }
        } else {
            constexpr int R = kWatchSlots;
            const int step = waves * kWave;
            for (int top = (n - 1) / (R * step) * (R * step) + wave * kWave; top >= 0;
                 top -= kWatchSteps * R * step) {
                uint64_t found = 0;
#pragma unroll 1
                for (int b = 0; b < kWatchSteps; ++b) {
                    const int v0 = top - b * R * step;
                    if (v0 < 0) break;
                    int s[R];
                    uint32_t f = 0;
#pragma unroll
                    for (int k = 0; k < R; ++k)
                        s[k] = wt_get(sup, min(v0 + k * step + lane_id(), n - 1));
#pragma unroll
                    for (int k = 0; k < R; ++k)
                        f |= (uint32_t)(wt_bit(bits, s[k]) && v0 + k * step + lane_id() < n) << k;
                    found |= (uint64_t)f << (kWatchSlots * b);
                }
                if (ballot(found != 0) == 0) continue;
                any = true;
                take(found, [&](int s) {
                    return top + (s % R - s / R * R) * step + lane_id();
                }, mine, run);
            }
        }
        return any;
    }

    // Passes until one hands no vertex back (kDone), until they and the forest
    // rounds would exceed `budget` (kStalled), or until more than `narrow_limit`
    // were narrow (kNarrow, with kCounted: go on by to_lists).  At the end the null vertex's bit
    // is set again.
    template <bool kCounted = false>
    __device__ __forceinline__ WatchEnd passes(int budget, int narrow_limit = INT_MAX) {
        const int null = null_vertex();
        if (null < 0) return kDone;   // nothing was removed before the sweep, nothing ever is
        if (rank() < 3) cnt[rank()] = 0;
        if (rank() == 0) bits[null >> 5] &= ~(1u << (null & 31));
        const int waves = size() / kWave;
        const int wave = __builtin_amdgcn_readfirstlane(kWaveGroup ? 0 : rank() / kWave);
        if constexpr (sizeof(Sup) == 2)
            for (int v = n + rank(); v < watch_padded(n, size()); v += size()) wt_set(sup, v, null);
        sync();
        Item* mine = list + wave * kWatchList;
        WatchEnd end = kDone;
        int narrow = 0;
        for (;; ++steps) {
            const uint32_t before = t.visited;
            const bool any = watch(mine, wave, waves, null);
            // flags rotate over three words, as the forest's; bit 1: many finds
            int* flag = cnt + steps % 3;
            if (any) {
                int bits_found = 1;
                if (kCounted && popc(ballot(t.visited != before)) > kNarrowLanes) bits_found = 3;
                if (lane_id() == 0) atomicOr(flag, bits_found);
            }
            sync_lds();
            const int more = __hip_atomic_load(flag, __ATOMIC_RELAXED, kWatchWG);
            if (rank() == 0) cnt[(steps + 2) % 3] = 0;
            if (!more) break;   // the same in every lane of the group
            if (steps + jumps >= budget) {
                end = kStalled;
                break;
            }
            narrow += more == 1;
            if (kCounted && __builtin_expect(narrow > narrow_limit, 0)) {
                end = kNarrow;
                ++steps;
                break;
            }
        }
        if (rank() == 0) bits[null >> 5] |= 1u << (null & 31);
        sync();
        return end;
    }

    // Every vertex left joins the list of its support (a plain exchange: nothing
    // is closed meanwhile); those whose support is removed resume their scans in
    // the first phase.  The positions may lie in m.l0, supports that are not in
    // LDS in m.l1; l.st is LDS that nothing uses by then (the supports' own place,
    // if they are there).
    __device__ __forceinline__ void to_lists(GroupLists<View, kWaveGroup>& l) {
        constexpr int U = 4;
        const ListArrays& m = l.m;
        const int rounds = (n + size() - 1) / size();
        uint32_t* lost = reinterpret_cast<uint32_t*>(list);   // a bitmap, as in the sweep
        for (int i = 0; i < rounds; ++i) {
            const int v = i * size() + rank();
            if (v >= n) break;
            const int h = wt_bit(bits, v) ? kDead : kEmpty;
            reinterpret_cast<int2*>(m.head)[v] = make_int2(h, h);
        }
        sync();
        for (int i = 0; i < rounds; i += U) {
            int v[U], s[U], p[U], e[U], old[U];
            bool live[U], gone[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                v[k] = (i + k) * size() + rank();
                const int x = min(v[k], n - 1);
                live[k] = v[k] < n && !wt_bit(bits, x);
                s[k] = wt_get(sup, x);
                p[k] = wt_get(cur, x);
                e[k] = g.end(x);
            }
#pragma unroll
            for (int k = 0; k < U; ++k) {
                gone[k] = live[k] && wt_bit(bits, s[k]);
                old[k] = kEmpty;
                if (live[k] && !gone[k])
                    old[k] = xchg_s<kWG>(m.head + 2 * s[k] + (p[k] + 1 == e[k]), v[k]);
            }
#pragma unroll
            for (int k = 0; k < U; ++k) {
                if (live[k]) st_s<kWG>(m.rec + v[k], pack_rec(old[k], p[k]));
                const uint64_t b = ballot(gone[k]);
                if (lane_id() == 0 && v[k] < n) {
                    lost[v[k] >> 5] = (uint32_t)b;
                    lost[(v[k] >> 5) + 1] = (uint32_t)(b >> 32);
                }
            }
        }
        sync();   // supports and positions are not read any more
        l.begin();
        sync();
        for (int i = 0; i < rounds; ++i) {
            const int v = i * size() + rank();
            const bool back = v < n && wt_bit(lost, v);
            t.visited += back;
            l.emit(back ? make_item(kOwnRescan, v) : kNone);
        }
        l.flush();
        sync();
    }
};

}  // namespace

}  // namespace trim
