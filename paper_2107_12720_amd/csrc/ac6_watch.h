// ac6_watch.h -- AC-6 of a large explicit graph by watching supports
// (Section 6.2; included by ac6.hip; the parts shared with the two-sided form
// in watch_rounds.h).
//
// As in watch.h, a vertex is handed back when a pass over the vertices finds
// its support removed, not by a walk over the support's list; the support
// searches and their counts are the same.  Joining a list costs a device-wide
// exchange at a random place for every vertex that keeps a successor: on
// R-MAT 22, 1.6 of 2.0 * 10^6 of them in a sweep of 0.2 ms, to hand back 53
// vertices; a round over all supports reads them in order and probes a bitmap
// that the L2s hold.
//
//   watch_init    statuses (two bitmaps: the sweep reads y1, everything later
//                 reads and sets `dead`), counters, filters;
//   watch_sweep   DoPost of every vertex; supports in sup[], positions in the
//                 high halves of rec[] where they are not the first, links and
//                 members for the forest collapse;
//   watch_counted, watch_collect
//                 (late registration, opts.rounds >= 2) the counted rounds, then
//                 the forest's links and members from the supports left;
//   ac6_jump      the forest collapse (forest_jump.h), setting statuses;
//   watch_round   one round: vertices whose support was removed resume their
//                 scans.  round_launches(n) launches; a round that removes
//                 nothing is the last, and what follows returns at once;
//   watch_tail    further rounds in one launch with grid barriers, up to
//                 watch_rounds(n) rounds in all or kNarrowRounds narrow ones;
//                 then the list heads;
//   watch_register
//                 if that did not end it (a deep, narrow remainder): every
//                 vertex left joins its support's list, and the propagation
//                 over lists finishes.
//
// What bounds it: the sweep by its gathers of row_off, col and statuses (50 us
// for R-MAT 22, edge factor 16; 200 with the exchanges), a round of all vertices
// by reading sup (12 us at 2^22) and by the latency of four dependent loads,
// about 5 us, plus 2 for the barrier in the tail.  R-MAT 22 with a chain of
// 2*10^5: 494 -> 210 us in all; core+tail of 10^5 vertices 402 -> 252, of 2^20
// 564 -> 381.  Late registration, R-MAT 26 with four counted rounds: 0.90 -> 0.78
// ms if three reach the fixed point, 3.80 -> 0.83 if not (5 * 10^7 list exchanges
// took 2.65).
#pragma once
#include "trim_device.h"
#include "block_append.h"
#include "grid_barrier.h"
#include "ac6_support.h"
#include "forest_jump.h"
#include "watch_rounds.h"

namespace trim {

namespace {

// How the first sweep records a vertex without a live successor: it is removed
// by the propagation (round 0), by the forest collapse, or by the first of the
// counted rounds of late registration.
enum WatchMode { kWatchStep, kWatchForest, kWatchCounted };

// A lane takes four vertices from one 16-byte load of the offsets when they
// are aligned (`wide`), a wavefront 256, whose eight words it assembles.
__global__ void watch_init(const int* row_off, int n, bool wide, const uint32_t* preset,
                           uint32_t* y1, uint32_t* dead, WatchFilter flt, int* ctr,
                           uint64_t* worker_edges, int P, trim_stats_t* stats, bool counted) {
    const int tid = blockIdx.x * blockDim.x + threadIdx.x;
    const int stride = gridDim.x * blockDim.x;
    if (tid < kCtrInts) ctr[tid] = counted && tid == kHyRounds ? 1 : 0;
    for (int p = tid; p < P; p += stride) worker_edges[p] = 0;
    if (stats && tid < (int)(sizeof(trim_stats_t) / 8)) ((uint64_t*)stats)[tid] = 0;
    for (int i = tid; i < 3 * flt.words(); i += stride) flt.f[i] = 0;
    const int ngroups = (n + 3) >> 2, nwords = (n + 31) >> 5;
    const int lane = lane_id(), waves = stride / kWave;
    for (int g0 = (tid / kWave) * kWave; g0 < ngroups; g0 += waves * kWave) {
        const int gi = g0 + lane, v = gi << 2;
        uint32_t nib = 0;
        if (wide && v + 4 <= n) {
            typedef int v4i __attribute__((ext_vector_type(4)));
            const v4i a = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(row_off) + gi);
            const int e4 = __builtin_nontemporal_load(row_off + v + 4);
            nib = (uint32_t)(a.x == a.y) | ((uint32_t)(a.y == a.z) << 1) |
                  ((uint32_t)(a.z == a.w) << 2) | ((uint32_t)(a.w == e4) << 3);
        } else {
            for (int j = 0; j < 4 && v + j < n; ++j)
                nib |= (uint32_t)(row_off[v + j] == row_off[v + j + 1]) << j;
        }
        uint32_t word = nib << (4 * (lane & 7));
        word |= __shfl_xor(word, 1);
        word |= __shfl_xor(word, 2);
        word |= __shfl_xor(word, 4);
        const int wi = (g0 >> 3) + (lane >> 3);
        if ((lane & 7) == 0 && wi < nwords) {
            if (preset) word |= preset[wi];
            y1[wi] = word;
            dead[wi] = word;
        }
    }
}

// kWatchForest: jp and jlist as in ac6_sweep.  Otherwise the vertices without a
// live successor are removed here.
template <WatchMode kMode>
__global__ __launch_bounds__(1024) void watch_sweep(WatchState a, long long m, const uint32_t* y1,
                                                    bool preset, int* jp, uint32_t* jlist,
                                                    uint64_t* part) {
    constexpr int U = kSweepFlight;
    constexpr bool kForest = kMode == kWatchForest;
    __shared__ int s_wave[1024 / kWave], s_base;
    __shared__ uint64_t red[16];
    uint64_t edges = 0, removed = 0;
    const int n = a.n, per = U * blockDim.x;
    const int steps = (n + per - 1) / per;
    for (int b0 = blockIdx.x; b0 < steps; b0 += gridDim.x) {
        const int st = step_of(b0, steps);
        const int base = ((a.sched & TRIM_SCHED_REVERSE) ? steps - 1 - st : st) * per;
        int b[U], e[U], p[U], w[U];
        bool ok[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int v = base + k * blockDim.x + threadIdx.x, x = min(v, n - 1);
            b[k] = __builtin_nontemporal_load(a.row_off + x);
            e[k] = __builtin_nontemporal_load(a.row_off + x + 1);
            ok[k] = v < n;
        }
        if (preset) {
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int v = base + k * blockDim.x + threadIdx.x;
                ok[k] = ok[k] && !status_bit(y1, min(v, n - 1));
            }
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            p[k] = b[k];
            w[k] = b[k] < e[k] ? __builtin_nontemporal_load(a.col + b[k]) : 0;
            if (!ok[k]) e[k] = b[k];   // removed already, or past the end
        }
#pragma unroll
        for (int k = 0; k < U; ++k) ok[k] = !status_bit(y1, w[k]) && b[k] < e[k];
        int c = 0;
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int v = base + k * blockDim.x + threadIdx.x;
            if (b[k] < e[k] && !ok[k]) {   // the rare scan past removed vertices
                for (++p[k]; p[k] < e[k]; ++p[k]) {
                    w[k] = __builtin_nontemporal_load(a.col + p[k]);
                    if (!status_bit(y1, w[k])) break;
                }
                ok[k] = p[k] < e[k];
            }
            if (ok[k]) {
                edges += (uint64_t)(p[k] - b[k] + 1);
                if (p[k] != b[k]) *rec_pos(a.rec, v) = p[k];
            } else {
                edges += (uint64_t)(e[k] - b[k]);
            }
            if (v < n) {
                a.sup[v] = ok[k] ? (w[k] | (p[k] == b[k] ? kSupFirst : 0)) : -1;
                if (kForest && b[k] < e[k])
                    jp[v] = !ok[k] ? ~v : p[k] + 1 == e[k] ? w[k] : v;
            }
            if (kForest) {
                c += b[k] < e[k] && (!ok[k] || p[k] + 1 == e[k]);
            } else if (b[k] < e[k] && !ok[k]) {
                atomicOr(a.dead + (v >> 5), 1u << (v & 31));
                if (kMode == kWatchCounted) a.flt.add(1, v);
                removed += 1;
            }
        }
        if constexpr (kForest) {
            int slot = block_append_base(c, a.ctr + kJCnt0, nullptr, s_wave, &s_base);
#pragma unroll
            for (int k = 0; k < U; ++k)
                if (b[k] < e[k] && (!ok[k] || p[k] + 1 == e[k]))
                    jlist[slot++] = (uint32_t)(base + k * (int)blockDim.x + (int)threadIdx.x) |
                                    (ok[k] ? 0u : kRootBit);
        }
    }
    edges = block_sum(edges, red);
    if (!kForest) removed = block_sum(removed, red);
    if (threadIdx.x == 0) {
        if (edges) add_dev(a.worker_edges + (blockIdx.x % a.P), edges);
        part[kPartSweep * kPartStride + blockIdx.x] = edges;
        part[kPartDeg * kPartStride + blockIdx.x] = blockIdx.x == 0 ? (uint64_t)m : 0;
        if (!kForest && removed) {
            add_dev(a.ctr + kHyDead0 + (kMode == kWatchCounted), (int)removed);
            if (kMode == kWatchStep)
                add_dev(reinterpret_cast<uint64_t*>(a.ctr + kWatchCloses), removed);
        }
    }
}

// The forest collapse's removal of v (round 0).  No list is handed back.
struct WatchKill {
    static constexpr bool kItems = false;
    static constexpr int kThreads = kRoundThreads, kUnroll = 1;
    int* sup;
    uint32_t* dead;
    __device__ __forceinline__ void operator()(int v) const {
        sup[v] = -1;
        atomicOr(dead + (v >> 5), 1u << (v & 31));
    }
};

// Round r over the thread's vertices; returns the removals.  sflt: the filter of
// round r - 1 in LDS, or NULL.
template <bool kFresh>
__device__ __forceinline__ uint32_t watch_vertices(const WatchState& a, int r,
                                                   const uint32_t* sflt, int* found,
                                                   WatchSums& t) {
    constexpr int U = kRoundFlight;
    found += threadIdx.x / kWave * (U * kWave);
    uint32_t removed = 0;
    const int n = a.n, runs = (n + 3) >> 2;
    const int blocks = (runs + (int)blockDim.x - 1) / (int)blockDim.x;
    for (int b0 = blockIdx.x; b0 < blocks; b0 += U / 4 * gridDim.x) {
        int s[U], q[U / 4];
        bool back[U];
#pragma unroll
        for (int g = 0; g < U / 4; ++g) {
            const int b = b0 + g * (int)gridDim.x;
            q[g] = b < blocks ? step_of(b, blocks) * (int)blockDim.x + (int)threadIdx.x : runs;
            const int4 y = reinterpret_cast<const int4*>(a.sup)[min(q[g], runs - 1)];
            s[4 * g] = y.x, s[4 * g + 1] = y.y, s[4 * g + 2] = y.z, s[4 * g + 3] = y.w;
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            back[k] = 4 * q[k >> 2] + (k & 3) < n && s[k] >= 0;
        }
        if (sflt) {
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const uint32_t h = a.flt.hash(s[k] & kSupMask);
                back[k] = back[k] && ((sflt[h >> 5] >> (h & 31)) & 1u);
            }
        }
        uint32_t x[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int w = s[k] & kSupMask;
            x[k] = 0;
            if (back[k]) x[k] = kFresh ? ld_dev(a.dead + (w >> 5)) : a.dead[w >> 5];
        }
#pragma unroll
        for (int k = 0; k < U; ++k) back[k] = back[k] && ((x[k] >> (s[k] & 31)) & 1u);
        const int cnt = watch_found(back, q, found);
        for (int i = lane_id(); i < cnt; i += kWave) {
            const int v = found[i];
            int pos, to;
            t.visited += 1;
            if (watch_scan<kFresh>(a, v, a.sup[v], pos, to, t.edges)) {
                a.sup[v] = to;
                *rec_pos(a.rec, v) = pos;
                t.joins += 1;
            } else {
                a.sup[v] = -1;
                atomicOr(a.dead + (v >> 5), 1u << (v & 31));
                a.flt.add(r, v);
                t.closes += 1;
                removed += 1;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    return removed;
}

// Late registration (opts.rounds = R): counted rounds 2 .. R, a vertex's support
// checked again in each.  Round r reads ycur, which holds the removals before
// it, and builds ynext from the bitmap of the round before last: the words of
// ycur and its own removals.  (The rounds and their counts are the sequential
// ones whatever the order of the lanes.)  True if round r need not run: a round
// before it removed nothing.
__device__ __forceinline__ bool counted_done(int* ctr, int r) {
    if (ld_dev(ctr + kHyStop)) return true;
    if (ld_dev(ctr + kHyDead0 + (r - 1) % 3) == 0) {
        if (blockIdx.x == 0 && threadIdx.x == 0) st_dev(ctr + kHyStop, 1);
        return true;
    }
    return false;
}

__global__ __launch_bounds__(kRoundThreads) void watch_counted(WatchState a, int r,
                                                               const uint32_t* ycur,
                                                               uint32_t* ynext) {
    constexpr int U = kRoundFlight;
    __shared__ __align__(8) uint32_t s_flt[WatchFilter::kMaxWords];
    __shared__ int s_found[kRoundThreads * U];
    __shared__ uint64_t red[16];
    if (counted_done(a.ctr, r)) return;
    const int before = ld_dev(a.ctr + kHyDead0 + (r - 1) % 3);
    const uint32_t* sflt = watch_stage<kRoundThreads, false>(a, r, before, s_flt);
    const int n = a.n, stride = gridDim.x * blockDim.x, runs = (n + 3) >> 2;
    const int blocks = (runs + (int)blockDim.x - 1) / (int)blockDim.x;
    const int tid = blockIdx.x * blockDim.x + threadIdx.x;
    int* found = s_found + threadIdx.x / kWave * (U * kWave);
    for (int i = tid; i < (n + 31) >> 5; i += stride) {
        const uint32_t b = ycur[i];
        if (b & ~ynext[i]) atomicOr(ynext + i, b);
    }
    WatchState now = a;
    now.dead = const_cast<uint32_t*>(ycur);
    uint64_t edges = 0;
    uint32_t removed = 0, entries = 0;
    for (int b0 = blockIdx.x; b0 < blocks; b0 += U / 4 * gridDim.x) {
        uint32_t x[U];
        int s[U], q[U / 4];
        bool back[U];
#pragma unroll
        for (int g = 0; g < U / 4; ++g) {
            const int b = b0 + g * (int)gridDim.x;
            q[g] = b < blocks ? step_of(b, blocks) * (int)blockDim.x + (int)threadIdx.x : runs;
            const int4 y = reinterpret_cast<const int4*>(a.sup)[min(q[g], runs - 1)];
            s[4 * g] = y.x, s[4 * g + 1] = y.y, s[4 * g + 2] = y.z, s[4 * g + 3] = y.w;
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            back[k] = 4 * q[k >> 2] + (k & 3) < n && s[k] >= 0;
            entries += back[k];
        }
        if (sflt) {
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const uint32_t h = a.flt.hash(s[k] & kSupMask);
                back[k] = back[k] && ((sflt[h >> 5] >> (h & 31)) & 1u);
            }
        }
#pragma unroll
        for (int k = 0; k < U; ++k) x[k] = back[k] ? ycur[(s[k] & kSupMask) >> 5] : 0;
#pragma unroll
        for (int k = 0; k < U; ++k) back[k] = back[k] && ((x[k] >> (s[k] & 31)) & 1u);
        const int cnt = watch_found(back, q, found);
        for (int i = lane_id(); i < cnt; i += kWave) {
            const int v = found[i];
            int pos, to;
            if (watch_scan<false>(now, v, a.sup[v], pos, to, edges)) {
                a.sup[v] = to;
                *rec_pos(a.rec, v) = pos;
            } else {
                a.sup[v] = -1;
                atomicOr(ynext + (v >> 5), 1u << (v & 31));
                a.flt.add(r, v);
                removed += 1;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    uint32_t* f = a.flt.slot(r + 1);
    for (int i = tid; i < a.flt.words(); i += stride) f[i] = 0;
    if (tid == 0) {
        st_dev(a.ctr + kHyDead0 + (r + 1) % 3, 0);
        st_dev(a.ctr + kHyRounds, r);
    }
    const uint64_t rem = block_sum(removed, red), ent = block_sum(entries, red);
    edges = block_sum(edges, red);
    if (threadIdx.x == 0) {
        add_dev(a.worker_edges + (blockIdx.x % a.P), edges + ent);
        if (ent) add_dev(reinterpret_cast<uint64_t*>(a.ctr + kHyWork), ent);
        if (rem) add_dev(a.ctr + kHyDead0 + r % 3, (int)rem);
    }
}

// After counted round R, which removed something: what watch_sweep leaves for the
// forest collapse, from the supports as they are now; vertices whose support
// round R removed resume their scans.  It reads a.dead only.
__global__ __launch_bounds__(1024) void watch_collect(WatchState a, int* jp, uint32_t* jlist) {
    constexpr int U = kSweepFlight;
    __shared__ int s_wave[1024 / kWave], s_base;
    __shared__ uint64_t red[16];
    if (counted_done(a.ctr, a.r1)) return;
    WatchSums t;
    const int n = a.n, per = U * blockDim.x, steps = (n + per - 1) / per;
    for (int b0 = blockIdx.x; b0 < steps; b0 += gridDim.x) {
        const int base = step_of(b0, steps) * per;
        int s[U], e[U], p[U];
        uint32_t x[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int v = base + k * blockDim.x + threadIdx.x, c = min(v, n - 1);
            s[k] = v < n ? a.sup[c] : -1;
            p[k] = __builtin_nontemporal_load(a.row_off + c);
            e[k] = __builtin_nontemporal_load(a.row_off + c + 1);
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int v = base + k * blockDim.x + threadIdx.x;
            x[k] = a.dead[(s[k] & kSupMask) >> 5 & (s[k] < 0 ? 0 : -1)];
            if (s[k] >= 0 && !(s[k] & kSupFirst)) p[k] = *rec_pos(a.rec, v);
        }
        int c = 0;
        uint32_t put = 0, root = 0;
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if (s[k] < 0) continue;
            const int v = base + k * blockDim.x + threadIdx.x;
            int w = s[k] & kSupMask;
            bool lost = false;
            if ((x[k] >> (w & 31)) & 1u) {
                t.visited += 1;
                lost = !watch_scan<false>(a, v, s[k], p[k], w, t.edges);
                if (!lost) {
                    *rec_pos(a.rec, v) = p[k];
                    t.joins += 1;
                }
                a.sup[v] = lost ? -1 : w;
            }
            const bool member = !lost && p[k] + 1 == e[k];
            jp[v] = lost ? ~v : member ? w : v;
            put |= (uint32_t)(lost || member) << k;
            root |= (uint32_t)lost << k;
        }
        c = __popc(put);
        int slot = block_append_base(c, a.ctr + kJCnt0, nullptr, s_wave, &s_base);
#pragma unroll
        for (int k = 0; k < U; ++k)
            if ((put >> k) & 1u)
                jlist[slot++] = (uint32_t)(base + k * (int)blockDim.x + (int)threadIdx.x) |
                                ((root >> k) & 1u ? kRootBit : 0u);
    }
    watch_sums(a, t, red);
}

template <bool kFilter>
__global__ __launch_bounds__(kRoundThreads) void watch_round(WatchState a, int r) {
    __shared__ __align__(8) uint32_t sflt[kFilter ? WatchFilter::kMaxWords : 2];
    __shared__ int found[kRoundThreads * kRoundFlight];
    __shared__ uint64_t red[16];
    if (ld_dev(a.ctr + kHyStop)) return;
    const int before = removed_before(a, r);
    if (before == 0) {   // the fixed point; workgroup 0 tells the later launches
        if (blockIdx.x == 0 && threadIdx.x == 0) st_dev(a.ctr + kHyStop, 1);
        return;
    }
    WatchSums t;
    const uint32_t removed =
        watch_vertices<false>(
        a, r, kFilter ? watch_stage<kRoundThreads, false>(a, r, before, sflt) : nullptr, found, t);
    watch_round_end(a, r, removed, red);
    watch_sums(a, t, red);
}

// Rounds r0 .. watch_rounds(n) in one launch of at most one workgroup per CU, all
// resident at once.  A vertex is the same thread's in every round.
__global__ __launch_bounds__(kRoundThreads) void watch_tail(WatchState a, int r0, int last,
                                                          int* head, int* ext, int budget) {
    __shared__ __align__(8) uint32_t sflt[WatchFilter::kMaxWords];
    __shared__ int found[kRoundThreads * kRoundFlight];
    __shared__ uint64_t red[16];
    if (ld_dev(a.ctr + kHyStop)) return;
    WatchSums t;
    int r = r0, narrow = 0;   // the same in every workgroup
    for (;; ++r) {
        const int before = removed_before(a, r);
        if (before == 0) {
            if (blockIdx.x == 0 && threadIdx.x == 0) st_dev(a.ctr + kHyStop, 1);
            break;
        }
        narrow += before <= narrow_removals(a.n);
        if (r > last || narrow > kNarrowRounds) {
            // the lists' heads; nothing reads the filters there any more
            for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < a.n;
                 v += gridDim.x * blockDim.x) {
                const int h = (ld_dev(a.dead + (v >> 5)) >> (v & 31)) & 1u ? kDead : kEmpty;
                reinterpret_cast<int2*>(head)[v] = make_int2(h, h);
                if (ext)
                    for (int j = 0; j < kMoreLists - 1; ++j)
                        ext[(kMoreLists - 1) * (long long)v + j] = h;
            }
            break;
        }
        // (the removals before the first round are in no filter)
        const uint32_t* f =
            r == a.r1 ? nullptr : watch_stage<kRoundThreads, true>(a, r, before, sflt);
        const uint32_t removed = watch_vertices<true>(a, r, f, found, t);
        watch_round_end(a, r, removed, red);
        if (!grid_barrier(a.ctr + kBarCount, a.ctr + kBarGen, a.ctr + kStall, budget)) break;
    }
    watch_sums(a, t, red);
}

// Every vertex left joins the list of its support, those whose support the last
// round removed that of the next live successor; those without one become close
// items.  Nothing is closed while this runs, so joining is a plain exchange.
__global__ __launch_bounds__(256) void watch_register(WatchState a, int* head, int* ext,
                                                      uint32_t* q) {
    constexpr int U = 4;
    __shared__ int s_wave[256 / kWave], s_base;
    __shared__ uint64_t red[16];
    // (after a stall the heads may not be there)
    if (ld_dev(a.ctr + kHyStop) || ld_dev(a.ctr + kStall)) return;
    WatchSums t;
    const int n = a.n, step = gridDim.x * blockDim.x * U;
    for (int base = blockIdx.x * blockDim.x * U; base < n; base += step) {
        int s[U], p[U], w[U], old[U], c = 0;
        bool lost[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int v = base + k * blockDim.x + threadIdx.x;
            s[k] = v < n ? a.sup[v] : -1;
            lost[k] = false;
            if (s[k] < 0) continue;
            w[k] = s[k] & kSupMask;
            p[k] = (s[k] & kSupFirst) ? a.row_off[v] : *rec_pos(a.rec, v);
            if (status_bit(a.dead, w[k])) {
                t.visited += 1;
                if (watch_scan<false>(a, v, s[k], p[k], w[k], t.edges)) {
                    t.joins += 1;
                } else {
                    lost[k] = true;
                    s[k] = -1;
                    c += 1;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int v = base + k * blockDim.x + threadIdx.x;
            if (s[k] >= 0)
                old[k] = xchg_dev(join_slot(head, ext, w[k], p[k] + 1 == a.row_off[v + 1], v), v);
        }
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (s[k] >= 0) a.rec[base + k * blockDim.x + threadIdx.x] = pack_rec(old[k], p[k]);
        int slot = block_append_base(c, a.ctr + kQTail, a.ctr + kPending, s_wave, &s_base);
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (lost[k]) q[slot++] = make_item(0, base + k * blockDim.x + threadIdx.x);
    }
    watch_sums(a, t, red);
}

}  // namespace

}  // namespace trim
