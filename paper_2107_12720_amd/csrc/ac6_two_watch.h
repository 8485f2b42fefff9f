// ac6_two_watch.h -- two-sided AC-6 trimming by watching supports (Section 4.1
// and 6.2; included by ac6_two.hip).
//
// As one-sided (ac6_watch.h): a vertex keeps its two supports in arrays, and a
// round over the vertices hands back those whose support on either side was
// removed, instead of both sides' lists joined in the first sweep by device-wide
// exchanges and walked afterwards.  If the rounds don't reach the fixed point,
// the vertices left join their lists and ac6t_propagate finishes.
//
// What bounds it: the sweep by its gathers on both sides, a round by reading both
// support arrays and four dependent loads.  R-MAT of edge factor 16 and 2^22
// vertices 518 -> 225 us a call (exchanges for 380 in the sweep), with a chain of
// 83,000 809 -> 303; core+tail of 32,768 vertices 418 -> 182, of 2^20 742 -> 350.
#pragma once
#include "trim_device.h"
#include "block_append.h"
#include "grid_barrier.h"
#include "ac6_support.h"
#include "forest_jump.h"
#include "watch_rounds.h"

namespace trim {

namespace {

// Both sides as one-sided states: `o` over G, `i` over G^T; the statuses, the
// filters and the counters are shared, o.sup[v] < 0 marks v removed.
struct TwoWatch {
    WatchState o, i;
};

__global__ void two_watch_init(TwoWatch t, const uint32_t* preset, uint32_t* y1,
                               trim_stats_t* stats) {
    const WatchState& a = t.o;
    const int tid = blockIdx.x * blockDim.x + threadIdx.x;
    const int stride = gridDim.x * blockDim.x, n = a.n;
    if (tid < kCtrInts) a.ctr[tid] = 0;
    for (int p = tid; p < a.P; p += stride) a.worker_edges[p] = 0;
    if (stats && tid < (int)(sizeof(trim_stats_t) / 8)) ((uint64_t*)stats)[tid] = 0;
    for (int i = tid; i < 3 * a.flt.words(); i += stride) a.flt.f[i] = 0;
    const int nwords = (n + 31) >> 5;
    for (int base = tid / kWave * kWave; base < n; base += stride) {
        const int v = base + lane_id(), x = min(v, n - 1);
        const bool d = t.o.row_off[x + 1] == t.o.row_off[x] ||
                       t.i.row_off[x + 1] == t.i.row_off[x] || (preset && status_bit(preset, x));
        const uint64_t m = ballot(v < n && d);
        const int w = (base >> 5) + lane_id();
        if (lane_id() < 2 && w < nwords) {
            const uint32_t word = (uint32_t)(m >> (32 * lane_id()));
            y1[w] = word;
            a.dead[w] = word;
        }
    }
}

// The first sweep: v's out-support and, only if there is one, its in-support;
// jp and jlist as in ac6t_sweep.  Without kForest the vertices without one of
// them are removed here (round 0).
template <bool kForest>
__global__ __launch_bounds__(1024) void two_watch_sweep(TwoWatch t, long long m,
                                                        const uint32_t* y1, int* jp,
                                                        uint32_t* jlist, uint64_t* part) {
    constexpr int U = 4;   // vertices per lane in flight
    __shared__ int s_wave[1024 / kWave], s_base;
    __shared__ uint64_t red[16];
    uint64_t edges = 0, removed = 0;
    const int n = t.o.n, per = U * blockDim.x;
    const int steps = (n + per - 1) / per;
    for (int b0 = blockIdx.x; b0 < steps; b0 += gridDim.x) {
        const int st = step_of(b0, steps);
        const int base = ((t.o.sched & TRIM_SCHED_REVERSE) ? steps - 1 - st : st) * per;
        int b[2][U], e[2][U], p[2][U], w[2][U];
        bool live[U], ok[2][U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int v = base + k * blockDim.x + threadIdx.x, x = min(v, n - 1);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int* off = s ? t.i.row_off : t.o.row_off;
                b[s][k] = __builtin_nontemporal_load(off + x);
                e[s][k] = __builtin_nontemporal_load(off + x + 1);
            }
            live[k] = v < n && !status_bit(y1, x);
        }
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                p[s][k] = b[s][k];
                w[s][k] = 0;
                const int* adj = s ? t.i.col : t.o.col;
                if (live[k]) w[s][k] = __builtin_nontemporal_load(adj + b[s][k]);
            }
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int s = 0; s < 2; ++s) ok[s][k] = live[k] && !status_bit(y1, w[s][k]);
        uint32_t put = 0, root = 0;
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int v = base + k * blockDim.x + threadIdx.x;
            // the rare scans past removed vertices, the in-side's only for a
            // vertex with an out-support
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                if (!live[k] || (s && !ok[0][k])) continue;
                if (!ok[s][k]) {
                    for (++p[s][k]; p[s][k] < e[s][k]; ++p[s][k]) {
                        w[s][k] = __builtin_nontemporal_load((s ? t.i.col : t.o.col) + p[s][k]);
                        if (!status_bit(y1, w[s][k])) break;
                    }
                    ok[s][k] = p[s][k] < e[s][k];
                }
                edges += (uint64_t)((ok[s][k] ? p[s][k] + 1 : e[s][k]) - b[s][k]);
                if (ok[s][k] && p[s][k] != b[s][k])
                    *rec_pos(s ? t.i.rec : t.o.rec, v) = p[s][k];
            }
            const bool keep = live[k] && ok[0][k] && ok[1][k], lost = live[k] && !keep;
            const bool member = keep && p[0][k] + 1 == e[0][k];
            if (v < n) {
                t.o.sup[v] = keep ? w[0][k] | (p[0][k] == b[0][k] ? kSupFirst : 0) : -1;
                if (keep) t.i.sup[v] = w[1][k] | (p[1][k] == b[1][k] ? kSupFirst : 0);
                if (kForest && live[k]) jp[v] = lost ? ~v : member ? w[0][k] : v;
            }
            put |= (uint32_t)(lost || member) << k;
            root |= (uint32_t)lost << k;
            if (!kForest && lost) {
                atomicOr(t.o.dead + (v >> 5), 1u << (v & 31));
                removed += 1;
            }
        }
        if constexpr (kForest) {
            int slot = block_append_base(__popc(put), t.o.ctr + kJCnt0, nullptr, s_wave, &s_base);
#pragma unroll
            for (int k = 0; k < U; ++k)
                if ((put >> k) & 1u)
                    jlist[slot++] = (uint32_t)(base + k * (int)blockDim.x + (int)threadIdx.x) |
                                    ((root >> k) & 1u ? kRootBit : 0u);
        }
    }
    edges = block_sum(edges, red);
    if (!kForest) removed = block_sum(removed, red);
    if (threadIdx.x == 0) {
        if (edges) add_dev(t.o.worker_edges + (blockIdx.x % t.o.P), edges);
        part[kPartSweep * kPartStride + blockIdx.x] = edges;
        part[kPartDeg * kPartStride + blockIdx.x] = blockIdx.x == 0 ? (uint64_t)m : 0;
        if (!kForest && removed) {
            add_dev(t.o.ctr + kHyDead0, (int)removed);
            add_dev(reinterpret_cast<uint64_t*>(t.o.ctr + kWatchCloses), removed);
        }
    }
}

// The forest collapse's removal of v.  No list is handed back.
struct TwoWatchKill {
    static constexpr bool kItems = false;
    static constexpr int kThreads = kRoundThreads, kUnroll = 1;
    int* sup;
    uint32_t* dead;
    __device__ __forceinline__ void operator()(int v) const {
        sup[v] = -1;
        atomicOr(dead + (v >> 5), 1u << (v & 31));
    }
};

constexpr int kTwoFlight = 4;   // vertices per lane in flight in a round

// Round r over the thread's vertices; returns the removals.  The hand-backs of a
// wavefront are gathered in `found` as in watch_found, with a bit per side.
template <bool kFresh>
__device__ __forceinline__ uint32_t two_watch_vertices(const TwoWatch& t, int r,
                                                       const uint32_t* sflt, uint32_t* found,
                                                       WatchSums& sum) {
    constexpr int U = kTwoFlight;
    found += threadIdx.x / kWave * (U * kWave);
    uint32_t removed = 0;
    const uint32_t* dead = t.o.dead;
    const int n = t.o.n, stride = gridDim.x * blockDim.x;
    for (int base = blockIdx.x * blockDim.x + threadIdx.x; base < n; base += U * stride) {
        int s[2][U];
        bool back[2][U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int v = base + k * stride, x = min(v, n - 1);
            s[0][k] = t.o.sup[x];
            s[1][k] = t.i.sup[x];
            back[0][k] = back[1][k] = v < n && s[0][k] >= 0;
        }
        if (sflt) {
#pragma unroll
            for (int k = 0; k < U; ++k)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const uint32_t h = t.o.flt.hash(s[j][k] & kSupMask);
                    back[j][k] = back[j][k] && ((sflt[h >> 5] >> (h & 31)) & 1u);
                }
        }
        uint32_t x[2][U];
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int w = s[j][k] & kSupMask;
                x[j][k] = 0;
                if (back[j][k]) x[j][k] = kFresh ? ld_dev(dead + (w >> 5)) : dead[w >> 5];
            }
        int cnt = 0;
#pragma unroll
        for (int k = 0; k < U; ++k) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
                back[j][k] = back[j][k] && ((x[j][k] >> (s[j][k] & 31)) & 1u);
            const bool any = back[0][k] || back[1][k];
            const uint64_t mask = ballot(any);
            if (any)
                found[cnt + popc(mask & lanes_below())] =
                    (uint32_t)(base + k * stride) | (uint32_t)back[0][k] << 30 |
                    (uint32_t)back[1][k] << 31;
            cnt += popc(mask);
        }
        __builtin_amdgcn_wave_barrier();
        for (int i = lane_id(); i < cnt; i += kWave) {
            const uint32_t f = found[i];
            const int v = (int)(f & kSupMask);
            bool keep = true;
            for (int j = 0; j < 2 && keep; ++j) {
                if (!((f >> (30 + j)) & 1u)) continue;
                const WatchState& a = j ? t.i : t.o;
                int pos, to;
                sum.visited += 1;
                keep = watch_scan<kFresh>(a, v, a.sup[v], pos, to, sum.edges);
                if (keep) {
                    a.sup[v] = to;
                    *rec_pos(a.rec, v) = pos;
                    sum.joins += 1;
                }
            }
            if (!keep) {
                t.o.sup[v] = -1;
                atomicOr(t.o.dead + (v >> 5), 1u << (v & 31));
                t.o.flt.add(r, v);
                sum.closes += 1;
                removed += 1;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    return removed;
}

template <bool kFilter>
__global__ __launch_bounds__(kRoundThreads) void two_watch_round(TwoWatch t, int r) {
    __shared__ __align__(8) uint32_t sflt[kFilter ? WatchFilter::kMaxWords : 2];
    __shared__ uint32_t found[kRoundThreads * kTwoFlight];
    __shared__ uint64_t red[16];
    const WatchState& a = t.o;
    if (ld_dev(a.ctr + kHyStop)) return;
    const int before = removed_before(a, r);
    if (before == 0) {   // the fixed point; workgroup 0 tells the later launches
        if (blockIdx.x == 0 && threadIdx.x == 0) st_dev(a.ctr + kHyStop, 1);
        return;
    }
    WatchSums sum;
    const uint32_t removed = two_watch_vertices<false>(
        t, r, kFilter ? watch_stage<kRoundThreads, false>(a, r, before, sflt) : nullptr, found,
        sum);
    watch_round_end(a, r, removed, red);
    watch_sums(a, sum, red);
}

// As watch_tail: rounds r0 .. last in one launch, then the heads of both sides.
__global__ __launch_bounds__(kRoundThreads) void two_watch_tail(TwoWatch t, int r0, int last,
                                                                int* hout, int* ext, int* hin,
                                                                int budget) {
    __shared__ __align__(8) uint32_t sflt[WatchFilter::kMaxWords];
    __shared__ uint32_t found[kRoundThreads * kTwoFlight];
    __shared__ uint64_t red[16];
    const WatchState& a = t.o;
    if (ld_dev(a.ctr + kHyStop)) return;
    WatchSums sum;
    for (int r = r0;; ++r) {
        const int before = removed_before(a, r);
        if (before == 0) {
            if (blockIdx.x == 0 && threadIdx.x == 0) st_dev(a.ctr + kHyStop, 1);
            break;
        }
        if (r > last) {
            for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < a.n;
                 v += gridDim.x * blockDim.x) {
                const int h = (ld_dev(a.dead + (v >> 5)) >> (v & 31)) & 1u ? kDead : kEmpty;
                reinterpret_cast<int2*>(hout)[v] = make_int2(h, h);
                reinterpret_cast<int2*>(hin)[v] = make_int2(h, h);
                if (ext)
                    for (int j = 0; j < kMoreLists - 1; ++j)
                        ext[(kMoreLists - 1) * (long long)v + j] = h;
            }
            break;
        }
        // (the removals before the first round are in no filter)
        const uint32_t* f =
            r == a.r1 ? nullptr : watch_stage<kRoundThreads, true>(a, r, before, sflt);
        const uint32_t removed = two_watch_vertices<true>(t, r, f, found, sum);
        watch_round_end(a, r, removed, red);
        if (!grid_barrier(a.ctr + kBarCount, a.ctr + kBarGen, a.ctr + kStall, budget)) break;
    }
    watch_sums(a, sum, red);
}

// Every vertex left joins the lists of its supports; those whose support the last
// round removed that of the next live neighbour, or become close items.  Nothing
// is closed while this runs, so joining is a plain exchange.
__global__ __launch_bounds__(256) void two_watch_register(TwoWatch t, int* hout, int* ext,
                                                          int* hin, uint32_t* q) {
    __shared__ int s_wave[256 / kWave], s_base;
    __shared__ uint64_t red[16];
    const WatchState& a = t.o;
    // (after a stall the heads may not be there)
    if (ld_dev(a.ctr + kHyStop) || ld_dev(a.ctr + kStall)) return;
    WatchSums sum;
    for (int base = blockIdx.x * blockDim.x; base < a.n; base += gridDim.x * blockDim.x) {
        const int v = base + threadIdx.x;
        int s[2] = {-1, -1}, p[2] = {0, 0}, w[2] = {0, 0};
        bool keep = false;
        if (v < a.n && (s[0] = t.o.sup[v]) >= 0) {
            s[1] = t.i.sup[v];
            keep = true;
            for (int j = 0; j < 2 && keep; ++j) {
                const WatchState& c = j ? t.i : t.o;
                w[j] = s[j] & kSupMask;
                p[j] = (s[j] & kSupFirst) ? c.row_off[v] : *rec_pos(c.rec, v);
                if (status_bit(a.dead, w[j])) {
                    sum.visited += 1;
                    keep = watch_scan<false>(c, v, s[j], p[j], w[j], sum.edges);
                    sum.joins += keep;
                }
            }
        }
        if (keep) {
            const bool lasto = p[0] + 1 == t.o.row_off[v + 1];
            const bool lasti = p[1] + 1 == t.i.row_off[v + 1];
            const int oldo = xchg_dev(join_slot(hout, ext, w[0], lasto, v), v);
            const int oldi = xchg_dev(hin + 2 * w[1] + lasti, v);
            t.o.rec[v] = pack_rec(oldo, p[0]);
            t.i.rec[v] = pack_rec(oldi, p[1]);
        }
        const bool lost = s[0] >= 0 && !keep;
        const int slot = block_append_base(lost, a.ctr + kQTail, a.ctr + kPending, s_wave, &s_base);
        if (lost) q[slot] = make_item(0, v);
    }
    watch_sums(a, sum, red);
}

// Live bitmap and the live vertices' checks after the rounds (see ac6t_pack).
__device__ __forceinline__ void two_watch_pack(const TwoWatch& t, uint32_t* bitmap,
                                               uint64_t& live_cnt, uint64_t& live_edges) {
    const int n = t.o.n, nwords = (n + 31) >> 5;
    const int waves = (gridDim.x * blockDim.x) / kWave;
    const int wid = (blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    for (int base = wid * kWave; base < n; base += waves * kWave) {
        const int v = base + lane_id();
        const int s = v < n ? t.o.sup[v] : -1;
        if (s >= 0) {
            live_edges += 2;
            if (!(s & kSupFirst)) live_edges += *rec_pos(t.o.rec, v) - t.o.row_off[v];
            if (!(t.i.sup[v] & kSupFirst)) live_edges += *rec_pos(t.i.rec, v) - t.i.row_off[v];
        }
        const uint64_t b = ballot(s >= 0);
        if (lane_id() == 0) {
            const int w = base >> 5;
            bitmap[w] = (uint32_t)b;
            if (w + 1 < nwords) bitmap[w + 1] = (uint32_t)(b >> 32);
            live_cnt += (uint64_t)popc(b);
        }
    }
}

}  // namespace

}  // namespace trim
