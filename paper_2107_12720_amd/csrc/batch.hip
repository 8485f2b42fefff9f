// batch.hip -- trim_batch: AC-6 over a batch of independent graphs, each graph
// owned by one workgroup or one wavefront (Section 6.2, Alg. par-ac-6-trim, run
// per graph).
//
// The graphs of a batch share nothing, so a graph needs no device-wide
// coordination at all: whoever claims it trims it start to finish and claims
// the next.  Claims go largest first (graphs ordered by the size class of
// n + m), so the biggest graphs start early and the small ones fill in behind
// them.  Graphs of up to kWatchMaxN vertices are trimmed as watch.h describes,
// their statuses in LDS: by a wavefront when they are small, else by the whole
// workgroup, with the supports in LDS, too, up to 65,536 vertices (somewhat fewer
// with opts.block no power of two).  What bounds
// the batch of 4,096 graphs (5.9 * 10^7 vertices) is the latency of a pass's
// resumed scans in the middling graphs; with supporting sets as lists in
// device memory it was the dependent accesses of every phase.
//
// Larger graphs are trimmed over lists (own_graph; group_lists.h): the first
// successor that is not a sink becomes a vertex's support, joined by an exchange
// of the support's S_more or S_last head, whichever its position selects;
// vertices with none start the phases.  Heads, records and the two phase lists of
// a graph live in device memory at the graph's own vertex range, where the
// workgroup's L2 keeps them for the graph's lifetime; there, too, a smaller graph
// finds its positions, its supports if the LDS does not hold them, and the lists
// of a deep, narrow remainder.
#include <climits>

#include "trim_internal.h"
#include "trim_device.h"
#include "trim_stats.h"
#include "ac6_support.h"
#include "watch.h"

namespace trim {
namespace {

constexpr int kOwnMaxBlock = 1024;
constexpr int kOwnUnroll = 2;     // sweep vertices per lane in flight
// LDS of a workgroup, shared out as the graph at hand needs it; a sixteenth for
// each wavefront with a graph of its own, which holds the statuses, supports
// and list of kOwnWaveN vertices.
constexpr int kOwnLds = 155648;
constexpr int kOwnWaveLds = kOwnLds / 16;
constexpr int kOwnWaveN = 4096;
static_assert(watch_fits(kOwnWaveN, kWave, kOwnWaveN) &&
              kOwnWaveN / 8 + kOwnWaveN * 2 + kWatchList * 2 <= kOwnWaveLds &&
              kWatchList * 2 >= kOwnWaveN / 8, "a wavefront's share");
static_assert(kWatchLdsN / 8 + kWatchLdsN * 2 + 16 * kWatchList * 2 <= kOwnLds,
              "statuses, supports and lists of the largest graph with supports in LDS");
static_assert(kWatchMaxN / 8 + 16 * kWatchList * 4 <= kOwnLds &&
              2 * (kWatchMaxN / 8) + sizeof(ListStage<16>) <= kOwnLds,
              "the same without the supports; a second bitmap and the stage of the lists");
static_assert(sizeof(ListStage<1>) <= kOwnWaveN * 2, "a wavefront's stage in its supports' place");
// A wavefront trims a graph alone up to this n + m (and kOwnWaveN vertices).
constexpr uint32_t kOwnWaveSize = 1u << 16;
constexpr int kKeys = 2 * 33;

// Size class of graph gi: larger graphs get smaller keys, those that a
// wavefront trims alone 33 and more.
__device__ __forceinline__ int size_key(const int64_t* vbase, const int* row_off, int gi) {
    const int64_t v0 = vbase[gi], v1 = vbase[gi + 1];
    const uint32_t size = (uint32_t)(row_off[v1] - row_off[v0]) + (uint32_t)(v1 - v0);
    return __clz(size > 0 ? size : 1u) + (v1 - v0 <= kOwnWaveN && size < kOwnWaveSize ? 33 : 0);
}

// One block: order[] = graph indices by descending size class; zeroes the
// control words and the statistics.
__global__ void batch_order(const int64_t* vbase, const int* row_off, int G, int* order, int* ctr,
                            trim_stats_t* stats) {
    __shared__ int hist[kKeys];
    for (int i = threadIdx.x; i < kCtrInts; i += blockDim.x) ctr[i] = 0;
    if (stats && threadIdx.x < (int)(sizeof(trim_stats_t) / 8))
        ((uint64_t*)stats)[threadIdx.x] = 0;
    if (threadIdx.x < kKeys) hist[threadIdx.x] = 0;
    __syncthreads();
    for (int gi = threadIdx.x; gi < G; gi += blockDim.x)
        atomicAdd(&hist[size_key(vbase, row_off, gi)], 1);
    __syncthreads();
    if (threadIdx.x == 0) {
        int run = 0;
        for (int k = 0; k < kKeys; ++k) {
            const int c = hist[k];
            hist[k] = run;
            run += c;
        }
    }
    __syncthreads();
    for (int gi = threadIdx.x; gi < G; gi += blockDim.x)
        order[atomicAdd(&hist[size_key(vbase, row_off, gi)], 1)] = gi;
}

// Shared state of an owned-graph kernel's workgroup (LDS).
struct OwnShared {
    __attribute__((aligned(16))) unsigned char raw[kOwnLds];
    int cnt[kOwnMaxBlock / kWave][kWatchCnt];   // per wavefront with a graph of its own; [0] for
                                                // the workgroup's
    int claim;
    uint64_t red[16];
};
// Per-thread running totals of the kernel.
struct OwnTotals {
    WatchTotals w;
    int max_phases = 0;
};

// The batch's arrays.
struct OwnArgs {
    const int64_t* vbase;
    const int* row_off;
    const int* col;
    const int64_t* bitmap_base;
    int total_m;
    int* head;
    uint64_t* rec;
    uint32_t* l0;
    uint32_t* l1;
    uint32_t* bitmaps;
    uint64_t* graph_edges;
    int sched;
};

// Graph gi's part of the arrays.
__device__ __forceinline__ CachedView own_view(const OwnArgs& a, int gi) {
    return CachedView{a.row_off + a.vbase[gi], a.col, a.total_m};
}
__device__ __forceinline__ ListArrays own_lists(const OwnArgs& a, int gi) {
    const int64_t vb = a.vbase[gi];
    return ListArrays{a.head + 2 * vb, a.rec + vb, a.l0 + vb, a.l1 + vb};
}

using OwnLists = GroupLists<CachedView, false>;

// The first list of graph gi, larger than watch.h takes, by the whole workgroup.
__device__ __forceinline__ void own_graph(const OwnArgs& a, int gi, OwnLists& l, OwnTotals& t) {
    const int n = (int)(a.vbase[gi + 1] - a.vbase[gi]);
    const int rank = threadIdx.x, size = blockDim.x;
    const CachedView& g = l.g;
    const ListArrays& m = l.m;
    uint64_t edges = 0;
    l.begin();
    // init: the heads of the graph's vertices
    for (int v = rank; v < n; v += size) {
        const int b = g.begin(v), e = g.end(v);
        const int h = b == e ? kDead : kEmpty;
        reinterpret_cast<int2*>(m.head)[v] = make_int2(h, h);
        t.w.deg += (uint64_t)(e - b);
    }
    l.sync();
    // sweep: only sinks are removed while it runs, so a target is live iff it
    // has a successor
    auto sink = [&](int w) { return g.begin(w) == g.end(w); };
    for (int base = 0; base < n; base += kOwnUnroll * size) {
        int v[kOwnUnroll], b[kOwnUnroll], e[kOwnUnroll], p[kOwnUnroll], w[kOwnUnroll];
        bool ok[kOwnUnroll];
#pragma unroll
        for (int k = 0; k < kOwnUnroll; ++k) {
            v[k] = base + k * size + rank;
            b[k] = e[k] = 0;
            if (v[k] < n) {
                b[k] = g.begin(v[k]);
                e[k] = g.end(v[k]);
            }
            p[k] = b[k];
            w[k] = b[k] < e[k] ? g.col[b[k]] : 0;
        }
#pragma unroll
        for (int k = 0; k < kOwnUnroll; ++k) {
            ok[k] = b[k] < e[k] && !sink(w[k]);
            if (b[k] < e[k] && !ok[k]) {
                for (++p[k]; p[k] < e[k]; ++p[k]) {
                    w[k] = g.col[p[k]];
                    if (!sink(w[k])) break;
                }
                ok[k] = p[k] < e[k];
            }
        }
        int old[kOwnUnroll];
#pragma unroll
        for (int k = 0; k < kOwnUnroll; ++k) {
            if (ok[k]) {
                if (a.sched & TRIM_SCHED_JITTER)
                    jitter_nap(((uint64_t)gi << 32) ^ (uint32_t)v[k]);
                old[k] = xchg_s<kWG>(m.head + 2 * w[k] + (p[k] + 1 == e[k]), v[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < kOwnUnroll; ++k) {
            uint32_t it = kNone;
            if (ok[k]) {
                st_s<kWG>(m.rec + v[k], pack_rec(old[k], p[k]));
                edges += (uint64_t)(p[k] - b[k] + 1);
            } else if (b[k] < e[k]) {
                it = make_item(kOwnClose, v[k]);
                edges += (uint64_t)(e[k] - b[k]);
            }
            l.emit(it);
        }
    }
    l.flush();
    t.w.sweep += edges;
    t.w.edges += edges;
    l.sync();
}

// Graph gi from its first list to its outputs; `before`: the totals' edges
// before the graph, `passes`: those it had.
__device__ __forceinline__ void own_finish(const OwnArgs& a, int gi, OwnLists& l, uint64_t before,
                                           int passes, OwnShared& sh, OwnTotals& t) {
    const int n = (int)(a.vbase[gi + 1] - a.vbase[gi]);
    const int rank = threadIdx.x, size = blockDim.x;
    const ListArrays& m = l.m;
    const int ph = passes + l.run(INT_MAX);
    t.max_phases = ph > t.max_phases ? ph : t.max_phases;
    // pack: the graph's bitmap words (bits past its n stay zero)
    const int64_t wb = a.bitmap_base[gi], we = a.bitmap_base[gi + 1];
    const int nwords = (n + 31) >> 5;
    for (int base = l.wave() * kWave; base < n; base += size) {
        const int v = base + lane_id();
        const uint64_t b = ballot(v < n && ld_s<kWG>(m.head + 2 * v) != kDead);
        if (lane_id() == 0) {
            const int wi = base >> 5;
            a.bitmaps[wb + wi] = (uint32_t)b;
            if (wi + 1 < nwords) a.bitmaps[wb + wi + 1] = (uint32_t)(b >> 32);
            t.w.live += (uint32_t)popc(b);
        }
    }
    for (int64_t wi = wb + nwords + rank; wi < we; wi += size) a.bitmaps[wi] = 0;
    const uint64_t edges = block_sum(t.w.edges - before, sh.red);
    if (rank == 0) a.graph_edges[gi] = edges;
    l.sync();
}

// LDS of own_watch: the statuses, then the supports when they are 16-bit, then
// the list.  Stage of the lists: the supports' place, or behind a second bitmap.
template <class Sup>
__device__ __forceinline__ unsigned char* own_stage(unsigned char* raw, int max_n) {
    return raw + (sizeof(Sup) == 2 ? 1 : 2) * (max_n / 8);
}

// Trim graph gi as watch.h describes: by the workgroup, or (kWaveGroup) by this
// wavefront.  Positions, and supports in device memory (32-bit), lie in the
// graph's own part of the two phase lists.  A workgroup leaves a deep, narrow
// remainder, its first list built, to own_finish (`end` kNarrow); returns the
// passes.
template <class Sup, class Item, bool kWaveGroup>
__device__ __forceinline__ int own_watch(const OwnArgs& a, int gi, unsigned char* raw, int max_n,
                                         int* cnt, OwnShared& sh, OwnTotals& t, WatchEnd& end) {
    const int n = (int)(a.vbase[gi + 1] - a.vbase[gi]);
    const CachedView g = own_view(a, gi);
    uint32_t* bits = reinterpret_cast<uint32_t*>(raw);
    unsigned char* rest = raw + max_n / 8;
    Sup* sup;
    if constexpr (sizeof(Sup) == 2) {
        sup = reinterpret_cast<uint16_t*>(rest);
        rest += max_n * 2;
    } else {
        sup = reinterpret_cast<int*>(own_lists(a, gi).l1);
    }
    const uint64_t before = t.w.edges;
    Watch<CachedView, Sup, int, Item, kWaveGroup> w{
        g, n, bits, sup, reinterpret_cast<int*>(own_lists(a, gi).l0), reinterpret_cast<Item*>(rest), cnt,
        a.sched, t.w};
    w.init(nullptr);
    w.template sweep<false>((int*)nullptr);
    end = w.template passes<true>(INT_MAX, kWaveGroup         ? kNarrowLds
                                           : sizeof(Sup) == 2 ? narrow_limit(n)
                                                              : kNarrowMem);
    if (__builtin_expect(end == kNarrow, 0)) {
        using Lists = GroupLists<CachedView, kWaveGroup>;
        Lists l{g, own_lists(a, gi), bits,
                *reinterpret_cast<ListStage<Lists::kWaves>*>(own_stage<Sup>(raw, max_n)), a.sched,
                t.w};
        w.to_lists(l);
        if constexpr (kWaveGroup)
            w.steps += l.run(INT_MAX);
        else
            return w.steps;
    }
    t.max_phases = w.steps > t.max_phases ? w.steps : t.max_phases;
    const int64_t wb = a.bitmap_base[gi], we = a.bitmap_base[gi + 1];
    const int nwords = (n + 31) >> 5;
    for (int64_t i = w.rank(); i < we - wb; i += w.size()) {
        const uint32_t word = i < nwords ? ~bits[i] : 0;   // the positions past n are set in bits
        a.bitmaps[wb + i] = word;
        t.w.live += (uint32_t)__popc(word);
    }
    const uint64_t edges = kWaveGroup ? wave_sum(t.w.edges - before)
                                      : block_sum(t.w.edges - before, sh.red);
    if (w.rank() == 0) a.graph_edges[gi] = edges;
    w.sync();
    return w.steps;
}

// Graphs are claimed in order (largest first).  A workgroup trims the larger
// ones together; once it claims one that a wavefront trims alone (all the
// later ones are), its wavefronts go their own ways: each trims that graph or
// graphs it claims itself, so up to one small graph per wavefront is in flight.
__global__ __launch_bounds__(kOwnMaxBlock) void ac6_owned(OwnArgs a, int G, const int* order,
                                                          int* ctr, uint64_t* wedges,
                                                          uint64_t* part) {
    __shared__ OwnShared sh;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    OwnTotals t;
    int first = -1;   // the small graph that ended the workgroup's part, if any
    for (;;) {
        if (threadIdx.x == 0) sh.claim = add_dev(ctr + kCursor, 1);
        __syncthreads();
        const int claim = sh.claim;
        __syncthreads();
        if (claim >= G) break;
        const int gi = order[claim];
        if (size_key(a.vbase, a.row_off, gi) >= 33) {
            first = gi;
            break;
        }
        const int64_t n = a.vbase[gi + 1] - a.vbase[gi];
        const uint64_t before = t.w.edges;
        WatchEnd end = kNarrow;
        int passes = 0;
        unsigned char* stage = sh.raw;
        if (watch_fits(n, (int)blockDim.x, kWatchLdsN)) {
            stage = own_stage<uint16_t>(sh.raw, kWatchLdsN);
            passes = own_watch<uint16_t, uint16_t, false>(a, gi, sh.raw, kWatchLdsN, sh.cnt[0], sh,
                                                          t, end);
        } else if (n <= kWatchMaxN) {
            stage = own_stage<int>(sh.raw, kWatchMaxN);
            passes =
                own_watch<int, uint32_t, false>(a, gi, sh.raw, kWatchMaxN, sh.cnt[0], sh, t, end);
        }
        if (__builtin_expect(end != kNarrow, 1)) continue;
        const CachedView g = own_view(a, gi);
        OwnLists l{g, own_lists(a, gi), n <= kWatchMaxN ? reinterpret_cast<uint32_t*>(sh.raw) : nullptr,
                   *reinterpret_cast<ListStage<16>*>(stage), a.sched, t.w};
        if (n > kWatchMaxN) own_graph(a, gi, l, t);
        own_finish(a, gi, l, before, passes, sh, t);
    }
    // wavefront part: wavefront 0 takes the graph that ended the workgroup part
    __syncthreads();   // the workgroup's LDS is free for the wavefronts
    for (int gi = (wv == 0) ? first : -1;;) {
        if (gi < 0) {
            int c = 0;
            if (lane_id() == 0) c = add_dev(ctr + kCursor, 1);
            c = __shfl(c, 0);
            if (c >= G) break;
            gi = order[c];
        }
        WatchEnd end;
        own_watch<uint16_t, uint16_t, true>(a, gi, sh.raw + wv * kOwnWaveLds, kOwnWaveN,
                                            sh.cnt[wv], sh, t, end);
        gi = -1;
    }
    __syncthreads();
    const uint64_t sweep = block_sum(t.w.sweep, sh.red);
    const uint64_t closes = block_sum(t.w.closes, sh.red);
    const uint64_t joins = block_sum(t.w.joins, sh.red);
    const uint64_t visited = block_sum(t.w.visited, sh.red);
    const uint64_t live = block_sum(t.w.live, sh.red);
    const uint64_t deg = block_sum(t.w.deg, sh.red);
    const uint64_t edges = block_sum(t.w.edges, sh.red);
    if (threadIdx.x == 0) {
        wedges[blockIdx.x] = edges;
        part[kPartSweep * kPartStride + blockIdx.x] = sweep;
        part[kPartDeg * kPartStride + blockIdx.x] = deg;
        part[kPartLive * kPartStride + blockIdx.x] = live;
        part[kPartLvCloses * kPartStride + blockIdx.x] = closes;
        part[kPartLvJoins * kPartStride + blockIdx.x] = joins;
        part[kPartLvVisited * kPartStride + blockIdx.x] = visited;
    }
    int mp = t.max_phases;
    for (int off = 32; off > 0; off >>= 1) mp = max(mp, __shfl_xor(mp, off));
    if (lane_id() == 0 && mp) atomicMax(ctr + kLvPhases, mp);
}

}  // namespace

int ac6_owned_blocks_per_cu(int block) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, ac6_owned, block, 0) != hipSuccess)
        return 1;
    return nb < 1 ? 1 : nb;
}

hipError_t ac6_batch_owned(int G, const int64_t* vbase, const int32_t* row_off,
                           const int32_t* col, int64_t total_n, int64_t total_m,
                           const int64_t* bitmap_base, const Work& w, const LaunchCfg& lc,
                           uint32_t* bitmaps, uint64_t* graph_edges, trim_stats_t* stats) {
    const int B = lc.block;
    int W = lc.workers > 0 ? lc.workers : lc.cus * ac6_owned_blocks_per_cu(B);
    if (W > kPartStride) W = kPartStride;
    {
        Timed t(lc, "batch_order");
        hipLaunchKernelGGL(batch_order, dim3(1), dim3(1024), 0, lc.stream, vbase, row_off, G, w.d,
                           w.ctr, stats);
    }
    {
        Timed t(lc, "ac6_owned");
        const OwnArgs a{vbase, row_off, col,     bitmap_base, (int)total_m, w.a,
                        w.b,   w.e,     w.e + w.cap, bitmaps,  graph_edges,  lc.schedule};
        hipLaunchKernelGGL(ac6_owned, dim3(W), dim3(B), 0, lc.stream, a, G, w.d, w.ctr, w.wedges,
                           w.part);
    }
    if (stats) {
        Timed t(lc, "finalize");
        hipLaunchKernelGGL(finalize_stats, dim3(1), dim3(1024), 0, lc.stream, (int)total_n, W, W,
                           0, W, 0, w.wedges, w.part, w.ctr, stats, 0, 0, W);
    }
    return hipGetLastError();
}

}  // namespace trim
