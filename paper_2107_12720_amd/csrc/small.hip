// small.hip -- AC-6 of a small graph by one workgroup (watch.h).
//
// The device-wide path (ac6.hip) takes seven launches and device-wide phases;
// on a graph of a few thousand vertices its persistent workers and barriers
// cost far more than the work.  One workgroup keeps every status and support
// in LDS instead and writes all outputs itself.  Three forms:
//   ac6_tiny    the graph itself is staged in LDS, too (16-bit ids and
//               positions): a resumed scan is two LDS reads instead of two
//               dependent loads from device memory, 2 us a pass;
//   ac6_small   one launch, the graph read through the caches;
//   fronted     from kFrontN vertices on, the status bits and the sweep, whose
//               loads one compute unit issues too slowly, run on all of them
//               (two launches more, about 5 us each), and ac6_small starts at
//               the forest collapse.
#include "trim_internal.h"
#include "trim_device.h"
#include "watch.h"

namespace trim {
namespace {

constexpr int kSmallBlock = 1024;
constexpr int kSmallWaves = kSmallBlock / kWave;
constexpr int kTinyN = 8192, kTinyM = 36864;
constexpr int kFrontN = 16384;
constexpr int kFrontBlock = 256;

// Table staging of the implicit view, as in the device-wide kernels.
template <class View>
struct StageSmall {
    static constexpr int kWords = 1;
    __device__ static void apply(View&, uint64_t*) {}
};
template <>
struct StageSmall<ImplicitView> {
    static constexpr int kWords = 256;
    __device__ static void apply(ImplicitView& g, uint64_t* lds) {
        for (int i = threadIdx.x; i < 256; i += blockDim.x) lds[i] = g.table[i];
        __syncthreads();
        g.table = lds;
    }
};

// A graph in LDS.
struct LdsView {
    const uint16_t* row_off;
    const uint16_t* col;
    __device__ __forceinline__ int vctx(int) const { return 0; }
    __device__ __forceinline__ int begin(int v) const { return row_off[v]; }
    __device__ __forceinline__ int end(int v) const { return row_off[v + 1]; }
    __device__ __forceinline__ int target(int, int p, int) const { return col[p]; }
};

struct SmallOut {
    uint32_t* bitmap;
    uint64_t* worker_edges;
    int P;
    trim_stats_t* stats;
    int* ctr;
};

enum { kEdges, kSweep, kDeg, kCloses, kJoins, kVisited, kForestN, kLive, kTotals };
struct SmallRed {
    uint32_t part[kTotals][kSmallWaves];
    uint32_t tot[kTotals];
};

// All outputs of the call.  The totals fit 32 bits: no graph here has more
// than 2^24 edges, and no edge is checked twice.
template <class W>
__device__ __forceinline__ void small_outputs(const W& a, WatchTotals& t, bool done,
                                              const SmallOut& out, SmallRed& red) {
    const int nwords = (a.n + 31) >> 5;
    for (int i = threadIdx.x; i < nwords; i += blockDim.x) {
        const uint32_t word = ~a.bits[i];
        out.bitmap[i] = word;
        t.live += (uint32_t)__popc(word);
    }
    for (int p = threadIdx.x; p < out.P; p += blockDim.x)
        if (p > 0) out.worker_edges[p] = 0;
    uint32_t x[kTotals] = {(uint32_t)t.edges, (uint32_t)t.sweep, (uint32_t)t.deg, t.closes,
                           t.joins, t.visited, t.forest, t.live};
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1)
#pragma unroll
        for (int q = 0; q < kTotals; ++q) x[q] += __shfl_xor(x[q], off);
    if (lane_id() == 0)
#pragma unroll
        for (int q = 0; q < kTotals; ++q) red.part[q][threadIdx.x / kWave] = x[q];
    __syncthreads();
    if (threadIdx.x >= kWave) return;
    if (threadIdx.x < kTotals) {
        uint32_t s = 0;
        for (int i = 0; i < (int)(blockDim.x / kWave); ++i) s += red.part[threadIdx.x][i];
        red.tot[threadIdx.x] = s;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    constexpr int kWords = sizeof(trim_stats_t) / 8;
    if (out.stats && threadIdx.x < kWords) {
        trim_stats_t s = {};
        s.edges_total = red.tot[kEdges];
        s.n_live = red.tot[kLive];
        s.n_dead = (uint64_t)(a.n - (int)red.tot[kLive]);
        s.edges_sweep = red.tot[kSweep];
        s.closes = red.tot[kCloses];
        s.joins = red.tot[kJoins];
        s.visited = red.tot[kVisited];
        s.graph_edges = red.tot[kDeg];
        s.stalled = done ? 0 : 1;
        s.forest = red.tot[kForestN];
        s.jump_rounds = (uint64_t)a.jumps;
        s.work_items = red.tot[kForestN];
        s.phases = (uint64_t)a.steps;
        const uint64_t* word = reinterpret_cast<const uint64_t*>(&s);
        uint64_t mine = 0;
#pragma unroll
        for (int i = 0; i < kWords; ++i) mine = (int)threadIdx.x == i ? word[i] : mine;
        reinterpret_cast<uint64_t*>(out.stats)[threadIdx.x] = mine;
    }
    if (threadIdx.x == 0) {
        if (out.P > 0) out.worker_edges[0] = red.tot[kEdges];
        out.ctr[kStall] = done ? 0 : 1;
    }
}

template <bool kForest>
__global__ __launch_bounds__(kSmallBlock) void ac6_tiny(const int* row_off, const int* col, int n,
                                                        int m, const uint32_t* preset,
                                                        SmallOut out, int sched, int budget) {
    __shared__ __attribute__((aligned(16))) uint32_t bits[kTinyN / 32];
    __shared__ __attribute__((aligned(16))) uint16_t sup[kTinyN];
    __shared__ uint16_t keep[kForest ? kTinyN : 1], cur[kTinyN];
    __shared__ __attribute__((aligned(16))) uint16_t list[kSmallWaves * kWatchList];
    __shared__ uint16_t s_off[kTinyN + 1], s_col[kTinyM];
    __shared__ int cnt[kWatchCnt];
    __shared__ SmallRed red;
    static_assert(sizeof list >= sizeof bits, "the list holds the sweep's second bitmap first");
    for (int i = threadIdx.x; i <= n; i += blockDim.x) s_off[i] = (uint16_t)row_off[i];
#pragma unroll 8
    for (int i = threadIdx.x; i < m; i += blockDim.x) s_col[i] = (uint16_t)col[i];
    __syncthreads();
    WatchTotals t;
    const LdsView g{s_off, s_col};
    Watch<LdsView, uint16_t, uint16_t, uint16_t, false> a{g, n, bits, sup, cur, list, cnt, sched, t};
    a.init(preset);
    a.template sweep<kForest>(keep);
    bool done = true;
    if (kForest) done = a.forest(keep, budget);
    if (done) done = a.passes(budget) == kDone;
    small_outputs(a, t, done, out, red);
}

// sup_g: n ints; the positions lie in m.l0.  With kFront the status bits (`gbits`), the second
// bitmap (`gnone`), the links and the per-workgroup sums come from the two
// front kernels.
struct Front {
    const uint32_t* bits;
    const uint32_t* none;
    const int* link;
    const uint64_t* part;
    int blocks;
};

template <class View, bool kForest, bool kFront>
__global__ __launch_bounds__(kSmallBlock) void ac6_small(View g, int n, const uint32_t* preset,
                                                         int* sup_g, ListArrays m, Front f,
                                                         SmallOut out, int sched, int budget) {
    __shared__ uint64_t table[StageSmall<View>::kWords];
    __shared__ __attribute__((aligned(16))) uint32_t bits[kWatchLdsN / 32];
    __shared__ __attribute__((aligned(16))) uint16_t sup[kWatchLdsN];
    // first the sweep's second bitmap
    __shared__ __attribute__((aligned(16))) uint16_t list[kSmallWaves * kWatchList];
    static_assert(sizeof list >= sizeof bits, "the list holds the sweep's second bitmap first");
    __shared__ int cnt[kWatchCnt];
    __shared__ SmallRed red;
    StageSmall<View>::apply(g, table);
    WatchTotals t;
    Watch<View, uint16_t, int, uint16_t, false> a{g, n, bits, sup, reinterpret_cast<int*>(m.l0),
                                                  list, cnt, sched, t};
    if constexpr (kFront) {
        const int nwords = (n + 31) >> 5, tid = threadIdx.x;
        if (tid < kWatchCnt) cnt[tid] = 0;
        __syncthreads();
        for (int i = tid; i < ((nwords + 1) & ~1); i += blockDim.x) {
            const uint32_t b = f.bits[i];
            const uint32_t real = i < nwords - 1 || !(n & 31) ? b : b & ((1u << (n & 31)) - 1u);
            const uint32_t x = i < nwords ? f.none[i] : 0;
            bits[i] = b | x;
            if (kForest) t.forest += __popc(x);
            else t.closes += __popc(x);
            if (i < nwords && real) cnt[3] = 32 * i + __ffs((int)real);
        }
        if (tid < f.blocks) {
            t.edges = t.sweep = f.part[kPartSweep * kPartStride + tid];
            t.deg = f.part[kPartDeg * kPartStride + tid];
        }
        __syncthreads();
        const int null = a.null_vertex();
        constexpr int U = 8;
        for (int i = 0; i < n; i += U * kSmallBlock) {
            int s[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int v = min(i + k * kSmallBlock + tid, n - 1);
                s[k] = (kForest ? f.link : sup_g)[v];
            }
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int v = i + k * kSmallBlock + tid;
                if (v < n) sup[v] = (uint16_t)(s[k] < 0 ? null : s[k]);
            }
        }
        __syncthreads();
    } else {
        a.init(preset);
        a.template sweep<kForest>(sup_g);
    }
    bool done = true;
    if (kForest) done = a.forest(sup_g, budget);
    if (done) {
        const WatchEnd end = a.template passes<kFront>(budget, narrow_limit(n));
        done = end != kStalled;
        if constexpr (kFront) {
            if (end == kNarrow) {
                GroupLists<View, false> l{g, m, bits, *reinterpret_cast<ListStage<16>*>(sup), sched, t};
                a.to_lists(l);
                const int left = budget - a.steps - a.jumps, ph = l.run(left);
                a.steps += ph;
                done = ph < left;
            }
        }
    }
    small_outputs(a, t, done, out, red);
}

// The status bits of the vertices removed before the sweep, set past n as well.
__global__ __launch_bounds__(kFrontBlock) void small_bits(const int* row_off, int n,
                                                          const uint32_t* preset, uint32_t* bits) {
    const int v = blockIdx.x * kFrontBlock + threadIdx.x;
    const bool gone = v >= n || row_off[v] == row_off[v + 1] ||
                      (preset && ((preset[v >> 5] >> (v & 31)) & 1u));
    const uint64_t m = ballot(gone);
    if (lane_id() == 0 && v < n) {
        bits[v >> 5] = (uint32_t)m;
        bits[(v >> 5) + 1] = (uint32_t)(m >> 32);
    }
}

// The sweep, one vertex per lane: supports (-1: none), positions, links and the
// bitmap of the vertices without a live successor.
__global__ __launch_bounds__(kFrontBlock) void small_sweep(const int* row_off, const int* col,
                                                           int n, const uint32_t* bits, int* sup_g,
                                                           int* cur, int* link, uint32_t* none,
                                                           uint64_t* part) {
    __shared__ uint64_t red[16];
    const int v = blockIdx.x * kFrontBlock + threadIdx.x;
    uint64_t edges = 0, deg = 0;
    bool lost = false;
    if (v < n) {
        const int b = row_off[v], e = row_off[v + 1];
        deg = (uint64_t)(e - b);
        int s = -1, p = b;
        if (!wt_bit(bits, v)) {
            constexpr int K = 4;
            for (; p < e && s < 0; p += K) {
                int w[K];
                bool live[K];
#pragma unroll
                for (int j = 0; j < K; ++j) w[j] = col[min(p + j, e - 1)];
#pragma unroll
                for (int j = 0; j < K; ++j) live[j] = !wt_bit(bits, w[j]);
#pragma unroll
                for (int j = K - 1; j >= 0; --j)
                    if (p + j < e && live[j]) {
                        s = w[j];
                        cur[v] = p + j;
                        link[v] = p + j + 1 == e ? s : v;
                        edges = (uint64_t)(p + j - b + 1);
                    }
            }
            lost = s < 0;
            if (lost) edges = deg;
        }
        sup_g[v] = s;
        if (s < 0) link[v] = v;
    }
    const uint64_t m = ballot(lost);
    if (lane_id() == 0 && v < n) {
        none[v >> 5] = (uint32_t)m;
        none[(v >> 5) + 1] = (uint32_t)(m >> 32);
    }
    edges = block_sum(edges, red);
    deg = block_sum(deg, red);
    if (threadIdx.x == 0) {
        part[kPartSweep * kPartStride + blockIdx.x] = edges;
        part[kPartDeg * kPartStride + blockIdx.x] = deg;
    }
}

int small_block(int n) {
    const int block = (n / 2 + kWave - 1) / kWave * kWave;
    return block < 256 ? 256 : block > kSmallBlock ? kSmallBlock : block;
}

}  // namespace

// Where the line lies: depth and list lengths divide one workgroup from the
// device-wide rounds, which the sizes do not tell, so it lies where neither is the
// faster over all kinds.  Twelve kinds of graph (core+tail of mean degree 6.5, 8 and
// 15, uniform of 1.1 to 16, R-MAT with and without a chain), device-wide over one
// workgroup, geometric mean (least, largest): 36,000 vertices 1.30 (0.87, 1.60),
// 50,000 1.06 (0.62, 1.47), 54,000 1.05 (0.60, 1.41), 58,000 0.99 (0.55, 1.46),
// 65,536 0.91 (0.56, 1.26).  A pass goes in batches of 8,192 supports; seven are
// below the crossing, the eighth starts there.  us, one workgroup / device-wide, at
// 54,000 and 65,536: core+tail 265 / 243 and 308 / 249, with lists of 15 857 / 511 and
// 999 / 556, uniform of 1.1 221 / 302 and 334 / 422, of 16 28 / 39 and 31 / 38, R-MAT
// of edge factor 16 43 / 50 and 47 / 50.  The edge limit keeps graphs of long lists
// away, whose scans one compute unit runs slowly: tails of 30 successors a vertex,
// nearly all of them removed, take 908 / 1,358 with 17,000 vertices, 2,302 / 1,430
// with 50,000.
constexpr long long kSmallMaxN = 7 * 8192;
static_assert(kSmallMaxN <= kWatchLdsN, "the LDS holds the supports");
bool ac6_small_ok(long long n, long long m, int rounds) {
    return rounds < 2 && n <= kSmallMaxN && m <= kSmallMaxM;
}
// A resumed scan of the implicit graph hashes its degree again: 2^14 vertices
// 114 / 190 us, 2^16 324 / 245.
bool ac6_small_implicit_ok(int log2n, int rounds) { return rounds < 2 && log2n <= 15; }

hipError_t ac6_small_csr(const trim_csr_t& g, const Work& w, const LaunchCfg& lc, uint32_t* bitmap,
                         uint64_t* worker_edges, trim_stats_t* stats, const uint32_t* preset) {
    const int n = g.n;
    const SmallOut out{bitmap, worker_edges, lc.workers, stats, w.ctr};
    hipStream_t st = lc.stream;
    if (n <= kTinyN && g.m <= kTinyM) {
        Timed t(lc, "ac6_small");
        const dim3 block(small_block(n));
        if (lc.forest)
            hipLaunchKernelGGL(ac6_tiny<true>, dim3(1), block, 0, st, g.row_off, g.col, n,
                               (int)g.m, preset, out, lc.schedule, lc.budget);
        else
            hipLaunchKernelGGL(ac6_tiny<false>, dim3(1), block, 0, st, g.row_off, g.col, n,
                               (int)g.m, preset, out, lc.schedule, lc.budget);
        return hipGetLastError();
    }
    const CachedView v{g.row_off, g.col, (int)g.m};
    // the lists' heads and records are made, if at all, when the rest is done with
    const ListArrays m{w.a, w.b, w.e, w.e + n};
    int* sup = reinterpret_cast<int*>(m.l1);
    if (n < kFrontN) {
        Timed t(lc, "ac6_small");
        if (lc.forest)
            hipLaunchKernelGGL((ac6_small<CachedView, true, false>), dim3(1), dim3(kSmallBlock), 0,
                               st, v, n, preset, sup, m, Front{}, out, lc.schedule, lc.budget);
        else
            hipLaunchKernelGGL((ac6_small<CachedView, false, false>), dim3(1), dim3(kSmallBlock),
                               0, st, v, n, preset, sup, m, Front{}, out, lc.schedule, lc.budget);
        return hipGetLastError();
    }
    uint32_t* bits = reinterpret_cast<uint32_t*>(w.c);
    uint32_t* none = bits + (n + 63) / 64 * 2;
    const int blocks = (n + kFrontBlock - 1) / kFrontBlock;
    {
        Timed t(lc, "ac6_init");
        hipLaunchKernelGGL(small_bits, dim3(blocks), dim3(kFrontBlock), 0, st, g.row_off, n,
                           preset, bits);
    }
    {
        Timed t(lc, "ac6_sweep");
        hipLaunchKernelGGL(small_sweep, dim3(blocks), dim3(kFrontBlock), 0, st, g.row_off, g.col,
                           n, bits, sup, reinterpret_cast<int*>(m.l0), w.jp, none, w.part);
    }
    Timed t(lc, "ac6_small");
    const Front f{bits, none, w.jp, w.part, blocks};
    if (lc.forest)
        hipLaunchKernelGGL((ac6_small<CachedView, true, true>), dim3(1), dim3(kSmallBlock), 0, st,
                           v, n, preset, sup, m, f, out, lc.schedule, lc.budget);
    else
        hipLaunchKernelGGL((ac6_small<CachedView, false, true>), dim3(1), dim3(kSmallBlock), 0, st,
                           v, n, preset, sup, m, f, out, lc.schedule, lc.budget);
    return hipGetLastError();
}

hipError_t ac6_small_implicit(const trim_implicit_t& g, const Work& w, const LaunchCfg& lc,
                              uint32_t* bitmap, uint64_t* worker_edges, trim_stats_t* stats) {
    const int n = 1 << g.log2n;
    const ImplicitView v{g.seed, g.zero_thr, g.deg_table, (uint32_t)(n - 1)};
    const SmallOut out{bitmap, worker_edges, lc.workers, stats, w.ctr};
    const ListArrays m{w.a, w.b, w.e, w.e + n};
    Timed t(lc, "ac6_small");
    if (lc.forest)
        hipLaunchKernelGGL((ac6_small<ImplicitView, true, false>), dim3(1), dim3(kSmallBlock), 0,
                           lc.stream, v, n, (const uint32_t*)nullptr, w.a, m, Front{}, out,
                           lc.schedule, lc.budget);
    else
        hipLaunchKernelGGL((ac6_small<ImplicitView, false, false>), dim3(1), dim3(kSmallBlock), 0,
                           lc.stream, v, n, (const uint32_t*)nullptr, w.a, m, Front{}, out,
                           lc.schedule, lc.budget);
    return hipGetLastError();
}

}  // namespace trim
