// ac4.hip -- AC-4-based graph trimming on gfx950 (Section 5.2, Alg. par-ac4trim).
//
// cnt[v] is the live out-degree counter, initialised from CSR offsets
// (AC4Trim*, Section 9.3: no edge is traversed to find it).  A removed vertex
// w decrements cnt[u] once for every edge u -> w, walking w's predecessors in
// the transposed graph.  The paper takes CAS(status, LIVE, DEAD) to enqueue a
// vertex once; here the fetch-and-add that brings cnt[u] from 1 to 0 returns
// 1 to exactly one lane, which makes that lane u's unique remover, so the
// status is simply cnt[u] == 0.
//
// Two-sided (Section 4.1, the in-degree check over G^T): cnt[n+v] also counts
// v's live predecessors, from the G^T offsets.  A removed w then decrements
// the out-counters of its predecessors and the in-counters of its successors;
// a vertex can reach zero on both counters, so the lane that brings either to
// zero removes it only if its exchange of dead[v] is the first one.  Every
// removed vertex walks both of its lists once.
//
// Kernels: ac4_init (counters), ac4_first (the vertices removed from the start,
// spread evenly over the device), ac4_long (their long lists, in pieces); those
// that their removal takes down are queued for ac4_propagate (persistent workers
// on per-wavefront LDS rings, WaveQueue; a lane walks a short predecessor list of
// its removed vertex eight at a time, with the eight decrements in flight
// together, and then goes on with one of the vertices it removed itself, depth
// first; long lists are walked by the whole wavefront), ac4_pack (bitmap from
// cnt > 0).
#include "trim_device.h"
#include "trim_stats.h"
#include "trim_internal.h"

namespace trim {

namespace {

// A preset vertex (removed before trimming) starts at cnt = 0: it is queued
// like an out-degree-0 vertex, and its counter only goes negative after that,
// so no decrement ever returns 1 for it.
template <bool kTwo>
__global__ void ac4_init(const int* row_off, const int* rrow_off, const uint32_t* preset, int n,
                         int* cnt, int* dead, int* ctr, uint64_t* worker_edges, int P,
                         trim_stats_t* stats) {
    const int tid = blockIdx.x * blockDim.x + threadIdx.x;
    if (tid < kCtrInts) ctr[tid] = 0;
    for (int p = tid; p < P; p += gridDim.x * blockDim.x) worker_edges[p] = 0;
    if (stats && tid < (int)(sizeof(trim_stats_t) / 8)) ((uint64_t*)stats)[tid] = 0;
    for (int v = tid; v < n; v += gridDim.x * blockDim.x) {
        const int d = row_off[v + 1] - row_off[v];
        cnt[v] = (preset && ((preset[v >> 5] >> (v & 31)) & 1u)) ? 0 : d;
        if (kTwo) {
            const int di = rrow_off[v + 1] - rrow_off[v];
            cnt[n + v] = di;
            dead[v] = (d == 0 || di == 0) ? 1 : 0;
        }
    }
}

// The lane whose decrement brought a counter of u to zero: u's remover?
template <bool kTwo>
__device__ __forceinline__ bool removes(int* dead, int u) {
    return !kTwo || xchg_dev(dead + u, 1) == 0;
}

constexpr int kBatch = 8;
constexpr int kCoop = 16;   // predecessor lists longer than this are walked by the wavefront
// Busy iterations between polls for waiting lanes elsewhere: 16, as for the
// AC-6 kernels on explicit graphs (measured at 512 workers: the 65,536-vertex
// core+tail graph 35 % and R-MAT 22 with half of its vertices preset 12 %
// faster than with 64, the R-MAT 22 chain workload unchanged).
constexpr int kShareEvery4 = 16;
// Queue slots a wavefront of ac4_propagate takes at first: on small graphs, whose
// few removals to start with all fit one or two wavefronts, fewer than its lanes.
// Core+tail of 12,000 vertices 209 us with 16, 237 with 64, of 36,000 273 and 321;
// R-MAT from 2^18 vertices on 3 to 12 % slower with 16.
constexpr int kSpreadTickets = 16, kSpreadN = 1 << 16;

// A wavefront's buffer in LDS to its reserved place.
template <class X>
__device__ __forceinline__ void write_out(const X* buf, X* to, int& fill) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int i = lane_id(); i < fill; i += kWave) to[i] = buf[i];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    fill = 0;
}
// One reservation for all wavefronts of the workgroup (256 lanes); each gets
// the place of its own k.
template <class Reserve>
__device__ __forceinline__ int block_reserve(int k, Reserve reserve) {
    __shared__ int s_k[256 / kWave], s_base;
    const int wv = threadIdx.x / kWave;
    __syncthreads();
    if (lane_id() == 0) s_k[wv] = k;
    __syncthreads();
    int before = 0, all = 0;
    for (int w = 0; w < 256 / kWave; ++w) {
        before += w < wv ? s_k[w] : 0;
        all += s_k[w];
    }
    if (threadIdx.x == 0 && all > 0) s_base = reserve(all);
    __syncthreads();
    return all > 0 ? s_base + before : 0;
}

// Items that a wavefront collects in LDS (room for kStepItems more after
// make_room), so that it makes one reservation in the queue for hundreds.  Its
// size, with the pieces', leaves room for eight workgroups a CU (with seven,
// 20 KB, ac4_first took 338 us on R-MAT 24).
constexpr int kStepItems = kWave * kBatch;   // removals of one step at most
struct ItemBuf {
    static constexpr int kItems = kStepItems + 256;
    uint32_t* buf;   // kItems words of LDS, the wavefront's own
    uint32_t* q;
    int* ctr;
    int fill = 0;    // the same in every lane
    __device__ __forceinline__ void make_room() {
        if (fill > kItems - kStepItems) flush();
    }
    __device__ __forceinline__ void push(bool has, int u) {
        const uint64_t m = ballot(has);
        if (has) buf[fill + popc(m & lanes_below())] = make_item(0, u);
        fill += popc(m);
    }
    __device__ __forceinline__ int reserve(int k) const {
        add_dev(ctr + kPending, k);
        return add_dev(ctr + kQTail, k);
    }
    __device__ __forceinline__ void flush() {
        int base = 0;
        if (lane_id() == 0) base = reserve(fill);
        write_out(buf, q + __shfl(base, 0), fill);
    }
    // At the kernel's end, by all of the workgroup.
    __device__ __forceinline__ void finish() {
        const int base = block_reserve(fill, [&](int k) { return reserve(k); });
        write_out(buf, q + base, fill);
    }
};

// One step of a walk: entries j < nb of `at` (stride apart) lose a neighbour on
// this side; the vertices whose last one it was are collected.
template <bool kTwo>
__device__ __forceinline__ void first_step(const int* at, int stride, int nb, int* ctr_of,
                                           int* dead, ItemBuf& out, int sched, uint64_t key) {
    int u[kBatch], old[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j)
        if (j < nb) u[j] = at[j * stride];
    if (sched & TRIM_SCHED_JITTER) jitter_nap(key);
    bool any = false;
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
        old[j] = 0;
        if (j < nb) old[j] = add_dev(ctr_of + u[j], -1);
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) any = any || old[j] == 1;
    if (!ballot(any)) return;
#pragma unroll
    for (int j = 0; j < kBatch; ++j) out.push(old[j] == 1 && removes<kTwo>(dead, u[j]), u[j]);
}

// The vertices removed from the start (no successors, with kTwo no predecessors
// either way, or preset; read off the offsets, since counters reach zero while
// this runs).  On a power-law graph they are most of all removals and nearly all
// have no list to walk or a short one: through the shared queue the 9.4 * 10^6 of
// R-MAT 24, 2.1 * 10^6 reverse edges in all, took 3.4 of 3.7 ms.  A lane takes a
// list of up to kBatch entries itself, in one step.  Longer ones are listed in
// pieces of `piece` entries (vertex, number of the piece) for ac4_long, which
// spreads them over the device: walked here, the hubs of an R-MAT graph, its low
// ids, met in few wavefronts (R-MAT 20 of edge factor 16 with 30 % of the vertices
// kept: 3,608 us here, 148 + 1,463 with ac4_long, 2,771 through the queue).
// (Two-sided, a vertex removed from the start has one list at most.)  Steps go to
// the workgroups by step_of: in turn 340 us on R-MAT 24, so 296.
constexpr int kLongBuf = 128;   // pieces a wavefront buffers

template <bool kTwo>
__global__ __launch_bounds__(256) void ac4_first(const int* rrow_off, const int* rcol,
                                                 const int* row_off, const int* col,
                                                 const uint32_t* preset, int n, int* cnt,
                                                 int* dead, uint32_t* q, int* ctr,
                                                 uint64_t* worker_edges, int P, int sched,
                                                 uint64_t* pieces, int piece) {
    __shared__ uint32_t items[256 / kWave][ItemBuf::kItems];
    __shared__ uint64_t longs[256 / kWave][kLongBuf];
    __shared__ uint64_t red[16];
    const int wv = threadIdx.x / kWave;
    ItemBuf out{items[wv], q, ctr};
    int nlong = 0;   // the same in every lane
    uint64_t edges = 0;
    const int steps = (int)((n + (long long)blockDim.x - 1) / blockDim.x);
    for (int b0 = blockIdx.x; b0 < steps; b0 += gridDim.x) {
        const int v = step_of(b0, steps) * (int)blockDim.x + (int)threadIdx.x;
        const int x = v < n ? v : n - 1;
        const int b = row_off[x], be = row_off[x + 1], rb = rrow_off[x], re = rrow_off[x + 1];
        const bool gone = v < n && (b == be || (kTwo && rb == re) ||
                                    (preset && ((preset[x >> 5] >> (x & 31)) & 1u)));
        if (!ballot(gone)) continue;
        const bool post = kTwo && rb == re;   // the list is the successors
        const int k = post ? b : rb, len = gone ? (post ? be : re) - k : 0;
        const uint64_t m = ballot(len > kBatch && len <= piece);
        if (m) {
            if (nlong > kLongBuf - kWave) {
                int base = 0;
                if (lane_id() == 0) base = add_dev(ctr + kA4Pieces, nlong);
                write_out(longs[wv], pieces + __shfl(base, 0), nlong);
            }
            if (len > kBatch && len <= piece)
                longs[wv][nlong + popc(m & lanes_below())] = (uint64_t)(uint32_t)v;
            nlong += popc(m);
        }
        if (len > piece) {
            const int c = (len - 1) / piece + 1, base = add_dev(ctr + kA4Pieces, c);
            for (int i = 0; i < c; ++i) pieces[base + i] = (uint64_t)i << 32 | (uint32_t)v;
        }
        const int nb = len <= kBatch ? len : 0;
        if (!ballot(nb > 0)) continue;
        out.make_room();
        edges += (uint64_t)nb;
        first_step<kTwo>((post ? col : rcol) + k, 1, nb, post ? cnt + n : cnt, dead, out, sched,
                         ((uint64_t)k << 16) ^ v);
    }
    out.finish();
    const int base = block_reserve(nlong, [&](int k) { return add_dev(ctr + kA4Pieces, k); });
    write_out(longs[wv], pieces + base, nlong);
    edges = block_sum(edges, red);
    if (threadIdx.x == 0 && edges) add_dev(worker_edges + (blockIdx.x % P), edges);
}

// The long lists of ac4_first, a piece per wavefront at a time.
template <bool kTwo>
__global__ __launch_bounds__(256) void ac4_long(const int* rrow_off, const int* rcol,
                                                const int* row_off, const int* col, int n,
                                                int* cnt, int* dead, uint32_t* q, int* ctr,
                                                uint64_t* worker_edges, int P, int sched,
                                                const uint64_t* pieces, int piece) {
    __shared__ uint32_t items[256 / kWave][ItemBuf::kItems];
    __shared__ uint64_t red[16];
    const int c = ctr[kA4Pieces];
    if (c == 0) return;
    const int waves = (int)(gridDim.x * blockDim.x / kWave);
    const int wave = (int)(blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    ItemBuf out{items[threadIdx.x / kWave], q, ctr};
    uint64_t edges = 0;
    for (int i = wave; i < c; i += waves) {
        const uint64_t x = pieces[i];
        const int v = (int)(uint32_t)x;
        const bool post = kTwo && rrow_off[v] == rrow_off[v + 1];
        const int* off = post ? row_off : rrow_off;
        const uint32_t e = off[v + 1];   // (unsigned: see step_index)
        const uint32_t p0 = off[v] + (uint32_t)(x >> 32) * (uint32_t)piece;
        const uint32_t p1 = min(e, p0 + (uint32_t)piece);
        if (lane_id() == 0) edges += p1 - p0;
        for (uint32_t p = p0; p < p1; p += kStepItems) {
            out.make_room();
            const int mine = (int)(p1 - p) - lane_id();   // entry j of the lane: j * kWave < mine
            first_step<kTwo>((post ? col : rcol) + p + lane_id(), kWave,
                             (mine + kWave - 1) / kWave, post ? cnt + n : cnt, dead, out, sched,
                             ((uint64_t)p << 20) ^ v);
        }
    }
    out.finish();
    edges = block_sum(edges, red);
    if (threadIdx.x == 0 && edges) add_dev(worker_edges + (blockIdx.x % P), edges);
}

// Phase 0 walks pre(w) over G^T and decrements out-counters (cnt[u]); with
// kTwo, phase 1 then walks post(w) over G and decrements in-counters
// (cnt[n + x]).
template <bool kTwo>
__global__ __launch_bounds__(256) void ac4_propagate(const int* rrow_off, const int* rcol,
                                                     const int* row_off, const int* col, int n,
                                                     int* cnt, int* dead, uint32_t* q, int* ctr,
                                                     uint64_t* worker_edges, uint64_t* part,
                                                     int sched, int budget, int tickets) {
    __shared__ uint32_t rings[256 / kWave][kLocalQ];
    __shared__ int ring_tail[256 / kWave];
    WaveQueue wq;
    const int wv = threadIdx.x / kWave;
    wq.init(rings[wv], &ring_tail[wv], q, ctr + kQHead, ctr + kQTail, ctr + kPending,
            ctr + kStall, budget, kShareEvery4);
    wq.claim(tickets);
    uint32_t item = kNone;
    int k = 0, e = 0, ph = 0;
    bool started = false;
    uint64_t edges = 0;
    while (wq.acquire(item)) {
        uint32_t out[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) out[j] = kNone;
        if (item != kNone && !started) {
            const int w = item_vertex(item);
            k = rrow_off[w];
            e = rrow_off[w + 1];
            ph = 0;
            started = true;
            edges += (uint64_t)(e - k);
            if (kTwo) edges += (uint64_t)(row_off[w + 1] - row_off[w]);
        }
        // Long predecessor lists: the whole wavefront walks them, one list at
        // a time, 64 x kBatch decrements in flight per round.
        for (uint64_t big = ballot(item != kNone && e - k > kCoop); big; big &= big - 1) {
            const int owner = __ffsll((unsigned long long)big) - 1;
            const uint32_t kb = __shfl(k, owner), eb = __shfl(e, owner);
            const int phb = kTwo ? __shfl(ph, owner) : 0;
            const int* adj = phb ? col : rcol;
            int* ctr_of = phb ? cnt + n : cnt;
            for (uint32_t base = kb; base < eb; base += kWave * kBatch) {
                int u[kBatch], old[kBatch];
                uint32_t o[kBatch];
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    const uint32_t p = base + j * kWave + lane_id();
                    if (p < eb) u[j] = adj[p];
                }
                if (sched & TRIM_SCHED_JITTER) jitter_nap(((uint64_t)kb << 20) ^ base);
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    const uint32_t p = base + j * kWave + lane_id();
                    if (p < eb) old[j] = add_dev(ctr_of + u[j], -1);
                }
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    const uint32_t p = base + j * kWave + lane_id();
                    o[j] = (p < eb && old[j] == 1 && removes<kTwo>(dead, u[j])) ? make_item(0, u[j])
                                                                               : kNone;
                }
#pragma unroll
                for (int j = 0; j < kBatch; j += 2) wq.push(o[j], o[j + 1]);
            }
            if (lane_id() == owner) {
                if (kTwo && ph == 0) {   // on to the successors of the owner's vertex
                    const int w = item_vertex(item);
                    k = row_off[w];
                    e = row_off[w + 1];
                    ph = 1;
                } else {
                    item = kNone;
                    started = false;
                }
            }
        }
        if (item != kNone) {
            const int nb = min(kBatch, e - k);
            const int* adj = (kTwo && ph) ? col : rcol;
            int* ctr_of = (kTwo && ph) ? cnt + n : cnt;
            int u[kBatch], old[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j)
                if (j < nb) u[j] = adj[k + j];
            if (sched & TRIM_SCHED_JITTER) jitter_nap(((uint64_t)k << 16) ^ item);
#pragma unroll
            for (int j = 0; j < kBatch; ++j)
                if (j < nb) old[j] = add_dev(ctr_of + u[j], -1);
#pragma unroll
            for (int j = 0; j < kBatch; ++j)   // u's last live neighbour on this side
                if (j < nb && old[j] == 1 && removes<kTwo>(dead, u[j])) out[j] = make_item(0, u[j]);
            k += nb;
            if (kTwo && k >= e && ph == 0) {   // on to the successors
                const int w = item_vertex(item);
                k = row_off[w];
                e = row_off[w + 1];
                ph = 1;
            }
            if (k >= e) {
                item = kNone;
                started = false;
                // depth first: go on with one vertex this lane has just
                // removed instead of handing it to the queue
#pragma unroll
                for (int j = 0; j < kBatch; ++j)
                    if (item == kNone && out[j] != kNone) {
                        item = out[j];
                        out[j] = kNone;
                    }
            }
        }
#pragma unroll
        for (int j = 0; j < kBatch; j += 2) wq.push(out[j], out[j + 1]);
        wq.rebalance();
    }
    edges = wave_sum(edges);
    if (lane_id() == 0 && edges) add_dev(worker_edges + blockIdx.x, edges);
    __shared__ int red[16];
    const int qhw = block_max(wq.hw, red);
    if (threadIdx.x == 0) part[kPartQhw * kPartStride + blockIdx.x] = (uint64_t)qhw;
}

struct Ac4Live {
    const int* cnt;
    __device__ __forceinline__ bool operator()(int v) const { return cnt[v] > 0; }
};
struct Ac4TwoLive {
    const int* dead;
    __device__ __forceinline__ bool operator()(int v) const { return dead[v] == 0; }
};

inline int grid_for(long long n, int block, int max_blocks = 1 << 20) {
    long long b = (n + block - 1) / block;
    if (b < 1) b = 1;
    if (b > max_blocks) b = max_blocks;
    return (int)b;
}

template <bool kTwo>
hipError_t ac4_run(const trim_csr_t& g, const Work& w, const LaunchCfg& lc, uint32_t* bitmap,
                   uint64_t* worker_edges, trim_stats_t* stats, const uint32_t* preset) {
    const int n = g.n, P = lc.workers;
    int pack_blocks = 0;
    uint64_t* pieces = reinterpret_cast<uint64_t*>(w.e);   // the three arrays of w.e and w.jp
    const int piece = piece_entries(n, g.m, kStepItems);
    {
        Timed t(lc, kTwo ? "ac4t_init" : "ac4_init");
        hipLaunchKernelGGL(ac4_init<kTwo>, dim3(grid_for(n, 256, 16384)), dim3(256), 0,
                           lc.stream, g.row_off, g.rrow_off, preset, n, w.a, w.d, w.ctr,
                           worker_edges, P, stats);
    }
    if (n > 0) {
        {
            Timed t(lc, kTwo ? "ac4t_first" : "ac4_first");
            hipLaunchKernelGGL(ac4_first<kTwo>, dim3(grid_for(n, 256, lc.cus * 8)), dim3(256), 0,
                               lc.stream, g.rrow_off, g.rcol, g.row_off, g.col, preset, n, w.a,
                               w.d, w.q, w.ctr, worker_edges, P, lc.schedule, pieces, piece);
        }
        {
            Timed t(lc, kTwo ? "ac4t_long" : "ac4_long");
            hipLaunchKernelGGL(ac4_long<kTwo>, dim3(lc.cus * 8), dim3(256), 0, lc.stream,
                               g.rrow_off, g.rcol, g.row_off, g.col, n, w.a, w.d, w.q, w.ctr,
                               worker_edges, P, lc.schedule, pieces, piece);
        }
        {
            Timed t(lc, kTwo ? "ac4t_propagate" : "ac4_propagate");
            hipLaunchKernelGGL(ac4_propagate<kTwo>, dim3(P), dim3(256), 0, lc.stream, g.rrow_off,
                               g.rcol, g.row_off, g.col, n, w.a, w.d, w.q, w.ctr, worker_edges,
                               w.part, lc.schedule, lc.budget, n <= kSpreadN ? kSpreadTickets : kWave);
        }
        Timed t(lc, kTwo ? "ac4t_pack" : "ac4_pack");
        pack_blocks = grid_for(n, 256, lc.cus * 4);
        if (kTwo)
            hipLaunchKernelGGL(pack_bitmap<Ac4TwoLive>, dim3(pack_blocks), dim3(256), 0, lc.stream,
                               Ac4TwoLive{w.d}, n, bitmap, w.part, w.ctr, w.q, w.qwords);
        else
            hipLaunchKernelGGL(pack_bitmap<Ac4Live>, dim3(pack_blocks), dim3(256), 0, lc.stream,
                               Ac4Live{w.a}, n, bitmap, w.part, w.ctr, w.q, w.qwords);
    }
    if (stats)
        hipLaunchKernelGGL(finalize_stats, dim3(1), dim3(1024), 0, lc.stream, n, P, 0, 0,
                           pack_blocks, n > 0 ? P : 0, worker_edges, w.part, w.ctr, stats, 0);
    return hipGetLastError();
}

}  // namespace

hipError_t ac4_csr(const trim_csr_t& g, const Work& w, const LaunchCfg& lc, uint32_t* bitmap,
                   uint64_t* worker_edges, trim_stats_t* stats, const uint32_t* preset) {
    return ac4_run<false>(g, w, lc, bitmap, worker_edges, stats, preset);
}

hipError_t ac4_two_csr(const trim_csr_t& g, const Work& w, const LaunchCfg& lc, uint32_t* bitmap,
                       uint64_t* worker_edges, trim_stats_t* stats) {
    return ac4_run<true>(g, w, lc, bitmap, worker_edges, stats, nullptr);
}

int ac4_max_workers_per_cu(int) {
    int nb = 0, nb2 = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, ac4_propagate<false>, 256, 0) !=
        hipSuccess)
        return 1;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb2, ac4_propagate<true>, 256, 0) ==
            hipSuccess &&
        nb2 < nb)
        nb = nb2;
    return nb < 1 ? 1 : nb;
}

}  // namespace trim
