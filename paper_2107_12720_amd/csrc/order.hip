// order.hip -- per-edge preprocessing (in-degrees, edge sources) and the
// reordering of successor lists by a per-edge key.
//
// AC-6 checks a vertex's successors in list order and keeps the first live
// one (Section 6.1), so reordering the lists changes the traversed edges but
// never the live set.  These kernels are edge-parallel: the edge array is cut
// into tiles of kTileE edges, one workgroup per tile, so a tile's work does
// not depend on how its edges fall into lists (a hub's list spreads over many
// tiles, a tile may hold thousands of short lists).
//
// Source of each edge of a tile: the source of the tile's first edge comes
// from a per-tile table; every later list that starts inside the tile stamps
// its vertex id at its start in LDS, and a prefix maximum fills the gaps.
//
// Reorder: a stable counting sort of every list into kBuckets levels, larger
// keys first.  With P(x, q) = number of edges before position x (over the
// whole edge array) at level q, edge p of list u = [s, e) at level k moves to
//   s + sum_{q<k} (P(e, q) - P(s, q)) + (P(p, k) - P(s, k)).
// P is an exclusive scan of per-tile level counts plus in-tile prefixes kept
// in LDS; a list start or end outside the tile costs one partial count over
// the tile it lies in (at most two per tile).
#include "trim_device.h"
#include "trim_internal.h"

namespace trim {

namespace {

constexpr int kTileT = 256;                 // threads of a tile workgroup
constexpr int kPerT = kTileE / kTileT;      // consecutive edges per thread
constexpr int kTileWaves = kTileT / kWave;
constexpr int kBuckets = 16;
static_assert(kPerT == 16, "in-tile prefixes assume 16 edges per thread");

// Level of edge p: 0 for keys at hi (placed first) .. kBuckets-1 at lo.
struct Levels {
    const float* key;
    float hi, scale;
    __device__ __forceinline__ int of(float x) const {
        const int k = (int)((hi - x) * scale);
        return k < 0 ? 0 : (k >= kBuckets ? kBuckets - 1 : k);
    }
    __device__ __forceinline__ int operator()(long long p) const { return of(key[p]); }
};

// kBuckets counters of 16 bits in four words (a count never exceeds kTileE).
struct Packed {
    uint64_t w[4];
    __device__ __forceinline__ void clear() { w[0] = w[1] = w[2] = w[3] = 0; }
    __device__ __forceinline__ void add_one(int k) {
        const uint64_t inc = 1ull << (16 * (k & 3));
        const int h = k >> 2;
        w[0] += h == 0 ? inc : 0;
        w[1] += h == 1 ? inc : 0;
        w[2] += h == 2 ? inc : 0;
        w[3] += h == 3 ? inc : 0;
    }
    __device__ __forceinline__ int get(int k) const {
        const int h = k >> 2;
        const uint64_t x = h == 0 ? w[0] : h == 1 ? w[1] : h == 2 ? w[2] : w[3];
        return (int)((x >> (16 * (k & 3))) & 0xFFFFu);
    }
};

__device__ __forceinline__ uint64_t shfl_up64(uint64_t x, int d) {
    const unsigned lo = __shfl_up((unsigned)x, d), hi = __shfl_up((unsigned)(x >> 32), d);
    return ((uint64_t)hi << 32) | lo;
}

// Exclusive scan of x over the workgroup; *total gets the sum.  `wtot` holds
// kTileWaves entries of LDS.
__device__ Packed block_exscan(const Packed& x, Packed* wtot, Packed* total) {
    const int l = lane_id(), wv = threadIdx.x / kWave;
    Packed inc = x;
    for (int d = 1; d < kWave; d <<= 1) {
        for (int i = 0; i < 4; ++i) {
            const uint64_t y = shfl_up64(inc.w[i], d);
            if (l >= d) inc.w[i] += y;
        }
    }
    __syncthreads();
    if (l == kWave - 1) wtot[wv] = inc;
    __syncthreads();
    Packed pre, tot;
    pre.clear();
    tot.clear();
    for (int w = 0; w < kTileWaves; ++w)
        for (int i = 0; i < 4; ++i) {
            if (w < wv) pre.w[i] += wtot[w].w[i];
            tot.w[i] += wtot[w].w[i];
        }
    *total = tot;
    Packed ex;
    for (int i = 0; i < 4; ++i) ex.w[i] = inc.w[i] - x.w[i] + pre.w[i];
    return ex;
}

__device__ Packed block_total(const Packed& x, Packed* wtot) {
    Packed tot;
    (void)block_exscan(x, wtot, &tot);
    return tot;
}

// tinfo[t] = (u, row_off[u], row_off[u + 1]) for the source u of edge
// t * kTileE: the list that holds the tile's first edge.
__global__ void tile_first(const int* row_off, int n, int* tinfo) {
    for (int u = blockIdx.x * blockDim.x + threadIdx.x; u < n; u += gridDim.x * blockDim.x) {
        const int b = row_off[u], e = row_off[u + 1];
        for (long long t = (b + (long long)kTileE - 1) / kTileE; t * kTileE < e; ++t) {
            tinfo[3 * t] = u;
            tinfo[3 * t + 1] = b;
            tinfo[3 * t + 2] = e;
        }
    }
}

// owner[j] = source of edge t0 + j for j < len; uf = source of edge t0.
__device__ void tile_owners(const int* row_off, int n, long long t0, int len, int uf, int* owner,
                            int* wmax) {
    for (int j = threadIdx.x; j < kTileE; j += kTileT) owner[j] = -1;
    __syncthreads();
    if (threadIdx.x == 0) owner[0] = uf;
    // lists after uf start after t0 (uf's own list reaches past t0)
    for (int u = uf + 1 + threadIdx.x; u < n; u += kTileT) {
        const long long x = row_off[u] - t0;
        if (x >= len) break;
        atomicMax(owner + x, u);
    }
    __syncthreads();
    const int l = lane_id(), wv = threadIdx.x / kWave;
    int run = -1;
    for (int i = 0; i < kPerT; ++i) run = max(run, owner[threadIdx.x * kPerT + i]);
    int inc = run;
    for (int d = 1; d < kWave; d <<= 1) {
        const int y = __shfl_up(inc, d);
        if (l >= d) inc = max(inc, y);
    }
    if (l == kWave - 1) wmax[wv] = inc;
    __syncthreads();
    int m = __shfl_up(inc, 1);
    if (l == 0) m = -1;
    for (int w = 0; w < wv; ++w) m = max(m, wmax[w]);
    for (int i = 0; i < kPerT; ++i) {
        m = max(m, owner[threadIdx.x * kPerT + i]);
        owner[threadIdx.x * kPerT + i] = m;
    }
    __syncthreads();
}

__device__ __forceinline__ int clamp_vertex(int u, int n) { return u < 0 ? 0 : (u >= n ? n - 1 : u); }

// src[e] = source of edge e.
__global__ __launch_bounds__(kTileT) void tile_sources(const int* row_off, int n, long long m,
                                                       const int* tinfo, int* src) {
    __shared__ int owner[kTileE];
    __shared__ int wmax[kTileWaves];
    const long long T = (m + kTileE - 1) / kTileE;
    for (long long t = blockIdx.x; t < T; t += gridDim.x) {
        const long long t0 = t * kTileE;
        const int len = (int)(m - t0 < kTileE ? m - t0 : kTileE);
        tile_owners(row_off, n, t0, len, clamp_vertex(tinfo[3 * t], n), owner, wmax);
        for (int j = threadIdx.x; j < len; j += kTileT) src[t0 + j] = owner[j];
        __syncthreads();
    }
}

// In-degrees by binning.  Counting at random places of an array of n counters
// is bound by those places: with one copy of the counters per XCD (below) R-MAT
// 24 took 13.7 ms, 51 ns for every thousand of its 2.7 * 10^8 edges, since the
// copies do not fit the L2s and hub counters queue.  Instead the edges' targets
// are dealt into bins of kBinV vertices, 16 bits each, and every bin is counted
// in LDS: 4 + 4 + 2 + 2 bytes of streamed traffic per edge.
//   bin_count    targets per (bin, slice of the edge array);
//   bin_scan     their exclusive scan over the slices, and the bins' totals;
//   bin_scatter  each slice's targets, a tile at a time sorted by bin in LDS, to
//                the slice's places in the bins;
//   bin_degrees  the counters of a bin, or of a part of a large one, in LDS.
// Up to kBinV vertices bin_degrees reads the targets themselves.
constexpr int kBinLog = 15;
constexpr int kBinV = 1 << kBinLog;
constexpr int kBinMax = 1024;               // bins
constexpr int kBinThreads = 512;
constexpr int kBinPer = 32;                 // targets per thread of a tile
constexpr int kBinTile = kBinThreads * kBinPer;
constexpr int kBinSlices = 1024;
constexpr long long kBinChunk = 1 << 21;    // targets one workgroup counts at most
// Fewer edges (in one bin, in several): the plain counters.  One bin, scores of
// R-MAT graphs of 30,000 vertices, plain / binned, us: edge factor 4 36 / 37, 16
// 79 / 47.  Several bins take 60 to 68 us up to 2 * 10^6 edges, trim_mlp_prepare
// plain / binned: 40,000 vertices, 560,000 edges 56 / 68, 640,000 62 / 67; 60,000,
// 600,000 59 / 65, 720,000 67 / 66; 90,000, 540,000 53 / 64, 720,000 63 / 63; 140,000,
// 560,000 57 / 62, 840,000 72 / 61; 260,000, 520,000 71 / 70.  (Just above one bin
// they meet sooner: 33,000 vertices, 400,000 edges 69 / 68.)
constexpr long long kBinMinM = 1 << 16;
constexpr long long kBinsMinM = 11 << 16;
constexpr int kBinCountThreads = 1024;
static_assert(kBinMax == 2 * kBinThreads && kBinMax == kBinCountThreads, "scans of the bins' totals");

struct Bins {
    uint16_t* id;   // m targets, by bin
    int* cnt;       // bins x slices
    int* tot;       // targets of each bin
    int bins, slices;
    int tiles;      // per slice
};

// Exclusive scan over the workgroup; *total gets the sum.  wtot: one word per
// wavefront.
__device__ __forceinline__ int block_scan(int x, int* wtot, int* total) {
    int inc = x;
    for (int d = 1; d < kWave; d <<= 1) {
        const int y = __shfl_up(inc, d);
        if (lane_id() >= d) inc += y;
    }
    const int wv = threadIdx.x / kWave, nw = blockDim.x / kWave;
    __syncthreads();
    if (lane_id() == kWave - 1) wtot[wv] = inc;
    __syncthreads();
    int pre = 0, sum = 0;
    for (int w = 0; w < nw; ++w) {
        if (w < wv) pre += wtot[w];
        sum += wtot[w];
    }
    *total = sum;
    return pre + inc - x;
}

__global__ __launch_bounds__(kBinThreads) void bin_count(const int* col, long long m, Bins b) {
    __shared__ int hist[kBinMax];
    for (int i = threadIdx.x; i < b.bins; i += kBinThreads) hist[i] = 0;
    __syncthreads();
    const long long t0 = (long long)blockIdx.x * b.tiles * kBinTile;
    const long long t1 = min(m, t0 + (long long)b.tiles * kBinTile);
    constexpr int U = 8;
    for (long long e0 = t0 + threadIdx.x; e0 < t1; e0 += U * kBinThreads) {
        int w[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const long long e = e0 + (long long)k * kBinThreads;
            w[k] = e < t1 ? __builtin_nontemporal_load(col + e) : -1;
        }
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (w[k] >= 0) atomicAdd(&hist[w[k] >> kBinLog], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < b.bins; i += kBinThreads)
        b.cnt[(long long)i * b.slices + blockIdx.x] = hist[i];
}

// One workgroup per bin.
__global__ __launch_bounds__(256) void bin_scan(Bins b) {
    __shared__ int wtot[256 / kWave];
    int* c = b.cnt + (long long)blockIdx.x * b.slices;
    constexpr int K = kBinSlices / 256;
    int x[K], sum = 0, total;
    for (int k = 0; k < K; ++k) {
        const int i = threadIdx.x * K + k;
        x[k] = i < b.slices ? c[i] : 0;
        sum += x[k];
    }
    int run = block_scan(sum, wtot, &total);
    for (int k = 0; k < K; ++k) {
        const int i = threadIdx.x * K + k;
        if (i < b.slices) c[i] = run;
        run += x[k];
    }
    if (threadIdx.x == 0) b.tot[blockIdx.x] = total;
}

__global__ __launch_bounds__(kBinThreads) void bin_scatter(const int* col, long long m, Bins b) {
    __shared__ int tile[kBinTile];          // targets sorted by bin
    __shared__ int hist[kBinMax], place[kBinMax], start[kBinMax];
    __shared__ int wtot[kBinThreads / kWave];
    const int t = threadIdx.x;
    int total;
    {   // place[p]: where this slice's next target of bin p goes
        const int x0 = 2 * t < b.bins ? b.tot[2 * t] : 0;
        const int x1 = 2 * t + 1 < b.bins ? b.tot[2 * t + 1] : 0;
        const int pre = block_scan(x0 + x1, wtot, &total);
        if (2 * t < b.bins) place[2 * t] = pre + b.cnt[(long long)(2 * t) * b.slices + blockIdx.x];
        if (2 * t + 1 < b.bins)
            place[2 * t + 1] = pre + x0 + b.cnt[(long long)(2 * t + 1) * b.slices + blockIdx.x];
    }
    for (int j = 0; j < b.tiles; ++j) {
        const long long t0 = ((long long)blockIdx.x * b.tiles + j) * kBinTile;
        if (t0 >= m) break;
        const int len = (int)min(m - t0, (long long)kBinTile);
        __syncthreads();   // the previous tile has been written
        hist[2 * t] = 0;
        hist[2 * t + 1] = 0;
        __syncthreads();
        int w[kBinPer], rank[kBinPer];
#pragma unroll
        for (int k = 0; k < kBinPer; ++k) {
            const int i = k * kBinThreads + t;
            w[k] = i < len ? __builtin_nontemporal_load(col + t0 + i) : -1;
        }
#pragma unroll
        for (int k = 0; k < kBinPer; ++k)
            rank[k] = w[k] >= 0 ? atomicAdd(&hist[w[k] >> kBinLog], 1) : 0;
        __syncthreads();
        const int h0 = hist[2 * t], h1 = hist[2 * t + 1];
        const int pre = block_scan(h0 + h1, wtot, &total);
        start[2 * t] = pre;
        start[2 * t + 1] = pre + h0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kBinPer; ++k)
            if (w[k] >= 0) tile[start[w[k] >> kBinLog] + rank[k]] = w[k];
        __syncthreads();
        for (int i = t; i < len; i += kBinThreads) {
            const int x = tile[i], p = x >> kBinLog;
            b.id[(uint32_t)(place[p] + (i - start[p]))] = (uint16_t)(x & (kBinV - 1));
        }
        __syncthreads();
        if (2 * t < b.bins) place[2 * t] += h0;
        if (2 * t + 1 < b.bins) place[2 * t + 1] += h1;
    }
}

// Workgroup i counts part i of the bins' parts in bin order, a bin of c targets
// having max(1, ceil(c / chunk)).  A bin of one part stores its counters, one of
// several adds them (indeg cleared before).  Without bins (b.id NULL) the one
// bin's targets are col itself.
__global__ __launch_bounds__(kBinCountThreads) void bin_degrees(const int* col, long long m, int n,
                                                                Bins b, long long chunk,
                                                                int* indeg) {
    __shared__ int deg[kBinV];
    __shared__ int wtot[kBinCountThreads / kWave];
    __shared__ long long s_from, s_to;
    __shared__ int s_bin, s_parts;
    const int t = threadIdx.x;
    if (t == 0) s_bin = -1;
    for (int i = t; i < kBinV; i += kBinCountThreads) deg[i] = 0;
    {
        const long long c = t < b.bins ? (b.id ? (long long)b.tot[t] : m) : 0;
        const int parts = t < b.bins ? (c > chunk ? (int)((c + chunk - 1) / chunk) : 1) : 0;
        int total;
        const int before = block_scan((int)c, wtot, &total);   // m < 2^31
        const int p0 = block_scan(parts, wtot, &total);
        const int mine = (int)blockIdx.x - p0;
        if (mine >= 0 && mine < parts) {
            s_bin = t;
            s_parts = parts;
            s_from = before + mine * chunk;
            s_to = min((long long)before + c, s_from + chunk);
        }
    }
    __syncthreads();
    if (s_bin < 0) return;   // the grid covers the largest possible number of parts
    const long long from = s_from, to = s_to;
    if (b.id) {
        // 16-byte loads from the aligned position at or before `from`
        const uint16_t* id = b.id;
        constexpr int U = 4;
        for (long long q = (from & ~7ll) + 8 * t; q < to; q += 8ll * U * kBinCountThreads) {
            uint4 x[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const long long at = q + 8ll * k * kBinCountThreads;
                if (at < to) x[k] = *reinterpret_cast<const uint4*>(id + at);
            }
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const long long at = q + 8ll * k * kBinCountThreads;
                const uint32_t y[4] = {x[k].x, x[k].y, x[k].z, x[k].w};
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (at + j >= from && at + j < to)
                        atomicAdd(&deg[(y[j >> 1] >> (16 * (j & 1))) & (kBinV - 1)], 1);
            }
        }
    } else {
        for (long long e = from + t; e < to; e += kBinCountThreads) atomicAdd(&deg[col[e]], 1);
    }
    __syncthreads();
    const int v0 = s_bin << kBinLog;
    const int len = min(kBinV, n - v0);
    if (s_parts == 1) {
        for (int i = t; i < len; i += kBinCountThreads) indeg[v0 + i] = deg[i];
    } else {
        for (int i = t; i < len; i += kBinCountThreads)
            if (deg[i]) atomicAdd(indeg + v0 + i, deg[i]);
    }
}

// In-degrees with one copy of the counters per XCD: graphs of more than
// kBinMax * kBinV vertices, and contexts whose memory cap leaves no room for the
// bins.  Every XCD counts into its own copy with workgroup-scope
// atomics, which its L2 executes (no other XCD touches that copy), and
// sum_copies adds the copies at the end.  A wave on an unexpected XCD id adds
// to indeg directly with device-wide atomics.
__global__ void in_degrees_xcd(const int* col, long long m, int n, int* copies, int* indeg) {
    const unsigned xcc = __builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20);   // XCC_ID[3:0]
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < m;
         e += (long long)gridDim.x * blockDim.x) {
        const int w = col[e];
        if (copies && xcc < kXcdCopies)
            __hip_atomic_fetch_add(copies + (long long)xcc * n + w, 1, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        else
            atomicAdd(indeg + w, 1);
    }
}

__global__ void sum_copies(const int* copies, int n, int* indeg) {
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        int s = indeg[v];
        for (int x = 0; x < kXcdCopies; ++x) s += copies[(long long)x * n + v];
        indeg[v] = s;
    }
}

__global__ void zero_ints(int* a, long long k) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < k;
         i += (long long)gridDim.x * blockDim.x)
        a[i] = 0;
}

// Out-degrees in two bytes (kDegMax: that or more), for edge_keys.
constexpr uint32_t kDegMax = 65535;
__global__ void short_degrees(const int* row_off, int n, uint16_t* deg) {
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x)
        deg[v] = (uint16_t)min((uint32_t)(row_off[v + 1] - row_off[v]), kDegMax);
}

// Keys for the reference orders: 0 = log1p(outdeg w) (larger first), 1 = a hash
// of (seed, e) (a random order).
__global__ void edge_keys(const int* row_off, const int* col, long long m, int kind, uint64_t seed,
                          float* key) {
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < m;
         e += gridDim.x * (long long)blockDim.x) {
        if (kind == 0) {
            const int w = col[e];
            key[e] = log1pf((float)(row_off[w + 1] - row_off[w]));
        } else {
            key[e] = (float)(mix64(seed ^ (uint64_t)e) >> 40) * (1.f / 16777216.f);
        }
    }
}

// Kind 0 for many edges.  The gather of the targets' degrees bounds it (a line
// from beyond the L2 for every one they miss): with the two offsets of every
// target it took 1.96 ms on R-MAT 24, from the table of two bytes a vertex, of
// which the L2s hold more, 1.75 ms with the table's making.  Targets and keys
// pass by the caches, which the table needs; graphs whose keys the ordering
// would find there still are taken by edge_keys.
__global__ void edge_keys_table(const int* row_off, const int* col, const uint16_t* deg,
                                long long m, float* key) {
    constexpr int U = 4;
    const long long stride = gridDim.x * (long long)blockDim.x;
    for (long long e0 = blockIdx.x * (long long)blockDim.x + threadIdx.x; e0 < m;
         e0 += U * stride) {
        int w[U], d[U];
#pragma unroll
        for (int k = 0; k < U; ++k)
            w[k] = __builtin_nontemporal_load(col + min(e0 + k * stride, m - 1));
#pragma unroll
        for (int k = 0; k < U; ++k) d[k] = (int)deg[w[k]];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if (d[k] == (int)kDegMax) d[k] = row_off[w[k] + 1] - row_off[w[k]];
            if (e0 + k * stride < m)
                __builtin_nontemporal_store(log1pf((float)d[k]), key + e0 + k * stride);
        }
    }
}

// tcnt[t][q] = edges of tile t at level q.
__global__ __launch_bounds__(kTileT) void order_count(long long m, Levels level, int* tcnt) {
    __shared__ Packed wtot[kTileWaves];
    const long long T = (m + kTileE - 1) / kTileE;
    for (long long t = blockIdx.x; t < T; t += gridDim.x) {
        const long long t0 = t * kTileE;
        const int len = (int)(m - t0 < kTileE ? m - t0 : kTileE);
        Packed c;
        c.clear();
        for (int j = threadIdx.x; j < len; j += kTileT) c.add_one(level(t0 + j));
        const Packed tot = block_total(c, wtot);
        if (threadIdx.x < kBuckets) tcnt[t * kBuckets + threadIdx.x] = tot.get(threadIdx.x);
        __syncthreads();
    }
}

// Exclusive scan of the tile counts, in place: tcnt[t][q] <- the sum of
// tcnt[t'][q] over t' < t, for t = 0..T (row T gets the totals; its input is
// ignored).  Rows are taken kScanRows at a time: scan_reduce sums each chunk,
// scan_rows scans the chunk sums (one workgroup), scan_apply rescans each
// chunk from its offset.
constexpr int kScanRows = 64;
constexpr int kScanT = 1024;

__device__ __forceinline__ int row_val(const int* a, long long rows_in, long long r, int q) {
    return r < rows_in ? a[r * kBuckets + q] : 0;
}

// 64 threads: thread (g, q) covers rows g*16 .. g*16+15 of the chunk, level q.
__global__ __launch_bounds__(kWave) void scan_reduce(const int* tcnt, long long T, int* csum) {
    __shared__ int part[4][kBuckets];
    const int q = threadIdx.x & 15, g = threadIdx.x >> 4;
    const long long r0 = blockIdx.x * (long long)kScanRows + g * 16;
    int acc = 0;
    for (int i = 0; i < 16; ++i) acc += row_val(tcnt, T, r0 + i, q);
    part[g][q] = acc;
    __syncthreads();
    if (g == 0) csum[blockIdx.x * kBuckets + q] = part[0][q] + part[1][q] + part[2][q] + part[3][q];
}

// One workgroup: the same exclusive scan over `rows` rows of a (the input of
// row `rows_in` and later is taken as 0).
__global__ __launch_bounds__(kScanT) void scan_rows(int* a, long long rows_in, long long rows) {
    __shared__ int wsum[kScanT / kWave][kBuckets];
    const int l = lane_id(), wv = threadIdx.x / kWave;
    const long long per = (rows + kScanT - 1) / kScanT;
    const long long r0 = threadIdx.x * per;
    const long long r1 = r0 + per < rows ? r0 + per : rows;
    int acc[kBuckets];
    for (int q = 0; q < kBuckets; ++q) acc[q] = 0;
    for (long long r = r0; r < r1; ++r)
        for (int q = 0; q < kBuckets; ++q) acc[q] += row_val(a, rows_in, r, q);
    int ex[kBuckets];
    for (int q = 0; q < kBuckets; ++q) {
        int inc = acc[q];
        for (int d = 1; d < kWave; d <<= 1) {
            const int y = __shfl_up(inc, d);
            if (l >= d) inc += y;
        }
        if (l == kWave - 1) wsum[wv][q] = inc;
        ex[q] = inc - acc[q];
    }
    __syncthreads();
    for (int w = 0; w < wv; ++w)
        for (int q = 0; q < kBuckets; ++q) ex[q] += wsum[w][q];
    for (long long r = r0; r < r1; ++r)
        for (int q = 0; q < kBuckets; ++q) {
            const int c = row_val(a, rows_in, r, q);
            a[r * kBuckets + q] = ex[q];
            ex[q] += c;
        }
}

__global__ __launch_bounds__(kWave) void scan_apply(int* tcnt, long long T, const int* csum) {
    __shared__ int part[4][kBuckets];
    const int q = threadIdx.x & 15, g = threadIdx.x >> 4;
    const long long r0 = blockIdx.x * (long long)kScanRows + g * 16;
    int v[16];
    int acc = 0;
    for (int i = 0; i < 16; ++i) {
        v[i] = row_val(tcnt, T, r0 + i, q);
        acc += v[i];
    }
    part[g][q] = acc;
    __syncthreads();
    int run = csum[blockIdx.x * kBuckets + q];
    for (int h = 0; h < g; ++h) run += part[h][q];
    for (int i = 0; i < 16; ++i) {
        if (r0 + i > T) break;
        tcnt[(r0 + i) * kBuckets + q] = run;
        run += v[i];
    }
}

// Edge j of the tile (position t0 + j) of list [s, e) at level k goes to
//   s + Lb(e, k) - Lb(s, k + 1) + (Lb(j, k + 1) - Lb(j, k)),
// where Lb(x, k) counts the tile's edges before t0 + x with level < k (the
// tile's scan entry cancels out of every difference).  One lane per edge: the
// tile is 64 chunks of 64 edges, and for every chunk the workgroup keeps, in
// LDS, the lane masks of "level < k" for k = 0..16 (from ballots) and the
// counts of such edges in the chunks before it, so Lb at any in-tile position
// is one mask, one count and a popcount.  A list's bounds come from the tile
// alone: starts of lists after the first are stamped as bits, the first list
// starts at row_off of the tile's first source, and the last one ends where
// the list holding the tile's last edge ends.  A start before the tile or an
// end after it uses counts over the part of the list outside the tile.
//
// What bounds it: vector instructions (196 a chunk of 64 edges, 1.34 ms for the
// 2.7 * 10^8 edges of R-MAT 24), and waiting while few workgroups fit the LDS.
// 1.75 ms there, 2.51 with keys and levels passed through LDS one load at a time,
// masks stored by single lanes and every edge written to its own place.
constexpr int kChunks = kTileE / kWave;             // 64
constexpr int kChunksPerWave = kChunks / kTileWaves;   // 16
static_assert(kChunks == kWave, "chunk prefixes are scanned one chunk per lane");

__device__ __forceinline__ uint64_t lanes_lt(int l) { return (1ull << l) - 1ull; }

__global__ __launch_bounds__(kTileT, 5) void order_place(const int* row_off, int n, long long m,
                                                      const int* col, Levels level,
                                                      const int* tinfo, const int* tpre,
                                                      int* col_out) {
    __shared__ int out[kTileE];                         // the lists that lie in the tile
    __shared__ uint64_t fm[kChunks];                    // bit = a list other than the first starts
    __shared__ uint64_t cm[kChunks][kBuckets + 1];      // lanes of the chunk with level < k
    __shared__ int cpre[kChunks + 1][kBuckets + 1];     // edges of earlier chunks with level < k
    __shared__ int lastst[kChunks], firstst[kChunks];   // last start before / first after the chunk
    __shared__ int wpart[kTileWaves][kBuckets];
    __shared__ int lout[2][kBuckets];
    __shared__ int loutc[2][kBuckets + 1];              // cumulative lout: level < k
    const int l = lane_id(), wv = threadIdx.x / kWave;
    const long long T = (m + kTileE - 1) / kTileE;
    for (long long t = blockIdx.x; t < T; t += gridDim.x) {
        const long long t0 = t * kTileE;
        const int len = (int)(m - t0 < kTileE ? m - t0 : kTileE);
        const long long t1 = t0 + len;
        // the wave's chunks, all their keys in flight; four bits a level
        float key[kChunksPerWave];
#pragma unroll
        for (int i = 0; i < kChunksPerWave; ++i)
            key[i] = level.key[t0 + min((wv * kChunksPerWave + i) * kWave + l, len - 1)];
        uint64_t lvl = 0;
#pragma unroll
        for (int i = 0; i < kChunksPerWave; ++i) lvl |= (uint64_t)level.of(key[i]) << (4 * i);
        if (threadIdx.x < kChunks) fm[threadIdx.x] = 0;
        const int uf = clamp_vertex(tinfo[3 * t], n);
        const long long sf = tinfo[3 * t + 1];
        long long el = t1;   // end of the list that holds edge t1 - 1
        if (t + 1 < T && tinfo[3 * t + 4] < t1) el = tinfo[3 * t + 5];
        __syncthreads();
        for (int u = uf + 1 + threadIdx.x; u < n; u += kTileT) {
            const long long x = row_off[u] - t0;
            if (x >= len) break;
            atomicOr((unsigned long long*)&fm[x >> 6], 1ull << (x & 63));
        }
        // lane k <= 16 works out "level < k" of a chunk from the ballots of the
        // levels' four bits (a compare, two moves and a store by one lane for
        // every k kept the LDS and the vector units busier)
        static_assert(kBuckets == 16, "levels of four bits");
#pragma unroll 1
        for (int i = 0; i < kChunksPerWave; ++i) {
            const int c = wv * kChunksPerWave + i;
            const int k = (int)(lvl >> (4 * i)) & (kBuckets - 1);
            const int left = len - c * kWave;
            uint64_t eq = left >= kWave ? ~0ull : left > 0 ? lanes_lt(left) : 0ull;
            uint64_t below = l == kBuckets ? eq : 0ull;
#pragma unroll
            for (int b = 3; b >= 0; --b) {
                const uint64_t plane = ballot((k >> b) & 1);
                const uint64_t mine = (l >> b) & 1 ? ~0ull : 0ull;
                below |= eq & mine & ~plane;
                eq &= ~(plane ^ mine);
            }
            if (l == kBuckets) below = left >= kWave ? ~0ull : left > 0 ? lanes_lt(left) : 0ull;
            if (l <= kBuckets) cm[c][l] = below;
        }
        __syncthreads();
        for (int k = wv; k <= kBuckets; k += kTileWaves) {   // lane = chunk
            const int cnt = popc(cm[l][k]);
            int inc = cnt;
            for (int d = 1; d < kWave; d <<= 1) {
                const int y = __shfl_up(inc, d);
                if (l >= d) inc += y;
            }
            cpre[l][k] = inc - cnt;
            if (l == kWave - 1) cpre[kChunks][k] = inc;
        }
        if (wv == 0) {   // lane = chunk
            const uint64_t f = fm[l];
            int lastv = f ? l * kWave + 63 - __clzll((long long)f) : 0;
            int firstv = f ? l * kWave + __ffsll((unsigned long long)f) - 1 : len;
            for (int d = 1; d < kWave; d <<= 1) {
                const int yl = __shfl_up(lastv, d), yf = __shfl_down(firstv, d);
                if (l >= d) lastv = max(lastv, yl);
                if (l + d < kWave) firstv = min(firstv, yf);
            }
            int ls = __shfl_up(lastv, 1), fs = __shfl_down(firstv, 1);
            if (l == 0) ls = 0;
            if (l == kWave - 1) fs = len;
            lastst[l] = ls;
            firstst[l] = fs;
        }
        __syncthreads();
        // The first list's start before the tile, the last list's end after
        // it: counted over the shorter of "from that position's tile start"
        // (with that tile's scan entry) or "between it and this tile".
        for (int side = 0; side < 2; ++side) {
            const long long x = side == 0 ? sf : el;
            if (side == 0 ? x >= t0 : x <= t1) continue;   // uniform over the workgroup
            const long long tx = x / kTileE;
            const long long fwd = x - tx * kTileE, near = side == 0 ? t0 - x : x - t1;
            const bool use_near = near < fwd;
            const long long p0 = use_near ? (side == 0 ? x : t1) : tx * kTileE;
            const long long p1 = use_near ? (side == 0 ? t0 : x) : x;
            int cq[kBuckets];
            for (int q = 0; q < kBuckets; ++q) cq[q] = 0;
            for (long long p = p0 + wv * kWave; p < p1; p += kTileT) {
                const int k = p + l < p1 ? level(p + l) : -1;
                for (int q = 0; q < kBuckets; ++q) cq[q] += popc(ballot(k == q));
            }
            if (l == 0)
                for (int q = 0; q < kBuckets; ++q) wpart[wv][q] = cq[q];
            __syncthreads();
            if (threadIdx.x < kBuckets) {
                const int q = threadIdx.x;
                int part = 0;
                for (int w = 0; w < kTileWaves; ++w) part += wpart[w][q];
                int v;
                if (!use_near) v = tpre[tx * kBuckets + q] - tpre[t * kBuckets + q] + part;
                else if (side == 0) v = -part;
                else v = cpre[kChunks][q + 1] - cpre[kChunks][q] + part;
                lout[side][q] = v;
            }
            __syncthreads();
            if (threadIdx.x <= kBuckets) {
                int acc = 0;
                for (int q = 0; q < (int)threadIdx.x; ++q) acc += lout[side][q];
                loutc[side][threadIdx.x] = acc;
            }
        }
        __syncthreads();
        auto Lb = [&](int x, int kk) {
            if (x >= len) return cpre[kChunks][kk];
            const int c = x >> 6;
            return cpre[c][kk] + popc(cm[c][kk] & lanes_lt(x & 63));
        };
        // lists that lie in the tile are put together in LDS and written in order;
        // the others' edges go where they belong one by one
        const int srel = (int)(sf - t0), erel = (int)(el - t0);
        const int from = sf < t0 ? (fm[0] ? __ffsll((unsigned long long)fm[0]) - 1 : firstst[0]) : 0;
        const int to = el > t1 ? (fm[kChunks - 1] ? kTileE - 1 - __clzll((long long)fm[kChunks - 1])
                                                  : lastst[kChunks - 1])
                               : len;
#pragma unroll 4
        for (int i = 0; i < kChunksPerWave; ++i) {
            const int c = wv * kChunksPerWave + i;
            const int j = c * kWave + l;
            const int w = col[t0 + min(j, len - 1)];
            if (j < len) {
                const int k = (int)(lvl >> (4 * i)) & (kBuckets - 1);
                const uint64_t f = fm[c];
                const uint64_t upto = f & (2 * (1ull << l) - 1), after = f ^ upto;
                const int s = upto ? c * kWave + 63 - __clzll((long long)upto) : lastst[c];
                const int e = after ? c * kWave + __ffsll((unsigned long long)after) - 1 : firstst[c];
                // positions from the tile's start (edges are numbered in 31 bits)
                const int sr = s == 0 ? srel : s, er = e == len ? erel : e;
                const int lbe = er > len ? loutc[1][k] : Lb(e, k);
                const int lbs = sr < 0 ? loutc[0][k + 1] : Lb(s, k + 1);
                const uint64_t same = cm[c][k + 1] & ~cm[c][k] & lanes_lt(l);
                const int pos = sr + lbe - lbs + cpre[c][k + 1] - cpre[c][k] + popc(same);
                if (pos >= sr && pos < er) {
                    if (j >= from && j < to)
                        out[pos] = w;
                    else
                        col_out[t0 + pos] = w;
                }
            }
        }
        __syncthreads();
        for (int j = from + threadIdx.x; j < to; j += kTileT) col_out[t0 + j] = out[j];
        __syncthreads();
    }
}

inline int grid_for(long long n, int block, int max_blocks) {
    long long b = (n + block - 1) / block;
    if (b < 1) b = 1;
    if (b > max_blocks) b = max_blocks;
    return (int)b;
}

inline int tile_grid(long long m) {
    const long long T = (m + kTileE - 1) / kTileE;
    return (int)(T < (1 << 20) ? (T < 1 ? 1 : T) : (1 << 20));
}

}  // namespace

bool bin_degrees_ok(long long n, long long m) {
    return n <= (long long)kBinMax * kBinV && m >= (n <= kBinV ? kBinMinM : kBinsMinM);
}

// Bytes of scratch: the binned targets (whole 16-byte words) and the counts.
// None up to kBinV vertices.
size_t bin_scratch_bytes(long long n, long long m) {
    if (n <= kBinV) return 0;
    const long long bins = (n + kBinV - 1) >> kBinLog;
    return (size_t)((m * 2 + 15) / 16 * 16 + (bins * kBinSlices + bins) * 4);
}

static void in_degrees_binned(const int* col, int n, long long m, int* indeg, void* scratch,
                              hipStream_t s) {
    Bins b{};
    b.bins = (int)(((long long)n + kBinV - 1) >> kBinLog);
    long long chunk = kBinChunk;
    if (b.bins > 1) {
        b.id = reinterpret_cast<uint16_t*>(scratch);
        b.cnt = reinterpret_cast<int*>(reinterpret_cast<char*>(scratch) + (m * 2 + 15) / 16 * 16);
        const long long tiles = (m + kBinTile - 1) / kBinTile;
        b.tiles = (int)((tiles + kBinSlices - 1) / kBinSlices);
        b.slices = (int)((tiles + b.tiles - 1) / b.tiles);
        b.tot = b.cnt + (long long)b.bins * b.slices;
        hipLaunchKernelGGL(bin_count, dim3(b.slices), dim3(kBinThreads), 0, s, col, m, b);
        hipLaunchKernelGGL(bin_scan, dim3(b.bins), dim3(256), 0, s, b);
        hipLaunchKernelGGL(bin_scatter, dim3(b.slices), dim3(kBinThreads), 0, s, col, m, b);
        // parts enough for the device, but no more adds than four a target
        while (chunk > 4 * kBinV && m / chunk + b.bins < 512) chunk >>= 1;
    } else {
        chunk = 4ll * n > 16384 ? 4ll * n : 16384;
    }
    const long long parts = b.bins + (m + chunk - 1) / chunk;
    hipLaunchKernelGGL(bin_degrees, dim3((unsigned)parts), dim3(kBinCountThreads), 0, s, col, m, n,
                       b, chunk, indeg);
}

hipError_t mlp_prepare(const int* row_off, const int* col, int n, long long m, int* indeg,
                       int* src, int* tinfo, int* copies, void* bins, hipStream_t s) {
    hipLaunchKernelGGL(zero_ints, dim3(grid_for(n, 256, 8192)), dim3(256), 0, s, indeg,
                       (long long)n);
    if (m > 0) {
        if (!copies && bin_degrees_ok(n, m)) {
            in_degrees_binned(col, n, m, indeg, bins, s);
        } else {
            if (copies)
                hipLaunchKernelGGL(zero_ints, dim3(grid_for((long long)n * kXcdCopies, 256, 16384)),
                                   dim3(256), 0, s, copies, (long long)n * kXcdCopies);
            hipLaunchKernelGGL(in_degrees_xcd, dim3(grid_for(m, 256, 16384)), dim3(256), 0, s, col,
                               m, n, copies, indeg);
            if (copies)
                hipLaunchKernelGGL(sum_copies, dim3(grid_for(n, 256, 16384)), dim3(256), 0, s,
                                   copies, n, indeg);
        }
        hipLaunchKernelGGL(tile_first, dim3(grid_for(n, 256, 16384)), dim3(256), 0, s, row_off, n,
                           tinfo);
        hipLaunchKernelGGL(tile_sources, dim3(tile_grid(m)), dim3(kTileT), 0, s, row_off, n, m,
                           tinfo, src);
    }
    return hipGetLastError();
}

hipError_t edge_keys_launch(const int* row_off, const int* col, int n, long long m, int kind,
                            uint64_t seed, float* key, uint16_t* deg, hipStream_t s) {
    if (m > 0) {
        if (kind == 0 && deg) {
            hipLaunchKernelGGL(short_degrees, dim3(grid_for(n, 256, 16384)), dim3(256), 0, s,
                               row_off, n, deg);
            hipLaunchKernelGGL(edge_keys_table, dim3(grid_for((m + 3) / 4, 256, 16384)), dim3(256),
                               0, s, row_off, col, deg, m, key);
        } else {
            hipLaunchKernelGGL(edge_keys, dim3(grid_for(m, 256, 16384)), dim3(256), 0, s, row_off,
                               col, m, kind, seed, key);
        }
    }
    return hipGetLastError();
}

hipError_t order_launch(const int* row_off, const int* col, int n, long long m, const float* key,
                        float lo, float hi, int* col_out, int* tinfo, int* tcnt,
                        hipStream_t s) {
    if (m <= 0) return hipGetLastError();
    const Levels lv{key, hi, hi > lo ? (float)kBuckets / (hi - lo) : 0.f};
    const long long T = (m + kTileE - 1) / kTileE;
    hipLaunchKernelGGL(tile_first, dim3(grid_for(n, 256, 16384)), dim3(256), 0, s, row_off, n,
                       tinfo);
    hipLaunchKernelGGL(order_count, dim3(tile_grid(m)), dim3(kTileT), 0, s, m, lv, tcnt);
    const long long B = (T + 1 + kScanRows - 1) / kScanRows;   // chunks of rows 0..T
    int* csum = tcnt + (T + 1) * kBuckets;
    hipLaunchKernelGGL(scan_reduce, dim3((unsigned)B), dim3(kWave), 0, s, tcnt, T, csum);
    hipLaunchKernelGGL(scan_rows, dim3(1), dim3(kScanT), 0, s, csum, B, B);
    hipLaunchKernelGGL(scan_apply, dim3((unsigned)B), dim3(kWave), 0, s, tcnt, T, csum);
    hipLaunchKernelGGL(order_place, dim3(tile_grid(m)), dim3(kTileT), 0, s, row_off, n, m, col,
                       lv, tinfo, tcnt, col_out);
    return hipGetLastError();
}

}  // namespace trim
