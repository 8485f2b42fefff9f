// watch_rounds.h -- what the device-wide rounds over watched supports share, one-
// sided (ac6_watch.h) and two-sided (ac6_two_watch.h).
//
// A vertex is handed back when a round over the vertices finds its support's
// status bit set.  Filters: a support that was live before round r - 1 is
// removed before round r iff round r - 1 removed it.  While those removals are
// few, a round tests a hashed filter of them in LDS and looks at the statuses
// only on a hit: in the rounds of one launch, where a status has to be read past
// the L2 (it may have changed since the line was cached), and, from the second
// round on, for graphs whose bitmap the L2s don't hold.
#pragma once
#include "trim_device.h"
#include "trim_internal.h"

namespace trim {

namespace {

constexpr int kSupFirst = 1 << 29;      // sup[]: the support is the first successor
constexpr int kSupMask = kSupFirst - 1;
// Rounds in launches of their own, which read statuses through clean caches; small
// graphs leave all to the tail (a launch that has nothing to do takes 2 us).
constexpr int round_launches(int n) { return n <= (1 << 17) ? 0 : n <= (1 << 18) ? 1 : 4; }
constexpr int kWatchRounds = 64;
// Rounds before the vertices left are registered in lists.  A round of the tail
// takes 6 to 9 us up to 2^20 vertices and 19 at 2^22, a phase over lists 5 (one
// removal) to 60 (thousands), registering 50 and 170.  Core+tail graphs of mean
// degree 30 and 2^20 vertices (some 60 rounds) take 2.4 ms with 64 rounds, with
// lists alone 3.8 (a limit of 40 cost 0.5 more).  Rounds that remove few end
// sooner: kNarrowRounds.
constexpr int watch_rounds(int n) {
    const int r = n <= (1 << 21) ? kWatchRounds : (int)(((long long)kWatchRounds << 21) / n);
    return r > 8 ? r : 8;
}
// Rounds of the tail that removed so few vertices that a phase over lists would
// have taken them sooner, of which so many register the rest: a round costs the
// same whatever it removes.  One path of 66 levels (every edge twice) among 2^17
// vertices 437 -> 328 us a call (lists from the start 353), 2^20 685 -> 498 (458),
// 2^22 1,225 -> 1,061 (907); five of them 454 -> 455 (518), 687 -> 547 (653), 1,259
// -> 1,107 (1,101).  With 12 rounds 2 to 3 % more, with 32 removals at 2^17 vertices
// uniform graphs of mean degree 1.1 lose 5 %, with 64 at 2^22 50 paths 3 %.
constexpr int kNarrowRounds = 8;
constexpr int narrow_removals(int n) { return n >> 17 > 1 ? n >> 17 : 1; }
constexpr int kSweepFlight = 8;         // vertices per lane in flight
constexpr int kRoundFlight = 8;
constexpr int kRoundThreads = 512;      // the tail: one workgroup per CU
constexpr int kTailPer = 2;

// Workgroups of the forest collapse over watched supports: one per 1,024 vertices
// (a bare path of 10^5: 121 us a call, with one per 8,192 359), at most one
// per CU.
inline int watch_jump_blocks(long long n, int cus) {
    const long long b = n / 1024;
    return (int)(b < 8 ? 8 : b > cus ? cus : b);
}

// Removals of three rounds in rotation, hashed into 2^log bits each.  (Small
// enough for every workgroup to stage a round's in a microsecond or two, and
// large enough that setting its bits does not queue at a few lines: with a
// second one of 2^12 bits, 30,000 removals a round cost 20 us.)
struct WatchFilter {
    static constexpr int kMaxWords = 1 << (18 - 5);
    uint32_t* f;
    int log;
    // graphs whose statuses cost more to read get a filter of more removals
    __host__ __device__ static constexpr int log_for(int n) { return n <= (1 << 20) ? 16 : 18; }
    __device__ __forceinline__ int words() const { return 1 << (log - 5); }
    __device__ __forceinline__ uint32_t* slot(int r) const { return f + (r % 3) * words(); }
    __device__ __forceinline__ uint32_t hash(int v) const {
        return ((uint32_t)v * 0x9E3779B1u) >> (32 - log);
    }
    __device__ __forceinline__ void add(int r, int v) const {
        const uint32_t h = hash(v);
        atomicOr(slot(r) + (h >> 5), 1u << (h & 31));
    }
    // whether a filter of that many removals answers most tests
    __device__ __forceinline__ bool useful(int removed) const { return removed <= words() * 8; }
};

struct WatchState {
    const int* row_off;
    const int* col;
    int n;
    int* sup;         // support and kSupFirst, or -1: removed
    uint64_t* rec;
    uint32_t* dead;
    WatchFilter flt;
    int* ctr;
    uint64_t* worker_edges;
    int P;
    int sched;
    int r1;           // the first round of the propagation: 1, after R counted ones R + 1
    bool forest;
};

__device__ __forceinline__ int* rec_pos(uint64_t* rec, int v) {
    return reinterpret_cast<int*>(rec + v) + 1;
}
__device__ __forceinline__ bool status_bit(const uint32_t* bm, int v) {
    return __builtin_amdgcn_ubfe(bm[v >> 5], (unsigned)v, 1) != 0;
}

// Removals whose supporters round r has to find: the round's before, and in
// front of the first those of the forest collapse or, without it, of the sweep
// or the last counted round.
__device__ __forceinline__ int removed_before(const WatchState& a, int r) {
    return r == a.r1 && a.forest ? ld_dev(a.ctr + kJKilled)
                                 : ld_dev(a.ctr + kHyDead0 + (r - 1) % 3);
}

struct WatchSums {
    uint64_t edges = 0;
    uint32_t closes = 0, joins = 0, visited = 0;
};

// The scan of v resumed after its removed support s: true with the position
// and the target, or false.  kFresh: statuses are read past the L2.
template <bool kFresh>
__device__ __forceinline__ bool watch_scan(const WatchState& a, int v, int s, int& pos, int& to,
                                           uint64_t& edges) {
    constexpr int K = 4;
    const int e = a.row_off[v + 1];
    const int p0 = ((s & kSupFirst) ? a.row_off[v] : *rec_pos(a.rec, v)) + 1;
    if (a.sched & TRIM_SCHED_JITTER) jitter_nap((uint64_t)v);
    for (uint32_t p = p0; p < (uint32_t)e; p += K) {
        int w[K];
        uint32_t x[K];
#pragma unroll
        for (int j = 0; j < K; ++j) w[j] = a.col[step_index(p, j, e)];
#pragma unroll
        for (int j = 0; j < K; ++j)
            x[j] = kFresh ? ld_dev(a.dead + (w[j] >> 5)) : a.dead[w[j] >> 5];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            if (p + j >= (uint32_t)e || ((x[j] >> (w[j] & 31)) & 1u)) continue;
            pos = (int)(p + j);
            edges += (uint64_t)(pos - p0 + 1);
            to = w[j];
            return true;
        }
    }
    edges += (uint64_t)(e - p0);
    return false;
}

// The wavefront's hand-backs among the U vertices of each lane, put side by side
// in its part of `found` (U * 64 entries): their scans, chains of four dependent
// loads, then run 64 at a time instead of a few lanes' at a time, U times.
// A lane polls runs of four vertices, the supports of each from one 16-byte load;
// vertex k is number k & 3 of run q[k >> 2].
template <int U>
__device__ __forceinline__ int watch_found(const bool (&back)[U], const int (&q)[U / 4],
                                           int* found) {
    int cnt = 0;
#pragma unroll
    for (int k = 0; k < U; ++k) {
        const uint64_t mask = ballot(back[k]);
        if (back[k]) found[cnt + popc(mask & lanes_below())] =
                4 * q[k >> 2] + (k & 3);
        cnt += popc(mask);
    }
    __builtin_amdgcn_wave_barrier();
    return cnt;
}

// What a round leaves for the next: the filter slot of round r + 1 cleared (it
// was last read by round r - 1), the counter after it, the round's removals.
__device__ __forceinline__ void watch_round_end(const WatchState& a, int r, uint32_t removed,
                                                uint64_t* red) {
    uint32_t* f = a.flt.slot(r + 1);
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < a.flt.words();
         i += gridDim.x * blockDim.x)
        st_dev(f + i, 0u);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st_dev(a.ctr + kHyDead0 + (r + 1) % 3, 0);
        add_dev(a.ctr + kLvPhases, 1);
    }
    const uint64_t sum = block_sum(removed, red);
    if (threadIdx.x == 0 && sum) add_dev(a.ctr + kHyDead0 + r % 3, (int)sum);
}

__device__ __forceinline__ void watch_sums(const WatchState& a, WatchSums& t, uint64_t* red) {
    const uint64_t e = block_sum(t.edges, red);
    const uint64_t x[3] = {block_sum(t.closes, red), block_sum(t.joins, red),
                           block_sum(t.visited, red)};
    if (threadIdx.x != 0) return;
    if (e) add_dev(a.worker_edges + (blockIdx.x % a.P), e);
    for (int i = 0; i < 3; ++i)
        if (x[i]) add_dev(reinterpret_cast<uint64_t*>(a.ctr + kWatchCloses) + i, x[i]);
}

// The filter of round r - 1, which removed `removed`, into LDS; NULL when it is
// of no use.
template <int kThreads, bool kFresh>
__device__ __forceinline__ const uint32_t* watch_stage(const WatchState& a, int r, int removed,
                                                       uint32_t* sflt) {
    const bool use = a.flt.useful(removed);
    if (use) {
        // 8-byte pieces, four in flight: a load past the L2 takes 1 us
        constexpr int K = 4;
        const uint64_t* f = reinterpret_cast<const uint64_t*>(a.flt.slot(r - 1));
        uint64_t* to = reinterpret_cast<uint64_t*>(sflt);
        const int words = a.flt.words() / 2;
        for (int base = threadIdx.x; base < words; base += K * kThreads) {
            uint64_t x[K];
#pragma unroll
            for (int i = 0; i < K; ++i) {
                const uint64_t* p = f + min(base + i * kThreads, words - 1);
                x[i] = kFresh ? ld_dev(p) : *p;
            }
#pragma unroll
            for (int i = 0; i < K; ++i)
                if (base + i * kThreads < words) to[base + i * kThreads] = x[i];
        }
    }
    __syncthreads();
    return use ? sflt : nullptr;
}

}  // namespace

}  // namespace trim
