// group_lists.h -- AC-6 propagation over support lists by one workgroup or one
// wavefront (Section 6.2): graphs too large for watch.h (batch.hip), and what a
// deep, narrow graph has left after many passes over all its supports.
//
// Phases: each takes the list the previous one built.  CLOSE(x) exchanges both
// heads of x with kDead and walks the two lists it got back: every S_last member
// is removed with x (a CLOSE item for the next phase), every S_more member
// resumes its scan after its old support (a RESCAN item).  RESCAN(x) resumes x's
// scan and closes x on the spot if it finds nothing.  A group barrier ends a
// phase; the graph is done when a phase builds an empty list.  A phase of one
// removal takes about 1.8 us, whatever the size of the graph.
//
// Every word of a graph's state is touched by its own group only, so
// workgroup-scope accesses keep it coherent.
#pragma once
#include "trim_device.h"
#include "ac6_support.h"

namespace trim {

namespace {

constexpr int kWG = __HIP_MEMORY_SCOPE_WORKGROUP;

// Per-lane totals of the graphs trimmed so far.
struct WatchTotals {
    uint64_t edges = 0, sweep = 0, deg = 0;
    uint32_t closes = 0, joins = 0, visited = 0, forest = 0, live = 0;
};

enum : uint32_t { kOwnClose = 0, kOwnRescan = 1 };

// LDS of a group of up to kWaves wavefronts: items staged per wavefront before
// one reservation, and the length of the list being built.
constexpr int kListStage = 128;
template <int kWaves>
struct ListStage {
    uint32_t item[kWaves][kListStage];
    int n[kWaves];
    int cnt;
};

// Device memory of a graph of n vertices (its own ids).
struct ListArrays {
    int* head;       // 2n
    uint64_t* rec;   // n
    uint32_t* l0;    // n
    uint32_t* l1;    // n
};

template <class View, bool kWaveGroup>
struct GroupLists {
    static constexpr int kWaves = kWaveGroup ? 1 : 1024 / kWave;
    const View& g;
    const ListArrays m;
    uint32_t* bits;   // the statuses in LDS, kept up to date, or NULL
    ListStage<kWaves>& st;
    const int sched;
    WatchTotals& t;
    uint32_t* out = nullptr;   // the list being built

    __device__ __forceinline__ int rank() const {
        return kWaveGroup ? lane_id() : (int)threadIdx.x;
    }
    __device__ __forceinline__ int size() const { return kWaveGroup ? kWave : (int)blockDim.x; }
    __device__ __forceinline__ int wave() const {
        return kWaveGroup ? 0 : (int)threadIdx.x / kWave;
    }
    __device__ __forceinline__ void sync() const {
        complete_mem();
        if (kWaveGroup) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else {
            __syncthreads();
        }
    }
    // Before the first item of the first list (barriers are the caller's).
    __device__ __forceinline__ void begin() {
        if (lane_id() == 0) st.n[wave()] = 0;
        if (rank() == 0) st.cnt = 0;
        out = m.l0;
    }
    // move this wavefront's staged items to the list being built (wave-uniform)
    __device__ __forceinline__ void flush() {
        const int k = st.n[wave()];
        if (k == 0) return;
        int base = 0;
        if (lane_id() == 0) base = atomicAdd(&st.cnt, k);
        base = __shfl(base, 0);
        for (int i = lane_id(); i < k; i += kWave) out[base + i] = st.item[wave()][i];
        __builtin_amdgcn_wave_barrier();
        if (lane_id() == 0) st.n[wave()] = 0;
        __builtin_amdgcn_wave_barrier();
    }
    // stage this lane's item, if any (wave-uniform)
    __device__ __forceinline__ void emit(uint32_t it) {
        const uint64_t mk = ballot(it != kNone);
        const int k = popc(mk);
        if (k == 0) return;
        if (st.n[wave()] + k > kListStage) flush();
        const int base = st.n[wave()];
        if (it != kNone) st.item[wave()][base + popc(mk & lanes_below())] = it;
        __builtin_amdgcn_wave_barrier();
        if (lane_id() == 0) st.n[wave()] = base + k;
        __builtin_amdgcn_wave_barrier();
    }
    // Phases from the flushed list in l0 (a barrier behind it) until one builds
    // none, at most `budget`: their number.
    __device__ __forceinline__ int run(int budget) {
        uint32_t* in = m.l0;
        out = m.l1;
        int ph = 0;
        for (int n_in = st.cnt; n_in > 0 && ph < budget; n_in = st.cnt) {
            sync();   // every thread has read the count
            if (rank() == 0) st.cnt = 0;
            sync();
            ++ph;
            for (int base = 0; base < n_in; base += size()) {
                const int i = base + rank();
                const uint32_t it = i < n_in ? (uint32_t)ld_s<kWG>((const int*)in + i) : kNone;
                int walk_last = -1, walk_more = -1, cx = -1;
                if (it != kNone) {
                    const int x = item_vertex(it);
                    if (item_kind(it) == kOwnRescan) {
                        // x is in no list until it joins again: its record is stable
                        const uint64_t r = ld_s<kWG>(m.rec + x);
                        if (sched & TRIM_SCHED_JITTER) jitter_nap((uint64_t)x);
                        if (resume<View, kWG>(g, x, rec_cursor(r) + 1, m.head, m.rec, t.edges,
                                              sched, nullptr, bits))
                            t.joins += 1;
                        else
                            cx = x;
                    } else {
                        cx = x;
                    }
                }
                if (cx >= 0) {
                    if (sched & TRIM_SCHED_JITTER) jitter_nap((uint64_t)cx << 8);
                    const int2 ab = xchg2_s<kWG>(m.head + 2 * cx, kDead, kDead);
                    if (bits) atomicOr(bits + (cx >> 5), 1u << (cx & 31));
                    t.closes += 1;
                    walk_more = ab.x;
                    walk_last = ab.y;
                }
                // a member's link is read before its item exists: its own
                // processing, in the next phase, is the only thing that can change
                // its record
                while (ballot(walk_last >= 0 || walk_more >= 0)) {
                    uint32_t e = kNone;
                    if (walk_last >= 0) {
                        const int nx = ld_s<kWG>(rec_link(m.rec, walk_last));
                        e = make_item(kOwnClose, walk_last);
                        walk_last = nx;
                    } else if (walk_more >= 0) {
                        const int nx = ld_s<kWG>(rec_link(m.rec, walk_more));
                        e = make_item(kOwnRescan, walk_more);
                        walk_more = nx;
                    }
                    t.visited += e != kNone;
                    emit(e);
                }
            }
            flush();
            sync();
            uint32_t* tmp = in;
            in = out;
            out = tmp;
        }
        return ph;
    }
};

}  // namespace

}  // namespace trim
