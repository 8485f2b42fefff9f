// mlp.hip -- learned successor order for AC-6 (BF16 MFMA, FP32 accumulation).
//
// AC-6 checks successors in CSR order and keeps the first live one as the
// support (Section 6.1); a live vertex costs (index of its first live
// successor + 1) checks.  A small network scores every edge u -> w by how
// likely w is to stay live, and each adjacency list is then reordered by that
// score, so AC-6 tries likely supports first.  The order changes only the
// traversed edges, never the live set (every order reaches the same greatest
// fixed point).
//
// Network: 8 edge features -> 32 -> 32 -> 1, ReLU, BF16 weights, BF16 inputs
// and layer-1 activations as MFMA operands (the FP32 layer-2 activations feed
// the 32-term output dot product directly), FP32 accumulation, FP32 master
// weights, Adam.  The backward pass rounds dZ2 and dZ1 to BF16 where they
// enter an MFMA.
// Features of u -> w at position i of u's list:
//   log1p(outdeg u), log1p(indeg u), log1p(outdeg w), log1p(indeg w),
//   log1p(outdeg u) - log1p(outdeg w)  (= log of the degree ratio),
//   three +-1 bits of a hash of i.
// Loss: binary cross-entropy of "w is live" over edges whose source is live
// (only those edges decide a support).
//
// MFMA layout (v_mfma_f32_32x32x8 bf16, 64 lanes): A[i][k] sits in lane
// i%32 + 32*(k/4), item k%4; B[k][j] in lane j + 32*(k/4), item k%4; D[i][j]
// in lane j + 32*((i/4)%2), register 4*(i/8) + i%4.  A 32-edge tile is
// computed transposed (hidden units x edges), so layer 1's output registers
// 4j..4j+3 are exactly the B operand of layer 2's k-block j.
// Contractions over 32 (layer 2 and its backward pass, the weight gradients
// over a tile's edges) use gfx950's double-K form v_mfma_f32_32x32x16 bf16:
// 8 items per lane, A[i][k] in lane i%32 + 32*(k/8), item k%8, the same D.
// Where its operands are two 8-deep blocks side by side (cat), both operands
// see the same order of k, and a sum over k does not depend on that order.
#include "trim_device.h"
#include "trim_internal.h"

namespace trim {

namespace {

typedef __attribute__((__vector_size__(4 * sizeof(short)))) short bf16x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr int kW1 = 0, kB1 = 256, kW2 = 288, kB2 = 1312, kW3 = 1344, kB3 = 1376;

__device__ __forceinline__ short f2bf(float f) {   // round to nearest even
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (short)(u >> 16);
}
__device__ __forceinline__ float bf2f(short h) {
    return __uint_as_float(((uint32_t)(uint16_t)h) << 16);
}
// row of D register r held by lane l
__device__ __forceinline__ int drow(int r, int l) { return 8 * (r >> 2) + 4 * (l >> 5) + (r & 3); }
__device__ __forceinline__ f32x16 mfma(bf16x4 a, bf16x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(a, b, c, 0, 0, 0);
}
typedef __attribute__((__vector_size__(8 * sizeof(short)))) short bf16x8;
typedef __bf16 bf16v8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ f32x16 mfma16(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16v8, a),
                                                   __builtin_bit_cast(bf16v8, b), c, 0, 0, 0);
}
__device__ __forceinline__ bf16x8 cat(bf16x4 lo, bf16x4 hi) {
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

struct Graph {
    const int* row_off;
    const int* col;
    const int* indeg;
    const int* src;
    long long m;
};

// This lane's four features (half 0: features 0-3, half 1: 4-7) of edge e.
__device__ __forceinline__ void features(const Graph& g, long long e, int half, float f[4],
                                         int& u, int& w) {
    u = g.src[e];
    w = g.col[e];
    const float lu = log1pf((float)(g.row_off[u + 1] - g.row_off[u]));
    const float lw = log1pf((float)(g.row_off[w + 1] - g.row_off[w]));
    const float iu = log1pf((float)g.indeg[u]);
    const float iw = log1pf((float)g.indeg[w]);
    if (half == 0) {
        f[0] = lu;
        f[1] = iu;
        f[2] = lw;
        f[3] = iw;
    } else {
        const uint64_t h = mix64((uint64_t)(e - g.row_off[u]));
        f[0] = lu - lw;
        f[1] = (h & 1) ? 1.f : -1.f;
        f[2] = (h & 2) ? 1.f : -1.f;
        f[3] = (h & 4) ? 1.f : -1.f;
    }
}

// Weights staged per wave as MFMA operands.
struct Weights {
    bf16x4 w1;        // A of layer 1: W1[l%32][4(l/32)+t]
    bf16x4 w2[4];     // A of layer 2, k-block j: W2[l%32][8j+4(l/32)+t]
    bf16x4 w2t[4];    // A of dH1 = W2^T dZ2, k-block j: W2[8j+4(l/32)+t][l%32]
    float b1[16], b2[16], w3[16];   // per D register
    float b3;
};

// p: the parameters, in LDS or device memory.
__device__ __forceinline__ void load_weights(const short* p, Weights& W) {
    const int l = lane_id();
    for (int t = 0; t < 4; ++t) W.w1[t] = p[kW1 + (l & 31) * 8 + 4 * (l >> 5) + t];
    for (int j = 0; j < 4; ++j)
        for (int t = 0; t < 4; ++t) {
            const int k = 8 * j + 4 * (l >> 5) + t;
            W.w2[j][t] = p[kW2 + (l & 31) * 32 + k];
            W.w2t[j][t] = p[kW2 + k * 32 + (l & 31)];
        }
    for (int r = 0; r < 16; ++r) {
        const int h = drow(r, l);
        W.b1[r] = bf2f(p[kB1 + h]);
        W.b2[r] = bf2f(p[kB2 + h]);
        W.w3[r] = bf2f(p[kW3 + h]);
    }
    W.b3 = bf2f(p[kB3]);
}

// Forward pass of a 32-edge tile (edge = l%32).  Returns the logit of this
// lane's edge; z1/z2 hold pre-activations, h1 the BF16 layer-1 activations.
__device__ __forceinline__ float forward(const Weights& W, const float f[4], f32x16& z1,
                                         f32x16& z2, bf16x4 h1[4], float h2[16]) {
    bf16x4 x;
    for (int t = 0; t < 4; ++t) x[t] = f2bf(f[t]);
    const f32x16 zero = {};
    z1 = mfma(W.w1, x, zero);
    for (int r = 0; r < 16; ++r) {
        z1[r] += W.b1[r];
        h1[r >> 2][r & 3] = f2bf(fmaxf(z1[r], 0.f));
    }
    z2 = mfma16(cat(W.w2[0], W.w2[1]), cat(h1[0], h1[1]), zero);
    z2 = mfma16(cat(W.w2[2], W.w2[3]), cat(h1[2], h1[3]), z2);
    float s = 0.f;
    for (int r = 0; r < 16; ++r) {
        z2[r] += W.b2[r];
        h2[r] = fmaxf(z2[r], 0.f);
        s += W.w3[r] * h2[r];
    }
    s += __shfl_xor(s, 32);   // the other half of the hidden units
    return s + W.b3;
}

__device__ __forceinline__ bool bit(const uint32_t* bm, int v) { return (bm[v >> 5] >> (v & 31)) & 1u; }

__device__ __forceinline__ long long sample_edge(const long long* ids, uint64_t seed, int step,
                                                 long long idx, long long m) {
    if (ids) return ids[idx];
    return (long long)(mix64(seed ^ ((uint64_t)step << 40) ^ (uint64_t)idx) % (uint64_t)m);
}

// Per-wave LDS tiles for the weight gradients, BF16 bits: hidden units x edges
// (x: features x edges).  A lane's eight operands of an MFMA over the edges lie
// side by side; the row length keeps them 16-byte aligned.
constexpr int kTileRow = 40;
struct Tiles {
    short a[32][kTileRow];
    short b[32][kTileRow];
    short x[8][kTileRow];
};
constexpr int kGradParams = 1378;   // the gradients and the loss
constexpr int kGradWaves = 8;

// Gradients of the mean loss over `count` sampled edges, accumulated into
// grad[0..1376]; grad[1377] accumulates the loss.  Edges are ids[k] when ids
// is given, else hashed samples.  Loss weight 1/count per edge, 0 when the
// source is not live.
//
// A step's few thousand edges leave a wavefront one tile, so the sums are the
// larger part of the work: with every wavefront adding its 1,378 to the same
// words, 16,384 edges took 94 us, most of it the queue at those words.  The
// wavefronts of a workgroup add up in LDS first, and the largest workgroup the
// registers allow (eight wavefronts of 256 registers) leaves 64 adds a word.
__global__ __launch_bounds__(kGradWaves * kWave) void mlp_grad(Graph g, const uint32_t* live,
                                                               const short* p,
                                                               const long long* ids,
                                                               long long count, uint64_t seed,
                                                               int step, float* grad) {
    union Lds {
        Tiles tiles[kGradWaves];
        float sums[kGradWaves][kGradParams];
    };
    __shared__ __attribute__((aligned(16))) Lds lds;
    __shared__ short wts[kGradParams];
    Tiles& T = lds.tiles[threadIdx.x / kWave];
    const int l = lane_id(), half = l >> 5, col = l & 31;
    for (int i = threadIdx.x; i < kGradParams - 1; i += blockDim.x) wts[i] = p[i];
    __syncthreads();
    Weights W;
    load_weights(wts, W);
    const f32x16 zero = {};
    f32x16 gw2 = zero, gw1 = zero;
    float gb1[16] = {}, gb2[16] = {}, gw3[16] = {};
    float gb3 = 0.f, loss = 0.f;
    const float inv = 1.f / (float)count;
    const long long tiles_total = (count + 31) / 32;
    const long long wave = (blockIdx.x * (long long)blockDim.x + threadIdx.x) / kWave;
    const long long nwaves = (gridDim.x * (long long)blockDim.x) / kWave;
    auto fence = [&]() {   // the wavefront's tiles, written by some lanes, read by others
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    };
    auto row8 = [](const short* q) { return *reinterpret_cast<const bf16x8*>(q); };
    for (long long t = wave; t < tiles_total; t += nwaves) {
        const long long k = t * 32 + col;
        float f[4] = {0.f, 0.f, 0.f, 0.f};
        float wgt = 0.f, y = 0.f;
        if (k < count) {
            const long long e = sample_edge(ids, seed, step, k, g.m);
            int u, w;
            features(g, e, half, f, u, w);
            wgt = bit(live, u) ? inv : 0.f;
            y = bit(live, w) ? 1.f : 0.f;
        }
        f32x16 z1, z2;
        bf16x4 h1[4];
        float h2[16];
        const float s = forward(W, f, z1, z2, h1, h2);
        // d(loss)/d(logit) for binary cross-entropy
        const float pr = 1.f / (1.f + expf(-s));
        const float gs = wgt * (pr - y);
        if (half == 0 && wgt != 0.f)
            loss += wgt * (fmaxf(s, 0.f) - s * y + log1pf(expf(-fabsf(s))));
        if (half == 0) gb3 += gs;
        float dz2[16];
        bf16x4 dz2b[4];
        for (int r = 0; r < 16; ++r) {
            gw3[r] += gs * h2[r];
            dz2[r] = z2[r] > 0.f ? gs * W.w3[r] : 0.f;
            gb2[r] += dz2[r];
            dz2b[r >> 2][r & 3] = f2bf(dz2[r]);
        }
        // dH1 = W2^T dZ2 (dZ2 registers 4j..4j+3 are the B operand of k-block j)
        f32x16 dh1 = mfma16(cat(W.w2t[0], W.w2t[1]), cat(dz2b[0], dz2b[1]), zero);
        dh1 = mfma16(cat(W.w2t[2], W.w2t[3]), cat(dz2b[2], dz2b[3]), dh1);
        // stage dZ2, H1 and X for the weight gradients (contraction over edges)
        for (int r = 0; r < 16; ++r) {
            T.a[drow(r, l)][col] = dz2b[r >> 2][r & 3];
            T.b[drow(r, l)][col] = h1[r >> 2][r & 3];
        }
        for (int t4 = 0; t4 < 4; ++t4) T.x[4 * half + t4][col] = f2bf(f[t4]);
        fence();
        // dW2[h_out][h_in] += sum_e dZ2[h_out][e] H1[h_in][e]
        for (int j = 0; j < 2; ++j)
            gw2 = mfma16(row8(&T.a[col][16 * j + 8 * half]), row8(&T.b[col][16 * j + 8 * half]), gw2);
        fence();
        // dZ1 = dH1 * relu'(Z1)
        for (int r = 0; r < 16; ++r) {
            const float dz1 = z1[r] > 0.f ? dh1[r] : 0.f;
            gb1[r] += dz1;
            T.a[drow(r, l)][col] = f2bf(dz1);
        }
        fence();
        // dW1[h][f] += sum_e dZ1[h][e] X[e][f]
        for (int j = 0; j < 2; ++j) {
            const bf16x8 none = {};
            const bf16x8 x = row8(&T.x[col & 7][16 * j + 8 * half]);
            gw1 = mfma16(row8(&T.a[col][16 * j + 8 * half]), col < 8 ? x : none, gw1);
        }
        fence();
    }
    // sums over the 32 edges of each half, then over the wavefronts, then one
    // atomic per parameter
    __syncthreads();   // the tiles are free
    float* mine = lds.sums[threadIdx.x / kWave];
    for (int r = 0; r < 16; ++r) {
        float a = gb1[r], b = gb2[r], c = gw3[r];
        for (int off = 16; off > 0; off >>= 1) {
            a += __shfl_xor(a, off);
            b += __shfl_xor(b, off);
            c += __shfl_xor(c, off);
        }
        if (col == 0) {
            mine[kB1 + drow(r, l)] = a;
            mine[kB2 + drow(r, l)] = b;
            mine[kW3 + drow(r, l)] = c;
        }
        mine[kW2 + drow(r, l) * 32 + col] = gw2[r];
        if (col < 8) mine[kW1 + drow(r, l) * 8 + col] = gw1[r];
    }
    for (int off = 16; off > 0; off >>= 1) {
        gb3 += __shfl_xor(gb3, off);
        loss += __shfl_xor(loss, off);
    }
    if (l == 0) {
        mine[kB3] = gb3;
        mine[kGradParams - 1] = loss;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kGradParams; i += blockDim.x) {
        float sum = 0.f;
        for (int w = 0; w < kGradWaves; ++w) sum += lds.sums[w][i];
        atomicAdd(grad + i, sum);
    }
}

// Adam on the FP32 master weights; writes the BF16 copy and clears the
// gradients.  c1 = 1 / (1 - beta1^t), c2 = 1 / (1 - beta2^t).
__global__ void mlp_adam(float* p32, short* pbf, float* m1, float* m2, float* grad, float lr,
                         float beta1, float beta2, float eps, float c1, float c2) {
    for (int i = threadIdx.x; i < 1377; i += blockDim.x) {
        const float gi = grad[i];
        const float a = beta1 * m1[i] + (1.f - beta1) * gi;
        const float b = beta2 * m2[i] + (1.f - beta2) * gi * gi;
        m1[i] = a;
        m2[i] = b;
        const float w = p32[i] - lr * (a * c1) / (sqrtf(b * c2) + eps);
        p32[i] = w;
        pbf[i] = f2bf(w);
        grad[i] = 0.f;
    }
    if (threadIdx.x == 0) grad[1377] = 0.f;
}

// Two floats as BF16 bits, nearest even, the first in the low half.
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    typedef __bf16 v2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{lo, hi}, v2));
}

// What scoring needs of a vertex, in the four bytes that a gather of targets at
// random places should cost at most: the out-degree (kOutMax: that or more)
// above a ten-bit code of the in-degree's feature, log1p of an integer below
// 2^31 as BF16, which is 0 or between bf16(log 2) and bf16(log 2^31).
constexpr uint32_t kOutMax = (1u << 22) - 1;
constexpr uint32_t kInBase = 0x3F00;
// The edges' sources come in order, so theirs may be wider: both features as
// BF16 (out-degree in the low half) and the out-degree's in FP32.
struct ScoreSource {
    uint32_t bf;
    float out;
};
// sv: an entry per vertex; su, if given, the sources' entries.
__global__ void score_vertices(const int* row_off, const int* indeg, int n, uint32_t* sv,
                               ScoreSource* su) {
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        const uint32_t d = (uint32_t)(row_off[v + 1] - row_off[v]);
        const uint32_t in = (uint32_t)(uint16_t)f2bf(log1pf((float)indeg[v]));
        sv[v] = (min(d, kOutMax) << 10) | (in ? in - kInBase : 0);
        if (su) {
            const float out = log1pf((float)(int)d);
            su[v] = ScoreSource{(pack_bf16(out, 0.f) & 0xFFFFu) | (in << 16), out};
        }
    }
}
// Both features of vertex v with entry x as BF16, the out-degree's in the low
// half, and that one in FP32 (`out`), for the difference.
__device__ __forceinline__ uint32_t score_features(uint32_t x, int v, const int* row_off,
                                                   float& out) {
    uint32_t d = x >> 10;
    if (d == kOutMax) d = (uint32_t)(row_off[v + 1] - row_off[v]);
    out = log1pf((float)(int)d);
    const uint32_t c = x & 0x3FFu;
    return (pack_bf16(out, 0.f) & 0xFFFFu) | ((min(c, 1u) * kInBase + c) << 16);
}

// The network's logit that the target of every edge stays live, in CSR
// order.  The logit, not the probability, is what the lists are ordered by:
// the logistic function saturates to exactly 1 in FP32 for logits above about
// 17, which would tie most live targets.
//
// Two things bound it on R-MAT 24 (2.7 * 10^8 edges, 8.4 * 10^6 tiles of 32,
// 3.73 ms at first): the targets' gathers, a fresh line for every one that the
// L2s miss, and, at four cycles an instruction, the 220 instructions of a tile
// (3 ms by themselves).  So what is gathered takes four bytes a vertex; a
// wavefront takes two tiles at a time, one edge per lane for the loads and the
// features (both halves used to make the same ones), and swaps halves of
// registers to get the tiles' operands; conversions go two values an
// instruction (the first ReLU does not: a maximum of packed 16-bit integers
// would pass a NaN, which fmaxf drops as in training); the second layer's biases enter as the MFMA's addend;
// and the position's hash bits, two 64-bit products, come from a table for the
// first kHashed positions of a list.
// The sources' features come from their own table (kWide) unless the context
// has no room for it: made from the four-byte entries, 3.05 instead of 2.64 ms.
constexpr int kHashed = 4096;

template <bool kWide>
__global__ __launch_bounds__(256) void mlp_score(const int* row_off, const int* col,
                                                 const int* src, long long m,
                                                 const uint32_t* sv, const ScoreSource* su,
                                                 const short* p, float* score) {
    __shared__ uint8_t hashed[kHashed];
    for (int i = threadIdx.x; i < kHashed; i += blockDim.x) hashed[i] = (uint8_t)(mix64(i) & 7);
    __syncthreads();
    const int l = lane_id();
    Weights W;
    load_weights(p, W);
    f32x16 b2;
    for (int r = 0; r < 16; ++r) b2[r] = W.b2[r];
    const f32x16 zero = {};
    const bf16x8 w2a = cat(W.w2[0], W.w2[1]), w2b = cat(W.w2[2], W.w2[3]);
    auto logit = [&](uint32_t x0, uint32_t x1) {
        const uint64_t x = ((uint64_t)x1 << 32) | x0;
        const f32x16 z1 = mfma(W.w1, __builtin_bit_cast(bf16x4, x), zero);
        uint32_t h[8];
#pragma unroll
        for (int r = 0; r < 8; ++r)
            h[r] = pack_bf16(fmaxf(z1[2 * r] + W.b1[2 * r], 0.f),
                             fmaxf(z1[2 * r + 1] + W.b1[2 * r + 1], 0.f));
        typedef uint32_t u4 __attribute__((ext_vector_type(4)));
        f32x16 z2 = mfma16(w2a, __builtin_bit_cast(bf16x8, u4{h[0], h[1], h[2], h[3]}), b2);
        z2 = mfma16(w2b, __builtin_bit_cast(bf16x8, u4{h[4], h[5], h[6], h[7]}), z2);
        float s = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) s += W.w3[r] * fmaxf(z2[r], 0.f);
        s += __shfl_xor(s, 32);   // the other half of the hidden units
        return s + W.b3;
    };
    const long long pairs = (m + 63) / 64;
    const long long wave = (blockIdx.x * (long long)blockDim.x + threadIdx.x) / kWave;
    const long long nwaves = (gridDim.x * (long long)blockDim.x) / kWave;
    // ids two tile pairs ahead, what they lead to one ahead
    struct Ids {
        int u, w;
        long long e;
    };
    struct Ends {
        ScoreSource a;     // !kWide: u's four-byte entry in `bf`
        uint32_t b, pos;   // w's entry
        int u, w;
    };
    auto ids_of = [&](long long t) {
        const long long e = t * 64 + l, ec = e < m ? e : m - 1;
        return Ids{__builtin_nontemporal_load(src + ec), __builtin_nontemporal_load(col + ec), ec};
    };
    auto ends_of = [&](const Ids& i) {
        return Ends{kWide ? su[i.u] : ScoreSource{sv[i.u], 0.f}, sv[i.w],
                    (uint32_t)(i.e - row_off[i.u]), i.u, i.w};
    };
    if (wave >= pairs) return;
    Ids ids = ids_of(wave);
    Ends next = ends_of(ids);
    ids = ids_of(wave + nwaves);
    for (long long t = wave; t < pairs; t += nwaves) {
        const Ends now = next;
        next = ends_of(ids);
        ids = ids_of(t + 2 * nwaves);
        const long long e = t * 64 + l;
        float a_out = now.a.out, b_out;
        const uint32_t a_bf =
            kWide ? now.a.bf : score_features(now.a.bf, now.u, row_off, a_out);
        const uint32_t b_bf = score_features(now.b, now.w, row_off, b_out);
        const uint32_t pos = now.pos;
        uint32_t h = hashed[pos & (kHashed - 1)];
        if (pos >= kHashed) h = (uint32_t)mix64(pos);
        // features 4-7: the difference and the signs of the three bits
        const uint32_t f45 = (pack_bf16(a_out - b_out, 0.f) & 0xFFFFu) |
                             (0xBF800000u ^ ((h & 1u) << 31));
        const uint32_t f67 = 0xBF80BF80u ^ ((h & 2u) << 14) ^ ((h & 4u) << 29);
        // lanes 0-31 hold edges 0-31: after the swaps, x0 x1 are the first
        // tile's operand (features 0-3 in the lower half, 4-7 in the upper)
        // and y0 y1 the second's
        const auto s0 = __builtin_amdgcn_permlane32_swap(a_bf, f45, false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(b_bf, f67, false, false);
        const float first = logit(s0[0], s1[0]), second = logit(s0[1], s1[1]);
        if (e < m) score[e] = l < 32 ? first : second;
    }
}

inline int grid_for(long long n, int block, int max_blocks) {
    long long b = (n + block - 1) / block;
    if (b < 1) b = 1;
    if (b > max_blocks) b = max_blocks;
    return (int)b;
}

}  // namespace

hipError_t mlp_grad_launch(const int* row_off, const int* col, const int* indeg, const int* src,
                           long long m, const uint32_t* live, const short* pbf,
                           const long long* ids, long long count, uint64_t seed, int step,
                           float* grad, int cus, hipStream_t s) {
    Graph g{row_off, col, indeg, src, m};
    const int blocks = grid_for((count + 31) / 32, kGradWaves, cus);
    hipLaunchKernelGGL(mlp_grad, dim3(blocks), dim3(kGradWaves * kWave), 0, s, g, live, pbf, ids,
                       count, seed, step, grad);
    return hipGetLastError();
}

hipError_t mlp_adam_launch(float* p32, short* pbf, float* m1, float* m2, float* grad, float lr,
                           float beta1, float beta2, float eps, int step, hipStream_t s) {
    // the bias corrections in double: 1 - beta2^t cancels badly in FP32
    // (beta2 = 0.999 loses about 15 bits at t = 2)
    const float c1 = (float)(1.0 / (1.0 - pow((double)beta1, (double)step)));
    const float c2 = (float)(1.0 / (1.0 - pow((double)beta2, (double)step)));
    hipLaunchKernelGGL(mlp_adam, dim3(1), dim3(256), 0, s, p32, pbf, m1, m2, grad, lr, beta1,
                       beta2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t mlp_score_launch(const int* row_off, const int* col, const int* indeg, const int* src,
                            int n, long long m, const short* pbf, float* score, uint32_t* sv,
                            bool wide, int cus, hipStream_t s) {
    if (m > 0) {
        ScoreSource* su = wide ? reinterpret_cast<ScoreSource*>(sv) : nullptr;
        if (wide) sv += 2 * (long long)n;
        hipLaunchKernelGGL(score_vertices, dim3(grid_for(n, 256, 16384)), dim3(256), 0, s,
                           row_off, indeg, n, sv, su);
        const dim3 grid(grid_for((m + 63) / 64, 4, cus * 16));
        if (wide)
            hipLaunchKernelGGL(mlp_score<true>, grid, dim3(256), 0, s, row_off, col, src, m, sv,
                               su, pbf, score);
        else
            hipLaunchKernelGGL(mlp_score<false>, grid, dim3(256), 0, s, row_off, col, src, m, sv,
                               su, pbf, score);
    }
    return hipGetLastError();
}

}  // namespace trim
