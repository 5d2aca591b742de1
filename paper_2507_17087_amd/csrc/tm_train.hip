// tm_train.hip -- the ranker's gradient (gfx950), three launches: k_forward_backward (a
// minibatch through the network and back, tile by tile), k_weight_grad (weight
// gradients over row ranges, the tiles' bias and head gradients) and k_reduce_grad or k_reduce_adam
// (the ranges summed in order; the Adam step).  Every sum has a fixed order: the same
// inputs give the same bits.
//
// Measured against the 22 launches before (per layer a data and a weight gradient, column
// sums and reductions, activations row-major between them): 4,096 rows 165 -> 25 us (14,
// 10 and 3), 34,833 rows 751 -> 137 us.  With weights and columns row-major (64-byte pieces
// of 16 lines per load) the two large launches took 25 and 16 us.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "tm_internal.h"
#include "tm_mfma.h"
#include "tm_ranker.h"

namespace tmk {

// a caller's rows: 16-byte loads at any 4-byte alignment
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kLd = kWidth + 8;   // bf16 elements per LDS row of activations (breaks bank aliasing)
constexpr int kLdX = kFeat + 8;   // the same of features
constexpr int kTrainThreads = 512;  // 8 waves: 32 output columns each

// Barrier for data passed through LDS only: __syncthreads also waits for the wave's global
// stores (the columns, that no one here reads back) and for the next layer's weights.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Weight fragments of this wave's 32 columns.
template <int K>
__device__ __forceinline__ void load_frags(u16x8 (&w)[K / 32][2], const uint16_t* __restrict__ F, int lane, int c0) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int ks = 0; ks < K / 32; ++ks)
            w[ks][b] = *reinterpret_cast<const u16x8*>(F + (((c0 / 16 + b) * (K / 32) + ks) * 64 + lane) * 8);
}

// acc[a][b]: rows 16a.., columns c0 + 16b.. of in (LDS, stride ld) times the fragments;
// transposed tiles, so a lane holds four consecutive columns of row 16a + (lane & 15).
template <int K, int RT>
__device__ __forceinline__ void tile_product(f32x4 (&acc)[RT][2], const uint16_t* in, int ld,
                                             const u16x8 (&w)[K / 32][2], int lane) {
    const int r16 = lane & 15, kq = (lane >> 4) * 8;
#pragma unroll
    for (int a = 0; a < RT; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    // all activations are requested before the first product waits for one
    u16x8 x[K / 32][RT];
#pragma unroll
    for (int ks = 0; ks < K / 32; ++ks)
#pragma unroll
        for (int a = 0; a < RT; ++a)
            x[ks][a] = *reinterpret_cast<const u16x8*>(in + (a * 16 + r16) * ld + ks * 32 + kq);
    if (RT == 1) __builtin_amdgcn_sched_group_barrier(0x100, K / 32, 0);
#pragma unroll
    for (int ks = 0; ks < K / 32; ++ks)
#pragma unroll
        for (int a = 0; a < RT; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) acc[a][b] = mfma16(w[ks][b], x[ks][a], acc[a][b]);
}

__device__ __forceinline__ uint2 pack4(float a, float b, float c, float d) {
    return make_uint2(pack_bf16(a, b), pack_bf16(c, d));
}

// This lane's biases of a layer: columns c0 + 16b + 4 (lane / 16) ..
__device__ __forceinline__ void load_bias(float (&o)[2][4], const float* __restrict__ bias, int lane, int c0) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int j = 0; j < 4; ++j) o[b][j] = bias[c0 + b * 16 + (lane >> 4) * 4 + j];
}

// bias + ReLU of the tile into LDS
template <int RT>
__device__ __forceinline__ void store_relu(uint16_t* out, const f32x4 (&acc)[RT][2], const float (&bias)[2][4],
                                           int lane, int c0) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int col = c0 + b * 16 + (lane >> 4) * 4;
        const float b0 = bias[b][0], b1 = bias[b][1], b2 = bias[b][2], b3 = bias[b][3];
#pragma unroll
        for (int a = 0; a < RT; ++a)
            *reinterpret_cast<uint2*>(out + (a * 16 + (lane & 15)) * kLd + col) =
                pack4(fmaxf(acc[a][b][0] + b0, 0.f), fmaxf(acc[a][b][1] + b1, 0.f), fmaxf(acc[a][b][2] + b2, 0.f),
                      fmaxf(acc[a][b][3] + b3, 0.f));
    }
}

// the tile where act is positive (the ReLU's derivative), into LDS
template <int RT>
__device__ __forceinline__ void store_masked(uint16_t* out, const f32x4 (&acc)[RT][2], const uint16_t* act, int lane,
                                             int c0) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int col = c0 + b * 16 + (lane >> 4) * 4;
#pragma unroll
        for (int a = 0; a < RT; ++a) {
            const int at = (a * 16 + (lane & 15)) * kLd + col;
            const uint2 h = *reinterpret_cast<const uint2*>(act + at);
            // activations are bf16 values >= 0: positive when any bit but the sign is set
            *reinterpret_cast<uint2*>(out + at) =
                pack4((h.x & 0x7fffu) ? acc[a][b][0] : 0.f, (h.x & 0x7fff0000u) ? acc[a][b][1] : 0.f,
                      (h.y & 0x7fffu) ? acc[a][b][2] : 0.f, (h.y & 0x7fff0000u) ? acc[a][b][3] : 0.f);
        }
    }
}

// The tile's columns in fragment order, the reduction index of the weight gradients being
// the row: 8 rows of a column per 16-byte store, whole 512-byte pieces per 16 rows.  each
// (column, first row, the 8 values) is called for every piece, with its result summed over
// the column's pieces (neighbouring lanes) for `sum`(column, total), once per column.
template <int R, class Each, class Sum>
__device__ __forceinline__ void store_columns(uint16_t* __restrict__ dst, int64_t steps, int64_t row0,
                                              const uint16_t* src, int ld, int cols, int tid, Each each, Sum sum) {
    for (int i = tid; i < cols * (R / 8); i += kTrainThreads) {
        const int c = (i / (2 * R)) * 16 + i % 16, r8 = (i / 16) % (R / 8) * 8;  // 16 columns, then the next 8 rows
        u16x8 v;
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = src[(r8 + j) * ld + c];
        *reinterpret_cast<u16x8*>(dst + frag_at(c, row0 + r8, steps)) = v;
        float2 t = each(c, r8, v);
#pragma unroll
        for (int o = 16; o < 2 * R; o <<= 1) {
            t.x += __shfl_xor(t.x, o, 64);
            t.y += __shfl_xor(t.y, o, 64);
        }
        if (r8 == 0) sum(c, t);
    }
}
template <int R>
__device__ __forceinline__ void store_columns(uint16_t* __restrict__ dst, int64_t steps, int64_t row0,
                                              const uint16_t* src, int ld, int cols, int tid) {
    store_columns<R>(dst, steps, row0, src, ld, cols, tid,
                     [](int, int, const u16x8&) { return make_float2(0.f, 0.f); }, [](int, float2) {});
}
// The same of a gradient, its column sums to part[column].
template <int R>
__device__ __forceinline__ void store_gradient(uint16_t* __restrict__ dst, int64_t steps, int64_t row0,
                                               const uint16_t* src, float* __restrict__ part, int tid) {
    store_columns<R>(
        dst, steps, row0, src, kLd, kWidth, tid,
        [](int, int, const u16x8& v) {
            float p = 0.f;
#pragma unroll
            for (int j = 0; j < 8; ++j) p += bf2f(v[j]);
            return make_float2(p, 0.f);
        },
        [&](int c, float2 t) { part[c] = t.x; });
}

// One workgroup per tile of 16 RT rows (zero rows past n): the forward pass, the head and
// its gradient, the data gradients back to the first layer, all activations in LDS.  Writes
// Y, the columns (store_columns) of X, H1..H3, dH1..dH3 and the tile's column sums of the
// gradients (bias gradients) and of H3 times dY (the head's).  Every layer's weights
// are read from L2 once per tile (544 KB in all) and requested before the barrier that the
// layer waits at.  Bound: that read, 64 bytes per clock and CU, and the chain of seven
// layers; 16-row tiles put 4,096 rows on all 256 CUs, above that 32-row tiles halve the
// reads.
template <int RT>
__global__ __launch_bounds__(kTrainThreads) void k_forward_backward(const TrainBatch B, const RankerWeights W, float s0,
                                                                    float s1, const TrainBuffers T) {
    constexpr int R = 16 * RT;
    __shared__ __attribute__((aligned(16))) uint16_t sx[R * kLdX];
    __shared__ __attribute__((aligned(16))) uint16_t h1[R * kLd], h2[R * kLd], h3[R * kLd], da[R * kLd], db[R * kLd];
    __shared__ __attribute__((aligned(16))) uint16_t s_w4[kOut * kWidth];  // head weights, transposed
    __shared__ float s_y[R][kOut];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, c0 = wid * 32;
    const int r16 = lane & 15, kq = (lane >> 4) * 8;
    const int64_t row0 = (int64_t)blockIdx.x * R, ks = T.npad / 32;
    // two layers' weight fragments: the next one's are in flight while one is used
    u16x8 w1[kFeat / 32][2], wa[kWidth / 32][2], wb[kWidth / 32][2];
    float bias1[2][4], bias2[2][4], bias3[2][4];
    f32x4 acc[RT][2];
    load_frags<kFeat>(w1, W.f1, lane, c0);
    load_frags<kWidth>(wa, W.f2, lane, c0);
    load_bias(bias1, W.b1, lane, c0);
    load_bias(bias2, W.b2, lane, c0);
    load_bias(bias3, W.b3, lane, c0);
    const float hb = W.b4[r16 < kOut ? r16 : 0];
    for (int i = tid; i < kOut * kWidth; i += kTrainThreads) s_w4[(i % kOut) * kWidth + i / kOut] = W.w4[i];
    // features (rows through the permutation when there is one) and targets
    for (int i = tid; i < R * (kFeat / 4); i += kTrainThreads) {
        const int r = i / (kFeat / 4), c4 = (i % (kFeat / 4)) * 4;
        f32x4u v = {0.f, 0.f, 0.f, 0.f};
        if (row0 + r < B.n) {
            const int64_t src = B.perm ? B.perm[B.first + row0 + r] : B.first + row0 + r;
            v = *reinterpret_cast<const f32x4u*>(B.feat + src * kFeat + c4);
        }
        *reinterpret_cast<uint2*>(sx + r * kLdX + c4) = pack4(v[0], v[1], v[2], v[3]);
    }
    float2 tgt = make_float2(0.f, 0.f);
    if (tid < R && row0 + tid < B.n) {
        const int64_t src = B.perm ? B.perm[B.first + row0 + tid] : B.first + row0 + tid;
        tgt = make_float2(B.target[src * kOut], B.target[src * kOut + 1]);
    }
    lds_barrier();
    load_frags<kWidth>(wb, W.f3, lane, c0);
    tile_product<kFeat, RT>(acc, sx, kLdX, w1, lane);
    store_relu<RT>(h1, acc, bias1, lane, c0);
    store_columns<R>(T.X, ks, row0, sx, kLdX, kFeat, tid);
    lds_barrier();
    tile_product<kWidth, RT>(acc, h1, kLd, wa, lane);
    load_frags<kWidth>(wa, W.g3, lane, c0);
    store_relu<RT>(h2, acc, bias2, lane, c0);
    store_columns<R>(T.H1, ks, row0, h1, kLd, kWidth, tid);
    lds_barrier();
    tile_product<kWidth, RT>(acc, h2, kLd, wb, lane);
    load_frags<kWidth>(wb, W.g2, lane, c0);
    store_relu<RT>(h3, acc, bias3, lane, c0);
    store_columns<R>(T.H2, ks, row0, h2, kLd, kWidth, tid);
    lds_barrier();
    // head: wave w takes rows 16w..16w+15; B columns 0, 1 are the two heads
    if (wid < RT) {
        f32x4 y = {0.f, 0.f, 0.f, 0.f};
        const u16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int k0 = 0; k0 < kWidth; k0 += 32) {
            const u16x8 af = *reinterpret_cast<const u16x8*>(h3 + (wid * 16 + r16) * kLd + k0 + kq);
            const u16x8 hw = *reinterpret_cast<const u16x8*>(s_w4 + (r16 < kOut ? r16 : 0) * kWidth + k0 + kq);
            y = mfma16(af, r16 < kOut ? hw : zero, y);
        }
        if (r16 < kOut) {
#pragma unroll
            for (int r = 0; r < 4; ++r) s_y[wid * 16 + (lane >> 4) * 4 + r][r16] = y[r] + hb;
        }
    }
    lds_barrier();
    // dY = scale (Y - target), 0 past n
    if (tid < R) {
        const bool on = row0 + tid < B.n;
        const float y0 = s_y[tid][0], y1 = s_y[tid][1];
        const float2 d = on ? make_float2(s0 * (y0 - tgt.x), s1 * (y1 - tgt.y)) : make_float2(0.f, 0.f);
        if (on) {
            *reinterpret_cast<float2*>(T.Y + (row0 + tid) * kOut) = make_float2(y0, y1);
            *reinterpret_cast<float2*>(T.T + (row0 + tid) * kOut) = tgt;
        }
        s_y[tid][0] = d.x;
        s_y[tid][1] = d.y;
    }
    lds_barrier();
    // the head's gradients of this tile: dW4 = H3^T dY, db4 = column sums of dY
    float* part = T.colpart + (int64_t)blockIdx.x * kColParts;
    store_columns<R>(
        T.H3, ks, row0, h3, kLd, kWidth, tid,
        [&](int, int r8, const u16x8& v) {
            float2 p = make_float2(0.f, 0.f);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                p.x += bf2f(v[j]) * s_y[r8 + j][0];
                p.y += bf2f(v[j]) * s_y[r8 + j][1];
            }
            return p;
        },
        [&](int c, float2 t) { *reinterpret_cast<float2*>(part + 3 * kWidth + c * kOut) = t; });
    if (tid < kOut) {
        float p = 0.f;
        for (int r = 0; r < R; ++r) p += s_y[r][tid];
        part[5 * kWidth + tid] = p;
    }
    // dH3 = (dY W4^T) where H3 > 0
    for (int i = tid; i < R * (kWidth / 8); i += kTrainThreads) {
        const int r = i / (kWidth / 8), k = i % (kWidth / 8) * 8;
        const float y0 = s_y[r][0], y1 = s_y[r][1];
        const u16x8 u = *reinterpret_cast<const u16x8*>(s_w4 + k), v = *reinterpret_cast<const u16x8*>(s_w4 + kWidth + k);
        const u16x8 h = *reinterpret_cast<const u16x8*>(h3 + r * kLd + k);
        float g[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) g[j] = (h[j] & 0x7fffu) ? y0 * bf2f(u[j]) + y1 * bf2f(v[j]) : 0.f;
        *reinterpret_cast<uint4*>(da + r * kLd + k) = make_uint4(pack_bf16(g[0], g[1]), pack_bf16(g[2], g[3]),
                                                                 pack_bf16(g[4], g[5]), pack_bf16(g[6], g[7]));
    }
    lds_barrier();
    tile_product<kWidth, RT>(acc, da, kLd, wa, lane);
    store_masked<RT>(db, acc, h2, lane, c0);
    store_gradient<R>(T.D3, ks, row0, da, part + 2 * kWidth, tid);
    lds_barrier();
    tile_product<kWidth, RT>(acc, db, kLd, wb, lane);
    store_masked<RT>(h3, acc, h1, lane, c0);  // H3 is no longer read
    store_gradient<R>(T.D2, ks, row0, db, part + kWidth, tid);
    lds_barrier();
    store_gradient<R>(T.D1, ks, row0, h3, part, tid);
}

// Weight gradients In^T dOut.  Blocks [0, 36 S): a 64 x 64 tile of W3, W2 or W1's gradient
// over one of S row ranges; its four waves take every fourth 32-row step (operands straight
// from memory, no LDS), their tiles are added in LDS in order.  The blocks after them add the
// tiles' column sums, the bias and head gradients, into grad.  Bound: latency
// of the operand reads.
constexpr int kColStep = 16;  // column sums in flight per thread
constexpr int kGradTiles = 36;  // 16 of W3, 16 of W2, 4 of W1
__global__ __launch_bounds__(256) void k_weight_grad(const TrainBuffers T, int64_t tiles, int splits, int64_t steps,
                                                     const RankerLayout L, float* __restrict__ part,
                                                     float* __restrict__ grad) {
    __shared__ float s_t[4][64 * 64];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int r16 = lane & 15;
    const int64_t ks = T.npad / 32;
    const int b = blockIdx.x;
    if (b < kGradTiles * splits) {
        const int t = b % kGradTiles, split = b / kGradTiles;
        const int layer = t < 16 ? 3 : (t < 32 ? 2 : 1), lt = layer == 1 ? t - 32 : t & 15;
        const int ti = layer == 1 ? 0 : lt >> 2, tn = lt & 3;  // tile (kin, kout)
        const uint16_t* In = (layer == 3 ? T.H2 : (layer == 2 ? T.H1 : T.X)) + ti * 4 * ks * 512 + lane * 8;
        const uint16_t* Do = (layer == 3 ? T.D3 : (layer == 2 ? T.D2 : T.D1)) + tn * 4 * ks * 512 + lane * 8;
        const int64_t ka = split * steps, kb = std::min(ks, ka + steps);
        f32x4 acc[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        // four steps' operands in flight: their latency (another XCD wrote them) is the cost
        for (int64_t k = ka + wid; k < kb; k += 16) {
            u16x8 x[4][4], d[4][4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t ku = k + 4 * u < kb ? k + 4 * u : k;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    x[u][i] = *reinterpret_cast<const u16x8*>(In + (i * ks + ku) * 512);
                    d[u][i] = *reinterpret_cast<const u16x8*>(Do + (i * ks + ku) * 512);
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (k + 4 * u >= kb) break;
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[i][j] = mfma16(x[u][i], d[u][j], acc[i][j]);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    s_t[wid][(i * 16 + (lane >> 4) * 4 + r) * 64 + j * 16 + r16] = acc[i][j][r];
        __syncthreads();
        const int64_t off = layer == 3 ? L.w3 : (layer == 2 ? L.w2 : L.w1);
        float* o = part + (int64_t)split * L.count + off;
        for (int i = tid; i < 64 * 16; i += 256) {
            const int r = i / 16, c = (i % 16) * 4;
            const float4 p0 = *reinterpret_cast<const float4*>(&s_t[0][r * 64 + c]);
            const float4 p1 = *reinterpret_cast<const float4*>(&s_t[1][r * 64 + c]);
            const float4 p2 = *reinterpret_cast<const float4*>(&s_t[2][r * 64 + c]);
            const float4 p3 = *reinterpret_cast<const float4*>(&s_t[3][r * 64 + c]);
            float* q = o + (int64_t)(ti * 64 + r) * kWidth + tn * 64 + c;
            q[0] = (p0.x + p1.x) + (p2.x + p3.x);
            q[1] = (p0.y + p1.y) + (p2.y + p3.y);
            q[2] = (p0.z + p1.z) + (p2.z + p3.z);
            q[3] = (p0.w + p1.w) + (p2.w + p3.w);
        }
        return;
    }
    // bias and head gradients: 16 of the tiles' column sums each, every 16th tile a thread
    const int q = (b - kGradTiles * splits) * 16 + (tid & 15);
    float a = 0.f;
    if (q < kColParts) {
        for (int64_t t = tid >> 4; t < tiles; t += 16 * kColStep) {
            float v[kColStep];
#pragma unroll
            for (int u = 0; u < kColStep; ++u) v[u] = t + 16 * u < tiles ? T.colpart[(t + 16 * u) * kColParts + q] : 0.f;
#pragma unroll
            for (int u = 0; u < kColStep; ++u) a += v[u];
        }
    }
    s_t[0][tid] = a;
    __syncthreads();
    if (tid >= 16 || q >= kColParts) return;
    a = 0.f;
    for (int t = 0; t < 16; ++t) a += s_t[0][t * 16 + tid];
    grad[q < kWidth ? L.b1 + q : (q < 2 * kWidth ? L.b2 + q - kWidth : (q < 3 * kWidth ? L.b3 + q - 2 * kWidth
                                                                                      : L.w4 + q - 3 * kWidth))] = a;
}
static_assert(ranker_layout().b4 == ranker_layout().w4 + kWidth * kOut, "the head's gradients are contiguous");

__device__ __forceinline__ bool in_matrix(int64_t i, const RankerLayout& L) {
    return i < L.b1 || (i >= L.w2 && i < L.b2) || (i >= L.w3 && i < L.b3);
}

// The gradient of parameter i: a matrix's row ranges in order (four partial sums), else
// what k_weight_grad wrote.
__device__ __forceinline__ float grad_at(int64_t i, const RankerLayout& L, const float* __restrict__ part, int splits,
                                         const float* __restrict__ grad) {
    if (!in_matrix(i, L)) return grad[i];
    float a[4] = {0.f, 0.f, 0.f, 0.f};
    int s = 0;
    for (; s + 4 <= splits; s += 4)
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] += part[(int64_t)(s + u) * L.count + i];
    for (; s < splits; ++s) a[0] += part[(int64_t)s * L.count + i];
    return (a[0] + a[1]) + (a[2] + a[3]);
}

__global__ __launch_bounds__(256) void k_reduce_grad(const RankerLayout L, const float* __restrict__ part, int splits,
                                                     float* __restrict__ grad) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < L.count && in_matrix(i, L)) grad[i] = grad_at(i, L, part, splits, grad);
}

// Adam on the fp32 master copy; refreshes the bf16 copies (in fragment order, of the matrices
// and of their transposes).  Parameter layout: see RankerLayout.
__global__ __launch_bounds__(256) void k_reduce_adam(float* __restrict__ p, const float* __restrict__ part, int splits,
                                                     const float* __restrict__ grad, float* __restrict__ m,
                                                     float* __restrict__ v, float lr, float b1, float b2, float eps,
                                                     float c1, float c2, const RankerWeights W) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= W.layout.count) return;
    const float gi = grad_at(i, W.layout, part, splits, grad);
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    p[i] = pi;
    publish_param(i, pi, W);
}

hipError_t launch_gradient(const TrainBatch& B, const RankerWeights& W, float s0, float s1, const TrainBuffers& T,
                           float* grad, hipStream_t s) {
    const int64_t npad = T.npad;  // a multiple of 32
    if (B.n <= kTrainSmallRows)
        hipLaunchKernelGGL(k_forward_backward<1>, dim3((unsigned)(npad / 16)), dim3(kTrainThreads), 0, s, B, W, s0, s1,
                           T);
    else
        hipLaunchKernelGGL(k_forward_backward<2>, dim3((unsigned)(npad / 32)), dim3(kTrainThreads), 0, s, B, W, s0, s1,
                           T);
    const int splits = grad_splits(B.n);
    const int64_t steps = (npad / 32 + splits - 1) / splits;
    const int blocks = kGradTiles * splits + (kColParts + 15) / 16;
    hipLaunchKernelGGL(k_weight_grad, dim3((unsigned)blocks), dim3(256), 0, s, T, npad / (B.n <= kTrainSmallRows ? 16 : 32), splits, steps, W.layout, T.part,
                       grad);
    return hipGetLastError();
}

hipError_t launch_reduce_grad(const RankerLayout& L, const TrainBuffers& T, int64_t n, float* grad, hipStream_t s) {
    hipLaunchKernelGGL(k_reduce_grad, dim3((unsigned)((L.count + 255) / 256)), dim3(256), 0, s, L, T.part,
                       grad_splits(n), grad);
    return hipGetLastError();
}

hipError_t launch_reduce_adam(float* p, const TrainBuffers& T, int64_t n, const float* grad, float* m, float* v, float lr,
                              float b1, float b2, float eps, int64_t t, const RankerWeights& W, hipStream_t s) {
    const float c1 = 1.f - powf(b1, (float)t), c2 = 1.f - powf(b2, (float)t);
    hipLaunchKernelGGL(k_reduce_adam, dim3((unsigned)((W.layout.count + 255) / 256)), dim3(256), 0, s, p, T.part,
                       grad_splits(n), grad, m, v, lr, b1, b2, eps, c1, c2, W);
    return hipGetLastError();
}

}  // namespace tmk
