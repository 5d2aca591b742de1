// tm_ranker.h -- internal interface of the learned ranker (kernels <-> host).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tm_internal.h"

namespace tmk {

constexpr int kFeat = 64;    // features per candidate
constexpr int kWidth = 256;  // hidden width (three hidden layers)
constexpr int kOut = 2;      // heads: log2(1 + bytes), log2(1 + inter-node bytes), standardised

// Offsets (in floats) of each tensor in the flat fp32 parameter vector.
struct RankerLayout {
    int64_t w1, b1, w2, b2, w3, b3, w4, b4, count;
};

constexpr RankerLayout ranker_layout() {
    RankerLayout L{};
    L.w1 = 0;                              // [kFeat][kWidth] row-major (in, out)
    L.b1 = L.w1 + kFeat * kWidth;          // [kWidth]
    L.w2 = L.b1 + kWidth;                  // [kWidth][kWidth]
    L.b2 = L.w2 + kWidth * kWidth;
    L.w3 = L.b2 + kWidth;                  // [kWidth][kWidth]
    L.b3 = L.w3 + kWidth * kWidth;
    L.w4 = L.b3 + kWidth;                  // [kWidth][kOut]
    L.b4 = L.w4 + kWidth * kOut;           // [kOut]
    L.count = L.b4 + kOut;
    return L;
}

// bf16 matrices the MFMA kernels read lie in fragment order: a matrix of C columns with
// the reduction index k as blocks of 16 columns x 32 k, each block the 1 KB that one
// fragment load of a wave takes, lane l's 16 bytes (column l % 16, k 8 (l / 16) ..) at
// 16 l.  A load then reads eight whole cache lines.
__host__ __device__ inline int64_t frag_at(int64_t c, int64_t k, int64_t blocks_k) {
    return ((c / 16 * blocks_k + k / 32) * 64 + (k % 32) / 8 * 16 + c % 16) * 8 + k % 8;
}

// Device views of the weights: bf16 fragments of each layer's product (f: output columns,
// reduced over inputs) and of its transpose (g: input columns, reduced over outputs);
// biases are read from the fp32 master vector.
struct RankerWeights {
    uint16_t *f1, *f2, *f3, *g2, *g3, *w4;
    const float *b1, *b2, *b3, *b4;
    RankerLayout layout;
};

// Writes the bf16 copies of master parameter i.
__device__ __forceinline__ void publish_param(int64_t i, float v, const RankerWeights& W) {
    uint32_t u = __float_as_uint(v);
    u += 0x7fffu + ((u >> 16) & 1u);
    const uint16_t h = (uint16_t)(u >> 16);
    const RankerLayout& L = W.layout;
    if (i >= L.w1 && i < L.b1) {
        const int64_t j = i - L.w1, r = j / kWidth, c = j % kWidth;
        W.f1[frag_at(c, r, kFeat / 32)] = h;
    } else if (i >= L.w2 && i < L.b2) {
        const int64_t j = i - L.w2, r = j / kWidth, c = j % kWidth;
        W.f2[frag_at(c, r, kWidth / 32)] = h;
        W.g2[frag_at(r, c, kWidth / 32)] = h;
    } else if (i >= L.w3 && i < L.b3) {
        const int64_t j = i - L.w3, r = j / kWidth, c = j % kWidth;
        W.f3[frag_at(c, r, kWidth / 32)] = h;
        W.g3[frag_at(r, c, kWidth / 32)] = h;
    } else if (i >= L.w4 && i < L.b4) {
        W.w4[i - L.w4] = h;
    }
}

// Row ranges of the weight gradients: about 512 rows each (288 workgroups on 4,096 rows),
// at most 16 (their partial gradients are written and read back).
constexpr int kMaxSplits = 16;
inline int grad_splits(int64_t n) {
    const int64_t s = (n + 511) / 512;
    return (int)(s < 1 ? 1 : (s > kMaxSplits ? kMaxSplits : s));
}
// Batches up to this many rows run 16-row tiles.
constexpr int64_t kTrainSmallRows = 4096;

// A minibatch: rows first + i, or perm[first + i], of the features and targets.
struct TrainBatch {
    const float *feat, *target;
    const int64_t* perm;
    int64_t first, n;
};
// Per-batch work buffers, rows padded to npad (a multiple of 32): the features,
// activations and their gradients in fragment order (their columns, reduced over rows);
// fp32 rows; per tile of at least 16 rows its column sums [kColParts] (b1, b2, b3, w4,
// b4); the matrices' gradients per row range [kMaxSplits][count].
constexpr int kColParts = 3 * kWidth + kWidth * kOut + kOut;
struct TrainBuffers {
    uint16_t *X, *H1, *H2, *H3, *D1, *D2, *D3;
    float *Y, *T;
    float *colpart, *part;
    int64_t npad;
};

constexpr int kMaxMrankCross = 8;  // node-crossing fractions kept per candidate
// The descriptor estimate of the ghost cells enters the features as
// log2(1 + est) / kBaseScale at kBaseFeat[0] (feature kBaseFeat[1], the inter-node
// head's base, is 0); the network learns the residual of log2(1 + exact bytes) over
// kBaseScale * feature, so the estimate keeps its fp32 precision instead of passing
// through bf16.
constexpr int kBaseFeat[kOut] = {23, 60};
constexpr float kBaseScale = 32.f;
struct FeatHalo {
    int32_t h[TM_MAX_LRANK];
};
// Features of n candidates: bf16 rows X, fp32 copies f32 (nullable), and the fp32 base of
// each one's score.
hipError_t launch_features(const DevFeat* feats, int64_t n, const FeatHalo& halo, float* base, uint16_t* X, float* f32,
                           hipStream_t s);
// A loaded batch as the block-model estimates read it.
struct EstimateBatch {
    const DevCand* cands;
    const DevEval* evals;
    int32_t max_vol;
    int32_t max_blocks;  // most blocks of all launch dims of a simple candidate
    int32_t halo[TM_MAX_LRANK];
    const int32_t* d_halo;
    bool all_simple;
};
// Block-model estimates of entries 0..n-1: candidate idx[i] (negative: skipped) or i
// without idx; to est[2i..] and, as the second stage's score, score[i] (nullable).
hipError_t launch_estimates(const EstimateBatch& b, const int64_t* idx, int64_t n, float lambda, double* est,
                            float* score, hipStream_t s);
// The ranking scores of rows with these bases (score == nullptr: outputs instead).
struct RankScore {
    const float* base;
    float mu[kOut], sigma[kOut], lambda;
    float* score;
};
// Network outputs Y, or scores, of n rows of bf16 features.
hipError_t launch_mlp_forward(const uint16_t* X, int64_t n, const RankerWeights& W, float* Y, const RankScore& S,
                              hipStream_t s);
// Forward and backward of one batch (s0, s1: the heads' scale of Y - target): Y, T and the
// columns; the bias and head gradients into grad, the matrices' into T.part.
hipError_t launch_gradient(const TrainBatch& B, const RankerWeights& W, float s0, float s1, const TrainBuffers& T,
                           float* grad, hipStream_t s);
// The matrices' gradients into grad; or the Adam step from them.
hipError_t launch_reduce_grad(const RankerLayout& L, const TrainBuffers& T, int64_t n, float* grad, hipStream_t s);
hipError_t launch_reduce_adam(float* p, const TrainBuffers& T, int64_t n, const float* grad, float* m, float* v, float lr,
                              float b1, float b2, float eps, int64_t t, const RankerWeights& W, hipStream_t s);
hipError_t launch_publish(const float* p, int64_t count, const RankerWeights& W, hipStream_t s);
// The k smallest (score, index) entries of each segment (k_select): sel[s*k ..)
// in index order, -1 after; stride > 0 takes segment s as the first
// min(stride, seg[s+1] - seg[s]) entries from s * stride; remap (nullable) maps an
// entry to the index written; n: entries of all segments.
hipError_t launch_select(const float* score, const int64_t* seg, int64_t nseg, int64_t n, int64_t stride, int k,
                         float margin, const int64_t* remap, int64_t* sel, hipStream_t s);

}  // namespace tmk
