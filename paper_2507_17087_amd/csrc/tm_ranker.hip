// tm_ranker.hip -- learned ranker kernels (gfx950): descriptor features, a 3-layer
// BF16 MLP (MFMA v_mfma_f32_16x16x32_bf16, FP32 accumulation) inference, the block-model
// estimates of a ranked search's second stage, and per-segment k-smallest selection.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "tm_chain.h"
#include "tm_groups.h"
#include "tm_internal.h"
#include "tm_mfma.h"
#include "tm_ranker.h"

namespace tmk {

// ------------------------------------------------------------------ features

__device__ __forceinline__ float lg2(double x) { return (float)log2(x); }

// ------------------------------------------------------------------ block-model estimates
//
// The second stage of a ranked search: per candidate the estimated ghost cells and
// inter-node ghost cells (volumes above kCrossMax: 0, 0).  When every launch dim is
// projected by blocks onto exactly one final dim (k_block_estimates), each cell boundary b
// along a launch dim is seen by the min(h, b) + min(h, l - b) cells within the halo of it,
// times the area of the face (the product of the other dims' block widths), counted where
// the owners (or nodes) on its two sides differ -- exact for bijective chains whose blocks
// are at least h wide.  Otherwise (k_crossing_estimates): per launch dim, the (cell,
// distinct foreign coordinate) pairs along it times the other extents times the largest
// fraction of adjacent final coordinates whose owners (nodes) differ.
constexpr int kCrossMax = 16384;
// Most block records in LDS, of one-wave and of four-wave workgroups (of the dims but the
// largest there are at most 130): few, so that workgroups are many.
constexpr int kEstRecordsWave = 256, kEstRecords = 4096;
constexpr int kStatsStage = 1024;     // launch dims up to this extent have their contributions staged in LDS
constexpr int kStatsSmallVol = 2048;  // owner-table words of the first (small-candidate) launch

// The second stage's scores of n estimates: log2(1 + cells) + lambda log2(1 + inter-node
// cells); +inf when that is not finite.  A launch of its own: in the estimates' workgroups
// one lane would run the two 64-bit logarithms for all.
__global__ __launch_bounds__(256) void k_estimate_scores(const double2* __restrict__ est, int64_t n, float lambda,
                                                         float* __restrict__ score) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double2 e = est[i];
    const float b0 = kBaseScale * (lg2(1.0 + e.x) / kBaseScale), b1 = kBaseScale * (lg2(1.0 + e.y) / kBaseScale);
    const float v = b0 + lambda * b1;
    score[i] = __builtin_isfinite(v) ? v : INFINITY;
}

typedef double f64x2 __attribute__((ext_vector_type(2), aligned(8)));  // a caller's rows

struct EstimateArgs {
    const DevEval* evals;
    const int64_t* idx;
    int64_t n;
    int32_t halo[TM_MAX_LRANK];
    int32_t vmin, vmax;  // volumes this launch takes: above vmin, up to vmax (kCrossMax: zeros beyond)
    int32_t cap;         // LDS words of keys: the largest volume it meets
    int32_t records;     // block records there is room for
    double* est;
};

// A workgroup per entry: the owner table and, per launch dim and block of it, a record in
// LDS -- cells of the block; offset to the final coordinate of the cell before it, and cells
// that see its boundary (none before the first block) -- then a thread per tuple of blocks.
// A block starts at cell ceil(a l / s), in closed form; every sum is of whole numbers below
// 2^53, exact in any order.  Bound: VALU issue (as the stencil evaluation).  Measured on
// 116,992 kept candidates: block tables in LDS and a descriptor of 960 bytes staged word by
// word 741 us, blocks and boundaries computed per final coordinate 285, these records 248,
// with 256 of them at most (six workgroups a CU more) and a shorter owner table 203.
template <int NT>
__global__ __launch_bounds__(NT) void k_block_estimates(const EstimateArgs A) {
    extern __shared__ __attribute__((aligned(16))) int32_t key[];  // owners, then the records
    __shared__ DevEval ev;
    __shared__ double dred[NT / 64][2];
    constexpr int NW = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63;
    i32x2* rec = reinterpret_cast<i32x2*>(key + A.cap);
    for (int64_t i = blockIdx.x; i < A.n; i += gridDim.x) {
        const int64_t ci = A.idx ? wave_uniform64(A.idx[i]) : i;
        if (ci < 0) continue;
        if (i != (int64_t)blockIdx.x) lds_sync(NW);  // the previous entry's LDS is no longer read
        stage_eval(&ev, A.evals + ci, tid);
        lds_sync(NW);
        const int32_t vol = wave_uniform(ev.vol);
        if (!(wave_uniform(ev.flags) & kEvalSimple)) continue;
        const bool beyond = vol > kCrossMax && A.vmax == kCrossMax;
        if (!beyond && (vol <= A.vmin || vol > A.vmax)) continue;
        double tot = 0, inter = 0;
        if (!beyond) {
            const int K = wave_uniform(ev.lrank), gb = wave_uniform(ev.gbits);
            owner_table(ev, key, 0, vol, -1, tid, NT);
            // per launch dim: its final dim's size and stride (one block without a projection)
            int32_t st[TM_MAX_LRANK], size[TM_MAX_LRANK], rest = 0, most = 0, D = 0;
#pragma unroll
            for (int d = 0; d < TM_MAX_LRANK; ++d) {
                const bool on = d < K && wave_uniform(ev.dim[d].nblk) > 0;
                const int j = on ? wave_uniform(ev.dim[d].first) : 0;
                size[d] = on ? wave_uniform(ev.pj[j].s) : 1;
                st[d] = on ? wave_uniform(ev.pj[j].stride) : 0;
                rest += d < K ? size[d] : 0;
                if (d < K && size[d] > most) {
                    most = size[d];
                    D = d;
                }
            }
            rest -= most;
            // the records of every dim, of the largest (D) as many at a time as there is room
            // for (A.records)
            const int32_t room = A.records - rest;
            for (int32_t g0 = 0; g0 < most; g0 += room) {
                if (g0 > 0) lds_sync(NW);  // the previous range's are no longer read
                int32_t sz[TM_MAX_LRANK], lo[TM_MAX_LRANK], first[TM_MAX_LRANK], all = 0;
                uint32_t tuples = 1;
                float rsz[TM_MAX_LRANK];
#pragma unroll
                for (int d = 0; d < TM_MAX_LRANK; ++d) {
                    lo[d] = d == D ? g0 : 0;
                    sz[d] = d == D ? (most - g0 < room ? most - g0 : room) : size[d];
                    rsz[d] = 1.0f / (float)sz[d];
                    first[d] = all;
                    all += d < K ? sz[d] : 0;
                    tuples *= (uint32_t)sz[d];
                }
                for (int32_t r = tid; r < all; r += NT) {
                    int d = 0;
                    int32_t f = -lo[0];
                    uint32_t h = (uint32_t)A.halo[0];
#pragma unroll
                    for (int e = 1; e < TM_MAX_LRANK; ++e)
                        if (e < K && r >= first[e]) {
                            d = e;
                            f = first[e] - lo[e];
                            h = (uint32_t)A.halo[e];
                        }
                    const LaneDim ld = lane_dim(ev, d, false);
                    const uint32_t x = (uint32_t)(r - f);
                    const double rs = ld.nblk ? ld.brs : 1.0, n0 = fma((double)x, (double)ld.l, ld.bs - 1.0);
                    const uint32_t x0 = div_wide(n0, rs), cells = div_wide(n0 + (double)ld.l, rs) - x0;
                    uint32_t seen = 0, off = 0;
                    if (x > 0 && cells > 0) {  // else no boundary, or an empty block
                        const uint32_t after = ld.l - x0;
                        seen = (h < x0 ? h : x0) + (h < after ? h : after);
                        off = (x - block_index(x0 - 1, ld.bs, ld.rl)) * ld.bst;
                    }
                    rec[r] = i32x2{(int32_t)cells, (int32_t)(off | seen << 16)};
                }
                lds_sync(NW);
                for (uint32_t t = tid; t < tuples; t += NT) {
                    uint32_t q = t;
                    int32_t v = 0;
                    i32x2 e[TM_MAX_LRANK];
                    double wd[TM_MAX_LRANK];
#pragma unroll
                    for (int d = TM_MAX_LRANK - 1; d >= 0; --d) {
                        wd[d] = 1;
                        if (d >= K) continue;
                        const uint32_t hi = d > 0 ? div_small(q, rsz[d]) : 0, x = q - __umul24(hi, (uint32_t)sz[d]);
                        q = hi;
                        e[d] = rec[first[d] + (int32_t)x];
                        v += (int32_t)__umul24(x + (uint32_t)lo[d], (uint32_t)st[d]);
                        wd[d] = (double)(uint32_t)e[d].x;
                    }
                    const int32_t kv = key[v];
#pragma unroll
                    for (int d = 0; d < TM_MAX_LRANK; ++d) {
                        if (d >= K) continue;
                        const int32_t kl = key[v - (e[d].y & 0xffff)];
                        const uint32_t seen = (uint32_t)e[d].y >> 16;
                        double w = 1;
#pragma unroll
                        for (int f = 0; f < TM_MAX_LRANK; ++f)
                            if (f != d && f < K) w *= wd[f];
                        tot = fma((double)(kl != kv ? seen : 0u), w, tot);
                        inter = fma((double)((kl >> gb) != (kv >> gb) ? seen : 0u), w, inter);
                    }
                }
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                tot += __shfl_xor(tot, o, 64);
                inter += __shfl_xor(inter, o, 64);
            }
            if (NW > 1) {
                if (lane == 0) {
                    dred[tid >> 6][0] = tot;
                    dred[tid >> 6][1] = inter;
                }
                __syncthreads();
                for (int w = 1; w < NW; ++w) {
                    tot += tid == 0 ? dred[w][0] : 0.0;
                    inter += tid == 0 ? dred[w][1] : 0.0;
                }
            }
        }
        if (tid == 0) *reinterpret_cast<f64x2*>(A.est + 2 * i) = f64x2{tot, inter};
    }
}

__global__ __launch_bounds__(256) void k_crossing_estimates(const DevCand* __restrict__ cands,
                                                            const int32_t* __restrict__ d_halo, EstimateArgs A) {
    __shared__ DevCand sc;
    // dynamic LDS: the owner keys (cap words), then a launch dim's contributions
    extern __shared__ __attribute__((aligned(16))) int32_t key[];
    int32_t* s_ct = key + A.cap;
    __shared__ int32_t red[kMaxMrankCross][4][2];  // per final dim and wave: node and owner changes
    __shared__ double dred[4][2];
    __shared__ float s_cross[2 * kMaxMrankCross];  // this candidate's crossing fractions
    __shared__ float s_rt[kRecipSlots];             // reciprocals of the inverse chain's divisors
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nw = blockDim.x >> 6;
    for (int64_t i = blockIdx.x; i < A.n; i += gridDim.x) {
        const int64_t ci = A.idx ? wave_uniform64(A.idx[i]) : i;
        if (ci < 0 || (wave_uniform(A.evals[ci].flags) & kEvalSimple)) continue;
        const int32_t v0 = wave_uniform(cands[ci].vol);
        const bool beyond = v0 > kCrossMax && A.vmax == kCrossMax;
        if (!beyond && (v0 <= A.vmin || v0 > A.vmax)) continue;
        double tot = 0, inter = 0;
        if (!beyond) {
            lds_sync(nw);
            stage_cand(&sc, &cands[ci]);
            lds_sync(nw);
            op_reciprocals(sc, s_rt, tid, blockDim.x);
            lds_sync(nw);
            const int32_t vol = sc.vol;
            const int K = wave_uniform(sc.lrank), gb = wave_uniform(sc.gbits), fr = wave_uniform(sc.frank);
            const int nj = fr < kMaxMrankCross ? fr : kMaxMrankCross;
            int32_t fs[kMaxMrankCross], fst[kMaxMrankCross];
            float rfs[kMaxMrankCross];
#pragma unroll
            for (int j = 0; j < kMaxMrankCross; ++j) {
                fs[j] = j < fr ? wave_uniform(sc.fshape[j]) : 1;
                fst[j] = j < fr ? wave_uniform(sc.fstride[j]) : 0;
                rfs[j] = j < fr ? s_rt[kRecipFinal + j] : 1.0f;
            }
            owner_keys_sized(sc, s_rt, key, 0, 0, vol, -1, tid, blockDim.x);
            lds_sync(nw);
            // per final dim the adjacent pairs (v, v + e_j) that change owner / node, as
            // owner changes << 16 | node changes (each at most the volume, below 2^16,
            // also summed over a wave)
            int32_t ch[kMaxMrankCross];
#pragma unroll
            for (int j = 0; j < kMaxMrankCross; ++j) ch[j] = 0;
            for (int32_t v = tid; v < vol; v += blockDim.x) {
                uint32_t rem = (uint32_t)v;
                const int32_t kv = key[v];
#pragma unroll
                for (int j = kMaxMrankCross - 1; j >= 0; --j) {
                    const uint32_t q = j < fr ? div24(rem, (uint32_t)fs[j], rfs[j]) : rem;
                    const int32_t a = j < fr ? (int32_t)(rem - __umul24(q, (uint32_t)fs[j])) : 0;
                    rem = q;
                    if (j < nj && a < fs[j] - 1) {
                        const int32_t kn = key[v + fst[j]];
                        ch[j] += ((kn != kv) << 16) | ((kn >> gb) != (kv >> gb));
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < kMaxMrankCross; ++j) {
                if (j < nj) {
#pragma unroll
                    for (int o2 = 32; o2 > 0; o2 >>= 1) ch[j] += __shfl_xor(ch[j], o2, 64);
                    if (lane == 0) {
                        red[j][wv][0] = ch[j] & 0xffff;
                        red[j][wv][1] = ch[j] >> 16;
                    }
                }
            }
            lds_sync(nw);
            if (tid < kMaxMrankCross) {
                float fn = 0.f, fp = 0.f;
                if (tid < nj) {
                    // pairs (v, v + e_j): the coordinates with a_j < S_j - 1
                    const int32_t Sj = sc.fshape[tid];
                    const int pairs = (Sj - 1) * (vol / Sj);
                    int dn = 0, dp = 0;
                    for (int w = 0; w < nw; ++w) {
                        dn += red[tid][w][0];
                        dp += red[tid][w][1];
                    }
                    const float inv = pairs ? 1.f / (float)pairs : 0.f;
                    fn = (float)dn * inv;
                    fp = (float)dp * inv;
                }
                s_cross[tid] = fn;
                s_cross[kMaxMrankCross + tid] = fp;
            }
            lds_sync(nw);
            for (int d = 0; d < K; ++d) {
                const int64_t l = sc.extent[d];
                const int h = d_halo[d];
                double part = 0;
                if (h > 0 && l <= 65536) {
                    const bool staged = l <= kStatsStage;  // uniform
                    if (staged) {
                        for (int32_t x = tid; x < (int32_t)l; x += blockDim.x) s_ct[x] = coord_value(sc, d, x);
                        lds_sync(nw);
                    }
                    for (int64_t x = tid; x < l; x += blockDim.x) {
                        const int32_t val = staged ? s_ct[x] : coord_value(sc, d, x);
                        int32_t found[2 * kMaxHalo];
                        int cnt = 0;
                        for (int sft = 1; sft <= h && sft <= kMaxHalo; ++sft)
                            for (int dir = 0; dir < 2; ++dir) {
                                const int64_t xx = dir ? x + sft : x - sft;
                                if (xx < 0 || xx >= l) continue;
                                const int32_t dv = (staged ? s_ct[xx] : coord_value(sc, d, xx)) - val;
                                bool seen = dv == 0;
                                for (int u = 0; u < cnt; ++u) seen = seen || found[u] == dv;
                                if (!seen) found[cnt++] = dv;
                            }
                        part += cnt;
                    }
                    if (staged) lds_sync(nw);  // the next dim rewrites s_ct
                }
                float cn = 0.f, cp = 0.f;
                for (int j = 0; j < sc.frank && j < kMaxMrankCross; ++j)
                    if (sc.proj_src[j] == d) {
                        cn = fmaxf(cn, s_cross[j]);
                        cp = fmaxf(cp, s_cross[kMaxMrankCross + j]);
                    }
                double pts = 1;
                for (int dd = 0; dd < K; ++dd)
                    if (dd != d) pts *= (double)sc.extent[dd];
                tot += part * pts * cp;
                inter += part * pts * cn;
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                tot += __shfl_xor(tot, o, 64);
                inter += __shfl_xor(inter, o, 64);
            }
            if (lane == 0) {
                dred[wv][0] = tot;
                dred[wv][1] = inter;
            }
            lds_sync(nw);
            tot = inter = 0;
            for (int w = 0; w < nw; ++w) {
                tot += dred[w][0];
                inter += dred[w][1];
            }
        }
        if (tid == 0) *reinterpret_cast<f64x2*>(A.est + 2 * i) = f64x2{tot, inter};
    }
}

hipError_t launch_estimates(const EstimateBatch& b, const int64_t* idx, int64_t n, float lambda, double* est,
                            float* score, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const unsigned g = (unsigned)std::min<int64_t>(n, int64_t(1) << 20);
    const int32_t top = std::max(1, std::min(b.max_vol, kCrossMax));
    EstimateArgs A{};
    A.evals = b.evals;
    A.idx = idx;
    A.n = n;
    for (int d = 0; d < TM_MAX_LRANK; ++d) A.halo[d] = b.halo[d];
    A.est = est;
    // most candidates are small: a first launch with a small owner table in LDS (more
    // workgroups per CU) takes the volumes up to kStatsSmallVol, a second one, sized for
    // the batch's largest, the rest; large batches take one-wave workgroups
    for (int pass = 0; pass < (top > kStatsSmallVol ? 2 : 1); ++pass) {
        A.vmin = pass ? kStatsSmallVol : 0;
        const bool last = pass || top <= kStatsSmallVol;
        A.vmax = last ? kCrossMax : kStatsSmallVol;
        A.cap = ((last ? top : kStatsSmallVol) + 3) & ~3;
        const size_t lds = (size_t)A.cap * 4;
        A.records = std::min({b.max_blocks, A.cap + TM_MAX_LRANK, n >= kSmallBlockBatch ? kEstRecordsWave : kEstRecords});
        const size_t records = (size_t)A.records * 8;
        if (n >= kSmallBlockBatch)
            hipLaunchKernelGGL(k_block_estimates<64>, dim3(g), dim3(64), lds + records, s, A);
        else
            hipLaunchKernelGGL(k_block_estimates<256>, dim3(g), dim3(256), lds + records, s, A);
        if (!b.all_simple)
            hipLaunchKernelGGL(k_crossing_estimates, dim3(g), dim3(n >= kSmallBlockBatch ? 64 : 256),
                               lds + kStatsStage * 4, s, b.cands, b.d_halo, A);
    }
    if (score)
        hipLaunchKernelGGL(k_estimate_scores, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                           reinterpret_cast<const double2*>(est), n, lambda, score);
    return hipGetLastError();
}

// A candidate's DevFeat unpacked.
struct FeatDesc {
    int k, nops, nodes, gpus, gbits, fr;
    int32_t ext[TM_MAX_LRANK];
    int32_t fsh[TM_MAX_MRANK];
    uint32_t proj, kinds, opa;
    int32_t opb[6];
    int32_t F[TM_MAX_LRANK];
    __device__ __forceinline__ int src(int j) const { return (int)(proj >> (4 * j)) & 7; }
    __device__ __forceinline__ bool cyclic(int j) const { return (proj >> (4 * j + 3)) & 1u; }
    __device__ __forceinline__ int kind(int t) const { return (int)(kinds >> (4 * t)) & 15; }
};

__device__ __forceinline__ FeatDesc unpack_feat(const int4* q) {
    FeatDesc d;
    const int4 e = q[0], m = q[1], s0 = q[2], s1 = q[3], b0 = q[4], b1 = q[5], f = q[6];
    d.ext[0] = e.x, d.ext[1] = e.y, d.ext[2] = e.z, d.ext[3] = e.w;
    d.nodes = m.x, d.gpus = m.y;
    d.k = m.z & 255, d.nops = (m.z >> 8) & 255, d.gbits = (m.z >> 16) & 255, d.fr = (m.z >> 24) & 255;
    d.kinds = (uint32_t)m.w;
    d.fsh[0] = s0.x, d.fsh[1] = s0.y, d.fsh[2] = s0.z, d.fsh[3] = s0.w;
    d.fsh[4] = s1.x, d.fsh[5] = s1.y, d.fsh[6] = s1.z, d.fsh[7] = s1.w;
    d.opb[0] = b0.x, d.opb[1] = b0.y, d.opb[2] = b0.z, d.opb[3] = b0.w, d.opb[4] = b1.x, d.opb[5] = b1.y;
    d.opa = (uint32_t)b1.z;
    d.proj = (uint32_t)b1.w;
    d.F[0] = f.x, d.F[1] = f.y, d.F[2] = f.z, d.F[3] = f.w;
    return d;
}

// Descriptor estimate of the ghost cells, from the shapes alone: if every change of
// the final coordinates projected from a launch dim changes the processor (a
// bijective chain), the processor changes along launch dim d at l - 1 coordinate
// boundaries when a final dim of size > 1 is projected onto it cyclically, and
// otherwise at the interior block starts of its block-projected final dims (at most
// the sum of their sizes less one each, and at most l - 1); every boundary puts 2h
// cells of each cross-section into the halo.  Exact for bijective chains with one
// final dim per launch dim whose blocks are at least h wide.
__device__ __forceinline__ double descriptor_estimate(const FeatDesc& c, const int32_t (&halo)[TM_MAX_LRANK]) {
    double cells = 0;
#pragma unroll
    for (int d = 0; d < TM_MAX_LRANK; ++d) {
        if (d >= c.k) continue;
        const int64_t l = c.ext[d];
        int64_t nb = 0;
        bool cyc = false;
#pragma unroll
        for (int j = 0; j < TM_MAX_MRANK; ++j) {
            if (j >= c.fr || c.src(j) != d) continue;
            if (c.cyclic(j)) cyc = cyc || c.fsh[j] > 1;
            else nb += c.fsh[j] - 1;
        }
        nb = cyc ? l - 1 : (nb < l - 1 ? nb : l - 1);
        double face = 1;
#pragma unroll
        for (int e = 0; e < TM_MAX_LRANK; ++e)
            if (e < c.k && e != d) face *= (double)c.ext[e];
        cells += 2.0 * halo[d] * (double)nb * face;
    }
    return cells;
}

// log2 in fp32 for the features other than the estimate's (they are compared with
// the fp64 reference at 1e-5 and stored in bf16)
__device__ __forceinline__ float lg2f(float x) { return log2f(x); }

// A thread per candidate: kFeat bf16 values (a row of X), the base of its score (the
// descriptor estimate in the target's log space; the inter-node head has none) and, when
// feat_f32 is given, the features in fp32.  A wave's descriptors come in, and its rows go
// out, as whole lines through LDS.
//
// Bound: HBM bytes, 260 a candidate.  1.03M candidates: 57 us (4.7 TB/s); reading the
// fields where they lie in the 960-byte descriptors, five to six lines of each, 162 us.
constexpr int kFeatStride = 36;  // LDS words of a row: 16-byte pieces of eight lanes on distinct banks
__global__ __launch_bounds__(64) void k_features(const DevFeat* __restrict__ feats, int64_t n, const FeatHalo halo,
                                                 float* __restrict__ base, uint16_t* __restrict__ X,
                                                 float* __restrict__ feat_f32) {
    __shared__ __attribute__((aligned(16))) int32_t rows[64 * kFeatStride];
    const int tid = threadIdx.x;
    const int64_t first = blockIdx.x * (int64_t)64, i = first + tid;
    const int here = (int)(n - first < 64 ? n - first : 64);
    constexpr int kPieces = (int)sizeof(DevFeat) / 16;
    static_assert(sizeof(DevFeat) == 128 && kFeat * 2 == 128, "a descriptor and a row of X are eight 16-byte pieces");
    const int4* src = reinterpret_cast<const int4*>(feats + first);
#pragma unroll
    for (int t = 0; t < kPieces; ++t) {
        const int p = t * 64 + tid;
        if (p < here * kPieces) *reinterpret_cast<int4*>(rows + (p >> 3) * kFeatStride + (p & 7) * 4) = src[p];
    }
    lds_sync(1);
    const FeatDesc c = unpack_feat(reinterpret_cast<const int4*>(rows + (tid < here ? tid : 0) * kFeatStride));
    lds_sync(1);
    // every index into f and the small arrays below is static once the loops are
    // unrolled (bounded by the ABI's maxima, the candidate's counts as predicates), so
    // all of them live in registers
    float f[kFeat];
#pragma unroll
    for (int t = 0; t < kFeat; ++t) f[t] = 0.f;
    const int k = c.k, fr = c.fr, nops = c.nops;
#pragma unroll
    for (int d = 0; d < TM_MAX_LRANK; ++d) f[d] = d == k - 1 ? 1.f : 0.f;
    // blocks per launch dim: the product of the final extents it projects onto
    double blocks[TM_MAX_LRANK] = {1, 1, 1, 1};
#pragma unroll
    for (int j = 0; j < TM_MAX_MRANK; ++j) {
        if (j < fr) {
            const int src = c.src(j);
            const double sh = (double)c.fsh[j];
#pragma unroll
            for (int d = 0; d < TM_MAX_LRANK; ++d) blocks[d] *= src == d ? sh : 1.0;
        }
    }
    int32_t hl[TM_MAX_LRANK];
#pragma unroll
    for (int d = 0; d < TM_MAX_LRANK; ++d) hl[d] = d < k ? halo.h[d] : 0;
    double vol_f = 0;
#pragma unroll
    for (int d = 0; d < TM_MAX_LRANK; ++d) {
        if (d < k) {
            const double l = (double)c.ext[d];
            const float ll = lg2f((float)l), lb = lg2f((float)blocks[d]);
            f[4 + d] = ll / 10.f;
            f[15 + d] = lb / 9.f;
            f[19 + d] = (ll - lb) / 10.f;
            vol_f += 2.0 * hl[d] * (c.F[d] - 1.0) / l;
            f[54 + d] = hl[d] / 4.f;
        }
    }
    f[8] = lg2f((float)c.nodes) / 6.f;
    f[9] = lg2f((float)c.gpus) / 3.f;
    f[10] = lg2f((float)c.nodes * (float)c.gpus) / 9.f;
#pragma unroll
    for (int m = 0; m < TM_MAX_LRANK; ++m)
        f[11 + m] = lg2f((float)c.F[m]) / 9.f;
    f[24] = lg2f((float)(1.0 + vol_f)) / 4.f;
#pragma unroll
    for (int t = 0; t < TM_MAX_OPS; ++t) {
        if (t < nops) {
            const int kd = c.kind(t);
#pragma unroll
            for (int q = 0; q < 5; ++q) f[25 + q] += kd == q + 1 ? 0.25f : 0.f;
            if (t < 6) {
                f[30 + t] = kd / 5.f;
                if (t < 3) f[39 + t] = (float)((c.opa >> (8 * t)) & 255u) / 8.f;
                f[42 + t] = kd == TM_DECOMPOSE ? 0.f : lg2f(1.f + (float)c.opb[t < 6 ? t : 0]) / 9.f;
            }
        }
    }
    f[48] = (nops > 0 && c.kind(0) == TM_SWAP) ? 1.f : 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (j < fr) f[49 + j] = c.cyclic(j) ? 1.f : 0.f;
    f[53] = fr / 8.f;
    f[58] = c.gbits / 3.f;
    f[59] = 1.f;
    // the descriptor estimate of the ghost cells in the log space of the target (the
    // inter-node head has no base: feature kBaseFeat[1] stays 0)
    f[kBaseFeat[0]] = lg2(1.0 + descriptor_estimate(c, hl)) / kBaseScale;
    if (tid < here) base[i] = f[kBaseFeat[0]];
#pragma unroll
    for (int t = 0; t < kFeat / 8; ++t) {
        uint4 w;
        w.x = pack_bf16(f[8 * t], f[8 * t + 1]);
        w.y = pack_bf16(f[8 * t + 2], f[8 * t + 3]);
        w.z = pack_bf16(f[8 * t + 4], f[8 * t + 5]);
        w.w = pack_bf16(f[8 * t + 6], f[8 * t + 7]);
        *reinterpret_cast<uint4*>(rows + tid * kFeatStride + t * 4) = w;
    }
    lds_sync(1);
    int4* dst = reinterpret_cast<int4*>(X + first * kFeat);
#pragma unroll
    for (int t = 0; t < kPieces; ++t) {
        const int p = t * 64 + tid;
        if (p < here * kPieces) dst[p] = *reinterpret_cast<const int4*>(rows + (p >> 3) * kFeatStride + (p & 7) * 4);
    }
    if (feat_f32 && tid < here) {
        float4* fo = reinterpret_cast<float4*>(feat_f32 + i * kFeat);
#pragma unroll
        for (int t = 0; t < kFeat / 4; ++t) fo[t] = make_float4(f[4 * t], f[4 * t + 1], f[4 * t + 2], f[4 * t + 3]);
    }
}

// ------------------------------------------------------------------ fused forward
//
// A workgroup of the forward pass (8 waves) takes 64 rows.  Activations stay in LDS
// (bf16); wave w computes output columns [32w, 32w + 32) of
// each hidden layer as 4 x 2 MFMA tiles, reading weight fragments straight from
// the bf16 weights in fragment order (16 contiguous bytes per lane).  Measured on
// 1M rows: 8 waves of 32 columns 0.58 ms, 4 of 64 columns 0.63 ms, 16 of 16
// columns 0.72 ms, 128-row workgroups 0.70 ms.  The tiles are computed
// transposed (weights as the first operand), so a lane ends with four consecutive
// columns of one row: the epilogue (bias, ReLU, round to bf16) writes them to LDS
// as one 8-byte store.
// The head (256 -> 2) is one more MFMA tile per wave against the two weight columns
// staged in LDS (the other 14 columns zero): bf16 products summed in fp32.

// What becomes of a row's two outputs: written to Y, or combined into a ranking score,
// predicted log2(1 + bytes) + lambda * predicted log2(1 + inter-node bytes), each the
// estimate's base (the same fp32 value training used; the inter-node head has none) plus
// the un-standardised residual; +inf when that is not finite: a score of diverged or
// corrupt parameters ranks last, by index, so that such candidates stay selectable and
// every instance keeps its survivors.  acc: rows row .. row + 3, output r16.
__device__ __forceinline__ void put_outputs(const f32x4& acc, float hb, int r16, const f32x4& base, int64_t row,
                                            int64_t n, float* __restrict__ Y, const RankScore& S) {
    if (S.score) {
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float y = acc[r] + hb, y1 = __shfl_down(y, 1, 64);
            const float b0 = kBaseScale * base[r], b1 = 0.f;
            const float p0 = b0 + S.mu[0] + S.sigma[0] * y, p1 = b1 + S.mu[1] + S.sigma[1] * y1;
            const float sc = p0 + S.lambda * p1;
            v[r] = __builtin_isfinite(sc) ? sc : INFINITY;
        }
        if (r16 == 0) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (row + r < n) S.score[row + r] = v[r];
        }
    } else if (r16 < kOut) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (row + r < n) Y[(row + r) * kOut + r16] = acc[r] + hb;
    }
}

// The bases of rows row .. row + 3.
__device__ __forceinline__ f32x4 score_bases(const RankScore& S, int64_t row, int64_t n) {
    f32x4 b = {0.f, 0.f, 0.f, 0.f};
    if (S.score) {
#pragma unroll
        for (int r = 0; r < 4; ++r) b[r] = S.base[row + r < n ? row + r : n - 1];
    }
    return b;
}

constexpr int kRowsMlp = 64;    // rows per workgroup of the forward pass
constexpr int kMlpThreads = 512;
constexpr int kMlpNB = kWidth / 16 / (kMlpThreads / 64);  // 16-column blocks per wave
constexpr int kMlpInferCus = 256;  // persistent inference workgroups (one per CU)

// Activations lie in LDS in fragment order too: row r, reduction index k of a tile at
// frag_at(r, k, blocks of k).  A fragment read and a wave's epilogue write (one 16-byte
// piece a lane) are then 1 KB in lane order, and no bank is asked twice in a cycle; rows of
// a padded stride cannot do that, since a 16-byte read takes its lanes in groups that mix
// the quarters of a fragment: half of the LDS cycles were conflicts.
constexpr int kActElems = kRowsMlp * kWidth;

// Row block a's fragment of reduction block ks, of nk.
__device__ __forceinline__ u16x8 act_frag(const uint16_t* __restrict__ lds, int a, int ks, int nk, int lane) {
    return *reinterpret_cast<const u16x8*>(lds + ((a * nk + ks) * 64 + lane) * 8);
}

// A wave's 32 output columns are dealt to its two column blocks in fours, so that a lane
// (quarter q of the fragment) ends with the eight columns cbase + 8 q ..: position i of
// block b is column cbase + 8 (i / 4) + 4 b + i % 4.
static_assert(kMlpNB == 2, "two blocks of 16 columns a wave");
__device__ __forceinline__ const uint16_t* weight_frag(const uint16_t* __restrict__ F, int b, int ks, int nk, int lane,
                                                       int cbase) {
    const int c = cbase + (lane & 12) * 2 + b * 4 + (lane & 3);
    return F + frag_at(c, ks * 32 + (lane >> 4) * 8, nk);
}

// max(x, 0), NaN -> 0, as fmaxf has it, in one instruction: fmaxf quiets its operand in
// another, and so does a median whose bound the compiler knows to be infinite.
__device__ __forceinline__ float relu(float x) {
    float top = INFINITY;
    asm("" : "+s"(top));
    return __builtin_amdgcn_fmed3f(x, 0.f, top);
}

// acc[a][b][r] (row a*16 + lane%16, column cbase + 8 (lane / 16) + 4 b + r) -> ReLU, bf16,
// to the next layer's activations, one 16-byte piece a row block.
__device__ __forceinline__ void layer_out(const f32x4 (&acc)[4][kMlpNB], uint16_t* __restrict__ out_lds, int lane,
                                          int cbase) {
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        uint4 w;
        w.x = pack_bf16(relu(acc[a][0][0]), relu(acc[a][0][1]));
        w.y = pack_bf16(relu(acc[a][0][2]), relu(acc[a][0][3]));
        w.z = pack_bf16(relu(acc[a][1][0]), relu(acc[a][1][1]));
        w.w = pack_bf16(relu(acc[a][1][2]), relu(acc[a][1][3]));
        *reinterpret_cast<uint4*>(out_lds + ((a * (kWidth / 32) + cbase / 32) * 64 + lane) * 8) = w;
    }
}

// The sums start from the biases (LDS).
__device__ __forceinline__ void layer_start(f32x4 (&acc)[4][kMlpNB], const float* __restrict__ bias, int lane,
                                            int cbase) {
#pragma unroll
    for (int b = 0; b < kMlpNB; ++b) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(bias + cbase + (lane >> 4) * 8 + b * 4);
#pragma unroll
        for (int a = 0; a < 4; ++a) acc[a][b] = v;
    }
}

template <int KIN>
__device__ __forceinline__ void layer_fwd(const uint16_t* __restrict__ in_lds, uint16_t* __restrict__ out_lds,
                                          const uint16_t* __restrict__ F, const float* __restrict__ bias,
                                          int lane, int cbase) {
    f32x4 acc[4][kMlpNB];
    layer_start(acc, bias, lane, cbase);
    // two k-steps in flight
#pragma unroll 2
    for (int ks = 0; ks < KIN / 32; ++ks) {
        u16x8 bf[kMlpNB];
#pragma unroll
        for (int b = 0; b < kMlpNB; ++b)
            bf[b] = *reinterpret_cast<const u16x8*>(weight_frag(F, b, ks, KIN / 32, lane, cbase));
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const u16x8 af = act_frag(in_lds, a, ks, KIN / 32, lane);
#pragma unroll
            for (int b = 0; b < kMlpNB; ++b) acc[a][b] = mfma16(bf[b], af, acc[a][b]);
        }
    }
    layer_out(acc, out_lds, lane, cbase);
}

// The head over 16 rows: B columns 0, 1 are the two heads.
__device__ __forceinline__ f32x4 head_rows(const uint16_t* __restrict__ h3, const uint16_t* __restrict__ w4, int rb,
                                           int lane) {
    const int r16 = lane & 15, kq = (lane >> 4) * 8;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const u16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < kWidth / 32; ++ks) {
        const u16x8 af = act_frag(h3, rb, ks, kWidth / 32, lane);
        const u16x8 wf = *reinterpret_cast<const u16x8*>(w4 + (r16 < kOut ? r16 : 0) * kWidth + ks * 32 + kq);
        acc = mfma16(af, r16 < kOut ? wf : zero, acc);
    }
    return acc;
}

// Head weights transposed and biases to LDS.
__device__ __forceinline__ void stage_small(uint16_t* __restrict__ w4, float* __restrict__ bias, const RankerWeights& W,
                                            int tid) {
    for (int i = tid; i < kOut * kWidth; i += kMlpThreads) w4[(i % kOut) * kWidth + i / kOut] = W.w4[i];
    for (int i = tid; i < kWidth; i += kMlpThreads) {
        bias[i] = W.b1[i];
        bias[kWidth + i] = W.b2[i];
        bias[2 * kWidth + i] = W.b3[i];
    }
}

__global__ __launch_bounds__(kMlpThreads) void k_mlp_forward(const uint16_t* __restrict__ X, int64_t n,
                                                             const RankerWeights W, float* __restrict__ Y, const RankScore S) {
    __shared__ __attribute__((aligned(16))) uint16_t sa[kActElems];
    __shared__ __attribute__((aligned(16))) uint16_t sb[kActElems];
    __shared__ __attribute__((aligned(16))) uint16_t s_w4[kOut * kWidth];
    __shared__ __attribute__((aligned(16))) float s_bias[3 * kWidth];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int cbase = wid * kMlpNB * 16;  // this wave's output columns
    stage_small(s_w4, s_bias, W, tid);
    const float hb = (lane & 15) < kOut ? W.b4[lane & 15] : 0.f;
    for (int64_t row0 = (int64_t)blockIdx.x * kRowsMlp; row0 < n; row0 += (int64_t)gridDim.x * kRowsMlp) {
        __syncthreads();
        // X tile -> sa (kRowsMlp x 64 bf16), zero rows past n
        static_assert(kRowsMlp * (kFeat / 8) == kMlpThreads && kFeat == 64, "one feature piece per thread");
        {
            const int r = (wid >> 1) * 16 + (lane & 15), c8 = (wid & 1) * 32 + (lane >> 4) * 8;
            u16x8 v = {0, 0, 0, 0, 0, 0, 0, 0};
            if (row0 + r < n) v = *reinterpret_cast<const u16x8*>(X + (row0 + r) * kFeat + c8);
            *reinterpret_cast<u16x8*>(sa + tid * 8) = v;
        }
        const f32x4 base = score_bases(S, row0 + (wid % 4) * 16 + (lane >> 4) * 4, n);
        __syncthreads();
        layer_fwd<kFeat>(sa, sb, W.f1, s_bias, lane, cbase);
        __syncthreads();
        layer_fwd<kWidth>(sb, sa, W.f2, s_bias + kWidth, lane, cbase);
        __syncthreads();
        layer_fwd<kWidth>(sa, sb, W.f3, s_bias + 2 * kWidth, lane, cbase);
        __syncthreads();
        if (wid < kRowsMlp / 16)
            put_outputs(head_rows(sb, s_w4, wid, lane), hb, lane & 15, base, row0 + wid * 16 + (lane >> 4) * 4, n, Y, S);
    }
}

// Inference over many rows: a persistent workgroup per CU
// keeps its waves' weight fragments in registers for every row tile it takes, so
// the weights are read from L2 once per workgroup instead of once per tile.
//
// Bound: the three phases of a layer in a workgroup of its own (two waves a SIMD: the
// weights fill the registers): products 299 of 650 thousand cycles of a run over 1.03M rows,
// epilogues 110, LDS reads, barriers and their latencies the rest.  278 us (1.13 PFLOP/s);
// before, 355: padded rows (351 in fragment order), fragments read just before use and
// biases from memory in each epilogue (292 with both mended and three barriers a tile
// instead of four), eight-byte writes and fmaxf (278).
template <int KIN>
__device__ __forceinline__ void load_wfrag(u16x8 (&wf)[KIN / 32][kMlpNB], const uint16_t* __restrict__ F, int lane,
                                           int cbase) {
#pragma unroll
    for (int b = 0; b < kMlpNB; ++b)
#pragma unroll
        for (int ks = 0; ks < KIN / 32; ++ks)
            wf[ks][b] = *reinterpret_cast<const u16x8*>(weight_frag(F, b, ks, KIN / 32, lane, cbase));
}

// A layer from the weights in registers.  The next k-step's fragments are read while this
// one's are multiplied, one read to kMlpNB products: left to itself the compiler reads each
// fragment just before its products and waits out the LDS latency 64 times a tile.
template <int KIN>
__device__ __forceinline__ void layer_reg(const uint16_t* __restrict__ in_lds, uint16_t* __restrict__ out_lds,
                                          const u16x8 (&wf)[KIN / 32][kMlpNB], const float* __restrict__ bias,
                                          int lane, int cbase) {
    constexpr int NK = KIN / 32;
    constexpr int kDsRead = 0x100, kMfma = 0x8;
    f32x4 acc[4][kMlpNB];
    u16x8 cur[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) cur[a] = act_frag(in_lds, a, 0, NK, lane);
    layer_start(acc, bias, lane, cbase);
    __builtin_amdgcn_sched_group_barrier(kDsRead, 4 + kMlpNB, 0);
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
        u16x8 nxt[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            if (ks + 1 < NK) nxt[a] = act_frag(in_lds, a, ks + 1, NK, lane);
#pragma unroll
            for (int b = 0; b < kMlpNB; ++b) acc[a][b] = mfma16(wf[ks][b], cur[a], acc[a][b]);
            if (ks + 1 < NK) __builtin_amdgcn_sched_group_barrier(kDsRead, 1, 0);
            __builtin_amdgcn_sched_group_barrier(kMfma, kMlpNB, 0);
        }
#pragma unroll
        for (int a = 0; a < 4; ++a) cur[a] = nxt[a];
    }
    layer_out(acc, out_lds, lane, cbase);
}

__global__ __launch_bounds__(kMlpThreads) void k_mlp_infer(const uint16_t* __restrict__ X, int64_t n,
                                                           const RankerWeights W, float* __restrict__ Y,
                                                           const RankScore S) {
    __shared__ __attribute__((aligned(16))) uint16_t sx[kRowsMlp * kFeat];
    __shared__ __attribute__((aligned(16))) uint16_t h1[kActElems], h2[kActElems], h3[kActElems];
    __shared__ __attribute__((aligned(16))) uint16_t s_w4[kOut * kWidth];
    __shared__ __attribute__((aligned(16))) float s_bias[3 * kWidth];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int cbase = wid * kMlpNB * 16;
    stage_small(s_w4, s_bias, W, tid);
    u16x8 w1[kFeat / 32][kMlpNB], w2[kWidth / 32][kMlpNB], w3[kWidth / 32][kMlpNB];
    load_wfrag<kFeat>(w1, W.f1, lane, cbase);
    load_wfrag<kWidth>(w2, W.f2, lane, cbase);
    load_wfrag<kWidth>(w3, W.f3, lane, cbase);
    const float hb = (lane & 15) < kOut ? W.b4[lane & 15] : 0.f;
    // one 16-byte piece of a 64 x 64 feature tile per thread; the next tile's piece is
    // loaded while the current tile runs through the layers
    static_assert(kRowsMlp * (kFeat / 8) == kMlpThreads, "one feature piece per thread");
    // (thread t's is the t-th of the tile in fragment order: no bank is written twice)
    const int xr = (wid >> 1) * 16 + (lane & 15), xc = (wid & 1) * 32 + (lane >> 4) * 8;
    static_assert(kFeat == 64, "two reduction blocks of features");
    uint16_t* const xp = sx + tid * 8;
    const int64_t step = (int64_t)gridDim.x * kRowsMlp;
    auto x_piece = [&](int64_t r0) {
        u16x8 v = {0, 0, 0, 0, 0, 0, 0, 0};
        if (r0 + xr < n) v = *reinterpret_cast<const u16x8*>(X + (r0 + xr) * kFeat + xc);
        return v;
    };
    // the head of a tile runs beside the next one's first layer: waves 0..3, 16 rows each
    const int rq = (wid % 4) * 16 + (lane >> 4) * 4;
    f32x4 base = {0.f, 0.f, 0.f, 0.f};
    auto head = [&](int64_t r0) {
        if (wid < kRowsMlp / 16)
            put_outputs(head_rows(h3, s_w4, wid, lane), hb, lane & 15, base, r0 + rq, n, Y, S);
    };
    int64_t row0 = (int64_t)blockIdx.x * kRowsMlp;
    *reinterpret_cast<u16x8*>(xp) = x_piece(row0);
    for (; row0 < n; row0 += step) {
        __syncthreads();  // this tile's features in sx; the previous one's last layer in h3
        const u16x8 xn = x_piece(row0 + step);
        if (row0 >= step) head(row0 - step);
        layer_reg<kFeat>(sx, h1, w1, s_bias, lane, cbase);
        __syncthreads();  // sx is free
        *reinterpret_cast<u16x8*>(xp) = xn;
        layer_reg<kWidth>(h1, h2, w2, s_bias + kWidth, lane, cbase);
        __syncthreads();
        base = score_bases(S, row0 + rq, n);  // for its head
        layer_reg<kWidth>(h2, h3, w3, s_bias + 2 * kWidth, lane, cbase);
    }
    __syncthreads();
    if (row0 >= step) head(row0 - step);
}

// Refresh all bf16 copies from the fp32 master (after loading or setting params).
__global__ __launch_bounds__(256) void k_publish(const float* __restrict__ p, int64_t count, const RankerWeights W) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= count) return;
    publish_param(i, p[i], W);
}

// ------------------------------------------------------------------ k smallest per segment
//
// One workgroup per segment chooses its k smallest (score, index) pairs by a radix
// select over the scores' order-preserving 32-bit keys: three passes of 11, 11 and
// 10 bits, each a histogram in LDS of the keys that share the digits found so far,
// give the k-th smallest key T and how many of the k equal it; one pass in index
// order then takes every key below T and the lowest-indexed keys equal to T.  The
// chosen entries are written in index order, then -1 up to k.  Segment s is
// [seg[s], seg[s+1]), or with stride > 0 the first min(stride, seg[s+1] - seg[s])
// entries from s * stride.  margin > 0 keeps of the chosen only those scoring at
// most `margin` above the segment's best.  remap (nullable) gives the index written
// for entry e (else e).  Scores are finite or +inf.
//
// Bound: latency, of a chain of passes.  Up to kSelKeys keys are kept in LDS after the
// first pass, so that the others do not wait for memory, and a workgroup has 16 waves
// where its segments are long (kSelWide): 457 segments of 2,261 scores 26.7 us, before
// (four waves, every pass from memory) 36.6; 457 of 256 scores 7.4 us with four waves.

__device__ __forceinline__ uint32_t order_key(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
// A key's score (order_key's inverse; NaN has none).
__device__ __forceinline__ float key_score(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? k ^ 0x80000000u : ~k);
}

constexpr int kSelBins = 2048;
constexpr uint32_t kSelKeys = 8192;

template <int NT>
__global__ __launch_bounds__(NT) void k_select(const float* __restrict__ score, const int64_t* __restrict__ seg,
                                               int64_t stride, int k, float margin, const int64_t* __restrict__ remap,
                                               int64_t* __restrict__ sel) {
    constexpr int kWaves = NT / 64, kPer = kSelBins / NT;
    __shared__ uint32_t keys[kSelKeys];
    __shared__ uint32_t hist[kSelBins];
    __shared__ uint32_t wa[kWaves], wb[kWaves];
    __shared__ float wmin[kWaves];
    __shared__ uint32_t s_bin, s_below;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t s = blockIdx.x;
    const int64_t len_s = seg[s + 1] - seg[s];
    const int64_t a = stride > 0 ? s * stride : seg[s];
    const uint32_t len = (uint32_t)(stride > 0 ? (len_s < stride ? len_s : stride) : len_s);
    int64_t* out = sel + s * (int64_t)k;
    const uint64_t lt_mask = (1ull << lane) - 1;
    auto key_at = [&](uint32_t i) { return i < kSelKeys ? keys[i] : order_key(score[a + i]); };
    // the segment's best score (the margin's reference)
    float best = INFINITY;
    for (uint32_t i = tid; i < len; i += NT) {
        const float v = score[a + i];
        best = fminf(best, v);
        if (i < kSelKeys) keys[i] = order_key(v);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) best = fminf(best, __shfl_xor(best, o, 64));
    if (lane == 0) wmin[wv] = best;
    for (int b = tid; b < kSelBins; b += NT) hist[b] = 0;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) best = fminf(best, wmin[w]);
    // the k-th smallest key T; rem = how many of the chosen have key T
    const bool all = len <= (uint32_t)k;
    uint32_t prefix = 0, pmask = 0, rem = all ? len : (uint32_t)k;
    if (!all) {
        for (int pass = 0; pass < 3; ++pass) {
            const int shift = pass == 0 ? 21 : (pass == 1 ? 10 : 0);
            const uint32_t dmask = pass == 2 ? 0x3ffu : 0x7ffu;
            for (uint32_t i = tid; i < len; i += NT) {
                const uint32_t kk = key_at(i);
                if ((kk & pmask) == prefix) atomicAdd(&hist[(kk >> shift) & dmask], 1u);
            }
            __syncthreads();
            uint32_t c[kPer], tsum = 0;
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                c[q] = hist[tid * kPer + q];
                tsum += c[q];
            }
            uint32_t incl = tsum;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t u = __shfl_up(incl, o, 64);
                incl += lane >= o ? u : 0u;
            }
            if (lane == 63) wa[wv] = incl;
            __syncthreads();
            uint32_t run = incl - tsum;
            for (int w = 0; w < wv; ++w) run += wa[w];
            // exactly one bin has run < rem <= run + count
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                if (run < rem && run + c[q] >= rem) {
                    s_bin = (uint32_t)(tid * kPer + q);
                    s_below = run;
                }
                run += c[q];
                hist[tid * kPer + q] = 0;  // for the next pass
            }
            __syncthreads();
            prefix |= s_bin << shift;
            pmask |= dmask << shift;
            rem -= s_below;
            __syncthreads();  // s_bin and s_below are rewritten by the next pass
        }
    }
    // in index order: keys below T, then the first rem keys equal to T
    const uint32_t T = prefix;
    uint32_t seen_eq = 0, written = 0;
    for (uint32_t i0 = 0; i0 < len; i0 += NT) {
        const uint32_t i = i0 + tid;
        bool in = false, eq = false;
        float sv = INFINITY;
        if (i < len) {
            const uint32_t kk = key_at(i);
            sv = key_score(kk);
            in = all || kk < T;
            eq = !all && kk == T;
        }
        const uint64_t beq = __ballot(eq);
        if (lane == 0) wa[wv] = (uint32_t)__popcll(beq);
        __syncthreads();
        uint32_t eq_rank = (uint32_t)__popcll(beq & lt_mask), chunk_eq = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            eq_rank += w < wv ? wa[w] : 0u;
            chunk_eq += wa[w];
        }
        const bool take = (in || (eq && seen_eq + eq_rank < rem)) && (margin <= 0.f || sv <= best + margin);
        const uint64_t bt = __ballot(take);
        if (lane == 0) wb[wv] = (uint32_t)__popcll(bt);
        __syncthreads();
        uint32_t pos = (uint32_t)__popcll(bt & lt_mask), chunk_t = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            pos += w < wv ? wb[w] : 0u;
            chunk_t += wb[w];
        }
        if (take && written + pos < (uint32_t)k) out[written + pos] = remap ? remap[a + i] : a + i;
        written += chunk_t;
        seen_eq += chunk_eq;
        __syncthreads();  // wa, wb are rewritten by the next chunk
    }
    for (int64_t r = (int64_t)written + tid; r < k; r += NT) out[r] = -1;
}

// ------------------------------------------------------------------ launchers

hipError_t launch_features(const DevFeat* feats, int64_t n, const FeatHalo& halo, float* base, uint16_t* X,
                           float* f32, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_features, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, s, feats, n, halo, base, X, f32);
    return hipGetLastError();
}

hipError_t launch_mlp_forward(const uint16_t* X, int64_t n, const RankerWeights& W, float* Y, const RankScore& S,
                              hipStream_t s) {
    if (n <= 0) return hipSuccess;
    int64_t grid = (n + kRowsMlp - 1) / kRowsMlp;
    if (grid > 4 * kMlpInferCus) {
        // many rows: persistent workgroups, weights in registers
        hipLaunchKernelGGL(k_mlp_infer, dim3((unsigned)kMlpInferCus), dim3(kMlpThreads), 0, s, X, n, W, Y, S);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)grid), dim3(kMlpThreads), 0, s, X, n, W, Y, S);
    return hipGetLastError();
}

hipError_t launch_publish(const float* p, int64_t count, const RankerWeights& W, hipStream_t s) {
    hipLaunchKernelGGL(k_publish, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, p, count, W);
    return hipGetLastError();
}

// 16 waves a workgroup for segments longer than this on average: their passes share more
// lanes, but every barrier waits for more waves.  The 64 smallest of 457 segments, 16 waves and
// four, us: 256 scores each 9.5 and 6.8, 768 10.2 and 9.4, 1,024 10.9 and 10.6, 1,536 12.5 and
// 13.2, 4,096 19.6 and 25.4; of 8 segments 512 6.9 and 6.8, 1,024 7.5 and 9.1, 4,096 12.7 and 21.6.
constexpr int64_t kSelWide = 1024;

hipError_t launch_select(const float* score, const int64_t* seg, int64_t nseg, int64_t n, int64_t stride, int k,
                         float margin, const int64_t* remap, int64_t* sel, hipStream_t s) {
    if (nseg <= 0) return hipSuccess;
    if ((stride > 0 ? stride : n / nseg) > kSelWide)
        hipLaunchKernelGGL(k_select<1024>, dim3((unsigned)nseg), dim3(1024), 0, s, score, seg, stride, k, margin, remap,
                           sel);
    else
        hipLaunchKernelGGL(k_select<256>, dim3((unsigned)nseg), dim3(256), 0, s, score, seg, stride, k, margin, remap,
                           sel);
    return hipGetLastError();
}

}  // namespace tmk
