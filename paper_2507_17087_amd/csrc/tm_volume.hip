// tm_volume.hip -- matmul tile fetches and redistribution volumes over coordinate groups,
// one launch per batch: the owner tables, the groups and the tuples of a candidate (of a
// pair) stay in one workgroup's LDS.
//
// Bound: latency.  A call's candidates are a few dozen to a few hundred, their tuples a
// few thousand; what counts is that nothing goes through memory between the phases.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "tm_compile.h"
#include "tm_groups.h"
#include "tm_volume.h"

namespace tmk {

// Contribution at x of a launch dim (in this lane's registers).
__device__ __forceinline__ uint32_t value_at(const DevEval& c, const LaneDim& d, uint32_t x, int flags) {
    return block_value(c, d, x, flags & kEvalExtra) +
           ((flags & kEvalCyclic) ? cyclic_value(c, d, x, flags & kEvalExtra) : 0u);
}

// Members x0 + r + k M of a segment [x0, x0 + len).
__device__ __forceinline__ uint32_t members(uint32_t len, uint32_t r, uint32_t M, double rM) {
    if (r >= len) return 0;
    return M > 1 ? div_wide((double)(len - 1 - r), rM) + 1 : len;
}

// ------------------------------------------------------------------ matmul tiles
//
// A tile of A (i, k) is fetched by every processor that owns some task (i, j, k): per pair
// of groups (of i, of k) the owners along j are the same for all its tiles, and each counts
// their number, the product of the groups' members.  The same for B (k, j) over i and
// C (i, j) over k.  Where distinct tuples of groups have distinct owners (kEvalDistinct) a
// processor owns one tuple and its counts are that tuple's products; else a thread takes a
// pair, marks the owners it has met along the reduction dim in a bitmap of its own and adds
// the pair's tiles at each new one.
//
// 57 mappings of a 256^3 matmul onto 64 processors: 7.7 us; the general kernel takes 26 us
// after a table build of 8 and before totals of 5.  64 mappings of 250^3 with cyclic grids
// 16 x 8 x 8: 8.4 us, there 6.2 ms (a class per coordinate); 64 folded ones of 1,024
// processors: 16 us, there 80.
__global__ __launch_bounds__(kMatmulThreads) void k_matmul_groups(const DevEval* __restrict__ evals,
                                                                  int64_t tile_bytes,
                                                                  tm_matmul_cost* __restrict__ out,
                                                                  int64_t* __restrict__ per_proc) {
    extern __shared__ __attribute__((aligned(16))) int32_t lds[];  // ids, counts, groups, bitmaps
    constexpr int NT = kMatmulThreads, NW = NT / 64;
    __shared__ DevEval ev;
    __shared__ unsigned long long s_sum[3][NW];
    __shared__ uint32_t s_max[3][NW];
    const int tid = threadIdx.x;
    stage_eval(&ev, evals + blockIdx.x, tid);
    lds_sync(NW);
    const int32_t vol = wave_uniform(ev.vol), P = wave_uniform(ev.procs), flags = wave_uniform(ev.flags);
    int32_t* T = lds;
    uint32_t* cnt = reinterpret_cast<uint32_t*>(lds + ((vol + 3) & ~3));  // matrix m's at m P
    i32x2* rec = reinterpret_cast<i32x2*>(cnt + ((3 * P + 3) & ~3));      // contribution, members
    int32_t G[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) G[d] = wave_uniform(ev.dim[d].G);
    const i32x2 *r0 = rec, *r1 = rec + G[0], *r2 = r1 + G[1];
    owner_table<true>(ev, T, 0, vol, -1, tid, NT);
    for (int32_t i = tid; i < 3 * P; i += NT) cnt[i] = 0;
    for (int32_t i = tid; i < G[0] + G[1] + G[2]; i += NT) {
        const int d = i < G[0] ? 0 : (i < G[0] + G[1] ? 1 : 2);
        const uint32_t g = (uint32_t)(i - (d > 0 ? G[0] : 0) - (d > 1 ? G[1] : 0));
        const LaneDim ld = lane_dim(ev, d, flags & kEvalCyclic);
        const uint32_t a = ld.M > 1 ? div_small(g, (float)ld.rM) : g, r = g - __umul24(a, ld.M);
        const uint32_t x0 = segment_start(ev, ld, a, flags & kEvalExtra),
                       x1 = segment_start(ev, ld, a + 1, flags & kEvalExtra);
        const uint32_t w = members(x1 - x0, ld.M > 1 ? r : 0, ld.M, ld.rM);
        rec[i] = i32x2{w ? (int32_t)value_at(ev, ld, x0 + (ld.M > 1 ? r : 0), flags) : 0, (int32_t)w};
    }
    lds_sync(NW);
    if (flags & kEvalDistinct) {
        const uint32_t n = (uint32_t)(G[0] * G[1] * G[2]);
        const float rg2 = 1.0f / (float)G[2], rg1 = 1.0f / (float)G[1];
        for (uint32_t t = tid; t < n; t += NT) {
            const uint32_t q = div_small(t, rg2), i0 = div_small(q, rg1);
            const i32x2 a = r0[i0], b = r1[q - __umul24(i0, (uint32_t)G[1])], c = r2[t - __umul24(q, (uint32_t)G[2])];
            if (!a.y || !b.y || !c.y) continue;
            const int32_t p = T[a.x + b.x + c.x];
            cnt[p] = (uint32_t)a.y * (uint32_t)c.y;
            cnt[P + p] = (uint32_t)c.y * (uint32_t)b.y;
            cnt[2 * P + p] = (uint32_t)a.y * (uint32_t)b.y;
        }
    } else {
        uint32_t* met = reinterpret_cast<uint32_t*>(rec + G[0] + G[1] + G[2]) + tid;  // word i at i NT
        const int32_t words = (P + 31) >> 5;
        for (int m = 0; m < 3; ++m) {
            // fixed dims and reduction dim: A = (0, 2; 1), B = (2, 1; 0), C = (0, 1; 2)
            const i32x2 *ra = m == 1 ? r2 : r0, *rb = m == 0 ? r2 : r1, *rr = m == 0 ? r1 : (m == 1 ? r0 : r2);
            const uint32_t Ga = m == 1 ? G[2] : G[0], Gb = m == 0 ? G[2] : G[1],
                           Gr = m == 0 ? G[1] : (m == 1 ? G[0] : G[2]);
            const float rgb = 1.0f / (float)Gb;
            for (uint32_t t = tid; t < Ga * Gb; t += NT) {
                const uint32_t q = div_small(t, rgb);
                const i32x2 a = ra[q], b = rb[t - __umul24(q, Gb)];
                const uint32_t tiles = (uint32_t)a.y * (uint32_t)b.y;
                if (!tiles) continue;
                for (int32_t i = 0; i < words; ++i) met[i * NT] = 0;
                for (uint32_t j = 0; j < Gr; ++j) {
                    const i32x2 r = rr[j];
                    if (!r.y) continue;
                    const uint32_t p = (uint32_t)T[a.x + b.x + r.x], bit = 1u << (p & 31);
                    uint32_t* w = met + (p >> 5) * NT;
                    const uint32_t old = *w;
                    if (old & bit) continue;
                    *w = old | bit;
                    atomicAdd(&cnt[m * P + p], tiles);
                }
            }
        }
    }
    lds_sync(NW);
    const int64_t first = wave_uniform64(ev.offset);
    if (per_proc)
        for (int32_t i = tid; i < 3 * P; i += NT) {
            const uint32_t p = div_small((uint32_t)i, 1.0f / 3.0f);
            per_proc[first * 3 + i] = (int64_t)cnt[(i - 3 * p) * P + p];
        }
    unsigned long long sum[3] = {0, 0, 0};
    uint32_t most[3] = {0, 0, 0};
    for (int32_t p = tid; p < P; p += NT)
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            sum[m] += cnt[m * P + p];
            most[m] = max(most[m], cnt[m * P + p]);
        }
#pragma unroll
    for (int m = 0; m < 3; ++m) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            sum[m] += __shfl_xor(sum[m], o, 64);
            most[m] = max(most[m], (uint32_t)__shfl_xor((int)most[m], o, 64));
        }
        if ((tid & 63) == 0) {
            s_sum[m][tid >> 6] = sum[m];
            s_max[m][tid >> 6] = most[m];
        }
    }
    lds_sync(NW);
    if (tid != 0) return;
    tm_matmul_cost c;
    int64_t all = 0;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        for (int w = 1; w < NW; ++w) {
            sum[m] += s_sum[m][w];
            most[m] = max(most[m], s_max[m][w]);
        }
        c.tiles[m] = (int64_t)sum[m];
        c.max_tiles[m] = (int64_t)most[m];
        all += c.tiles[m];
    }
    c.bytes = all * tile_bytes;
    out[blockIdx.x] = c;
}

int32_t matmul_words(const DevEval& e) {
    int64_t groups = 0;
    for (int d = 0; d < 3; ++d) groups += e.dim[d].G;
    const bool distinct = e.flags & kEvalDistinct;
    const int64_t w = ((int64_t)(e.vol + 3) & ~3) + ((3 * e.procs + 3) & ~3) + 2 * groups +
                      (distinct ? 0 : (int64_t)kMatmulThreads * ((e.procs + 31) / 32));
    return w <= kMaxLdsWords ? (int32_t)w : 0;
}

hipError_t launch_matmul_groups(const DevEval* evals, int64_t n, int32_t lds_words, int64_t tile_bytes,
                                tm_matmul_cost* out, int64_t* per_proc, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_matmul_groups, dim3((unsigned)n), dim3(kMatmulThreads), (size_t)lds_words * 4, s, evals,
                       tile_bytes, out, per_proc);
    return hipGetLastError();
}

// ------------------------------------------------------------------ redistribution
//
// A cell moves when its owners under the pair's mappings differ, and both are fixed by its
// coordinates' contributions to the two final indices: the joint groups of a launch dim
// hold those of one pair of contributions, and the moved cells are a sum over tuples of
// joint groups, one owner comparison each, weighted by the cells it stands for.  Both
// indices stay below 2^15 and are added up as the halves of one word.
//
// 108 transposes of 512^3 on 128 processors: 12.3 us; the general kernels take 33.7 us in
// four launches.  4,320 of them 41 us, there 166; 198 on 1,024 processors 105 us, there 117.

// First cell of joint segment a (0 <= a <= nseg): see segment_start; the search starts from
// sum s x / l, of which the number of change points up to x falls short by less than one
// per block size.
__device__ __forceinline__ uint32_t joint_start(const JointDim& d, uint32_t a) {
    if (d.ident || a == 0) return a;
    const uint32_t l = (uint32_t)d.l;
    if (a >= (uint32_t)d.nseg) return l;
    if (d.nblk == 1) return div_wide(fma((double)a, (double)l, (double)d.s[0] - 1.0), d.rs);
    uint32_t lo = (uint32_t)((double)a * (double)l * d.rsum), hi = (uint32_t)((double)(a + d.nblk) * (double)l * d.rsum) + 2;
    lo = lo > 1 ? lo - 1 : 1;
    hi = hi < l ? hi : l;
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        uint32_t cnt = 0;
        for (int j = 0; j < d.nblk; ++j) cnt += block_index(mid, (double)d.s[j], d.rl);
        if (cnt >= a) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

template <int NT>
__global__ __launch_bounds__(NT) void k_pairs(const DevPair* __restrict__ pairs, int32_t most_parts,
                                               int64_t elem_bytes, tm_redist_cost* __restrict__ out) {
    extern __shared__ __attribute__((aligned(16))) int32_t lds[];  // a's owners, b's owners, joint groups
    __shared__ DevPair pr;
    __shared__ unsigned long long s_m[NT / 64], s_i[NT / 64];
    const int tid = threadIdx.x;
    const uint32_t pair = most_parts > 1 ? blockIdx.x / (uint32_t)most_parts : blockIdx.x;
    const int32_t part = most_parts > 1 ? (int32_t)(blockIdx.x - pair * (uint32_t)most_parts) : 0;
    if (tid < (int)(sizeof(DevPair) / 16))
        reinterpret_cast<i32x4v*>(&pr)[tid] = reinterpret_cast<const i32x4v*>(pairs + pair)[tid];
    lds_sync(NT / 64);
    const int32_t parts = wave_uniform(pr.parts);
    if (part >= parts) return;
    const int32_t va = wave_uniform(pr.a.vol), vb = wave_uniform(pr.b.vol), K = wave_uniform(pr.a.lrank);
    const int32_t D = wave_uniform(pr.dim_d), gb = wave_uniform(pr.a.gbits);
    const int32_t *TA = lds, *TB = lds + ((va + 3) & ~3);
    i32x2* rec = reinterpret_cast<i32x2*>(lds + ((va + 3) & ~3) + ((vb + 3) & ~3));  // contributions, members
    if (tid < NT / 2) owner_table(pr.a, lds, 0, va, -1, tid, NT / 2);
    else owner_table(pr.b, lds + ((va + 3) & ~3), 0, vb, -1, tid - NT / 2, NT / 2);
    // the dims' groups, of dim D this part's
    int32_t G[TM_MAX_LRANK], g0[TM_MAX_LRANK], all = 0;
    uint32_t n = 1;
#pragma unroll
    for (int d = 0; d < TM_MAX_LRANK; ++d) {
        const int32_t g = d < K ? wave_uniform(pr.dim[d].G) : 1;
        g0[d] = 0;
        G[d] = g;
        if (d == D && parts > 1) {
            g0[d] = (int32_t)((int64_t)g * part / parts);
            G[d] = (int32_t)((int64_t)g * (part + 1) / parts) - g0[d];
        }
        n *= (uint32_t)G[d];
        all += d < K ? G[d] : 0;
    }
    const int fa = wave_uniform(pr.a.flags), fb = wave_uniform(pr.b.flags);
    for (int32_t i = tid; i < all; i += NT) {
        int d = 0, f = 0;
        uint32_t g = (uint32_t)(i + g0[0]);
#pragma unroll
        for (int e = 1; e < TM_MAX_LRANK; ++e) {
            f += G[e - 1];
            if (e < K && i >= f) {
                d = e;
                g = (uint32_t)(i - f + g0[e]);
            }
        }
        const JointDim& jd = pr.dim[d];
        const uint32_t M = (uint32_t)jd.M, a = M > 1 ? div_small(g, (float)jd.rM) : g, r = M > 1 ? g - __umul24(a, M) : 0;
        const uint32_t x0 = joint_start(jd, a), w = members(joint_start(jd, a + 1) - x0, r, M, jd.rM);
        uint32_t v = 0;
        if (w) {
            const LaneDim la = lane_dim(pr.a, d, fa & kEvalCyclic), lb = lane_dim(pr.b, d, fb & kEvalCyclic);
            v = value_at(pr.a, la, x0 + r, fa) | value_at(pr.b, lb, x0 + r, fb) << 16;
        }
        rec[i] = i32x2{(int32_t)v, (int32_t)w};
    }
    lds_sync(NT / 64);
    float rG[TM_MAX_LRANK];
#pragma unroll
    for (int d = 1; d < TM_MAX_LRANK; ++d) rG[d] = 1.0f / (float)G[d];
    unsigned long long mv = 0, iv = 0;
    for (uint32_t t = tid; t < n; t += NT) {
        uint32_t q = t, v = 0, f = (uint32_t)all;
        unsigned long long w = 1;
#pragma unroll
        for (int d = TM_MAX_LRANK - 1; d >= 0; --d) {
            if (d >= K) continue;
            f -= (uint32_t)G[d];
            const uint32_t hi = d > 0 ? div_small(q, rG[d]) : 0;
            const i32x2 e = rec[f + q - __umul24(hi, (uint32_t)G[d])];
            q = hi;
            v += (uint32_t)e.x;
            w *= (uint32_t)e.y;
        }
        const int32_t oa = TA[v & 0xffff], ob = TB[v >> 16];
        mv += oa != ob ? w : 0;
        iv += (oa >> gb) != (ob >> gb) ? w : 0;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        mv += __shfl_xor(mv, o, 64);
        iv += __shfl_xor(iv, o, 64);
    }
    if ((tid & 63) == 0) {
        s_m[tid >> 6] = mv;
        s_i[tid >> 6] = iv;
    }
    lds_sync(NT / 64);
    if (tid != 0) return;
    for (int w = 1; w < NT / 64; ++w) {
        mv += s_m[w];
        iv += s_i[w];
    }
    const unsigned long long eb = (unsigned long long)elem_bytes;
    if (parts == 1) {
        tm_redist_cost c;
        c.moved_cells = (int64_t)mv;
        c.inter_cells = (int64_t)iv;
        c.bytes = (int64_t)(mv * eb);
        c.inter_bytes = (int64_t)(iv * eb);
        out[pair] = c;
    } else if (mv) {
        atomicAdd(reinterpret_cast<unsigned long long*>(&out[pair].moved_cells), mv);
        atomicAdd(reinterpret_cast<unsigned long long*>(&out[pair].inter_cells), iv);
        atomicAdd(reinterpret_cast<unsigned long long*>(&out[pair].bytes), mv * eb);
        atomicAdd(reinterpret_cast<unsigned long long*>(&out[pair].inter_bytes), iv * eb);
    }
}

__global__ void k_zero_moves(tm_redist_cost* __restrict__ out, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = tm_redist_cost{};
}

// Joint dim k of candidates a and b; false: more block sizes than JointDim lists.
static bool fill_joint(const CandView& a, const CandView& b, int k, JointDim* g) {
    const int64_t l = a.extent[k];
    int64_t m = 1, sizes[2 * TM_MAX_MRANK];
    int ns = 0;
    for (const CandView* c : {&a, &b}) {
        const uint64_t bits = projection_bits(*c);
        for (uint32_t m8 = cyclics_of(bits, k); m8; m8 &= m8 - 1) m = lcm_upto(m, c->fshape[__builtin_ctz(m8)], l);
        for (uint32_t m8 = blocks_of(bits, k); m8; m8 &= m8 - 1) sizes[ns++] = c->fshape[__builtin_ctz(m8)];
    }
    int64_t changes = 0, sum = 0;
    g->nblk = 0;
    for (int i = 0; i < ns; ++i) {
        bool covered = false;  // by a larger size, or the same one listed before
        for (int j = 0; j < ns; ++j)
            covered = covered || (j != i && sizes[j] % sizes[i] == 0 && (sizes[j] > sizes[i] || j < i));
        if (covered) continue;
        if (g->nblk == TM_MAX_MRANK) return false;
        g->s[g->nblk++] = (int32_t)sizes[i];
        changes += std::min(sizes[i], l) - 1;
        sum += sizes[i];
    }
    const int64_t nseg = changes + 1;
    const int64_t longest = g->nblk == 1 ? (l + g->s[0] - 1) / g->s[0] : l, r = std::min(m, longest);
    g->ident = nseg >= l || nseg * r >= l ? 1 : 0;
    g->l = (int32_t)l;
    g->nseg = (int32_t)(g->ident ? l : nseg);
    g->M = (int32_t)(g->ident ? 1 : m);
    const int64_t G = (int64_t)g->nseg * g->M;
    g->G = (int32_t)std::min<int64_t>(G, INT32_MAX);
    for (int i = g->nblk; i < TM_MAX_MRANK; ++i) g->s[i] = 1;
    g->pad[0] = g->pad[1] = 0;
    g->rl = 1.0 / (double)l;
    g->rM = 1.0 / (double)g->M;
    g->rs = 1.0 / (double)g->s[0];
    g->rsum = 1.0 / (double)std::max<int64_t>(sum, 1);
    return true;
}

bool fill_pair(const CandView& a, const CandView& b, DevPair* p, int32_t* words) {
    int64_t groups = 0, tuples = 1;
    p->dim_d = 0;
    for (int k = 0; k < a.lrank; ++k) {
        if (!fill_joint(a, b, k, &p->dim[k])) return false;
        groups += p->dim[k].G;
        if (groups > kMaxLdsWords) return false;
        tuples *= p->dim[k].G;
        if (p->dim[k].G > p->dim[p->dim_d].G) p->dim_d = k;
    }
    const int64_t w = ((a.vol + 3) & ~3) + ((b.vol + 3) & ~3) + 2 * groups, g = p->dim[p->dim_d].G;
    if (w > kMaxLdsWords || tuples / g > kPairRowTuples) return false;
    p->parts = (int32_t)std::max<int64_t>(1, std::min<int64_t>((tuples + kPairTuples - 1) / kPairTuples, g));
    p->pad[0] = p->pad[1] = 0;
    *words = (int32_t)w;
    return true;
}

hipError_t launch_pairs(const DevPair* pairs, int64_t n, int32_t parts, int32_t lds_words, int64_t elem_bytes,
                        tm_redist_cost* out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (parts > 1) {
        hipLaunchKernelGGL(k_zero_moves, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 1024)), dim3(256), 0, s, out, n);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (n * parts <= kPairWide) {
        hipLaunchKernelGGL(k_pairs<1024>, dim3((unsigned)(n * parts)), dim3(1024), (size_t)lds_words * 4, s, pairs, parts,
                           elem_bytes, out);
        return hipGetLastError();
    }
    const int64_t most = kMaxGrid / parts;  // pairs a launch (parts: at most the groups that fit the LDS)
    for (int64_t a = 0; a < n; a += most) {
        const int64_t m = std::min(n - a, most);
        hipLaunchKernelGGL(k_pairs<256>, dim3((unsigned)(m * parts)), dim3(256), (size_t)lds_words * 4, s, pairs + a, parts,
                           elem_bytes, out + a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace tmk
