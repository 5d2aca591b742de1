// tm_eval.hip -- the exact stencil evaluation: one kernel per batch, no tables in memory.
//
// Along launch dim d, coordinates with the same contribution to the linear final index
// form a group (DevDim); the cells of a tuple of groups, one per dim, share their owner.
// A cell's star neighbours sit at its index plus the offsets its coordinates see, so
//   sum over the tuple's cells of the distinct foreign owners of their neighbours
//     = sum over distinct foreign owners p of (cells that see some offset owned by p)
//     = sum over p of (W - prod_d N_d(p)),
// W the cells of the tuple and N_d(p) the members of group d that see no offset owned by
// p (the dims are independent: a cell misses p iff each of its coordinates does).  When
// every transformation is a bijection, distinct offsets have distinct owners and the sum
// is over offsets: (members that see it) x (cells of the other dims).  Exactly the
// per-cell count, regrouped; the tuples number at most the final space's volume, however
// large the domain and however the projections cycle.
//
// A workgroup takes one candidate (or one part of a large one: a range of the groups of
// its dim with the most groups), builds the owner table and the group records in LDS and
// counts; nothing but the 896-byte descriptor is read and nothing but the 32-byte cost
// row is written.  Records that do not fit the launch's LDS are
// built a range of that dim's groups at a time.
//
// Bound: VALU issue and LDS latency, about 1,400 vector instructions and 120 LDS accesses
// per wave on a search candidate (249 owners); small batches: the latency of one
// candidate, 8 us.  One-wave workgroups for large batches keep 20 candidates in flight per
// CU, and persistent ones taking several candidates in turn were slower (1.03-1.1 ms
// against 0.90 on the search).  Measured, against a table build into memory and a count
// over runs of equal coordinates read back from it: 219,424 search candidates 0.58 ms
// (6.30), 4,096 random ones 27 us (150), with a quarter of the projections cyclic 36 us
// (3,200), 300 two-level mappings of 512^3 at halo 2 20 us (23,350), 1,440 2-D mappings
// with rows of up to 640,000 cells 12 us (5,100), 216 mappings of 512^3 10.5 us (51).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "tm_compile.h"
#include "tm_eval.h"
#include "tm_groups.h"
#include "tm_internal.h"

namespace tmk {

// The records of one tuple loop, per dim.
struct GroupDims {
    int32_t G[TM_MAX_LRANK];     // groups in range
    int32_t base[TM_MAX_LRANK];  // LDS words of their first record
    float rG[TM_MAX_LRANK];
};

__device__ __forceinline__ int32_t low16(int32_t w) { return (int32_t)(int16_t)(w & 0xffff); }

// Record positions, heads, members and the contribution of tuple t (C order).  Members
// are doubles: weights are products of at most 2^40 in all and counts at most 48 times
// that, whole numbers that doubles hold exactly, and a double product costs half a 64-bit
// integer one.
template <int K>
__device__ __forceinline__ int32_t tuple_at(const int32_t* lds, const GroupDims& D, int32_t stride, uint32_t t,
                                            int32_t (&r)[K], uint32_t (&ne)[K], uint32_t (&W)[K]) {
#pragma unroll
    for (int d = K - 1; d >= 0; --d) {
        uint32_t k = t;
        if (d > 0) {
            const uint32_t q = div_small(t, D.rG[d]);
            k = t - __umul24(q, (uint32_t)D.G[d]);
            t = q;
        }
        r[d] = D.base[d] + (int32_t)__umul24(k, (uint32_t)stride);
    }
    int32_t v = 0;
#pragma unroll
    for (int d = 0; d < K; ++d) {
        const i32x2 w = *reinterpret_cast<const i32x2*>(lds + r[d]);
        ne[d] = (uint32_t)w.x >> 24;
        W[d] = (uint32_t)w.y;
        v += w.x & 0xffffff;
    }
    return v;
}

// Distinct owners per offset (bijective chains): offsets counted one by one.  An unused
// slot (0) reads the tuple's own owner and counts nothing.  Per dim the slots' counts are
// summed as (edge members | interior << 8).
template <int K, int U, int NT>
__device__ __forceinline__ void count_bijective(const int32_t* lds, const GroupDims& D, int32_t stride, int gb,
                                                uint32_t n, int tid, double& tot, double& inter) {
    const int32_t* T = lds;
    for (uint32_t t = tid; t < n; t += NT) {
        int32_t r[K];
        uint32_t ne[K], W[K];
        const int32_t v = tuple_at<K>(lds, D, stride, t, r, ne, W);
        const int32_t node = T[v] >> gb;
        uint32_t cs[K], is[K];
#pragma unroll
        for (int d = 0; d < K; ++d) {
            cs[d] = is[d] = 0;
#pragma unroll 4
            for (int u = 0; u < U; u += 2) {
                const i32x2 e = *reinterpret_cast<const i32x2*>(lds + r[d] + 2 + u);
                const int32_t p = T[v + low16(e.x)], q = T[v + low16(e.y)];
                const uint32_t a = (uint32_t)e.x >> 16, b = (uint32_t)e.y >> 16;
                cs[d] += a + b;
                is[d] += ((p >> gb) != node ? a : 0u) + ((q >> gb) != node ? b : 0u);
            }
        }
#pragma unroll
        for (int d = 0; d < K; ++d) {
            double wo = 1;
#pragma unroll
            for (int e = 0; e < K; ++e)
                if (e != d) wo *= (double)W[e];
            const double ni = (double)(W[d] - ne[d]);  // interior members
            tot = fma(fma((double)(cs[d] >> 8), ni, (double)(cs[d] & 0xff)), wo, tot);
            inter = fma(fma((double)(is[d] >> 8), ni, (double)(is[d] & 0xff)), wo, inter);
        }
    }
}

// The cells of a tuple that see some slot of `same` (bits d U + u), all of them slots of
// one owner: W - prod_d (members that see none of dim d's), from the members' masks.
template <int K, int U>
__device__ __forceinline__ double cells_seeing(const int32_t* lds, const int32_t (&r)[K], const uint32_t (&ne)[K],
                                               const uint32_t (&W)[K], uint64_t same, double all) {
    double miss = 1;
#pragma unroll
    for (int d = 0; d < K; ++d) {
        const uint32_t m = (uint32_t)(same >> (d * U)) & ((1u << U) - 1u);
        uint32_t nm = W[d];
        if (m) {
            const uint16_t* mk = reinterpret_cast<const uint16_t*>(lds + r[d] + 2 + U);
            nm = (mk[0] & m) ? 0u : W[d] - ne[d];
            for (uint32_t e = 1; e <= ne[d]; ++e) nm += (mk[e] & m) ? 0u : 1u;
        }
        miss *= (double)nm;
    }
    return all - miss;
}

// Slots whose owners are compared in registers: one-wave workgroups (large batches) keep
// five waves per SIMD up to halo 2, where 24 slots would spill (non-cyclic 2-D mappings 16.0
// and 18.3 us); at halos of 3 and 4, 4,096 random candidates take 251 us with 12 slots and
// 100 with 24.
constexpr int owners_in_regs(int nt, int h) { return nt == 64 && h <= 2 ? 12 : 24; }

// The general case.  A foreign owner of one slot counts that slot's members, as above;
// one of several slots counts, at its first slot, the cells that see any of them.  Up to R
// slots their owners are compared in registers (on the search's chains few tuples
// have such owners); else every slot looks at all the others.
template <int K, int U, int NT, int R>
__device__ __forceinline__ void count_general(const int32_t* lds, const GroupDims& D, int32_t stride, int gb,
                                              uint32_t n, int tid, double& tot, double& inter) {
    const int32_t* T = lds;
    constexpr int S = K * U;
    for (uint32_t t = tid; t < n; t += NT) {
        int32_t r[K];
        uint32_t ne[K], W[K];
        const int32_t v = tuple_at<K>(lds, D, stride, t, r, ne, W);
        const int32_t o = T[v], node = o >> gb;
        double all = 1;
#pragma unroll
        for (int d = 0; d < K; ++d) all *= (double)W[d];
        // one owner's slots (its bits), from slot i's
        auto slots_of = [&](int32_t p) {
            uint64_t same = 0;
#pragma unroll
            for (int d = 0; d < K; ++d)
#pragma unroll 2
                for (int u = 0; u < U; ++u)
                    same |= T[v + low16(lds[r[d] + 2 + u])] == p ? 1ull << (d * U + u) : 0ull;
            return same;
        };
        auto owner_at = [&](int i) {
            const int d = i / U;
            int32_t rd = r[0];
#pragma unroll
            for (int e = 1; e < K; ++e) {
                rd = d == e ? r[e] : rd;
                // else r[] lies in scratch memory, stored on every tuple (8,192 random candidates:
                // 38.5 us, 37.4 without)
                asm("" : "+v"(rd));
            }
            return T[v + low16(lds[rd + 2 + i - d * U])];
        };
        if (S <= R) {
            int32_t p[S];
#pragma unroll
            for (int d = 0; d < K; ++d)
#pragma unroll
                for (int u = 0; u < U; u += 2) {
                    const i32x2 e = *reinterpret_cast<const i32x2*>(lds + r[d] + 2 + u);
                    p[d * U + u] = T[v + low16(e.x)];
                    p[d * U + u + 1] = T[v + low16(e.y)];
                }
            uint32_t multi = 0;  // the first of several slots of one foreign owner
#pragma unroll
            for (int d = 0; d < K; ++d) {
                uint32_t cs = 0, is = 0;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    // 0 where an earlier (a later) slot has this owner; kept out of compares,
                    // whose results would take a pair of scalar registers each
                    const int i = d * U + u;
                    uint32_t before = ~0u, after = ~0u;
                    int32_t q = p[i];
                    asm("" : "+v"(q));  // a copy of its own: no pair's difference is kept for its mirror
#pragma unroll
                    for (int j = 0; j < S; ++j) {
                        if (j < i) before = min(before, (uint32_t)(q ^ p[j]));
                        if (j > i) after = min(after, (uint32_t)(q ^ p[j]));
                    }
                    const uint32_t k = min(min(before, after), (uint32_t)(q ^ o)) ? (uint32_t)lds[r[d] + 2 + u] >> 16 : 0u;
                    cs += k;
                    is += (q >> gb) != node ? k : 0u;
                    multi |= q != o && before && !after ? 1u << i : 0u;
                }
                double wo = 1;
#pragma unroll
                for (int e = 0; e < K; ++e)
                    if (e != d) wo *= (double)W[e];
                const double ni = (double)(W[d] - ne[d]);
                tot = fma(fma((double)(cs >> 8), ni, (double)(cs & 0xff)), wo, tot);
                inter = fma(fma((double)(is >> 8), ni, (double)(is & 0xff)), wo, inter);
            }
            while (multi) {
                const int i = __builtin_ctz(multi);
                multi &= multi - 1;
                const int32_t q = owner_at(i);
                const double cells = cells_seeing<K, U>(lds, r, ne, W, slots_of(q), all);
                tot += cells;
                inter += (q >> gb) != node ? cells : 0.0;
            }
        } else {
            for (int i = 0; i < S; ++i) {
                const int32_t p = owner_at(i);
                if (p == o) continue;  // unused slots too
                const uint64_t same = slots_of(p);
                if (same & ((1ull << i) - 1ull)) continue;  // counted at an earlier slot
                const double cells = cells_seeing<K, U>(lds, r, ne, W, same, all);
                tot += cells;
                inter += (p >> gb) != node ? cells : 0.0;
            }
        }
    }
}

// Counts one part of candidate c: records, tuples.  LDS: the owner table (being written),
// the records of every dim but D, then a range of D's.  Launch ranks below the tuple
// loop's K take dims of one group of one coordinate (the record at `one`).
template <int NT, int H, bool CYC>
__device__ __forceinline__ void eval_part(const DevEval& c, const EvalArgs& A, int32_t* lds, int32_t one, int part,
                                          int parts, int tid, double& tot, double& inter) {
    constexpr int NW = NT / 64, U = CYC ? 4 * H : 2 * H, R = owners_in_regs(NT, H);
    const int32_t vol = wave_uniform(c.vol);
    const int gb = wave_uniform(c.gbits), K = wave_uniform(c.lrank), D = wave_uniform(c.dim_d);
    const int32_t flags = wave_uniform(c.flags);
    const bool masks = A.node_level || !wave_uniform(c.bij), extra = flags & kEvalExtra;
    const int32_t stride = group_stride(CYC, H, masks), t0 = (vol + 3) & ~3;
    int32_t G[TM_MAX_LRANK], rest = 0;  // groups per dim; of all dims but D
#pragma unroll
    for (int d = 0; d < TM_MAX_LRANK; ++d) {
        G[d] = d < K ? wave_uniform(c.dim[d].G) : 1;
        rest += d < K && d != D ? G[d] : 0;
    }
    int32_t GD = G[0];
#pragma unroll
    for (int d = 1; d < TM_MAX_LRANK; ++d) GD = d == D ? G[d] : GD;
    const int32_t ga = parts > 1 ? (int32_t)((int64_t)GD * part / parts) : 0,
                  gz = parts > 1 ? (int32_t)((int64_t)GD * (part + 1) / parts) : GD;
    const int32_t fit = (A.lds_words - t0) / stride - rest, room = fit > 1 ? fit : 1;
    for (int32_t g0 = ga; g0 < gz; g0 += room) {
        const int32_t g1 = gz < g0 + room ? gz : g0 + room;
        if (g0 > ga) lds_sync(NW);  // the previous range's records are no longer read
        // one lane per record: the other dims' (first range only), then D's range
        for (int32_t i = (g0 > ga ? rest : 0) + tid; i < rest + g1 - g0; i += NT) {
            int d = D, h = A.halo[D];
            uint32_t g = (uint32_t)(i - rest + g0);
            if (i < rest) {
                int32_t f = 0;
#pragma unroll
                for (int e = 0; e < TM_MAX_LRANK; ++e) {
                    if (e >= K || e == D) continue;
                    if (i >= f) {
                        d = e;
                        g = (uint32_t)(i - f);
                        h = A.halo[e];
                    }
                    f += G[e];
                }
            }
            const LaneDim ld = lane_dim(c, d, CYC);
            build_group<H, CYC>(c, ld, h, masks, extra, g, lds + t0 + i * stride);
        }
        lds_sync(NW);
        GroupDims g;
        uint32_t n = 1;
        int32_t f = 0;
#pragma unroll
        for (int d = 0; d < TM_MAX_LRANK; ++d) {
            g.G[d] = d == D ? g1 - g0 : G[d];
            g.base[d] = d < K ? t0 + (d == D ? rest : f) * stride : one;
            f += d < K && d != D ? G[d] : 0;
            g.rG[d] = 1.0f / (float)g.G[d];
            n *= (uint32_t)g.G[d];
        }
        if (masks) {
            if (K <= 2) count_general<2, U, NT, R>(lds, g, stride, gb, n, tid, tot, inter);
            else if (K == 3) count_general<3, U, NT, R>(lds, g, stride, gb, n, tid, tot, inter);
            else count_general<4, U, NT, R>(lds, g, stride, gb, n, tid, tot, inter);
        } else if (K <= 2) count_bijective<2, U, NT>(lds, g, stride, gb, n, tid, tot, inter);
        else if (K == 3) count_bijective<3, U, NT>(lds, g, stride, gb, n, tid, tot, inter);
        else count_bijective<4, U, NT>(lds, g, stride, gb, n, tid, tot, inter);
    }
}

__device__ __forceinline__ bool cost_less(int64_t b, int64_t i, int64_t x, int64_t b2, int64_t i2, int64_t x2) {
    return b < b2 || (b == b2 && (i < i2 || (i == i2 && x < x2)));
}

// The index minimising (bytes, inter_bytes, index) of n cost rows that other workgroups
// of this launch wrote (read at device scope) -> *best; with ids, its owner table as
// processor ids, at its place there (ev: LDS for its descriptor).
template <int NT>
__device__ __forceinline__ void select_rows(const tm_stencil_cost* out, int64_t n, int64_t* best,
                                            const DevEval* evals, int32_t* ids, DevEval& ev) {
    __shared__ int64_t sb[NT / 64], si[NT / 64], sx[NT / 64], s_best;
    const int t = threadIdx.x;
    int64_t kb = INT64_MAX, ki = INT64_MAX, kx = INT64_MAX;
    for (int64_t i0 = t; i0 < n; i0 += 4 * NT) {  // four rows in flight; past the end the last one again
        int64_t b[4], ib[4], x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            x[u] = i0 + u * NT < n ? i0 + u * NT : n - 1;
            int64_t* o = reinterpret_cast<int64_t*>(const_cast<tm_stencil_cost*>(&out[x[u]]));
            b[u] = __hip_atomic_load(o + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ib[u] = __hip_atomic_load(o + 3, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (cost_less(b[u], ib[u], x[u], kb, ki, kx)) {
                kb = b[u];
                ki = ib[u];
                kx = x[u];
            }
    }
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
        const int64_t b = __shfl_xor(kb, s, 64), ib = __shfl_xor(ki, s, 64), x = __shfl_xor(kx, s, 64);
        if (cost_less(b, ib, x, kb, ki, kx)) {
            kb = b;
            ki = ib;
            kx = x;
        }
    }
    if ((t & 63) == 0) {
        sb[t >> 6] = kb;
        si[t >> 6] = ki;
        sx[t >> 6] = kx;
    }
    __syncthreads();
    if (t == 0) {
        for (int w = 1; w < NT / 64; ++w)
            if (cost_less(sb[w], si[w], sx[w], kb, ki, kx)) {
                kb = sb[w];
                ki = si[w];
                kx = sx[w];
            }
        *best = n > 0 ? kx : -1;
        s_best = kx;
    }
    if (!ids || n <= 0) return;
    __syncthreads();
    stage_eval(&ev, evals + wave_uniform64(s_best), t);
    __syncthreads();
    owner_ids(ev, ids + wave_uniform64(ev.offset), wave_uniform(ev.vol), t, NT);
}

// The item of a workgroup's turn.  Workgroups go to the eight XCDs in turn, and batches are
// often menus of chains whose length is a multiple of eight, so that an XCD would take the
// same few chains of every menu, cheap or expensive ones: each group of eight is rotated by
// its place.  219,424 search candidates (menus of 32): 893 us in order (the CUs busy 62% of
// it), 598 rotated.
__device__ __forceinline__ int64_t spread_item(int64_t turn, int64_t items) {
    if (turn >= (items & ~int64_t(7))) return turn;
    return (turn & ~int64_t(7)) | ((turn + (turn >> 3) + (turn >> 6) + (turn >> 9)) & 7);
}

constexpr int kOneRecord = 2 + 4 * kMaxHalo;  // words of the largest record without masks

// Waves a SIMD: the registers of an instance without scratch memory.  At four, the four-wave
// one of halo 2 (256 work items or so: one workgroup a CU) kept 21 registers there: 216
// mappings of 512^3 with their selection 11.6 us at four and 10.5 at three, 300 random ones
// 17.9 and 16.5, 3,000 33.9 and 33.5.
constexpr int waves_per_simd(int nt, int h) { return nt == 64 && h <= 2 ? 5 : (h == 1 ? 4 : 3); }

template <int NT, int H>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(waves_per_simd(NT, H)))) void k_eval(const EvalArgs A) {
    extern __shared__ __attribute__((aligned(16))) int32_t lds[];
    __shared__ DevEval ev;
    __shared__ double s_sum[NT / 64][2];
    __shared__ int s_last;
    constexpr int NW = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t items = A.n * A.parts;
    // the record of a dim of one coordinate: {0, 1}, no offsets
    if (tid < kOneRecord) lds[A.lds_words + tid] = tid == 1 ? 1 : 0;
    for (int64_t turn = blockIdx.x; turn < items; turn += gridDim.x) {
        const int64_t item = spread_item(turn, items);
        const int64_t row = A.parts == 1 ? item : item / A.parts;
        const int part = (int)(item - row * A.parts);
        const int64_t ci = A.idx ? wave_uniform64(A.idx[row]) : row;
        if (ci < 0) continue;
        if (turn != (int64_t)blockIdx.x) lds_sync(NW);  // the previous item's LDS is no longer read
        stage_eval(&ev, A.evals + ci, tid);
        lds_sync(NW);
        const int32_t words = wave_uniform(ev.words), own = wave_uniform(ev.parts);
        const int parts = own < A.parts ? own : A.parts;
        if (words <= A.min_words || words > A.max_words || part >= parts) continue;  // another launch's, or no such part
        double tot = 0, inter = 0;
        // node-level tables keep the node of each owner (GPU bits cleared)
        owner_table(ev, lds, 0, wave_uniform(ev.vol), A.node_level ? ~((1 << wave_uniform(ev.gbits)) - 1) : -1, tid, NT);
        if (wave_uniform(ev.flags) & kEvalCyclic)
            eval_part<NT, H, true>(ev, A, lds, A.lds_words, part, parts, tid, tot, inter);
        else
            eval_part<NT, H, false>(ev, A, lds, A.lds_words, part, parts, tid, tot, inter);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            tot += __shfl_xor(tot, o, 64);
            inter += __shfl_xor(inter, o, 64);
        }
        if (NW > 1) {
            if (lane == 0) {
                s_sum[tid >> 6][0] = tot;
                s_sum[tid >> 6][1] = inter;
            }
            __syncthreads();
        }
        if (tid == 0) {
            if (NW > 1) {
                for (int w = 1; w < NW; ++w) {
                    tot += s_sum[w][0];
                    inter += s_sum[w][1];
                }
            }
            tm_stencil_cost* o = &A.out[row];
            const int64_t gc = (int64_t)tot, ic = (int64_t)inter;
            if (A.parts == 1) {
                *o = tm_stencil_cost{gc, ic, gc * A.elem_bytes, ic * A.elem_bytes};
            } else {
                atomicAdd(reinterpret_cast<unsigned long long*>(&o->ghost_cells), (unsigned long long)gc);
                atomicAdd(reinterpret_cast<unsigned long long*>(&o->inter_cells), (unsigned long long)ic);
            }
        }
    }
    if (!A.best) return;
    // the last workgroup to finish selects; the count wraps to the 0 it started from
    __syncthreads();
    if (tid == 0) {
        __threadfence();  // this workgroup's rows are visible before it reports done
        s_last = atomicInc(A.counter, gridDim.x - 1) == gridDim.x - 1;
    }
    __syncthreads();
    if (!s_last) return;
    __threadfence();
    select_rows<NT>(A.out, A.n, A.best, A.evals, A.best_ids, ev);
}

static hipError_t launch_eval(const EvalArgs& A, int H, bool wave, int64_t grid, hipStream_t s) {
    const size_t lds = (size_t)(A.lds_words + kOneRecord + 2) * 4;
#define TM_EVAL(nt, h) hipLaunchKernelGGL((k_eval<nt, h>), dim3((unsigned)grid), dim3(nt), lds, s, A)
#define TM_EVAL_H(nt)                   \
    do {                                \
        if (H <= 1) TM_EVAL(nt, 1);     \
        else if (H <= 2) TM_EVAL(nt, 2); \
        else TM_EVAL(nt, 4);            \
    } while (0)
    if (wave) TM_EVAL_H(64);
    else TM_EVAL_H(256);
#undef TM_EVAL_H
#undef TM_EVAL
    return hipGetLastError();
}

// ------------------------------------------------------------------ the evaluation's descriptors

__global__ __launch_bounds__(64) void k_fill_evals(const DevCand* __restrict__ cands, int64_t n, EvalShape shape,
                                                   DevEval* __restrict__ evals, DevFeat* __restrict__ feats,
                                                   unsigned int* __restrict__ counters) {
    static_assert(kCounters == 64, "one a thread of the first workgroup");
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (blockIdx.x == 0) counters[threadIdx.x] = 0;
    if (i >= n) return;
    fill_eval(cands[i], shape, &evals[i]);
    fill_feat(cands[i], &feats[i]);
}

hipError_t launch_fill_evals(const EvalPlan& p, const DevCand* cands, DevEval* evals, DevFeat* feats,
                             unsigned int* counters, hipStream_t s) {
    if (p.n <= 0) return hipSuccess;
    const EvalShape shape{p.H, p.node_level, p.per_item, p.fill};
    hipLaunchKernelGGL(k_fill_evals, dim3((unsigned)((p.n + 63) / 64)), dim3(64), 0, s, cands, p.n, shape, evals,
                       feats, counters);
    return hipGetLastError();
}

// ------------------------------------------------------------------ rows and selection

__global__ __launch_bounds__(256) void k_zero_costs(int64_t* __restrict__ o, int64_t words) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < words; i += (int64_t)gridDim.x * blockDim.x)
        o[i] = 0;
}

hipError_t launch_zero_costs(tm_stencil_cost* out, int64_t n, hipStream_t s) {
    const int64_t g = std::min<int64_t>(std::max<int64_t>((4 * n + 255) / 256, 1), 4096);
    hipLaunchKernelGGL(k_zero_costs, dim3((unsigned)g), dim3(256), 0, s, reinterpret_cast<int64_t*>(out), 4 * n);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_cost_bytes(tm_stencil_cost* __restrict__ out, int64_t n, int64_t eb) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        out[i].bytes = out[i].ghost_cells * eb;
        out[i].inter_bytes = out[i].inter_cells * eb;
    }
}

// The selection of select_rows in a launch of its own, over the rows of earlier launches: one
// chain of latencies (four rows in flight a thread, two reductions by shuffles), so a row is one
// plain 16-byte load (two at device scope before) and the waves' winners go over the lanes of
// every wave (one thread after the other before).  An evaluation with this selection, before
// and now: 256 rows 9.8 and 9.4 us, 1,440 12.4 and 11.8, 8,192 40.1 and 38.2.
typedef int64_t i64x2 __attribute__((ext_vector_type(2), aligned(8)));  // a caller's rows

__global__ __launch_bounds__(1024) void k_select_rows(const tm_stencil_cost* __restrict__ out, int64_t n,
                                                      int64_t* __restrict__ best, const DevEval* __restrict__ evals,
                                                      int32_t* __restrict__ ids) {
    constexpr int NT = 1024, NW = NT / 64;
    __shared__ DevEval ev;
    __shared__ int64_t sb[NW], si[NW], sx[NW];
    const int t = threadIdx.x;
    int64_t kb = INT64_MAX, ki = INT64_MAX, kx = INT64_MAX;
    auto take = [&](int64_t b, int64_t ib, int64_t x) {
        if (cost_less(b, ib, x, kb, ki, kx)) {
            kb = b;
            ki = ib;
            kx = x;
        }
    };
    for (int64_t i0 = t; i0 < n; i0 += 4 * NT) {  // past the end the last row again
        i64x2 v[4];
        int64_t x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            x[u] = i0 + u * NT < n ? i0 + u * NT : n - 1;
            v[u] = *reinterpret_cast<const i64x2*>(&out[x[u]].bytes);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) take(v[u].x, v[u].y, x[u]);
    }
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) take(__shfl_xor(kb, s, 64), __shfl_xor(ki, s, 64), __shfl_xor(kx, s, 64));
    if ((t & 63) == 0) {
        sb[t >> 6] = kb;
        si[t >> 6] = ki;
        sx[t >> 6] = kx;
    }
    __syncthreads();
    kb = sb[t % NW];
    ki = si[t % NW];
    kx = sx[t % NW];
#pragma unroll
    for (int s = NW / 2; s > 0; s >>= 1) take(__shfl_xor(kb, s, 64), __shfl_xor(ki, s, 64), __shfl_xor(kx, s, 64));
    if (t == 0) *best = n > 0 ? kx : -1;
    if (!ids || n <= 0) return;
    stage_eval(&ev, evals + wave_uniform64(kx), t);
    __syncthreads();
    owner_ids(ev, ids + wave_uniform64(ev.offset), wave_uniform(ev.vol), t, NT);
}

static hipError_t launch_select_rows(const tm_stencil_cost* out, int64_t n, int64_t* best, const DevEval* evals,
                                     int32_t* ids, hipStream_t s) {
    hipLaunchKernelGGL(k_select_rows, dim3(1), dim3(1024), 0, s, out, n, best, evals, ids);
    return hipGetLastError();
}

hipError_t launch_bytes_select(tm_stencil_cost* out, int64_t n, int64_t elem_bytes, int64_t* best, hipStream_t s,
                               const DevEval* evals, int32_t* ids) {
    const int64_t g = std::min<int64_t>(std::max<int64_t>((n + 255) / 256, 1), 2048);
    hipLaunchKernelGGL(k_cost_bytes, dim3((unsigned)g), dim3(256), 0, s, out, n, elem_bytes);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && best) e = launch_select_rows(out, n, best, evals, ids, s);
    return e;
}

hipError_t launch_eval_batch(const EvalPlan& p, const DevEval* evals, tm_stencil_cost* out, int64_t* best,
                             unsigned int* counter, int cus, hipStream_t s, const int64_t* idx, int64_t nidx,
                             int32_t* best_ids) {
    const int64_t n = idx ? nidx : p.n;
    if (n <= 0) return hipSuccess;
    const int32_t parts = idx ? 1 : p.parts;
    EvalArgs A{};
    A.evals = evals;
    A.idx = idx;
    A.n = n;
    A.out = out;
    A.counter = counter;
    A.elem_bytes = p.elem_bytes;
    A.node_level = p.node_level;
    A.parts = parts;
    for (int d = 0; d < TM_MAX_LRANK; ++d) A.halo[d] = p.halo[d];
    // the last workgroup of a single launch over few rows selects; else a launch of its own
    const bool fin = best && parts == 1 && n <= kFinInCount && (p.words[0] == 0 || p.words[1] == 0);
    if (fin) A.best = best;
    if (fin) A.best_ids = best_ids;
    hipError_t e = parts > 1 ? launch_zero_costs(out, n, s) : hipSuccess;
    int64_t grid = std::min<int64_t>(n * parts, kMaxGrid);  // workgroups take the items beyond in turn
    if (p.wg_per_cu > 0) grid = std::min<int64_t>(grid, (int64_t)p.wg_per_cu * cus);
    for (int b = 0; b < 2 && e == hipSuccess; ++b) {
        if (p.words[b] == 0) continue;
        A.min_words = b == 0 ? 0 : p.split;
        A.max_words = b == 0 ? p.split : INT32_MAX;
        A.lds_words = p.words[b];
        e = launch_eval(A, p.H, idx ? n >= eval_wave_batch(p.H) : p.wave, grid, s);
    }
    if (e == hipSuccess && parts > 1) return launch_bytes_select(out, n, p.elem_bytes, best, s, evals, best_ids);
    if (e == hipSuccess && best && !fin) e = launch_select_rows(out, n, best, evals, best_ids, s);
    return e;
}

// ------------------------------------------------------------------ class tuples

// Sorted distinct non-zero offsets to the in-domain neighbours of x; their number.
__device__ int sorted_offsets(const DevCand& c, int k, int64_t x, int h, int32_t* o) {
    const int64_t l = c.extent[k];
    const int32_t v = coord_value(c, k, x);
    int n = 0;
    for (int s = 1; s <= h; ++s)
        for (int dir = 0; dir < 2; ++dir) {
            const int64_t y = dir ? x + s : x - s;
            if (y < 0 || y >= l) continue;
            const int32_t dv = coord_value(c, k, y) - v;
            int at = 0;
            while (at < n && o[at] < dv) ++at;
            if (dv == 0 || (at < n && o[at] == dv)) continue;
            for (int i = n; i > at; --i) o[i] = o[i - 1];
            o[at] = dv;
            ++n;
        }
    return n;
}

// One workgroup per candidate: along each launch dim the runs of coordinates with equal
// contribution and equal offsets, their product added to the total.  A diagnostic, off
// the evaluation's path.
__global__ __launch_bounds__(256) void k_class_tuples(const DevCand* __restrict__ cands, int64_t n, int32_t h0,
                                                      int32_t h1, int32_t h2, int32_t h3,
                                                      unsigned long long* __restrict__ total) {
    __shared__ unsigned int s_runs;
    const int32_t hs[TM_MAX_LRANK] = {h0, h1, h2, h3};
    unsigned long long acc = 0;
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
        const DevCand& c = cands[i];
        unsigned long long prod = 1;
        for (int k = 0; k < c.lrank; ++k) {
            const int64_t l = c.extent[k];
            const int h = hs[k];
            __syncthreads();
            if (threadIdx.x == 0) s_runs = 0;
            __syncthreads();
            unsigned int runs = 0;
            for (int64_t x = threadIdx.x; x < l; x += blockDim.x) {
                bool start = x == 0 || coord_value(c, k, x) != coord_value(c, k, x - 1);
                if (!start) {
                    int32_t a[2 * kMaxHalo], b[2 * kMaxHalo];
                    const int na = sorted_offsets(c, k, x, h, a), nb = sorted_offsets(c, k, x - 1, h, b);
                    start = na != nb;
                    for (int u = 0; u < na && !start; ++u) start = a[u] != b[u];
                }
                runs += start ? 1 : 0;
            }
            atomicAdd(&s_runs, runs);
            __syncthreads();
            prod *= s_runs;
        }
        acc += prod;
    }
    if (threadIdx.x == 0 && acc) atomicAdd(total, acc);
}

hipError_t launch_class_tuples(const DevCand* cands, int64_t n, const int32_t* halo, unsigned long long* total,
                               hipStream_t s) {
    const int64_t grid = std::min<int64_t>(std::max<int64_t>(n, 1), 65536);
    hipLaunchKernelGGL(k_class_tuples, dim3((unsigned)grid), dim3(256), 0, s, cands, n, halo[0], halo[1], halo[2],
                       halo[3], total);
    return hipGetLastError();
}

}  // namespace tmk
