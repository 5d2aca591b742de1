// tm_groups.h -- device functions of the evaluation over coordinate groups: a
// candidate's owner table from its packed inverse ops, contributions of coordinates,
// and the records of its launch dims' groups (DevDim, tm_internal.h).
//
// The descriptor (DevEval) sits in LDS: every phase is a chain of dependent reads of a
// few of its fields, and an LDS read is several times nearer than a scalar load that
// misses the 16 KB scalar cache (some 40 waves of a CU pair share it).  Measured on
// 219,424 search candidates, one wave each, before later steps: fields by scalar loads
// 2.69 ms, from LDS 1.95 ms.
#pragma once

#include <hip/hip_runtime.h>

#include "tm_chain.h"
#include "tm_internal.h"

namespace tmk {

typedef int32_t i32x2 __attribute__((ext_vector_type(2)));
typedef int32_t i32x4v __attribute__((ext_vector_type(4)));

// Copies a DevEval into LDS (16 bytes per thread; the caller synchronises).
__device__ __forceinline__ void stage_eval(DevEval* dst, const DevEval* e, int tid) {
    if (tid < (int)(sizeof(DevEval) / 16))
        reinterpret_cast<i32x4v*>(dst)[tid] = reinterpret_cast<const i32x4v*>(e)[tid];
}

// ------------------------------------------------------------------ exact quotients
//
// The exact quotient n / d lies at least 1/(2d) away from the integers once half is added
// to n; a float product with the rounded reciprocal is off by less than that while
// (n + 0.5) 2^-23 < 0.5, that is for n < 2^22, and needs no correction.  The owner table
// lives in LDS, so every index here is below 2^15.
__device__ __forceinline__ uint32_t div_small(uint32_t n, float r) { return (uint32_t)fmaf((float)n, r, 0.5f * r); }

// floor(x s / l) for 0 <= x < l < 2^31, s <= 2^15, r = 1/l: the product is exact in double;
// a quotient that is no integer is at least 2^-31 below the next one and the rounding
// error is below 2^-35, so the floor of (quotient + 2^-33) is exact.
__device__ __forceinline__ uint32_t block_index(uint32_t x, double s, double r) {
    return (uint32_t)fma((double)x * s, r, 0x1p-33);
}

// floor(n / d) for 0 <= n < 2^47 with a quotient below 2^31, d <= 2^15, r = 1/d: the
// distance to the next integer is at least 2^-15, the error below 2^-20.
__device__ __forceinline__ uint32_t div_wide(double n, double r) { return (uint32_t)fma(n, r, 0x1p-18); }

// ------------------------------------------------------------------ owner table

// Owner keys (node << gbits) | gpu of the final-space coordinates [v0, v1) (v1 <= 2^15),
// AND keep, written to out (IDS: processor ids, node * gpus + gpu, instead): each undoes
// the ops on the linear index, last op first, down to Machine(GPU); uniform branches skip the divisions that an op's place makes trivial
// (nothing after or before its range, adjacent dims, factors of 1).  A thread takes KPT
// coordinates per pass, so an op's constants are read once per pass.
template <int KPT, bool IDS>
__device__ __forceinline__ void owner_table_pass(const DevEval& c, int32_t* __restrict__ out, int32_t v0, int32_t v1,
                                                 int32_t keep, int tid, int nt) {
    const uint32_t g = (uint32_t)c.gpus;
    const int gb = wave_uniform(c.gbits), nops = wave_uniform(c.nops);
    const float rg = c.rgpus;
    {
        uint32_t m[KPT], l0[KPT], h[KPT];
#pragma unroll
        for (int i = 0; i < KPT; ++i) {
            const int32_t v = v0 + tid + i * nt;
            m[i] = (uint32_t)(v < v1 ? v : v1 - 1);  // out-of-range slots repeat a valid index
            l0[i] = h[i] = 0;
        }
        // op 0 reaches Machine(GPU) = (nodes, gpus), so a merge there is of its two dims
        const bool fused = nops > 0 && (wave_uniform(c.inv[0].kind) & kOpKind) == TM_MERGE;
        for (int t = nops - 1; t >= (fused ? 1 : 0); --t) {
            const DevOp& op = c.inv[t];
            const int32_t kf = wave_uniform(op.kind), kind = kf & kOpKind;
            const uint32_t lo = op.lo, wi = op.wi, wo = op.wo;
            if (!(kf & kOpNoLo)) {
                const float rlo = op.rlo;
#pragma unroll
                for (int i = 0; i < KPT; ++i) {
                    const uint32_t q = div_small(m[i], rlo);
                    l0[i] = m[i] - __umul24(q, lo);
                    m[i] = q;
                }
            }
            if (!(kf & kOpNoHi)) {
                const float rwo = op.rwo;
#pragma unroll
                for (int i = 0; i < KPT; ++i) {
                    h[i] = div_small(m[i], rwo);
                    m[i] -= __umul24(h[i], wo);
                }
            }
            if (kind == TM_SPLIT || kind == TM_BALANCE_SPLIT) {
                // output digits (a, a1) of extents (b, cc), x = a * cc + a1; input a + a1 * b;
                // balance_split folds that onto the input extent, floor(v wi / wo): the
                // product is below 2^30 and the float quotient within one
                const uint32_t b = op.u[0], cc = op.u[1];
                const float rc = op.f[1];
#pragma unroll
                for (int i = 0; i < KPT; ++i) {
                    const uint32_t aa = div_small(m[i], rc), a1 = m[i] - __umul24(aa, cc);
                    m[i] = aa + __umul24(a1, b);
                }
                if (kind == TM_BALANCE_SPLIT) {
                    const float rwo = op.rwo;
#pragma unroll
                    for (int i = 0; i < KPT; ++i) {
                        const uint32_t n = m[i] * wi, q = (uint32_t)((float)n * rwo);
                        const int32_t r = (int32_t)(n - __umul24(q, wo));
                        m[i] = r < 0 ? q - 1 : (r >= (int32_t)wo ? q + 1 : q);
                    }
                }
            } else if (kind == TM_MERGE) {
                // output (a of extent sp * sq, mid); input (a mod sp, mid, a / sp)
                const uint32_t mid = op.u[0], sp = op.u[1], sq = op.u[2];
                const float rsp = op.f[1];
                uint32_t xm[KPT];
#pragma unroll
                for (int i = 0; i < KPT; ++i) xm[i] = 0;
                if (wave_uniform((int32_t)mid) > 1) {
                    const float rmid = op.f[0];
#pragma unroll
                    for (int i = 0; i < KPT; ++i) {
                        const uint32_t aa = div_small(m[i], rmid);
                        xm[i] = m[i] - __umul24(aa, mid);
                        m[i] = aa;
                    }
                }
#pragma unroll
                for (int i = 0; i < KPT; ++i) {
                    const uint32_t ahi = div_small(m[i], rsp), alo = m[i] - __umul24(ahi, sp);
                    m[i] = __umul24(__umul24(alo, mid) + xm[i], sq) + ahi;
                }
            } else if (kind == TM_SWAP) {
                // output (y_lo of extent shi, mid, y_hi of extent slo); input (y_hi, mid, y_lo)
                const uint32_t ms = op.u[0], slo = op.u[1], shi = op.u[2], mid = op.u[3];
                const float rms = op.f[0];
                uint32_t xm[KPT], ylo[KPT];
#pragma unroll
                for (int i = 0; i < KPT; ++i) {
                    ylo[i] = div_small(m[i], rms);
                    m[i] -= __umul24(ylo[i], ms);
                    xm[i] = 0;
                }
                if (wave_uniform((int32_t)mid) > 1) {
                    const float rslo = op.f[1];
#pragma unroll
                    for (int i = 0; i < KPT; ++i) {
                        xm[i] = div_small(m[i], rslo);
                        m[i] -= __umul24(xm[i], slo);
                    }
                }
#pragma unroll
                for (int i = 0; i < KPT; ++i) m[i] = __umul24(__umul24(m[i], mid) + xm[i], shi) + ylo[i];
            } else {  // TM_DECOMPOSE: output digits d_j in C order; input sum_j d_j prod_{i < j} f_i
                uint32_t r[KPT], w = __umul24(__umul24(op.u[0], op.u[1]), op.u[2]);
#pragma unroll
                for (int i = 0; i < KPT; ++i) r[i] = 0;
#pragma unroll
                for (int j = TM_MAX_LRANK - 1; j >= 1; --j) {
                    const uint32_t f = op.u[j];
                    if (wave_uniform((int32_t)f) > 1) {  // factors past their number are 1
                        const float rf = op.f[j];
#pragma unroll
                        for (int i = 0; i < KPT; ++i) {
                            const uint32_t q = div_small(m[i], rf);
                            r[i] += __umul24(m[i] - __umul24(q, f), w);
                            m[i] = q;
                        }
                    }
                    w = j == 3 ? __umul24(op.u[0], op.u[1]) : op.u[0];
                }
#pragma unroll
                for (int i = 0; i < KPT; ++i) m[i] += r[i];
            }
            if (!(kf & kOpNoHi)) {
#pragma unroll
                for (int i = 0; i < KPT; ++i) m[i] += __umul24(h[i], wi);
            }
            if (!(kf & kOpNoLo)) {
#pragma unroll
                for (int i = 0; i < KPT; ++i) m[i] = __umul24(m[i], lo) + l0[i];
            }
        }
        // m: the processor, or where the merge is fused its index with the node fastest
        const uint32_t d = fused ? c.inv[0].u[1] : g;
        const float rd = fused ? c.inv[0].f[1] : rg;
#pragma unroll
        for (int i = 0; i < KPT; ++i) {
            const int32_t v = v0 + tid + i * nt;
            if (IDS && !fused) {
                if (v < v1) out[v] = (int32_t)m[i];
                continue;
            }
            const uint32_t q = div_small(m[i], rd), r = m[i] - __umul24(q, d);
            const uint32_t node = fused ? r : q, gpu = fused ? q : r;
            if (v < v1) out[v] = IDS ? (int32_t)(__umul24(node, g) + gpu) : (int32_t)((node << gb) | gpu) & keep;
        }
    }
}

// The whole range: passes of four coordinates a thread, the rest in one of as many as are
// left (on 219,424 search candidates of 245 coordinates each 4.5 a thread on average; with
// passes of one, two or four 5.2).
template <bool IDS = false>
__device__ __forceinline__ void owner_table(const DevEval& c, int32_t* __restrict__ out, int32_t v0, int32_t v1,
                                            int32_t keep, int tid, int nt) {
    for (; v0 < v1; v0 += 4 * nt) {
        const int32_t len = v1 - v0;
        if (len <= nt) owner_table_pass<1, IDS>(c, out, v0, v1, keep, tid, nt);
        else if (len <= 2 * nt) owner_table_pass<2, IDS>(c, out, v0, v1, keep, tid, nt);
        else if (len <= 3 * nt) owner_table_pass<3, IDS>(c, out, v0, v1, keep, tid, nt);
        else owner_table_pass<4, IDS>(c, out, v0, v1, keep, tid, nt);
    }
}

// Processor ids of all coordinates, in little code (beside another table in a kernel: the
// instruction cache holds 64 KB).
__device__ __forceinline__ void owner_ids(const DevEval& c, int32_t* __restrict__ out, int32_t vol, int tid, int nt) {
    for (int32_t v0 = 0; v0 < vol; v0 += nt) owner_table_pass<1, true>(c, out, v0, vol, -1, tid, nt);
}

// ------------------------------------------------------------------ coordinates

// One launch dim in a lane's registers (lanes may hold different dims): its first block
// and first cyclic entry (size 1 where there is none); the others are read when
// kEvalExtra is set.
struct LaneDim {
    uint32_t l, M, nseg, ident;
    int32_t first, nblk, ncyc;
    double rl, rM, bs, brs, crs;
    uint32_t bst, cs, cst;
};

__device__ __forceinline__ LaneDim lane_dim(const DevEval& c, int d, bool cyclic) {
    const DevDim& q = c.dim[d];
    LaneDim x;
    x.l = (uint32_t)q.l;
    x.M = (uint32_t)q.M;
    x.nseg = (uint32_t)q.nseg;
    x.first = q.first;
    x.nblk = q.nblk;
    x.ncyc = q.ncyc;
    x.ident = (uint32_t)q.ident;
    x.rl = q.rl;
    x.rM = q.rM;
    // first + nblk is at most the number of entries: clamped, the entry itself unused
    const DevProj& b = c.pj[x.first & (TM_MAX_MRANK - 1)];
    x.bs = x.nblk ? (double)b.s : 1.0;
    x.bst = x.nblk ? (uint32_t)b.stride : 0u;
    x.brs = b.rs;
    x.cs = 1;
    x.cst = 0;
    x.crs = 1.0;
    if (cyclic) {
        const DevProj& y = c.pj[(x.first + x.nblk) & (TM_MAX_MRANK - 1)];
        x.cs = x.ncyc ? (uint32_t)y.s : 1u;
        x.cst = x.ncyc ? (uint32_t)y.stride : 0u;
        x.crs = x.ncyc ? y.rs : 1.0;
    }
    return x;
}

// Contribution of the cyclic projections at x (which may lie a halo past the extent) and
// of the block projections at x.  extra: the candidate's flag (uniform).
__device__ __forceinline__ uint32_t cyclic_value(const DevEval& c, const LaneDim& d, uint32_t x, bool extra) {
    uint32_t v = (x - div_wide((double)x, d.crs) * d.cs) * d.cst;
    if (extra)
        for (int j = 1; j < d.ncyc; ++j) {
            const DevProj& p = c.pj[d.first + d.nblk + j];
            v += (x - div_wide((double)x, p.rs) * (uint32_t)p.s) * (uint32_t)p.stride;
        }
    return v;
}
__device__ __forceinline__ uint32_t block_value(const DevEval& c, const LaneDim& d, uint32_t x, bool extra) {
    uint32_t v = block_index(x, d.bs, d.rl) * d.bst;
    if (extra)
        for (int j = 1; j < d.nblk; ++j) {
            const DevProj& p = c.pj[d.first + j];
            v += block_index(x, (double)p.s, d.rl) * (uint32_t)p.stride;
        }
    return v;
}

// First cell of segment a (0 <= a <= nseg).  One block projection of s blocks: ceil(a l /
// s).  Several: the smallest cell with at least a change points at or before it (binary
// search over their closed-form counts).
__device__ __forceinline__ uint32_t segment_start(const DevEval& c, const LaneDim& d, uint32_t a, bool extra) {
    if (d.ident || a == 0) return a;
    if (a >= d.nseg) return d.l;
    if (!extra || d.nblk == 1) return div_wide(fma((double)a, (double)d.l, d.bs - 1.0), d.brs);
    uint32_t lo = 1, hi = d.l;  // the answer lies in [lo, hi]
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        uint32_t cnt = 0;
        for (int j = 0; j < d.nblk; ++j) cnt += block_index(mid, (double)c.pj[d.first + j].s, d.rl);
        if (cnt >= a) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

// ------------------------------------------------------------------ group records

// A group's members differ only in which neighbours they have: the interior ones (at
// least h from both ends of their segment) all see the same offsets, the others are at
// most 2h edge members.  Record (int32 words, group_stride), U = 2H slots without cyclic
// projections, 4H with:
//   [0] contribution | edge members << 24
//   [1] members
//   U slots, one per distinct non-zero offset, the rest 0: offset & 0xffff | edge members
//       that see it << 16 | interior members see it << 24
//   with masks: 2h + 1 16-bit masks over the slots -- which offsets a member sees -- of
//       the interior members, then of each edge member
// Contributions and offsets stay below 2^15 (the owner table is held in LDS).

// The unions of the first i of H masks of U bits each, for i = 0..H, packed so that i may
// differ per lane.
template <int H, int U>
struct PrefixMasks {
    uint64_t packed = 0;
    uint32_t last = 0;
    __device__ __forceinline__ void set(const uint32_t (&bit)[U], int first) {
#pragma unroll
        for (int s = 0; s < H; ++s) {
            last |= bit[first + s];
            packed |= (uint64_t)last << (U * s);
        }
    }
    __device__ __forceinline__ uint32_t at(int i) const {
        const uint32_t m = (uint32_t)(packed >> (U * (i > 0 ? i - 1 : 0))) & ((1u << U) - 1u);
        return i > 0 ? m : 0u;
    }
};

// Record of group g of dim d (in this lane's registers) with halo h <= H, at o.
template <int H, bool CYC>
__device__ __forceinline__ void build_group(const DevEval& c, const LaneDim& d, int h, bool masks, bool extra,
                                            uint32_t g, int32_t* __restrict__ o) {
    constexpr int U = CYC ? 4 * H : 2 * H;
    uint32_t a = g, r = 0;
    if (CYC) {
        a = div_small(g, (float)d.rM);
        r = g - __umul24(a, d.M);
    }
    const uint32_t x0 = segment_start(c, d, a, extra), x1 = segment_start(c, d, a + 1, extra), len = x1 - x0;
    const bool none = r >= len;  // no such coordinate: an empty record
    auto value = [&](uint32_t x) {
        return block_value(c, d, x, extra) + (CYC ? cyclic_value(c, d, x, extra) : 0u);
    };
    const uint32_t cv = none ? 0u : value(x0 + r);
    uint32_t W = none ? 0u : len;
    // the members x0 + r + k M; jf: how far the last one is from the segment's last cell
    uint32_t jf = 0;
    if (CYC && !none && d.M > 1) {
        const uint32_t k = div_wide((double)(len - 1 - r), d.rM);
        W = k + 1;
        jf = len - 1 - r - k * d.M;
    }
    // offsets: [0, H) to the cells before the segment (nearest first), [H, 2H) to those
    // after it, then within the segment s back and s forward; 0 = none
    int32_t dv[U];
#pragma unroll
    for (int s = 0; s < H; ++s) {
        dv[s] = !none && s < h && x0 > (uint32_t)s ? (int32_t)(value(x0 - 1 - s) - cv) : 0;
        dv[H + s] = !none && s < h && x1 + s < d.l ? (int32_t)(value(x1 + s) - cv) : 0;
    }
    if (CYC) {
        const bool on = !none && d.M > 1;
        const uint32_t cy = cyclic_value(c, d, x0 + r, extra);
#pragma unroll
        for (int s = 0; s < H; ++s) {
            uint32_t y = x0 + r;  // s + 1 back, whole periods on where that is before the first cell
            while (y < (uint32_t)s + 1) y += d.M;
            y -= s + 1;
            dv[(CYC ? 2 : 0) * H + s] = on && s < h ? (int32_t)(cyclic_value(c, d, y, extra) - cy) : 0;
            dv[(CYC ? 3 : 0) * H + s] =
                on && s < h ? (int32_t)(cyclic_value(c, d, x0 + r + s + 1, extra) - cy) : 0;
        }
    }
    // every distinct non-zero one takes the slot of its first occurrence
    uint32_t bit[U];
#pragma unroll
    for (int i = 0; i < U; ++i) {
        uint32_t b = dv[i] ? 1u << i : 0u;
#pragma unroll
        for (int j = i - 1; j >= 0; --j) b = dv[j] == dv[i] ? bit[j] : b;
        bit[i] = b;
    }
    // unions: before / after the segment, back / forward inside it
    PrefixMasks<H, U> ml, mr, il, ir;
    ml.set(bit, 0);
    mr.set(bit, H);
    if (CYC) {
        il.set(bit, (CYC ? 2 : 0) * H);
        ir.set(bit, (CYC ? 3 : 0) * H);
    }
    const uint32_t imask = il.last | ir.last;
    uint16_t* mk = reinterpret_cast<uint16_t*>(o + 2 + U);
    uint32_t ne = 0, cnt[U];  // edge members; those that see slot i
#pragma unroll
    for (int i = 0; i < U; ++i) cnt[i] = 0;
    auto edge = [&](bool in, uint32_t m) {
        ne += in ? 1u : 0u;
        m = in ? m : 0u;
        if (masks && in) mk[ne] = (uint16_t)m;
#pragma unroll
        for (int i = 0; i < U; ++i) cnt[i] += (m >> i) & 1u;
    };
    // members i cells from the segment's first cell, then those j cells from its last
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const bool in = !none && i < h && (uint32_t)i < len &&
                        (!CYC || ((uint32_t)i >= r && (d.M == 1 || (uint32_t)i == r || (uint32_t)i - r == d.M)));
        const uint32_t j = len - 1 - i;
        edge(in, il.at(i) | ml.at(h - i) | (j < (uint32_t)h ? ir.at((int)j) | mr.at(h - (int)j) : ir.last));
    }
#pragma unroll
    for (int j = 0; j < H; ++j) {
        const bool in = !none && j < h && (uint32_t)j + (uint32_t)h < len &&
                        (!CYC || ((uint32_t)j >= jf && (d.M == 1 || (uint32_t)j == jf || (uint32_t)j - jf == d.M)));
        edge(in, ir.at(j) | mr.at(h - j) | il.last);
    }
    o[0] = (int32_t)(cv | ne << 24);
    o[1] = (int32_t)W;
    if (masks) mk[0] = (uint16_t)imask;
#pragma unroll
    for (int i = 0; i < U; ++i)
        o[2 + i] = bit[i] == 1u << i
                       ? (int32_t)(((uint32_t)dv[i] & 0xffffu) | cnt[i] << 16 | ((imask >> i) & 1u) << 24)
                       : 0;
}

}  // namespace tmk
