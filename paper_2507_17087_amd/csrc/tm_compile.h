// tm_compile.h -- a compiled candidate's view for the stencil evaluation (DevEval), on
// the host for single calls and on the GPU, a thread per candidate, for plans (whose
// descriptors then go up once, as DevCand).
#pragma once

#include <stdint.h>

#include "tm_eval.h"
#include "tm_internal.h"

namespace tmk {

// An op of a candidate with the products its inverse needs (see DevCand): the dims it
// touches (sa, sb: their extents), the ones after (lo), and whether none are before.
struct OpView {
    int32_t kind, a, b, nf;
    const int32_t* f;
    int32_t sa, sb, lo, wi, wo, mid, c;
    bool first;
};

// The inverse of an op as the kernels apply it (see DevOp).
__host__ __device__ inline void fill_inverse(const OpView& v, DevOp* o) {
    int kind = v.kind;
    if (kind == TM_BALANCE_SPLIT && v.wi == v.wo) kind = TM_SPLIT;
    o->kind = kind | (v.lo == 1 ? kOpNoLo : 0) | (v.first ? kOpNoHi : 0);
    o->lo = (uint32_t)v.lo;
    o->wi = (uint32_t)v.wi;
    o->wo = (uint32_t)v.wo;
    o->rlo = 1.0f / (float)o->lo;
    o->rwo = 1.0f / (float)o->wo;
    uint32_t u[5] = {1, 1, 1, 1, 1};
    if (kind == TM_SPLIT || kind == TM_BALANCE_SPLIT) {
        u[0] = (uint32_t)v.b;
        u[1] = (uint32_t)v.c;
    } else if (kind == TM_MERGE) {
        u[0] = (uint32_t)v.mid;
        u[1] = (uint32_t)v.sa;
        u[2] = (uint32_t)v.sb;
    } else if (kind == TM_SWAP) {
        u[1] = (uint32_t)(v.a < v.b ? v.sa : v.sb);
        u[2] = (uint32_t)(v.a < v.b ? v.sb : v.sa);
        u[3] = (uint32_t)v.mid;
        u[0] = u[3] * u[1];
    } else {
        for (int j = 0; j < TM_MAX_LRANK; ++j)
            if (j < v.nf) u[j] = (uint32_t)v.f[j];
    }
    for (int j = 0; j < 5; ++j) {
        o->u[j] = u[j];
        o->f[j] = 1.0f / (float)u[j];
    }
}

// Op t of a compiled candidate.
__host__ __device__ inline OpView op_view(const DevCand& d, int t) {
    OpView v;
    v.kind = d.op_kind[t];
    v.a = d.op_a[t];
    v.b = d.op_b[t];
    v.nf = d.op_nf[t];
    v.f = d.op_f[t];
    const bool pair = v.kind == TM_MERGE || v.kind == TM_SWAP;
    v.sa = d.shape[t][v.a];
    v.sb = pair ? d.shape[t][v.b] : 1;
    const int lo = pair && v.b < v.a ? v.b : v.a;
    int64_t before = 1;
    for (int u = 0; u < lo; ++u) before *= d.shape[t][u];
    v.first = before == 1;
    v.lo = d.inv_lo[t];
    v.wi = d.inv_win[t];
    v.wo = d.inv_wout[t];
    v.mid = d.inv_mid[t];
    v.c = d.inv_c[t];
    return v;
}

// The projections of a candidate (DevCand or CandView) that change anything, as bits: final
// dim j projected in blocks (cyclically) from launch dim k is bit 8 k + j (32 + 8 k + j).
template <class C>
__host__ __device__ inline uint64_t projection_bits(const C& d) {
    uint64_t m = 0;
    for (int j = 0; j < d.frank; ++j)
        m |= (uint64_t)(d.fshape[j] != 1) << (8 * (d.proj_src[j] + (d.proj_mode[j] == TM_CYCLIC ? TM_MAX_LRANK : 0)) + j);
    return m;
}
__host__ __device__ inline uint32_t blocks_of(uint64_t bits, int k) { return (uint32_t)(bits >> (8 * k)) & 0xffu; }
__host__ __device__ inline uint32_t cyclics_of(uint64_t bits, int k) { return blocks_of(bits, k + TM_MAX_LRANK); }

// The least common multiple of m and s, at most l: from l on every coordinate is its own
// residue.
__host__ __device__ inline int64_t lcm_upto(int64_t m, int64_t s, int64_t l) {
    int64_t a = m, b = s;
    while (b) {
        const int64_t r = a % b;
        a = b;
        b = r;
    }
    if (m < l) m = m / a * s;
    return m < l ? m : l;
}

// Segments, residues and groups of launch dim k (see DevDim), from its projections.
template <class C>
__host__ __device__ inline void count_groups(const C& d, int k, uint64_t bits, DevDim* g) {
    const int64_t l = d.extent[k];
    int64_t changes = 0, m = 1, longest = l;
    int nblk = 0, ncyc = 0;
    for (uint32_t c = cyclics_of(bits, k); c; c &= c - 1, ++ncyc) m = lcm_upto(m, d.fshape[__builtin_ctz(c)], l);
    for (uint32_t c = blocks_of(bits, k); c; c &= c - 1) {
        const int64_t s = d.fshape[__builtin_ctz(c)];
        changes += s < l ? s - 1 : l - 1;
        longest = nblk++ == 0 ? (int64_t)((uint32_t)(l + s - 1) / (uint32_t)s) : l;
    }
    // groups per segment: m, or every coordinate of one no longer than that; then there
    // are at least as many groups as coordinates
    const int64_t nseg = changes + 1, r = m < longest ? m : longest;
    g->ident = nseg >= l || nseg * r >= l ? 1 : 0;
    g->l = (int32_t)l;
    g->nseg = (int32_t)(g->ident ? l : nseg);
    g->M = (int32_t)(g->ident ? 1 : m);
    g->G = g->nseg * g->M;
    g->nblk = nblk;
    g->ncyc = ncyc;
}

// Whether distinct final coordinates always have distinct owners.
__host__ __device__ inline bool is_bijective(const DevCand& d) {
    for (int t = 0; t < d.nops; ++t)
        if (d.op_kind[t] == TM_BALANCE_SPLIT && d.inv_win[t] != d.inv_wout[t]) return false;
    return true;
}

// Whether every launch dim is projected by blocks onto exactly one final dim.
template <class C>
__host__ __device__ inline bool is_simple(const C& d) {
    uint32_t seen = 0;
    for (int j = 0; j < d.frank; ++j) {
        if (d.proj_mode[j] != TM_BLOCK || ((seen >> d.proj_src[j]) & 1u)) return false;
        seen |= 1u << d.proj_src[j];
    }
    return d.frank == d.lrank;
}

// What a launch layout asks of a candidate: halos up to H, node-level counting, work
// items of about per_item tuples (0: fill parts of at least kEvalPartTuples at most).
struct EvalShape {
    int32_t H, node_level;
    int64_t per_item, fill;
};

// LDS words a candidate needs -- its owner table, the group records of every dim but the
// one with the most groups (dim_d), and at least 64 of that one's (one pass of a wave) --
// the words of all records, and its parts.
struct EvalNeed {
    int32_t words, whole, parts, dim_d;
};
__host__ __device__ inline EvalNeed eval_need(const DevDim* dim, int lrank, int32_t vol, bool cyclic, bool bij,
                                              const EvalShape& e) {
    EvalNeed n;
    int64_t groups = 0, tuples = 1;
    n.dim_d = 0;
    for (int k = 0; k < lrank; ++k) {
        if (dim[k].G > dim[n.dim_d].G) n.dim_d = k;
        groups += dim[k].G;
        tuples *= dim[k].G;
    }
    const int64_t g = dim[n.dim_d].G, st = group_stride(cyclic, halo_class(e.H), e.node_level || !bij);
    const int64_t w = ((vol + 3) & ~3) + (groups - (g < 64 ? 0 : g - 64)) * st;
    n.words = (int32_t)((w + 3) & ~int64_t(3));
    const int64_t whole = (w + (g < 64 ? 0 : g - 64) * st + 3) & ~int64_t(3);
    n.whole = (int32_t)(whole < INT32_MAX ? whole : INT32_MAX);
    int64_t parts;
    if (e.per_item > 0) {
        parts = (tuples + e.per_item - 1) / e.per_item;
    } else {
        parts = (tuples + kEvalPartTuples - 1) / kEvalPartTuples;
        parts = parts < e.fill ? parts : e.fill;
    }
    parts = parts < g ? parts : g;
    n.parts = (int32_t)(parts < 1 ? 1 : parts);
    return n;
}

// Everything but the ops and the machine.
template <class C>
__host__ __device__ inline EvalNeed fill_dims(const C& d, bool bij, const EvalShape& shape, DevEval* e) {
    e->vol = d.vol;
    e->lrank = d.lrank;
    e->nops = d.nops;
    e->bij = bij;
    int flags = is_simple(d) ? kEvalSimple : 0;
    e->points = d.npoints;
    e->offset = 0;
    bool distinct = bij;
    const uint64_t bits = projection_bits(d);
    int next = 0;
    for (int k = 0; k < d.lrank; ++k) {
        DevDim& g = e->dim[k];
        count_groups(d, k, bits, &g);
        g.first = next;
        g.rl = 1.0 / (double)g.l;
        g.rM = 1.0 / (double)g.M;
        for (int cyc = 0; cyc < 2; ++cyc)
            for (uint32_t c = cyc ? cyclics_of(bits, k) : blocks_of(bits, k); c; c &= c - 1) {
                const int j = __builtin_ctz(c);
                DevProj& p = e->pj[next++];
                p.s = d.fshape[j];
                p.stride = d.fstride[j];
                p.rs = 1.0 / (double)p.s;
            }
        distinct = distinct && !(g.ident && g.nblk > 1);
        flags |= (g.ncyc ? kEvalCyclic : 0) | (g.nblk > 1 || g.ncyc > 1 ? kEvalExtra : 0);
    }
    flags |= distinct ? kEvalDistinct : 0;
    e->flags = flags;
    const EvalNeed n = eval_need(e->dim, d.lrank, d.vol, flags & kEvalCyclic, bij, shape);
    e->words = n.words;
    e->parts = n.parts;
    e->dim_d = n.dim_d;
    return n;
}

__host__ __device__ inline void fill_eval(const DevCand& d, const EvalShape& shape, DevEval* e) {
    e->gbits = d.gbits;
    e->gpus = d.gpus;
    e->rgpus = 1.0f / (float)d.gpus;
    e->procs = d.nodes * d.gpus;
    for (int t = 0; t < d.nops; ++t) fill_inverse(op_view(d, t), &e->inv[t]);
    fill_dims(d, is_bijective(d), shape, e);
    e->offset = d.arena_off;
}

__host__ __device__ inline void fill_feat(const DevCand& d, DevFeat* f) {
    uint32_t kinds = 0, opa = 0, proj = 0;
    int first = -1;  // decompose
    for (int t = 0; t < d.nops; ++t) {
        kinds |= (uint32_t)d.op_kind[t] << (4 * t);
        if (t < 3) opa |= (uint32_t)d.op_a[t] << (8 * t);
        if (first < 0 && d.op_kind[t] == TM_DECOMPOSE) first = t;
    }
    for (int j = 0; j < d.frank; ++j)
        proj |= ((uint32_t)d.proj_src[j] | (d.proj_mode[j] == TM_BLOCK ? 0u : 8u)) << (4 * j);
    f->nodes = d.nodes;
    f->gpus = d.gpus;
    f->counts = (uint32_t)d.lrank | (uint32_t)d.nops << 8 | (uint32_t)d.gbits << 16 | (uint32_t)d.frank << 24;
    f->kinds = kinds;
    f->opa = opa;
    f->proj = proj;
    for (int k = 0; k < TM_MAX_LRANK; ++k) {
        f->ext[k] = (int32_t)d.extent[k];
        f->F[k] = first >= 0 && k < d.op_nf[first] ? d.op_f[first][k] : 1;
    }
    for (int j = 0; j < TM_MAX_MRANK; ++j) f->fshape[j] = d.fshape[j];
    for (int t = 0; t < 6; ++t) f->opb[t] = d.op_b[t];
}

// A validated candidate without the tables' layout: what the calls that go straight to
// DevEval need of it.
struct CandView {
    int32_t lrank, frank, vol, nops;
    int64_t npoints, rows;
    int64_t extent[TM_MAX_LRANK];
    int32_t fshape[TM_MAX_MRANK], fstride[TM_MAX_MRANK];
    int8_t proj_src[TM_MAX_MRANK], proj_mode[TM_MAX_MRANK];
};

// Validates c and fills v and e (tm_host.cpp).  False: c is invalid, or larger than the
// evaluation's workgroups take; the general path tells which.
bool compile_eval(const tm_candidate* c, const EvalShape& shape, CandView* v, DevEval* e, EvalNeed* need);

}  // namespace tmk
