// tm_compile.h -- a compiled candidate's view for the stencil evaluation (DevEval), on
// the host for single calls and on the GPU, a thread per candidate, for plans (whose
// descriptors then go up once, as DevCand).
#pragma once

#include <stdint.h>

#include "tm_eval.h"
#include "tm_internal.h"

namespace tmk {

// The inverse of op t as the kernels apply it (see DevOp).
__host__ __device__ inline void fill_inverse(const DevCand& d, int t, DevOp* o) {
    const int pa = d.op_a[t], pb = d.op_b[t], plo = pa < pb ? pa : pb, phi = pa < pb ? pb : pa;
    int kind = d.op_kind[t];
    const bool pair = kind == TM_MERGE || kind == TM_SWAP;
    int64_t before = 1;
    for (int u = 0; u < (pair ? plo : pa); ++u) before *= d.shape[t][u];
    if (kind == TM_BALANCE_SPLIT && d.inv_win[t] == d.inv_wout[t]) kind = TM_SPLIT;
    o->kind = kind | (d.inv_lo[t] == 1 ? kOpNoLo : 0) | (before == 1 ? kOpNoHi : 0);
    o->lo = (uint32_t)d.inv_lo[t];
    o->wi = (uint32_t)d.inv_win[t];
    o->wo = (uint32_t)d.inv_wout[t];
    o->rlo = 1.0f / (float)o->lo;
    o->rwo = 1.0f / (float)o->wo;
    uint32_t u[5] = {1, 1, 1, 1, 1};
    if (kind == TM_SPLIT || kind == TM_BALANCE_SPLIT) {
        u[0] = (uint32_t)pb;
        u[1] = (uint32_t)d.inv_c[t];
    } else if (kind == TM_MERGE) {
        u[0] = (uint32_t)d.inv_mid[t];
        u[1] = (uint32_t)d.shape[t][pa];
        u[2] = (uint32_t)d.shape[t][pb];
    } else if (kind == TM_SWAP) {
        u[1] = (uint32_t)d.shape[t][plo];
        u[2] = (uint32_t)d.shape[t][phi];
        u[3] = (uint32_t)d.inv_mid[t];
        u[0] = u[3] * u[1];
    } else {
        for (int j = 0; j < TM_MAX_LRANK; ++j)
            if (j < d.op_nf[t]) u[j] = (uint32_t)d.op_f[t][j];
    }
    for (int j = 0; j < 5; ++j) {
        o->u[j] = u[j];
        o->f[j] = 1.0f / (float)u[j];
    }
}

// Segments, residues and groups of launch dim k (see DevDim), from its projections.
__host__ __device__ inline void count_groups(const DevCand& d, int k, DevDim* g) {
    const int64_t l = d.extent[k];
    int64_t changes = 0, m = 1, longest = l;
    int nblk = 0, ncyc = 0;
    for (int j = 0; j < d.frank; ++j) {
        const int64_t s = d.fshape[j];
        if (d.proj_src[j] != k || s == 1) continue;
        if (d.proj_mode[j] == TM_CYCLIC) {
            ++ncyc;
            int64_t a = m, b = s;
            while (b) {
                const int64_t r = a % b;
                a = b;
                b = r;
            }
            if (m < l) m = m / a * s;
            if (m > l) m = l;  // from l on every coordinate is its own residue
        } else {
            changes += s < l ? s - 1 : l - 1;
            longest = nblk++ == 0 ? (l + s - 1) / s : l;
        }
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
__host__ __device__ inline bool is_simple(const DevCand& d) {
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

__host__ __device__ inline void fill_eval(const DevCand& d, const EvalShape& shape, DevEval* e) {
    e->vol = d.vol;
    e->lrank = d.lrank;
    e->nops = d.nops;
    e->gbits = d.gbits;
    e->gpus = d.gpus;
    e->rgpus = 1.0f / (float)d.gpus;
    e->bij = is_bijective(d);
    e->flags = is_simple(d) ? kEvalSimple : 0;
    e->procs = d.nodes * d.gpus;
    e->points = d.npoints;
    e->first_proc = 0;
    bool distinct = e->bij;
    for (int t = 0; t < d.nops; ++t) fill_inverse(d, t, &e->inv[t]);
    int next = 0;
    for (int k = 0; k < d.lrank; ++k) {
        DevDim& g = e->dim[k];
        count_groups(d, k, &g);
        g.first = next;
        g.rl = 1.0 / (double)g.l;
        g.rM = 1.0 / (double)g.M;
        for (int cyc = 0; cyc < 2; ++cyc)
            for (int j = 0; j < d.frank; ++j) {
                if (d.proj_src[j] != k || (d.proj_mode[j] == TM_CYCLIC) != (cyc == 1) || d.fshape[j] == 1) continue;
                DevProj& p = e->pj[next++];
                p.s = d.fshape[j];
                p.stride = d.fstride[j];
                p.rs = 1.0 / (double)p.s;
            }
        distinct = distinct && !(g.ident && g.nblk > 1);
        e->flags |= (g.ncyc ? kEvalCyclic : 0) | (g.nblk > 1 || g.ncyc > 1 ? kEvalExtra : 0);
    }
    e->flags |= distinct ? kEvalDistinct : 0;
    const EvalNeed n = eval_need(e->dim, d.lrank, d.vol, e->flags & kEvalCyclic, e->bij, shape);
    e->words = n.words;
    e->parts = n.parts;
    e->dim_d = n.dim_d;
}

}  // namespace tmk
