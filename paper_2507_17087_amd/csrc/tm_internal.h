// tm_internal.h -- structures shared by the host side and the kernels of libtaskmap.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

#include "taskmap.h"

namespace tmk {

// One transformation as the kernels undo it, on linear indices (C order) of the
// processor space: the dims it touches form a contiguous range of its input shape
// (swap and merge: from the lower to the higher position; the others: one dim), inside
// which it maps the range's digits; the dims before and after pass through.  lo: the
// product of the dims after the range; wi / wo: volume of the range in the input /
// output shape; then per kind (u, and in f the reciprocals of its divisors):
//   split, balance_split  u = {b, c}: output digits (a of extent b, a1 of extent c)
//   merge                 u = {mid, s_p, s_q}; f = {1/mid, 1/s_p}
//   swap                  u = {mid * s_lo, s_lo, s_hi, mid}; f = {1/(mid * s_lo), 1/s_lo}
//   decompose             u = the factors (1 past their number); f = 1/u
// A balance_split whose factor divides is recorded as the split it equals.  One 64-byte
// record: four 16-byte LDS reads.
struct DevOp {
    int32_t kind;                 // tm_op_kind | kOpNoLo / kOpNoHi: lo == 1 / nothing before the range
    uint32_t lo, wi, wo;
    float rlo, rwo;               // 1/lo, 1/wo
    uint32_t u[5];
    float f[5];
};
constexpr int32_t kOpKind = 0xff, kOpNoLo = 0x100, kOpNoHi = 0x200;

// A final dim of size above 1 as a launch dim's coordinates see it.
struct DevProj {
    int32_t s, stride;            // its size and its stride in the final space
    double rs;                    // 1/s
};

// Coordinate groups of one launch dim.  Coordinates with the same contribution to the
// final index form a group.  The block projections' change points (cells where one of
// their block indices steps) cut [0, l) into segments in which they are constant; within
// a segment the contribution depends only on x modulo M, the least common multiple of
// the cyclic sizes.  Group g = a M + r holds segment a's coordinates x0 + r, x0 + r + M,
// ... .  When that would give no fewer groups than coordinates, every coordinate is a
// segment of its own (ident: nseg = l, M = 1).  Coinciding change points of several
// block projections give empty segments.  48 bytes: three 16-byte LDS reads.
struct DevDim {
    int32_t l, M;                 // extent, residues
    int32_t nseg, G;              // segments; groups: nseg * M
    int32_t first, nblk, ncyc;    // its entries of DevEval::pj: the block ones, then the cyclic ones
    int32_t ident;
    double rl;                    // 1/l
    double rM;                    // 1/M
};

// What the stencil evaluation reads of a candidate: 896 bytes, staged in LDS with one
// 16-byte load per lane.
struct alignas(16) DevEval {
    int32_t vol, lrank, nops, gbits;
    int32_t gpus;
    float rgpus;                  // 1/gpus
    int32_t bij;                  // every op is a bijection: distinct coordinates, distinct owners
    int32_t flags;                // kEval*
    int32_t words, parts, dim_d;  // LDS words the evaluation needs, its workgroups; the dim with the most groups
    int32_t procs;                // nodes * gpus
    int64_t points;               // of the launch domain
    int64_t offset;               // matmul batches: processors of the candidates before this one;
                                  // plans: its owner table's first word among the batch's (maps)
    DevDim dim[TM_MAX_LRANK];
    DevProj pj[TM_MAX_MRANK];
    DevOp inv[TM_MAX_OPS];
};
// kEvalCyclic: some launch dim has a cyclic projection; kEvalExtra: some has several
// block or several cyclic ones; kEvalSimple: every launch dim is projected by blocks onto
// exactly one final dim
constexpr int32_t kEvalCyclic = 1, kEvalExtra = 2, kEvalSimple = 4, kEvalDistinct = 8;
static_assert(sizeof(DevEval) == 896, "staged by the first 56 lanes of a wave");

// Compiled candidate as the kernels read it.  The host fills in the shapes of the
// processor space before every transformation (validation computes them anyway);
// the table-build kernel derives everything per coordinate from these.
struct DevCand {
    int32_t lrank, nops, nodes, gpus;
    int32_t gbits, frank, vol, words;   // gpu bits of the owner key; final rank and volume; table words
    int64_t extent[TM_MAX_LRANK];
    int64_t npoints;
    int64_t arena_off;                  // word offset of this candidate's tables
    int64_t item_first;                 // first work item of this candidate
    int64_t rows;                       // points / extent[lrank-1]
    int32_t L, pad1;                    // row length = last extent
    int32_t coord_off[TM_MAX_LRANK];    // table offsets of the per-dim coordinate tables
    int32_t cls_off[TM_MAX_LRANK];      // table offsets of the per-dim coordinate-class blocks
    int32_t cls_cap[TM_MAX_LRANK];      // class capacity of each dim (an upper bound on the class count)
    int32_t cls_base, cls_words;        // class record (four class counts) + the blocks: offset and words
    int32_t lds_words, pad2;            // owner table and, where it fits the LDS, the last dim's coordinate table
    int32_t citems, pad3;               // counting work items
    int32_t fshape[TM_MAX_MRANK], fstride[TM_MAX_MRANK];
    int8_t proj_src[TM_MAX_MRANK], proj_mode[TM_MAX_MRANK];
    int32_t rank[TM_MAX_OPS];                    // rank before op t
    int32_t shape[TM_MAX_OPS][TM_MAX_MRANK];     // shape before op t
    int32_t op_kind[TM_MAX_OPS], op_a[TM_MAX_OPS], op_b[TM_MAX_OPS], op_nf[TM_MAX_OPS];
    int32_t op_f[TM_MAX_OPS][TM_MAX_LRANK];
    // Inverse of op t on linear indices: the dims the op touches form a contiguous
    // range of its input shape (swap and merge: from the lower to the higher
    // position; the others: one dim), inside which the op maps the range's digits;
    // the dims before and after the range pass through.  inv_lo: product of the
    // input dims after the range; inv_win / inv_wout: volume of the range in the
    // input / output shape; inv_mid: product of the dims strictly inside a swap or
    // merge range; inv_c: the second output extent of a split or balance_split.
    int32_t inv_lo[TM_MAX_OPS], inv_win[TM_MAX_OPS], inv_wout[TM_MAX_OPS], inv_mid[TM_MAX_OPS],
        inv_c[TM_MAX_OPS];
};

// What the ranker's features read of a candidate: one cache line.
struct alignas(16) DevFeat {
    int32_t ext[TM_MAX_LRANK];  // 0 past the launch rank
    int32_t nodes, gpus;
    uint32_t counts;            // launch rank | ops << 8 | gpu bits << 16 | final rank << 24
    uint32_t kinds;             // of op t: bits 4 t
    int32_t fshape[TM_MAX_MRANK];
    int32_t opb[6];
    uint32_t opa;               // of op t < 3: bits 8 t
    uint32_t proj;              // of final dim j: source in bits 4 j, cyclic in bit 4 j + 3
    int32_t F[TM_MAX_LRANK];    // the factors of the first decompose (1 past them)
    int32_t pad[4];
};

// Batch header: one per plan, in device memory.
struct DevHeader {
    int64_t n;            // candidates
    int32_t halo[TM_MAX_LRANK];
    int32_t elem_bytes, lrank;
};

// Host-side result of validation: the rank and the extents (with ones up to 8) before
// each op and after the last.
struct Shapes {
    int32_t rank[TM_MAX_OPS + 1];
    int32_t size[TM_MAX_OPS + 1][TM_MAX_MRANK];
};

// An entry of a per-dim coordinate table holds the contribution of that coordinate
// to the linear final-space index (volumes are at most 2^24).
//
// Coordinate classes.  Along launch dim d, coordinate x has a
// contribution C_d[x] and a set of distinct non-zero index offsets C_d[x +- s] -
// C_d[x] to its in-domain star neighbours (1 <= s <= h_d).  A class is a maximal run of
// consecutive coordinates with equal contribution and equal offset set.  Matmul batches
// too large for the LDS build them with a zero halo (runs of equal contribution): class k's
// entry and first coordinate (k = R is the extent, so the run length is start[k+1] -
// start[k]).  For stencil batches the layout with classes is only a measure: of the scratch
// that tm_eval_stencil_batch_noalloc counts and of the run that a map needs before it.
constexpr int32_t kMaxLdsWords = 32768;
constexpr int kMaxHalo = 4;

// Upper bound on the class count of launch dim d (its block capacity): a class
// boundary at x needs a change of contribution within the halo of x (at some c with
// x - h <= c <= x + h), so there are at most 1 + changes * (2h + 1) classes, and
// never more than the extent.  Block projections change at most s - 1 times along
// the dim, cyclic ones at every step.
__host__ __device__ inline int64_t class_cap(const DevCand& c, int d, int h) {
    const int64_t l = c.extent[d];
    int64_t ch = 0;
    for (int j = 0; j < c.frank; ++j) {
        if (c.proj_src[j] != d) continue;
        const int64_t s = c.fshape[j];
        ch += c.proj_mode[j] == TM_BLOCK ? (s - 1 < l - 1 ? s - 1 : l - 1) : l - 1;
    }
    if (ch > l - 1) ch = l - 1;
    const int64_t r = 1 + ch * (2 * (int64_t)h + 1);
    return r < l ? r : l;
}

// Counting work items of a candidate: its class-tuple bound (product of the
// capacities) split into items of about `per_item` tuples (at least one item).
__host__ __device__ inline int32_t count_items(const DevCand& c, int64_t per_item) {
    int64_t b = 1;
    for (int d = 0; d < c.lrank; ++d) {
        b *= c.cls_cap[d] > 0 ? c.cls_cap[d] : 1;
        if (b > (int64_t(1) << 50)) b = int64_t(1) << 50;
    }
    if (per_item < 1) per_item = 1;
    const int64_t it = (b + per_item - 1) / per_item;
    return (int32_t)(it < 1 ? 1 : (it > (int64_t(1) << 30) ? (int64_t(1) << 30) : it));
}

// Stride (int32 words) of the stencil evaluation's group records (tm_groups.h) for halos
// up to h, with cyclic projections, with masks.
__host__ __device__ inline int32_t group_stride(bool cyclic, int32_t h, bool masks) {
    return 2 + (cyclic ? 4 : 2) * h + (masks ? (h + 2) & ~1 : 0);
}
// The records are laid out for halos up to 1, 2 or 4.
__host__ __device__ inline int32_t halo_class(int32_t h) { return h <= 1 ? 1 : (h <= 2 ? 2 : 4); }

// Most workgroups of a launch of at most 256 threads each: a grid dimension holds fewer than
// 2^32 threads.
constexpr int64_t kMaxGrid = INT32_MAX / 256;

int set_error(int code, const char* fmt, ...);
// TM_ENOMEM for a HIP allocation, whose own error the next launch's check would report.
template <class... A>
int no_memory(const char* fmt, A... args) {
    (void)hipGetLastError();
    return set_error(TM_ENOMEM, fmt, args...);
}
int validate_shapes(const tm_candidate* c, Shapes* sh);
int fill_devcand(const tm_candidate* c, const Shapes& sh, DevCand* d);

// Kernel launchers (tm_kernels.hip).  All enqueue on `s` and return hipError_t.
// Owner and coordinate tables; with runs also the coordinates' runs of equal contribution.
hipError_t launch_build_tables(const DevHeader* hdr, const DevCand* cands, int64_t n, int32_t* arena, int32_t runs,
                               hipStream_t s);
// Batches up to this many candidates select inside the evaluation launch: its last
// workgroup finds the best row, for which every workgroup makes its row visible to the other
// XCDs, some 20 ns each; a launch of its own costs about as much as 80 of that.  With the
// selection inside and in its own launch: 1 candidate 7.9 and 9.3 us, 64 8.9 and 9.7, 96 9.4
// and 9.6, 128 9.9 and 9.5.
constexpr int64_t kFinInCount = 96;
// Per segment the best cost row: of rows [seg[s], seg[s+1]), or with idx (row -> candidate,
// negative: no row) of the k rows from s k; best_cost may be null.
hipError_t launch_select_segments(const tm_stencil_cost* costs, const int64_t* seg, int64_t nseg, const int64_t* idx,
                                  int64_t k, int64_t* best, tm_stencil_cost* best_cost, hipStream_t s);
hipError_t launch_chain_table(const DevCand* cand, const int32_t* arena, int32_t* out, hipStream_t s);
// Batches of at least this many candidates run the per-candidate table and
// statistics kernels with one-wave workgroups (more candidates in flight per CU).
constexpr int64_t kSmallBlockBatch = 8192;
// Batches of at most this many candidates build their tables with one workgroup per
// (candidate, launch dim) instead of one per candidate.
constexpr int64_t kSplitBuildBatch = 1024;

// Matmul work blocks: kMatmulTiles class pairs of one matrix each.  A matrix over
// launch dims (a, b) has cls_cap[a] * cls_cap[b] class pairs at most; A = (0, 2),
// B = (2, 1), C = (0, 1).
constexpr int kMatmulTiles = 4096;
__host__ __device__ inline int64_t matmul_pair_blocks(int64_t ca, int64_t cb) {
    return (ca * cb + kMatmulTiles - 1) / kMatmulTiles;
}
__host__ __device__ inline int64_t matmul_blocks(const DevCand& d) {
    return matmul_pair_blocks(d.cls_cap[0], d.cls_cap[2]) + matmul_pair_blocks(d.cls_cap[2], d.cls_cap[1]) +
           matmul_pair_blocks(d.cls_cap[0], d.cls_cap[1]);
}

// Redistribution of npair pairs (joint classes, then counting over a work queue,
// then bytes); the arena holds both mappings' tables and each pair's class block.
hipError_t launch_redist(const DevCand* cands, int64_t npair, int32_t* arena, int64_t item_tab, int64_t items,
                         int64_t elem_bytes, tm_redist_cost* out, unsigned long long* counter, int grid,
                         int lds_words, hipStream_t s);
hipError_t launch_matmul(const DevCand* cands, int64_t n, const int32_t* arena, int words_max,
                         int pmax, const int64_t* proc_off, unsigned long long* per_proc,
                         int64_t total_blocks, const int64_t* block_first, hipStream_t s);
hipError_t launch_matmul_finalize(const DevCand* cands, int64_t n, const int64_t* proc_off,
                                  const unsigned long long* per_proc, int64_t tile_bytes,
                                  tm_matmul_cost* out, int64_t* out_per_proc, hipStream_t s);

}  // namespace tmk
