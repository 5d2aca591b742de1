// tm_eval.h -- launch interface of the stencil evaluation (tm_eval.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tm_internal.h"

namespace tmk {

// One launch: candidates that need words in (min_words, max_words], with lds_words of LDS,
// in up to `parts` workgroups each.  parts == 1: whole cost rows are stored; else the cells are added to
// rows the caller zeroed (bytes follow in another launch).  best (parts == 1, one launch
// for all candidates): the last workgroup also selects; counter starts at 0 and is left
// so, each launch in flight having one of its own.
struct EvalArgs {
    const DevEval* evals;
    const int64_t* idx;  // row i evaluates candidate idx[i] (negative: no row); null: i
    int64_t n;
    tm_stencil_cost* out;
    int64_t* best;
    int32_t* best_ids;  // nullable: the selected candidate's owner table, as processor ids, goes to its DevEval::offset here
    unsigned int* counter;
    int64_t elem_bytes;
    int32_t halo[TM_MAX_LRANK];
    int32_t node_level, parts, min_words, max_words, lds_words;
};

// A batch's launches.
struct EvalPlan {
    int64_t n = 0, items = 0, elem_bytes = 0;
    int64_t per_item = 0, fill = 1;  // the caller's tuples per work item, or the parts to fill the GPU with
    int32_t halo[TM_MAX_LRANK] = {0, 0, 0, 0};
    int32_t H = 0, parts = 1, node_level = 0;
    int32_t split = 0;          // candidates needing at most this many LDS words: the first launch
    int32_t words[2] = {0, 0};  // LDS words of the two launches (0: no such candidate)
    bool wave = false;          // one-wave workgroups
    bool all_simple = true;     // every candidate is simple (kEvalSimple)
    int32_t wg_per_cu = 0;      // at most this many workgroups per CU (0: one per item)
};

// Evaluates the batch into out (n rows) and, with best, selects into *best.  counter: a
// device word of this launch's own that holds 0 before it (and after it).  With idx, the nidx candidates idx[i] instead
// (whole ones; rows of negative entries are left alone).  best_ids: the selected candidate's
// owner table as processor ids (for its map), written at its offset by the workgroup that selects.
// cus: the GPU's, used with wg_per_cu.
hipError_t launch_eval_batch(const EvalPlan& p, const DevEval* evals, tm_stencil_cost* out, int64_t* best,
                             unsigned int* counter, int cus, hipStream_t s, const int64_t* idx = nullptr,
                             int64_t nidx = 0, int32_t* best_ids = nullptr);
// The evaluation's view of n compiled candidates; and a plan's counters set to 0.
constexpr int kCounters = 64;
hipError_t launch_fill_evals(const EvalPlan& p, const DevCand* cands, DevEval* evals, DevFeat* feats,
                             unsigned int* counters, hipStream_t s);
// The rows zeroed; and the bytes of rows that hold cells, with the selection.
hipError_t launch_zero_costs(tm_stencil_cost* out, int64_t n, hipStream_t s);
hipError_t launch_bytes_select(tm_stencil_cost* out, int64_t n, int64_t elem_bytes, int64_t* best, hipStream_t s,
                               const DevEval* evals = nullptr, int32_t* ids = nullptr);
// Sum over the candidates of the product of their class counts (tm_plan_class_tuples).
hipError_t launch_class_tuples(const DevCand* cands, int64_t n, const int32_t* halo, unsigned long long* total,
                               hipStream_t s);

// Batches of at least eval_wave_batch candidates run one-wave workgroups, of at least
// kEvalWaveSmall where no owner table is larger than kEvalWaveVol: with few candidates the
// largest one's latency decides, the longer the more slots a tuple has.  One wave and four,
// us.  Halo 1: random ones (tables to 900) 2,048 candidates 26.6 and 21.2, 4,096 27.0 and 30.3;
// the search's (to 512) 4,096 39.5 and 36.1, 8,192 44 and 61.  Halo 2: random 4,096 49 and 44,
// 6,144 62 and 58, 8,192 62 and 72; the search's 4,096 78 and 57, 8,192 79 and 90.  Halo 4:
// random 8,192 144 and 103, 16,384 171 and 174, 24,576 255 and 250; the search's 16,384 333 and
// 239.  The 2-D study's (to 128) at halos 1, 2 and 4: 512 10.1 and 10.0, 11.1 and 10.7, 13.3
// and 11.8; 1,024 11.2 and 11.9, 12.2 and 16.1, 14.3 and 18.2.
constexpr int64_t eval_wave_batch(int H) { return H <= 1 ? 4096 : (H <= 2 ? 8192 : 24576); }
constexpr int64_t kEvalWaveSmall = 1024;
constexpr int32_t kEvalWaveVol = 128;

// LDS words of a launch: records share the LDS up to kEvalSmall* words (5 KB per one-wave
// workgroup keeps 26 of them on a CU, 20 KB per four-wave one 8); all candidates go in one
// launch up to kEvalMost*.  Measured on 4,096 random candidates, largest need 1,350 words:
// one launch 32 us, two (1,280 words and the rest) 50 us.
constexpr int32_t kEvalSmallWave = 1280, kEvalMostWave = 2048;
constexpr int32_t kEvalSmallBlock = 5120, kEvalMostBlock = 8192;
// Without a caller's item size, batches smaller than this many workgroups split their
// candidates into parts of at least kEvalPartTuples tuples.
constexpr int64_t kEvalFill = 512, kEvalPartTuples = 1024;

}  // namespace tmk
