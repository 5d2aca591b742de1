// tm_plan.h -- internal view of batch plans (shared by the plan and search code).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "tm_eval.h"
#include "tm_internal.h"
#include "tm_ranker.h"

namespace tmk {

// A validated batch: compiled descriptors (host copy) and its sizes.
struct Compiled {
    std::vector<DevCand> cands;
    DevHeader hdr{};
    int64_t arena_words = 0, points = 0, max_points = 0;
    int32_t max_vol = 0;        // largest final-space volume
    int32_t max_blocks = 0;     // most blocks of all launch dims of a candidate (estimates' records)
    int32_t min_row = INT32_MAX;  // shortest row (last extent)
    int32_t cnt_words = 0;      // most LDS words of an owner table with its class blocks that fit (matmul batches)
    int64_t map_words = 0;      // plans: words of all owner tables (each candidate's arena_off is among them)
    EvalPlan eval;              // the evaluation's launches
    int H = 1;
};

// Device buffers of a search over a loaded plan (grown on demand).
struct SearchBufs {
    int64_t cap_n = 0, cap_sc = 0, cap_pre = 0, cap_sel = 0, cap_seg = 0, cap_all = 0;
    uint16_t* X = nullptr;          // [n][kFeat] bf16 features
    float* base = nullptr;          // [n] the scores' bases
    float* score = nullptr;         // [cap_sc] ranking scores (both stages)
    double* est = nullptr;          // [nseg*prefilter][2] their block-model estimates
    int64_t* pre = nullptr;         // [nseg*prefilter] candidates kept by the network's scores
    int64_t* seg = nullptr;         // [nseg+1] instance segments
    int64_t* sel = nullptr;         // [nseg*k] chosen candidate indices
    tm_stencil_cost* sub_out = nullptr;  // [nseg*k] their exact costs
    tm_stencil_cost* all_out = nullptr;  // [n] exhaustive costs
    int64_t nseg = 0, k = 0;
};

}  // namespace tmk

struct tm_plan {
    int device = 0;
    int64_t cap_cands = 0;
    int64_t cap_arena = 0;            // words of d_arena
    int64_t reserved = 0;             // of them asked for at creation
    tmk::DevCand* d_cands = nullptr;
    tmk::DevEval* d_evals = nullptr;  // the evaluation's view of the batch
    tmk::DevFeat* d_feats = nullptr;  // the features'
    int32_t* d_arena = nullptr;       // owner tables (processor ids) of the candidates mapped so far
    std::vector<int32_t*> outgrown;   // earlier ones, replaced during a capture
    tmk::DevHeader* d_hdr = nullptr;
    unsigned int* d_counter = nullptr;  // [kCounters] finished workgroups of the runs in flight
    unsigned int runs = 0, captured = 0;  // whose words are taken in turn
    tmk::DevCand* h_cands = nullptr;  // pinned staging
    tmk::DevHeader* h_hdr = nullptr;
    int64_t* h_seg = nullptr;         // pinned staging for search segments
    int64_t cap_hseg = 0;
    hipEvent_t up_ev = nullptr;
    bool up_pending = false;
    tmk::Compiled cp;  // the loaded batch
    bool loaded = false;
    bool ran = false;  // some batch of it was evaluated
    int64_t cells_per_item = 0;
    int wg_per_cu = 0;
    tmk::SearchBufs sb;
};

namespace tmk {

// Validates and compiles n candidates on the host (st == nullptr: tables without
// classes; need_lds: every owner table must fit the kernels' LDS budget).
int compile_batch(const tm_candidate* c, int64_t n, const tm_stencil* st, bool need_lds, Compiled& cp);
// Words that tm_eval_stencil_batch_noalloc counts for the tables and the work items of a
// compiled stencil batch against its scratch.
int64_t counted_words(const Compiled& cp);
// Lays out the evaluation of a compiled stencil batch (per-candidate LDS words, dim and
// parts; the launches).  node_level: the node-level volume.
void layout_eval(Compiled& cp, int64_t tuples_per_item, bool node_level);

bool capturing(hipStream_t s);
// While it lives, this thread may allocate, free and wait for events although a stream is
// capturing, on this thread or another (which otherwise fails, and ends the capture).
struct AnytimeMemory {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    AnytimeMemory() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~AnytimeMemory() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    AnytimeMemory(const AnytimeMemory&) = delete;
};
hipError_t malloc_anytime(void** p, size_t bytes);
// TM_ENOTSUP while s is capturing: for calls whose descriptors do not outlive them.
int refuse_capture(hipStream_t s);

int64_t plan_size(const tm_plan* p);
const DevFeat* plan_feats(const tm_plan* p);
EstimateBatch plan_estimates(const tm_plan* p);
FeatHalo plan_halo(const tm_plan* p);
int plan_features(const tm_plan* p, float* d_feat, hipStream_t s);
int plan_block_estimates(const tm_plan* p, double* d_est, hipStream_t s);
int plan_search_prepare(tm_plan* p, const int64_t* seg, int64_t nseg, int32_t prefilter, int32_t topk, bool ranked,
                        SearchBufs** out, hipStream_t s);
hipError_t plan_eval_chosen(tm_plan* p, SearchBufs* sb, int64_t* d_best, tm_stencil_cost* d_best_cost, hipStream_t s);
int plan_exhaustive_search(tm_plan* p, const int64_t* seg, int64_t nseg, int64_t* d_best,
                           tm_stencil_cost* d_best_cost, hipStream_t s);

}  // namespace tmk
