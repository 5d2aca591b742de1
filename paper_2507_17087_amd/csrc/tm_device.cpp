// tm_device.cpp -- device entry points of libtaskmap: single-shot evaluation calls
// and batch plans (descriptors kept on the device, runs launched directly).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <vector>

#include "tm_compile.h"
#include "tm_eval.h"
#include "tm_internal.h"
#include "tm_map.h"
#include "tm_plan.h"
#include "tm_ranker.h"
#include "tm_volume.h"

namespace tmk {

#define TM_HIP(expr)                                                                                 \
    do {                                                                                             \
        hipError_t e_ = (expr);                                                                      \
        if (e_ != hipSuccess) return set_error(TM_EDEVICE, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

// Class tuples per counted work item (counted_words): about 16 items per CU over the
// batch's class-tuple bound, between 2^10 and 2^16 tuples.
static int num_cus();
static int64_t default_tuples_per_item(int64_t tuples) {
    const int64_t target = tuples / (int64_t(num_cus()) * 16);
    int64_t c = int64_t(1) << 10;
    while (c < target && c < (int64_t(1) << 16)) c <<= 1;
    return c;
}
// Largest work item accepted from a caller.
constexpr int64_t kMaxCellsPerItem = int64_t(1) << 26;
// ------------------------------------------------------------------ batch compilation

static int64_t up4(int64_t x) { return (x + 3) & ~int64_t(3); }

// Arena layout of one candidate: owner table T, the last dim's coordinate table
// (16-byte aligned, padded to whole 512-entry chunks), the other dims'
// coordinate tables, then (halo != nullptr) the class record (the
// class count of each dim, written by the table build) and each dim's class block
// (entries, starts, and the room of offset lists of 2H words; capacities from class_cap).
static int layout_tables(DevCand& d, int H, const int32_t* halo) {
    const int K = d.lrank;
    int64_t off = up4(d.vol);
    const int64_t t_end = off + 4;
    d.coord_off[K - 1] = (int32_t)std::min<int64_t>(off, INT32_MAX);
    off += (d.extent[K - 1] + 511) & ~int64_t(511);  // zero-padded to whole 512-entry chunks
    const int64_t c_end = off + 4;                   // slack for the last four-entry read of a ragged row
    off = std::max(off, c_end);
    for (int k = 0; k < K - 1; ++k) {
        d.coord_off[k] = (int32_t)std::min<int64_t>(off, INT32_MAX);
        off += d.extent[k];
    }
    for (int k = 0; k < TM_MAX_LRANK; ++k) d.cls_off[k] = d.cls_cap[k] = 0;
    d.cls_base = d.cls_words = 0;
    if (halo) {
        off = up4(off);
        const int64_t cb = off;
        off += 4;
        for (int k = 0; k < K; ++k) {
            const int64_t cap = class_cap(d, k, halo[k]);
            if (off > INT32_MAX || cap > INT32_MAX / std::max(1, 2 * H)) return TM_EOVERFLOW;
            d.cls_cap[k] = (int32_t)cap;
            d.cls_off[k] = (int32_t)off;
            off += up4(cap) + up4(cap + 1) + up4(cap * 2 * H);
        }
        if (off - cb > INT32_MAX) return TM_EOVERFLOW;
        d.cls_base = (int32_t)cb;
        d.cls_words = (int32_t)(off - cb);
    }
    const int64_t staged = c_end <= kMaxLdsWords ? c_end : t_end;
    const int64_t words = up4(std::max(off, staged));  // the next candidate's tables start 16-byte aligned
    if (words > INT32_MAX) return TM_EOVERFLOW;
    d.lds_words = (int32_t)staged;
    d.words = (int32_t)words;
    return TM_OK;
}

// Blocks of all launch dims where each is projected onto at most one final dim, one for a
// dim without a projection.
static int32_t blocks_and_dims(const DevCand& d) {
    int64_t n = d.lrank;
    for (int j = 0; j < d.frank; ++j) n += d.fshape[j];
    return (int32_t)std::min<int64_t>(n, INT32_MAX);
}

int64_t counted_words(const Compiled& cp) {
    int64_t tuples = 0, items = 0;
    for (const auto& d : cp.cands) {
        int64_t b = 1;
        for (int k = 0; k < d.lrank; ++k) b = std::min<int64_t>(b * d.cls_cap[k], int64_t(1) << 50);
        tuples += b;
    }
    const int64_t per = default_tuples_per_item(tuples);
    for (const auto& d : cp.cands) items += count_items(d, per);
    return cp.arena_words + up4(items);
}

// Validates and compiles n candidates.  st == nullptr: tables without classes.
// need_lds: every candidate's tables must fit the LDS budget of the kernels.
int compile_batch(const tm_candidate* c, int64_t n, const tm_stencil* st, bool need_lds, Compiled& cp) {
    if (n < 0) return set_error(TM_EINVAL, "n = %lld", (long long)n);
    if (n > 0 && !c) return set_error(TM_EINVAL, "null candidate array");
    cp.cands.resize((size_t)n);
    cp.hdr = DevHeader{};
    cp.hdr.n = n;
    if (st) {
        if (st->lrank < 1 || st->lrank > TM_MAX_LRANK) return set_error(TM_EINVAL, "stencil lrank %d", st->lrank);
        if (st->elem_bytes < 0) return set_error(TM_EINVAL, "elem_bytes %d", st->elem_bytes);
        int hmax = 0;
        for (int d = 0; d < st->lrank; ++d) {
            if (st->halo[d] < 0 || st->halo[d] > TM_MAX_HALO) return set_error(TM_EINVAL, "halo[%d] = %d", d, st->halo[d]);
            hmax = std::max(hmax, st->halo[d]);
            cp.hdr.halo[d] = st->halo[d];
        }
        if (hmax > kMaxHalo) return set_error(TM_ENOTSUP, "halo %d above the kernels' limit of %d", hmax, kMaxHalo);
        cp.H = std::max(1, hmax);
        cp.hdr.elem_bytes = st->elem_bytes;
        cp.hdr.lrank = st->lrank;
    }
    int64_t words = 0;
    for (int64_t i = 0; i < n; ++i) {
        Shapes sh;
        int rc = validate_shapes(&c[i], &sh);
        if (rc != TM_OK) return set_error(rc, "candidate %lld: %s", (long long)i, tm_last_error());
        // a candidate of launch rank k takes the stencil's first k halo widths
        if (st && c[i].lrank > st->lrank)
            return set_error(TM_EINVAL, "candidate %lld: lrank %d but the stencil has %d", (long long)i, c[i].lrank,
                             st->lrank);
        DevCand& d = cp.cands[(size_t)i];
        rc = fill_devcand(&c[i], sh, &d);
        if (rc == TM_OK) rc = layout_tables(d, st ? cp.H : 0, st ? cp.hdr.halo : nullptr);
        if (rc != TM_OK) return set_error(rc, "candidate %lld: tables too large", (long long)i);
        if (need_lds && d.lds_words > kMaxLdsWords)
            return set_error(TM_ENOTSUP, "candidate %lld: %d table words exceed the LDS budget of %d", (long long)i,
                             d.lds_words, kMaxLdsWords);
        // row indices are 32-bit in the kernels, with room to step past the last row
        if (d.rows > (int64_t(1) << 30))
            return set_error(TM_ENOTSUP, "candidate %lld: more than 2^30 rows", (long long)i);
        d.arena_off = words;
        words += d.words;
        if (st) {
            const int64_t cw = up4(d.vol) + d.cls_words;  // staged when it fits, else read in place
            if (cw <= kMaxLdsWords) cp.cnt_words = std::max<int32_t>(cp.cnt_words, (int32_t)cw);
        }
        cp.points += d.npoints;
        cp.max_points = std::max(cp.max_points, d.npoints);
        cp.max_vol = std::max(cp.max_vol, d.vol);
        cp.max_blocks = std::max(cp.max_blocks, blocks_and_dims(d));
        cp.min_row = std::min(cp.min_row, d.L);
    }
    cp.arena_words = words;
    return TM_OK;
}

// The evaluation's launches.  One launch takes all candidates when the largest need
// (eval_need) is small, else those above kEvalSmall* go in a launch of their own, so that
// they do not cost the others their occupancy; a candidate gets as many more records than
// it needs as fit its launch's words.  Candidates are added one by one.
struct EvalLayout {
    EvalPlan& e;
    int32_t small, most;
    int32_t words[2] = {0, 0}, whole[2] = {0, 0}, largest = 0;  // of the needs up to small, above it

    // max_vol: of all candidates, or more where that is not known yet
    EvalLayout(EvalPlan& plan, int64_t n, int32_t max_vol, const tm_stencil& st, int H, int64_t tuples_per_item,
               bool node_level)
        : e(plan) {
        e = EvalPlan{};
        e.n = n;
        e.elem_bytes = st.elem_bytes;
        for (int k = 0; k < TM_MAX_LRANK; ++k) e.halo[k] = k < st.lrank ? st.halo[k] : 0;
        e.H = H;
        e.node_level = node_level ? 1 : 0;
        e.per_item = tuples_per_item;
        e.fill = std::max<int64_t>(1, kEvalFill / std::max<int64_t>(n, 1));
        e.wave = n >= eval_wave_batch(H) || (n >= kEvalWaveSmall && max_vol <= kEvalWaveVol);
        small = e.wave ? kEvalSmallWave : kEvalSmallBlock;
        most = e.wave ? kEvalMostWave : kEvalMostBlock;
    }
    EvalShape shape() const { return EvalShape{e.H, e.node_level, e.per_item, e.fill}; }
    void add(const EvalNeed& n, bool simple) {
        e.items += n.parts;
        e.parts = std::max(e.parts, n.parts);
        largest = std::max(largest, n.words);
        e.all_simple = e.all_simple && simple;
        const int b = n.words > small ? 1 : 0;
        words[b] = std::max(words[b], n.words);
        whole[b] = std::max(whole[b], n.whole);
    }
    void finish() {
        if (largest <= most) {
            e.split = largest;
            e.words[0] = std::max(largest, std::min(std::max(whole[0], whole[1]), small));
        } else {
            e.split = small;
            e.words[0] = std::max(words[0], std::min(whole[0], small));
            e.words[1] = words[1];
        }
    }
};

void layout_eval(Compiled& cp, int64_t tuples_per_item, bool node_level) {
    tm_stencil st{};
    st.lrank = TM_MAX_LRANK;
    st.elem_bytes = cp.hdr.elem_bytes;
    for (int k = 0; k < TM_MAX_LRANK; ++k) st.halo[k] = cp.hdr.halo[k];
    EvalLayout lay(cp.eval, (int64_t)cp.cands.size(), cp.max_vol, st, cp.H, tuples_per_item, node_level);
    const EvalShape shape = lay.shape();
    for (auto& c : cp.cands) {
        DevDim dim[TM_MAX_LRANK];
        bool cyclic = false;
        const uint64_t bits = projection_bits(c);
        for (int k = 0; k < c.lrank; ++k) {
            count_groups(c, k, bits, &dim[k]);
            cyclic = cyclic || dim[k].ncyc > 0;
        }
        lay.add(eval_need(dim, c.lrank, c.vol, cyclic, is_bijective(c), shape), is_simple(c));
    }
    lay.finish();
}

// ------------------------------------------------------------------ staging

bool capturing(hipStream_t s) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    return hipStreamIsCapturing(s, &cap) == hipSuccess && cap != hipStreamCaptureStatusNone;
}

hipError_t malloc_anytime(void** p, size_t bytes) {
    AnytimeMemory anytime;
    return hipMalloc(p, bytes);
}

// A single call's descriptors live until its work is done; the replays of a graph that
// recorded it come later, when their memory holds other calls' descriptors or is gone.
int refuse_capture(hipStream_t s) {
    if (!capturing(s)) return TM_OK;
    return set_error(TM_ENOTSUP, "the stream is capturing: single calls cannot be recorded (a loaded plan's runs and maps can)");
}

// Per-thread pinned staging for descriptor uploads; reused once the previous copy
// out of it has completed.
struct Staging {
    void* ptr = nullptr;
    size_t cap = 0;
    hipEvent_t ev = nullptr;
    int device = -1;
    bool pending = false;
};
static thread_local Staging g_stage;

static int staging_acquire(size_t bytes, void** out) {
    int dev = 0;
    TM_HIP(hipGetDevice(&dev));
    AnytimeMemory anytime;
    if (g_stage.pending) {
        TM_HIP(hipEventSynchronize(g_stage.ev));
        g_stage.pending = false;
    }
    if (g_stage.device != dev) {
        if (g_stage.ev) (void)hipEventDestroy(g_stage.ev);
        g_stage.ev = nullptr;
        g_stage.device = dev;
    }
    if (!g_stage.ev) TM_HIP(hipEventCreateWithFlags(&g_stage.ev, hipEventDisableTiming));
    if (g_stage.cap < bytes) {
        if (g_stage.ptr) TM_HIP(hipHostFree(g_stage.ptr));
        g_stage.ptr = nullptr;
        g_stage.cap = 0;
        const size_t cap = std::max<size_t>(bytes, 1 << 20);
        if (hipHostMalloc(&g_stage.ptr, cap, hipHostMallocDefault) != hipSuccess)
            return no_memory("pinned staging of %zu bytes", cap);
        g_stage.cap = cap;
    }
    *out = g_stage.ptr;
    return TM_OK;
}

static int staging_release(hipStream_t s) {
    TM_HIP(hipEventRecord(g_stage.ev, s));
    g_stage.pending = true;
    return TM_OK;
}

// Per-thread slots of pinned memory that kernels read descriptors from in place, and a
// piece of device scratch each: a call takes the next one once the work that used it last
// is done.  Bounded (kSlots x kSlotBytes a thread) and freed with the thread.  A small
// call's allocation, copy and free cost more than its kernel: 300 descriptors (269 KB) read
// in place 11.8 us a call (launch, event, GPU time of the reads), copied into a
// stream-ordered allocation 61.5 us.
constexpr int kSlots = 4;
constexpr size_t kSlotBytes = size_t(1) << 20;
constexpr size_t kSlotScratch = sizeof(DevEval) + (size_t)kMaxLdsWords * 4;  // a descriptor, an owner table

struct SlotRing {
    int device = -1;
    char* host = nullptr;
    char* scratch = nullptr;
    hipEvent_t ev[kSlots] = {};
    bool pending[kSlots] = {};
    int next = 0;

    // Also at the thread's end, when another thread may be capturing.
    void drop() {
        if (!host) return;
        AnytimeMemory anytime;
        for (int i = 0; i < kSlots; ++i) {
            if (pending[i]) (void)hipEventSynchronize(ev[i]);
            if (ev[i]) (void)hipEventDestroy(ev[i]);
            ev[i] = nullptr;
            pending[i] = false;
        }
        (void)hipHostFree(host);
        if (scratch) (void)hipFree(scratch);
        host = scratch = nullptr;
        device = -1;
    }
    ~SlotRing() { drop(); }
};
static thread_local SlotRing g_ring;

struct Slot {
    int index;
    char* host;
    char* scratch;
};

static int slot_acquire(bool scratch, Slot* out) {
    int dev = 0;
    TM_HIP(hipGetDevice(&dev));
    SlotRing& r = g_ring;
    if (r.device != dev) r.drop();
    r.device = dev;
    if (!r.host || (scratch && !r.scratch)) {
        AnytimeMemory anytime;
        if (!r.host && hipHostMalloc((void**)&r.host, kSlots * kSlotBytes, hipHostMallocDefault) != hipSuccess) {
            r.host = nullptr;
            return no_memory("pinned staging of %zu bytes", kSlots * kSlotBytes);
        }
        if (scratch && !r.scratch && hipMalloc((void**)&r.scratch, kSlots * kSlotScratch) != hipSuccess) {
            r.scratch = nullptr;
            return no_memory("scratch of %zu bytes", kSlots * kSlotScratch);
        }
    }
    const int i = r.next;
    if (!r.ev[i]) TM_HIP(hipEventCreateWithFlags(&r.ev[i], hipEventDisableTiming));
    if (r.pending[i]) {
        AnytimeMemory anytime;
        TM_HIP(hipEventSynchronize(r.ev[i]));
    }
    r.pending[i] = false;
    *out = Slot{i, r.host + (size_t)i * kSlotBytes, r.scratch ? r.scratch + (size_t)i * kSlotScratch : nullptr};
    return TM_OK;
}

// After the last launch that uses the slot.
static int slot_release(const Slot& slot, hipStream_t s) {
    SlotRing& r = g_ring;
    if (hipEventRecord(r.ev[slot.index], s) == hipSuccess) r.pending[slot.index] = true;
    else TM_HIP(hipStreamSynchronize(s));
    r.next = (slot.index + 1) % kSlots;
    return TM_OK;
}

// Descriptors that fill writes, for launch to read: in a slot, or larger ones in a device
// copy.  fill's result: TM_OK, an error, or kGeneral (nothing is launched).  *memory: the
// error of getting the memory; then the result is kGeneral, since the records come first
// (the general path has them validated before it meets the same error).
constexpr int kGeneral = 1;
template <class Fill, class Launch>
static int with_descriptors(size_t bytes, hipStream_t s, const char* what, int* memory, Fill fill, Launch launch) {
    hipError_t e = hipSuccess;
    int rc;
    *memory = refuse_capture(s);
    if (*memory != TM_OK) return kGeneral;
    if (bytes <= kSlotBytes) {
        Slot slot;
        *memory = slot_acquire(false, &slot);
        rc = *memory == TM_OK ? fill((void*)slot.host) : kGeneral;
        if (rc != TM_OK) return rc;
        e = launch((const void*)slot.host);
        rc = slot_release(slot, s);
    } else {
        void *stg = nullptr, *d = nullptr;
        *memory = staging_acquire(bytes, &stg);
        rc = *memory == TM_OK ? fill(stg) : kGeneral;
        if (rc != TM_OK) return rc;
        TM_HIP(hipMallocAsync(&d, bytes, s));
        e = hipMemcpyAsync(d, stg, bytes, hipMemcpyHostToDevice, s);
        if (e == hipSuccess) rc = staging_release(s);
        if (rc == TM_OK && e == hipSuccess) e = launch((const void*)d);
        (void)hipFreeAsync(d, s);
    }
    if (rc == TM_OK && e != hipSuccess) rc = set_error(TM_EDEVICE, "%s launch: %s", what, hipGetErrorString(e));
    return rc;
}

// Device copies of a compiled batch in stream-ordered allocations.
struct DeviceBatch {
    DevCand* cands = nullptr;
    DevHeader* hdr = nullptr;
    int32_t* arena = nullptr;
    unsigned long long* counter = nullptr;
};

static int upload_batch(const Compiled& cp, DeviceBatch& db, hipStream_t s) {
    int rc = refuse_capture(s);
    if (rc != TM_OK) return rc;
    const size_t nc = cp.cands.size() * sizeof(DevCand);
    TM_HIP(hipMallocAsync((void**)&db.cands, std::max<size_t>(nc, 64), s));
    TM_HIP(hipMallocAsync((void**)&db.hdr, sizeof(DevHeader) + 64, s));
    TM_HIP(hipMallocAsync((void**)&db.arena, std::max<size_t>((size_t)cp.arena_words * 4, 64), s));
    TM_HIP(hipMallocAsync((void**)&db.counter, 64, s));
    void* stg = nullptr;
    rc = staging_acquire(nc + sizeof(DevHeader), &stg);
    if (rc != TM_OK) return rc;
    std::memcpy(stg, &cp.hdr, sizeof(DevHeader));
    if (nc) std::memcpy((char*)stg + sizeof(DevHeader), cp.cands.data(), nc);
    TM_HIP(hipMemcpyAsync(db.hdr, stg, sizeof(DevHeader), hipMemcpyHostToDevice, s));
    if (nc) TM_HIP(hipMemcpyAsync(db.cands, (char*)stg + sizeof(DevHeader), nc, hipMemcpyHostToDevice, s));
    return staging_release(s);
}

static void free_batch(DeviceBatch& db, hipStream_t s) {
    if (db.cands) (void)hipFreeAsync(db.cands, s);
    if (db.hdr) (void)hipFreeAsync(db.hdr, s);
    if (db.arena) (void)hipFreeAsync(db.arena, s);
    if (db.counter) (void)hipFreeAsync(db.counter, s);
    db = DeviceBatch{};
}

static int num_cus() {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return 256;
    return n;
}
// The CUs that a launch bounded by them asks for.
static int eval_cus(const EvalPlan& p) { return p.wg_per_cu > 0 ? num_cus() : 0; }

}  // namespace tmk

using namespace tmk;

// ------------------------------------------------------------------ single-shot calls

extern "C" int tm_chain_table(const tm_candidate* c, int32_t* d_out, int64_t cap, int64_t* count, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    Compiled cp;
    int rc = compile_batch(c, 1, nullptr, false, cp);
    if (rc != TM_OK) return rc;
    if (count) *count = cp.cands[0].vol;
    if (cap < cp.cands[0].vol) return set_error(TM_ECAPACITY, "chain table has %d entries", cp.cands[0].vol);
    if (!d_out) return set_error(TM_EINVAL, "null output");
    DeviceBatch db;
    rc = upload_batch(cp, db, s);
    if (rc == TM_OK) {
        hipError_t e = launch_build_tables(db.hdr, db.cands, 1, db.arena, 0, s);
        if (e == hipSuccess) e = launch_chain_table(db.cands, db.arena, d_out, s);
        if (e != hipSuccess) rc = set_error(TM_EDEVICE, "chain table launch: %s", hipGetErrorString(e));
    }
    free_batch(db, s);
    return rc;
}

extern "C" int tm_proc_map(const tm_candidate* c, int32_t* d_map, int64_t len, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    Compiled cp;
    int rc = compile_batch(c, 1, nullptr, true, cp);
    if (rc != TM_OK) return rc;
    const DevCand& c0 = cp.cands[0];
    if (len != c0.npoints)
        return set_error(TM_ECAPACITY, "map length %lld but the domain has %lld points", (long long)len,
                         (long long)c0.npoints);
    if (!d_map) return set_error(TM_EINVAL, "null output");
    const EvalShape shape{1, 0, 0, 1};
    const MapShape m = map_shape(c0.vol, c0.npoints, c0.L);
    rc = refuse_capture(s);
    if (rc != TM_OK) return rc;
    Slot slot;
    rc = slot_acquire(true, &slot);
    if (rc != TM_OK) return rc;
    DevEval *h = reinterpret_cast<DevEval*>(slot.host), *d = reinterpret_cast<DevEval*>(slot.scratch);
    int32_t* ids = reinterpret_cast<int32_t*>(d + 1);
    fill_eval(c0, shape, h);
    // every workgroup of the map reads the descriptor: it goes to device memory on the way
    hipError_t e = launch_map_ids(h, 1, nullptr, 0, c0.vol, ids, s, d);
    if (e == hipSuccess) e = launch_map(m, d, 1, nullptr, 0, ids, d_map, s);
    rc = slot_release(slot, s);
    if (rc == TM_OK && e != hipSuccess) rc = set_error(TM_EDEVICE, "map launch: %s", hipGetErrorString(e));
    return rc;
}

// The halo slots of a stencil the kernels take (0: none; compile_batch tells why).
static int stencil_slots(const tm_stencil& st) {
    if (st.lrank < 1 || st.lrank > TM_MAX_LRANK || st.elem_bytes < 0) return 0;
    int h = 1;
    for (int d = 0; d < st.lrank; ++d) {
        if (st.halo[d] < 0) return 0;
        h = std::max(h, (int)st.halo[d]);
    }
    return h <= kMaxHalo ? h : 0;
}

static int eval_stencil(const tm_candidate* c, int64_t n, const tm_stencil* st, tm_stencil_cost* d_out,
                        hipStream_t s, bool node_level) {
    if (!st) return set_error(TM_EINVAL, "null stencil");
    EvalPlan plan;
    auto launch = [&](const void* d) {
        return launch_eval_batch(plan, static_cast<const DevEval*>(d), d_out, nullptr, nullptr, 0, s);
    };
    const int H = stencil_slots(*st);
    int memory = TM_OK;
    if (H > 0 && c && n > 0) {
        // straight from the records to the evaluation's descriptors
        const int rc = with_descriptors((size_t)n * sizeof(DevEval), s, "stencil", &memory, [&](void* stg) {
            DevEval* e = static_cast<DevEval*>(stg);
            EvalLayout lay(plan, n, INT32_MAX, *st, H, 0, node_level);
            const EvalShape shape = lay.shape();
            for (int64_t i = 0; i < n; ++i, ++e) {
                CandView v;
                EvalNeed need;
                if (c[i].lrank > st->lrank || !compile_eval(&c[i], shape, &v, e, &need)) return kGeneral;
                lay.add(need, e->flags & kEvalSimple);
            }
            lay.finish();
            return d_out ? TM_OK : set_error(TM_EINVAL, "null output");
        }, launch);
        if (rc != kGeneral) return rc;
    }
    Compiled cp;
    int rc = compile_batch(c, n, st, true, cp);
    if (rc != TM_OK) return rc;
    if (n == 0) return TM_OK;
    if (!d_out) return set_error(TM_EINVAL, "null output");
    layout_eval(cp, 0, node_level);
    plan = cp.eval;
    rc = with_descriptors((size_t)n * sizeof(DevEval), s, "stencil", &memory, [&](void* stg) {
        const EvalShape shape{plan.H, plan.node_level, plan.per_item, plan.fill};
        for (int64_t i = 0; i < n; ++i) fill_eval(cp.cands[(size_t)i], shape, static_cast<DevEval*>(stg) + i);
        return TM_OK;
    }, launch);
    return rc == kGeneral ? memory : rc;
}

extern "C" int tm_eval_stencil_batch(const tm_candidate* c, int64_t n, const tm_stencil* st,
                                     tm_stencil_cost* d_out, void* stream) {
    return eval_stencil(c, n, st, d_out, (hipStream_t)stream, false);
}

extern "C" int tm_eval_stencil_node_batch(const tm_candidate* c, int64_t n, const tm_stencil* st,
                                          tm_stencil_cost* d_out, void* stream) {
    return eval_stencil(c, n, st, d_out, (hipStream_t)stream, true);
}

// Pairs (src[i], dst[i]) over joint groups, when the tables of all of them fit a
// workgroup's LDS (else kGeneral).
static int redistribution_groups(const tm_candidate* src, const tm_candidate* dst, int64_t n, int64_t elem_bytes,
                                 tm_redist_cost* d_out, hipStream_t s) {
    int memory, parts = 1;
    int32_t words = 0;
    auto fill = [&](void* stg) {
        const EvalShape shape{1, 0, 0, 1};
        DevPair* p = static_cast<DevPair*>(stg);
        for (int64_t i = 0; i < n; ++i, ++p) {
            CandView a, b;
            EvalNeed need;
            int32_t w = 0;
            if (!compile_eval(&src[i], shape, &a, &p->a, &need) || !compile_eval(&dst[i], shape, &b, &p->b, &need) ||
                !fill_pair(a, b, p, &w))
                return kGeneral;
            words = std::max(words, w);
            parts = std::max(parts, p->parts);
        }
        return d_out ? TM_OK : set_error(TM_EINVAL, "null output");
    };
    return with_descriptors((size_t)n * sizeof(DevPair), s, "redistribution", &memory, fill, [&](const void* d) {
        return launch_pairs(static_cast<const DevPair*>(d), n, parts, words, elem_bytes, d_out, s);
    });
}

// Whether a matrix of the domain has more tiles than its counts hold.
static bool tiles_overflow(const int64_t* extent) {
    return extent[0] * extent[1] > INT32_MAX || extent[1] * extent[2] > INT32_MAX || extent[0] * extent[2] > INT32_MAX;
}
constexpr int64_t kMatmulProcs = 1024;

// Matmul tiles over coordinate groups, when all candidates are for that kernel (else
// kGeneral).
static int matmul_groups(const tm_candidate* c, int64_t n, int64_t tile_bytes, int64_t* d_per_proc,
                         tm_matmul_cost* d_out, hipStream_t s) {
    int memory;
    int32_t words = 0;
    int64_t procs = 0;
    auto fill = [&](void* stg) {
        DevEval* e = static_cast<DevEval*>(stg);
        for (int64_t i = 0; i < n; ++i, ++e) {
            CandView v;
            EvalNeed need;
            if (!compile_eval(&c[i], EvalShape{1, 0, 0, 1}, &v, e, &need) || v.lrank != 3 ||
                e->procs > kMatmulProcs || tiles_overflow(v.extent))
                return kGeneral;
            e->offset = procs;
            procs += e->procs;
            const int32_t w = matmul_words(*e);
            if (w == 0) return kGeneral;
            words = std::max(words, w);
        }
        if (n > INT32_MAX) return kGeneral;
        return d_out ? TM_OK : set_error(TM_EINVAL, "null output");
    };
    return with_descriptors((size_t)n * sizeof(DevEval), s, "matmul", &memory, fill, [&](const void* d) {
        return launch_matmul_groups(static_cast<const DevEval*>(d), n, words, tile_bytes, d_out, d_per_proc, s);
    });
}

extern "C" int tm_eval_redistribution_batch(const tm_candidate* src, const tm_candidate* dst, int64_t n,
                                            int64_t elem_bytes, tm_redist_cost* d_out, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    if (n < 0) return set_error(TM_EINVAL, "n = %lld", (long long)n);
    if (elem_bytes < 0) return set_error(TM_EINVAL, "elem_bytes %lld", (long long)elem_bytes);
    if (n > 0 && (!src || !dst)) return set_error(TM_EINVAL, "null candidate array");
    for (int64_t i = 0; i < n; ++i) {
        const tm_candidate &a = src[i], &b = dst[i];
        bool same = a.lrank == b.lrank && a.nodes == b.nodes && a.gpus_per_node == b.gpus_per_node;
        for (int d = 0; same && d < a.lrank && d < TM_MAX_LRANK; ++d) same = a.extent[d] == b.extent[d];
        if (!same) return set_error(TM_EINVAL, "pair %lld: different launch domains or machines", (long long)i);
    }
    if (n > 0) {
        const int rc = redistribution_groups(src, dst, n, elem_bytes, d_out, s);
        if (rc != kGeneral) return rc;
    }
    std::vector<tm_candidate> both((size_t)(2 * n));
    if (n > 0) {
        std::memcpy(both.data(), src, (size_t)n * sizeof(tm_candidate));
        std::memcpy(both.data() + n, dst, (size_t)n * sizeof(tm_candidate));
    }
    Compiled cp;
    int rc = compile_batch(both.data(), 2 * n, nullptr, false, cp);
    if (rc != TM_OK) return rc;
    if (n == 0) return TM_OK;
    if (!d_out) return set_error(TM_EINVAL, "null output");
    // each pair's joint-class block goes into its a-side table block: the record, then
    // per dim the a entries, the b entries and the run starts of its classes; a dim's
    // joint classes start where either mapping's contribution changes, so there are at
    // most 1 + changes_a + changes_b of them.  Work items split the pair's class-tuple
    // bound; the item table follows the tables.
    const int64_t tuples_per_item = int64_t(1) << 12;
    int64_t words = 0, items = 0;
    int32_t lds_words = 0;
    for (int64_t i = 0; i < 2 * n; ++i) {
        DevCand& d = cp.cands[(size_t)i];
        if (i < n) {
            const DevCand& b = cp.cands[(size_t)(n + i)];
            int64_t off = up4(d.words), bound = 1;
            d.cls_base = (int32_t)std::min<int64_t>(off, INT32_MAX);
            off += 4;
            for (int k = 0; k < d.lrank; ++k) {
                const int64_t cap = std::min<int64_t>(d.extent[k], class_cap(d, k, 0) + class_cap(b, k, 0) - 1);
                d.cls_cap[k] = (int32_t)cap;
                d.cls_off[k] = (int32_t)std::min<int64_t>(off, INT32_MAX);
                off += 2 * up4(cap) + up4(cap + 1);
                bound = std::min<int64_t>(bound * cap, int64_t(1) << 50);
            }
            if (off > INT32_MAX) return set_error(TM_EOVERFLOW, "pair %lld: tables too large", (long long)i);
            d.cls_words = (int32_t)(off - d.cls_base);
            d.words = (int32_t)off;
            d.citems = (int32_t)std::min<int64_t>(std::max<int64_t>((bound + tuples_per_item - 1) / tuples_per_item, 1),
                                                  int64_t(1) << 30);
            d.item_first = items;
            items += d.citems;
            const int64_t need = up4(d.vol) + up4(b.vol) + d.cls_words;  // staged when it fits the budget
            if (need <= kMaxLdsWords) lds_words = std::max<int32_t>(lds_words, (int32_t)need);
        }
        d.arena_off = words;
        words += d.words;
    }
    const int64_t item_tab = words;
    cp.arena_words = words + up4(items);
    DeviceBatch db;
    rc = upload_batch(cp, db, s);
    if (rc == TM_OK) {
        const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(items, (int64_t)num_cus() * 8));
        hipError_t e = launch_build_tables(db.hdr, db.cands, 2 * n, db.arena, 0, s);
        if (e == hipSuccess)
            e = launch_redist(db.cands, n, db.arena, item_tab, items, elem_bytes, d_out, db.counter, grid, lds_words, s);
        if (e != hipSuccess) rc = set_error(TM_EDEVICE, "redistribution launch: %s", hipGetErrorString(e));
    }
    free_batch(db, s);
    return rc;
}

extern "C" int tm_eval_matmul_batch(const tm_candidate* c, int64_t n, const tm_matmul* mm, int64_t* d_per_proc,
                                    tm_matmul_cost* d_out, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    if (!mm || mm->tile_bytes < 0) return set_error(TM_EINVAL, "bad matmul descriptor");
    if (c && n > 0) {
        const int rc = matmul_groups(c, n, mm->tile_bytes, d_per_proc, d_out, s);
        if (rc != kGeneral) return rc;
    }
    // coordinate classes with a zero halo: runs of coordinates with equal contributions
    tm_stencil zs{};
    zs.lrank = TM_MAX_LRANK;
    Compiled cp;
    int rc = compile_batch(c, n, &zs, false, cp);
    if (rc != TM_OK) return rc;
    if (n == 0) return TM_OK;
    if (!d_out) return set_error(TM_EINVAL, "null output");
    std::vector<int64_t> proc_off((size_t)n + 1), block_first((size_t)n + 1);
    int64_t procs = 0, blocks = 0;
    int pmax = 0;
    for (int64_t i = 0; i < n; ++i) {
        const DevCand& d = cp.cands[(size_t)i];
        if (d.lrank != 3) return set_error(TM_EINVAL, "candidate %lld: matmul needs launch rank 3", (long long)i);
        const int64_t P = (int64_t)d.nodes * d.gpus;
        if (P > kMatmulProcs)
            return set_error(TM_ENOTSUP, "candidate %lld: %lld processors (limit %lld)", (long long)i, (long long)P,
                             (long long)kMatmulProcs);
        if (tiles_overflow(d.extent))
            return set_error(TM_ENOTSUP, "candidate %lld: more than 2^31 tiles in a matrix", (long long)i);
        pmax = std::max<int>(pmax, (int)P);
        proc_off[(size_t)i] = procs;
        block_first[(size_t)i] = blocks;
        procs += P;
        blocks += matmul_blocks(d);
    }
    proc_off[(size_t)n] = procs;
    block_first[(size_t)n] = blocks;
    DeviceBatch db;
    rc = upload_batch(cp, db, s);
    int64_t *d_off = nullptr, *d_bf = nullptr;
    unsigned long long* d_pp = nullptr;
    if (rc == TM_OK) {
        hipError_t e = hipMallocAsync((void**)&d_off, (size_t)(n + 1) * 8, s);
        if (e == hipSuccess) e = hipMallocAsync((void**)&d_bf, (size_t)(n + 1) * 8, s);
        if (e == hipSuccess) e = hipMallocAsync((void**)&d_pp, (size_t)std::max<int64_t>(procs, 1) * 24, s);
        void* stg = nullptr;
        if (e == hipSuccess) {
            // the descriptor upload above used the staging buffer; reuse waits for it
            rc = staging_acquire((size_t)(n + 1) * 16, &stg);
            if (rc == TM_OK) {
                std::memcpy(stg, proc_off.data(), (size_t)(n + 1) * 8);
                std::memcpy((char*)stg + (n + 1) * 8, block_first.data(), (size_t)(n + 1) * 8);
                e = hipMemcpyAsync(d_off, stg, (size_t)(n + 1) * 8, hipMemcpyHostToDevice, s);
                if (e == hipSuccess)
                    e = hipMemcpyAsync(d_bf, (char*)stg + (n + 1) * 8, (size_t)(n + 1) * 8, hipMemcpyHostToDevice, s);
                if (e == hipSuccess) rc = staging_release(s);
            }
        }
        if (rc == TM_OK && e == hipSuccess) e = hipMemsetAsync(d_pp, 0, (size_t)std::max<int64_t>(procs, 1) * 24, s);
        if (rc == TM_OK && e == hipSuccess) e = launch_build_tables(db.hdr, db.cands, n, db.arena, 1, s);
        if (rc == TM_OK && e == hipSuccess)
            e = launch_matmul(db.cands, n, db.arena, cp.cnt_words, pmax, d_off, d_pp, blocks, d_bf, s);
        if (rc == TM_OK && e == hipSuccess)
            e = launch_matmul_finalize(db.cands, n, d_off, d_pp, mm->tile_bytes, d_out, d_per_proc, s);
        if (rc == TM_OK && e != hipSuccess) rc = set_error(TM_EDEVICE, "matmul launch: %s", hipGetErrorString(e));
    }
    if (d_off) (void)hipFreeAsync(d_off, s);
    if (d_bf) (void)hipFreeAsync(d_bf, s);
    if (d_pp) (void)hipFreeAsync(d_pp, s);
    free_batch(db, s);
    return rc;
}

extern "C" int tm_select_best(const tm_stencil_cost* d_costs, const int64_t* seg, int64_t nseg, int64_t* d_best,
                              void* stream) {
    hipStream_t s = (hipStream_t)stream;
    if (nseg < 0 || (nseg > 0 && (!seg || !d_best))) return set_error(TM_EINVAL, "bad segments");
    if (nseg == 0) return TM_OK;
    for (int64_t i = 0; i < nseg; ++i)
        if (seg[i] < 0 || seg[i + 1] < seg[i]) return set_error(TM_EINVAL, "segment %lld is not ordered", (long long)i);
    if (seg[nseg] > 0 && !d_costs) return set_error(TM_EINVAL, "null costs");
    int rc = refuse_capture(s);
    if (rc != TM_OK) return rc;
    int64_t* d_seg = nullptr;
    TM_HIP(hipMallocAsync((void**)&d_seg, (size_t)(nseg + 1) * 8, s));
    void* stg = nullptr;
    rc = staging_acquire((size_t)(nseg + 1) * 8, &stg);
    if (rc == TM_OK) {
        std::memcpy(stg, seg, (size_t)(nseg + 1) * 8);
        hipError_t e = hipMemcpyAsync(d_seg, stg, (size_t)(nseg + 1) * 8, hipMemcpyHostToDevice, s);
        if (e == hipSuccess) rc = staging_release(s);
        if (rc == TM_OK && e == hipSuccess) e = launch_select_segments(d_costs, d_seg, nseg, nullptr, 0, d_best, nullptr, s);
        if (rc == TM_OK && e != hipSuccess) rc = set_error(TM_EDEVICE, "select launch: %s", hipGetErrorString(e));
    }
    (void)hipFreeAsync(d_seg, s);
    return rc;
}

// ------------------------------------------------------------------ batch plans

namespace tmk {

static void search_free(SearchBufs& b) {
    void* ptrs[] = {b.X, b.base, b.score, b.est, b.pre, b.seg, b.sel, b.sub_out, b.all_out};
    for (void* q : ptrs)
        if (q) (void)hipFree(q);
    b = SearchBufs{};
}

static void plan_free(tm_plan* p) {
    search_free(p->sb);
    if (p->d_cands) (void)hipFree(p->d_cands);
    if (p->d_evals) (void)hipFree(p->d_evals);
    if (p->d_feats) (void)hipFree(p->d_feats);
    if (p->d_arena) (void)hipFree(p->d_arena);
    for (int32_t* a : p->outgrown) (void)hipFree(a);
    p->outgrown.clear();
    if (p->d_hdr) (void)hipFree(p->d_hdr);
    if (p->d_counter) (void)hipFree(p->d_counter);
    if (p->h_cands) (void)hipHostFree(p->h_cands);
    if (p->h_hdr) (void)hipHostFree(p->h_hdr);
    if (p->h_seg) (void)hipHostFree(p->h_seg);
    p->d_cands = nullptr;
    p->d_evals = nullptr;
    p->d_feats = nullptr;
    p->d_arena = nullptr;
    p->d_hdr = nullptr;
    p->d_counter = nullptr;
    p->h_cands = nullptr;
    p->h_hdr = nullptr;
    p->h_seg = nullptr;
    p->cap_hseg = 0;
    p->cap_cands = 0;
    p->cap_arena = 0;
    p->reserved = 0;
}

// Descriptor buffers for up to `cands` candidates (the owner tables' memory is allocated
// separately, on first use, by plan_ensure_arena).
static int plan_alloc(tm_plan* p, int64_t cands) {
    plan_free(p);
    cands = std::max<int64_t>(cands, 1);
    if (hipMalloc((void**)&p->d_cands, (size_t)cands * sizeof(DevCand)) != hipSuccess ||
        hipMalloc((void**)&p->d_evals, (size_t)cands * sizeof(DevEval)) != hipSuccess ||
        hipMalloc((void**)&p->d_feats, (size_t)cands * sizeof(DevFeat)) != hipSuccess ||
        hipMalloc((void**)&p->d_hdr, sizeof(DevHeader)) != hipSuccess ||
        hipMalloc((void**)&p->d_counter, kCounters * sizeof(unsigned int)) != hipSuccess ||
        hipHostMalloc((void**)&p->h_cands, (size_t)cands * sizeof(DevCand), hipHostMallocDefault) != hipSuccess ||
        hipHostMalloc((void**)&p->h_hdr, sizeof(DevHeader), hipHostMallocDefault) != hipSuccess) {
        plan_free(p);
        return no_memory("plan buffers for %lld candidates", (long long)cands);
    }
    p->cap_cands = cands;
    return TM_OK;
}

// A place for every candidate's owner table: a map writes its candidate's, and maps of
// several candidates may be in flight on several streams.
static void layout_maps(Compiled& cp) {
    int64_t words = 0;
    for (auto& d : cp.cands) {
        d.arena_off = words;
        words += map_ids_words(d.vol);
    }
    cp.map_words = words;
}

// Device memory for the batch's owner tables; grows (after draining `s`) when needed.  A
// capture can neither wait nor free: there the old memory stays until the plan's end, so that
// the first map of a batch can be recorded too.
static int plan_ensure_arena(tm_plan* p, hipStream_t s) {
    const int64_t words = std::max<int64_t>(p->cp.map_words, 4);
    if (p->d_arena && p->cap_arena >= words) return TM_OK;
    if (capturing(s)) {
        if (p->d_arena) p->outgrown.push_back(p->d_arena);
    } else {
        TM_HIP(hipStreamSynchronize(s));
        if (p->d_arena) (void)hipFree(p->d_arena);
    }
    p->d_arena = nullptr;
    p->cap_arena = 0;
    if (malloc_anytime((void**)&p->d_arena, (size_t)words * 4) != hipSuccess)
        return no_memory("owner tables of %lld words", (long long)words);
    p->cap_arena = words;
    return TM_OK;
}

// The batch's descriptors to the device; loaded once they are on their way.
static int plan_upload(tm_plan* p, hipStream_t s) {
    p->loaded = false;
    if (p->up_pending) {
        TM_HIP(hipEventSynchronize(p->up_ev));
        p->up_pending = false;
    }
    const size_t nc = p->cp.cands.size() * sizeof(DevCand);
    std::memcpy(p->h_hdr, &p->cp.hdr, sizeof(DevHeader));
    if (nc) std::memcpy(p->h_cands, p->cp.cands.data(), nc);
    TM_HIP(hipMemcpyAsync(p->d_hdr, p->h_hdr, sizeof(DevHeader), hipMemcpyHostToDevice, s));
    if (nc) TM_HIP(hipMemcpyAsync(p->d_cands, p->h_cands, nc, hipMemcpyHostToDevice, s));
    TM_HIP(hipEventRecord(p->up_ev, s));
    p->up_pending = true;
    TM_HIP(launch_fill_evals(p->cp.eval, p->d_cands, p->d_evals, p->d_feats, p->d_counter, s));
    p->loaded = true;
    return TM_OK;
}

// The word in which a run counts its finished workgroups.  Runs of one plan may overlap on
// several streams, so each takes the next one; the replays of a graph keep the word of its
// capture, which no run outside a graph takes.
static unsigned int* plan_counter(tm_plan* p, hipStream_t s) {
    constexpr unsigned int kHalf = kCounters / 2;
    if (capturing(s)) return p->d_counter + kHalf + p->captured++ % kHalf;
    return p->d_counter + p->runs++ % kHalf;
}

// Enqueues a run (stage -1) or one stage of it on stream s: one launch up to kFinInCount
// candidates, else two or three.  A launch costs the host 2.4 us; replaying a graph of one
// 18.2 us (and its capture at every change of an output).  Stage 2 on its own repeats the
// selection (idempotent).
static hipError_t plan_enqueue(tm_plan* p, int stage, tm_stencil_cost* out, int64_t* best, hipStream_t s,
                               int32_t* best_ids = nullptr) {
    const Compiled& cp = p->cp;
    if (stage == 0) return launch_zero_costs(out, cp.hdr.n, s);
    if (stage == 2) return launch_bytes_select(out, cp.hdr.n, cp.hdr.elem_bytes, best, s);
    return launch_eval_batch(cp.eval, p->d_evals, out, best, best ? plan_counter(p, s) : nullptr, eval_cus(cp.eval), s,
                             nullptr, 0, best_ids);
}

// Maps and class tuples are given once a batch of the plan was evaluated (by a run, a stage, an
// exhaustive search or the autotuner), or where the words reserved at creation hold all
// the tables of the batch's compiled candidates (DevCand::words).
static bool plan_ready(const tm_plan* p) { return p->ran || p->reserved >= p->cp.arena_words; }

// Map launch for a device-side index: fits every loaded candidate.
static MapShape plan_map_shape(const tm_plan* p) { return map_shape(p->cp.max_vol, p->cp.max_points, p->cp.min_row); }

}  // namespace tmk

extern "C" int tm_plan_create(int64_t max_cands, int64_t max_words, tm_plan** out) {
    if (!out) return set_error(TM_EINVAL, "null output");
    *out = nullptr;
    tm_plan* p = new (std::nothrow) tm_plan();
    if (!p) return no_memory("plan");
    (void)hipGetDevice(&p->device);
    int rc = plan_alloc(p, max_cands);
    if (rc == TM_OK && max_words > 0) {
        if (hipMalloc((void**)&p->d_arena, (size_t)max_words * 4) != hipSuccess) rc = no_memory("arena");
        else p->reserved = p->cap_arena = max_words;
    }
    if (rc == TM_OK && hipEventCreateWithFlags(&p->up_ev, hipEventDisableTiming) != hipSuccess)
        rc = set_error(TM_EDEVICE, "event");
    if (rc != TM_OK) {
        tm_plan_destroy(p);
        return rc;
    }
    *out = p;
    return TM_OK;
}

extern "C" int tm_plan_destroy(tm_plan* p) {
    if (!p) return TM_OK;
    if (p->up_pending) (void)hipEventSynchronize(p->up_ev);
    (void)hipDeviceSynchronize();
    plan_free(p);
    if (p->up_ev) (void)hipEventDestroy(p->up_ev);
    delete p;
    return TM_OK;
}

extern "C" int tm_plan_load(tm_plan* p, const tm_candidate* c, int64_t n, const tm_stencil* st,
                            int64_t cells_per_item, void* stream) {
    if (!p) return set_error(TM_EINVAL, "null plan");
    if (!st) return set_error(TM_EINVAL, "null stencil");
    if (cells_per_item < 0 || cells_per_item > kMaxCellsPerItem)
        return set_error(TM_EINVAL, "cells_per_item %lld (at most 2^26)", (long long)cells_per_item);
    hipStream_t s = (hipStream_t)stream;
    Compiled cp;
    int rc = compile_batch(c, n, st, true, cp);
    if (rc != TM_OK) return rc;
    if (n > p->cap_cands) {
        // grow: wait for work that may still read the old buffers
        TM_HIP(hipStreamSynchronize(s));
        p->loaded = false;  // its buffers go, whether or not larger ones come
        rc = plan_alloc(p, std::max(n, p->cap_cands));
        if (rc != TM_OK) return rc;
        p->up_pending = false;
    }
    if (cells_per_item > 0) p->cells_per_item = cells_per_item;
    layout_eval(cp, p->cells_per_item, false);
    layout_maps(cp);
    cp.eval.wg_per_cu = p->wg_per_cu;
    p->cp = std::move(cp);
    return plan_upload(p, s);
}

extern "C" int tm_plan_run(tm_plan* p, tm_stencil_cost* d_out, int64_t* d_best, void* stream) {
    if (!p || !p->loaded) return set_error(TM_EINVAL, "plan not loaded");
    if (p->cp.hdr.n > 0 && !d_out) return set_error(TM_EINVAL, "null output");
    if (p->cp.hdr.n == 0) return TM_OK;
    TM_HIP(plan_enqueue(p, -1, d_out, d_best, (hipStream_t)stream));
    p->ran = true;
    return TM_OK;
}

extern "C" int tm_plan_run_map(tm_plan* p, tm_stencil_cost* d_out, int64_t* d_best, int32_t* d_map, int64_t cap,
                               void* stream) {
    if (!p || !p->loaded) return set_error(TM_EINVAL, "plan not loaded");
    if (p->cp.hdr.n == 0) return set_error(TM_EINVAL, "empty batch");
    if (!d_out || !d_best || !d_map) return set_error(TM_EINVAL, "null output");
    if (cap < p->cp.max_points) return set_error(TM_ECAPACITY, "map needs %lld entries", (long long)p->cp.max_points);
    hipStream_t s = (hipStream_t)stream;
    const int rc = plan_ensure_arena(p, s);
    if (rc != TM_OK) return rc;
    TM_HIP(plan_enqueue(p, -1, d_out, d_best, s, p->d_arena));
    TM_HIP(launch_map(plan_map_shape(p), p->d_evals, p->cp.hdr.n, d_best, 0, p->d_arena, d_map, s));
    p->ran = true;
    return TM_OK;
}

extern "C" int tm_plan_run_stage(tm_plan* p, int32_t stage, tm_stencil_cost* d_out, int64_t* d_best,
                                 void* stream) {
    if (!p || !p->loaded) return set_error(TM_EINVAL, "plan not loaded");
    if (stage < 0 || stage > 2) return set_error(TM_EINVAL, "stage %d", stage);
    if (p->cp.hdr.n > 0 && !d_out) return set_error(TM_EINVAL, "null output");
    if (p->cp.hdr.n == 0) return TM_OK;
    TM_HIP(plan_enqueue(p, stage, d_out, d_best, (hipStream_t)stream));
    p->ran = true;
    return TM_OK;
}

extern "C" int tm_plan_materialize(tm_plan* p, const int64_t* d_index, int64_t host_index, int32_t* d_map,
                                   int64_t cap, void* stream) {
    if (!p || !p->loaded) return set_error(TM_EINVAL, "plan not loaded");
    if (!d_map) return set_error(TM_EINVAL, "null output");
    const Compiled& cp = p->cp;
    if (cp.hdr.n == 0) return set_error(TM_EINVAL, "empty batch");
    int64_t need = cp.max_points;
    MapShape shape;
    if (!d_index) {
        if (host_index < 0 || host_index >= cp.hdr.n) return set_error(TM_EINVAL, "index %lld", (long long)host_index);
        const DevCand& c = cp.cands[(size_t)host_index];
        need = c.npoints;
        shape = map_shape(c.vol, c.npoints, c.L);
    } else {
        shape = plan_map_shape(p);
    }
    if (cap < need) return set_error(TM_ECAPACITY, "map needs %lld entries", (long long)need);
    if (!plan_ready(p)) return set_error(TM_EINVAL, "not run yet: run the plan before materialising a map");
    const int rc = plan_ensure_arena(p, (hipStream_t)stream);
    if (rc != TM_OK) return rc;
    hipStream_t s = (hipStream_t)stream;
    hipError_t e = launch_map_ids(p->d_evals, cp.hdr.n, d_index, host_index, cp.max_vol, p->d_arena, s);
    if (e == hipSuccess) e = launch_map(shape, p->d_evals, cp.hdr.n, d_index, host_index, p->d_arena, d_map, s);
    if (e != hipSuccess) return set_error(TM_EDEVICE, "map launch: %s", hipGetErrorString(e));
    return TM_OK;
}

extern "C" int tm_plan_info(const tm_plan* p, int64_t* n, int64_t* items, int64_t* points) {
    if (!p) return set_error(TM_EINVAL, "null plan");
    if (n) *n = p->loaded ? p->cp.hdr.n : 0;
    if (items) *items = p->loaded ? p->cp.eval.items : 0;
    if (points) *points = p->loaded ? p->cp.points : 0;
    return TM_OK;
}

extern "C" int tm_plan_class_tuples(tm_plan* p, int64_t* tuples, void* stream) {
    if (!p || !p->loaded) return set_error(TM_EINVAL, "plan not loaded");
    if (!tuples) return set_error(TM_EINVAL, "null output");
    *tuples = 0;
    if (p->cp.hdr.n == 0) return TM_OK;
    if (!plan_ready(p)) return set_error(TM_EINVAL, "not run yet: run the plan first");
    hipStream_t s = (hipStream_t)stream;
    unsigned long long* d_tot = nullptr;
    TM_HIP(hipMallocAsync((void**)&d_tot, 8, s));
    unsigned long long h = 0;
    hipError_t e = hipMemsetAsync(d_tot, 0, 8, s);
    if (e == hipSuccess) e = launch_class_tuples(p->d_cands, p->cp.hdr.n, p->cp.hdr.halo, d_tot, s);
    if (e == hipSuccess) e = hipMemcpyAsync(&h, d_tot, 8, hipMemcpyDeviceToHost, s);
    (void)hipFreeAsync(d_tot, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return set_error(TM_EDEVICE, "class tuples: %s", hipGetErrorString(e));
    *tuples = (int64_t)h;
    return TM_OK;
}

// A launch configuration for the loaded batch (cells_per_item 0: the default).
static int plan_relayout(tm_plan* p, int64_t cells_per_item, int wg_per_cu, hipStream_t s) {
    p->cells_per_item = cells_per_item;
    p->wg_per_cu = wg_per_cu;
    if (p->cp.hdr.n == 0) return TM_OK;
    layout_eval(p->cp, cells_per_item, false);
    p->cp.eval.wg_per_cu = wg_per_cu;
    return plan_upload(p, s);
}

extern "C" int tm_plan_autotune(tm_plan* p, tm_stencil_cost* d_out, int64_t* cells_per_item, int32_t* wg_per_cu,
                                void* stream) {
    if (!p || !p->loaded) return set_error(TM_EINVAL, "plan not loaded");
    if (p->cp.hdr.n == 0) return TM_OK;
    if (!d_out) return set_error(TM_EINVAL, "null output");
    hipStream_t s = (hipStream_t)stream;
    hipEvent_t e0, e1;
    TM_HIP(hipEventCreate(&e0));
    TM_HIP(hipEventCreate(&e1));
    const int64_t cells_opts[] = {1 << 10, 1 << 12, 1 << 14};
    const int wg_opts[] = {0, 2, 1};
    float best_ms = 1e30f;
    int64_t best_c = cells_opts[0];
    int best_w = 0;
    int rc = TM_OK;
    for (int64_t cpi : cells_opts) {
        layout_eval(p->cp, cpi, false);
        rc = plan_upload(p, s);
        for (int w : wg_opts) {
            p->cp.eval.wg_per_cu = w;
            float tot = 0.f;
            for (int rep = 0; rep < 3 && rc == TM_OK; ++rep) {
                hipError_t e = hipEventRecord(e0, s);
                if (e == hipSuccess) e = plan_enqueue(p, 1, d_out, nullptr, s);
                if (e == hipSuccess) e = hipEventRecord(e1, s);
                if (e == hipSuccess) e = hipEventSynchronize(e1);
                float ms = 0.f;
                if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
                if (e != hipSuccess) rc = set_error(TM_EDEVICE, "autotune: %s", hipGetErrorString(e));
                if (rep > 0) tot += ms;
            }
            if (rc != TM_OK) break;
            if (tot < best_ms) {
                best_ms = tot;
                best_c = cpi;
                best_w = w;
            }
        }
        if (rc != TM_OK) break;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc != TM_OK) return rc;
    p->ran = true;
    rc = plan_relayout(p, best_c, best_w, s);
    if (cells_per_item) *cells_per_item = best_c;
    if (wg_per_cu) *wg_per_cu = best_w;
    return rc;
}

extern "C" int tm_plan_set_launch(tm_plan* p, int64_t cells_per_item, int32_t wg_per_cu, void* stream) {
    if (!p || !p->loaded) return set_error(TM_EINVAL, "plan not loaded");
    if (cells_per_item < 0 || cells_per_item > kMaxCellsPerItem || wg_per_cu < 0)
        return set_error(TM_EINVAL, "cells_per_item %lld (at most 2^26), wg_per_cu %d", (long long)cells_per_item,
                         wg_per_cu);
    return plan_relayout(p, cells_per_item, wg_per_cu, (hipStream_t)stream);
}

// ------------------------------------------------------------------ search support

namespace tmk {

int64_t plan_size(const tm_plan* p) { return p->cp.hdr.n; }
const DevFeat* plan_feats(const tm_plan* p) { return p->d_feats; }
FeatHalo plan_halo(const tm_plan* p) {
    const int32_t* h = p->cp.hdr.halo;
    return FeatHalo{{h[0], h[1], h[2], h[3]}};
}

// Ranker buffers: features and bases of n rows; scores of max(n, m) entries (m: the
// second stage's survivors of a ranked search).
static int ensure_rank_bufs(SearchBufs& b, int64_t n, int64_t m, hipStream_t s) {
    const int64_t sc = std::max<int64_t>(std::max(n, m), 1);
    if (b.cap_n < n) {
        TM_HIP(hipStreamSynchronize(s));
        if (b.X) (void)hipFree(b.X);
        if (b.base) (void)hipFree(b.base);
        b.X = nullptr;
        b.base = nullptr;
        b.cap_n = 0;
        if (hipMalloc((void**)&b.X, (size_t)std::max<int64_t>(n, 1) * kFeat * 2) != hipSuccess ||
            hipMalloc((void**)&b.base, (size_t)std::max<int64_t>(n, 1) * 4) != hipSuccess)
            return no_memory("feature buffers");
        b.cap_n = n;
    }
    if (b.cap_sc < sc) {
        TM_HIP(hipStreamSynchronize(s));
        if (b.score) (void)hipFree(b.score);
        b.score = nullptr;
        b.cap_sc = 0;
        if (hipMalloc((void**)&b.score, (size_t)sc * 4) != hipSuccess)
            return no_memory("score buffers");
        b.cap_sc = sc;
    }
    return TM_OK;
}

int plan_features(const tm_plan* p, float* d_feat, hipStream_t s) {
    if (!p || !p->loaded) return set_error(TM_EINVAL, "plan not loaded");
    if (!d_feat) return set_error(TM_EINVAL, "null output");
    tm_plan* q = const_cast<tm_plan*>(p);
    SearchBufs& b = q->sb;
    const int64_t n = p->cp.hdr.n;
    const int rc = ensure_rank_bufs(b, n, 0, s);
    if (rc != TM_OK) return rc;
    TM_HIP(launch_features(p->d_feats, n, plan_halo(p), b.base, b.X, d_feat, s));
    return TM_OK;
}

int plan_block_estimates(const tm_plan* p, double* d_est, hipStream_t s) {
    if (!p || !p->loaded) return set_error(TM_EINVAL, "plan not loaded");
    if (!d_est) return set_error(TM_EINVAL, "null output");
    TM_HIP(launch_estimates(plan_estimates(p), nullptr, p->cp.hdr.n, 0.f, d_est, nullptr, s));
    return TM_OK;
}

EstimateBatch plan_estimates(const tm_plan* p) {
    const EvalPlan& e = p->cp.eval;
    return EstimateBatch{p->d_cands, p->d_evals, p->cp.max_vol, p->cp.max_blocks, {e.halo[0], e.halo[1], e.halo[2], e.halo[3]},
                         p->d_hdr->halo, e.all_simple};
}

int plan_search_prepare(tm_plan* p, const int64_t* seg, int64_t nseg, int32_t prefilter, int32_t topk, bool ranked,
                        SearchBufs** out, hipStream_t s) {
    if (!p || !p->loaded) return set_error(TM_EINVAL, "plan not loaded");
    if (nseg < 1 || !seg) return set_error(TM_EINVAL, "no segments");
    const int64_t n = p->cp.hdr.n;
    if (seg[0] != 0 || seg[nseg] != n) return set_error(TM_EINVAL, "segments must cover the loaded batch");
    for (int64_t i = 0; i < nseg; ++i) {
        if (seg[i + 1] < seg[i]) return set_error(TM_EINVAL, "segment %lld is not ordered", (long long)i);
        if (seg[i + 1] - seg[i] > INT32_MAX) return set_error(TM_EINVAL, "segment %lld is too long", (long long)i);
    }
    if (ranked && (topk < 1 || topk > 4096)) return set_error(TM_EINVAL, "topk %d not in 1..4096", topk);
    if (ranked && prefilter != 0 && (prefilter < topk || prefilter > 65536))
        return set_error(TM_EINVAL, "prefilter %d not 0 or in topk..65536", prefilter);
    SearchBufs& b = p->sb;
    const int64_t nsel = ranked ? nseg * (int64_t)topk : 0;
    const int64_t npre = ranked ? nseg * (int64_t)prefilter : 0;
    auto grow = [&](bool need) -> int {
        if (!need) return TM_OK;
        TM_HIP(hipStreamSynchronize(s));
        return TM_OK;
    };
    if (ranked) {
        int rc = ensure_rank_bufs(b, n, npre, s);
        if (rc != TM_OK) return rc;
        if (b.cap_pre < npre) {
            TM_HIP(hipStreamSynchronize(s));
            if (b.pre) (void)hipFree(b.pre);
            if (b.est) (void)hipFree(b.est);
            b.pre = nullptr;
            b.est = nullptr;
            b.cap_pre = 0;
            if (hipMalloc((void**)&b.pre, (size_t)npre * 8) != hipSuccess ||
                hipMalloc((void**)&b.est, (size_t)npre * 2 * sizeof(double)) != hipSuccess)
                return no_memory("prefilter buffer");
            b.cap_pre = npre;
        }
        if (b.cap_sel < nsel) {
            int rc = grow(true);
            if (rc != TM_OK) return rc;
            if (b.sel) (void)hipFree(b.sel);
            if (b.sub_out) (void)hipFree(b.sub_out);
            b.sel = nullptr;
            b.sub_out = nullptr;
            b.cap_sel = 0;
            if (hipMalloc((void**)&b.sel, (size_t)nsel * 8) != hipSuccess ||
                hipMalloc((void**)&b.sub_out, (size_t)nsel * sizeof(tm_stencil_cost)) != hipSuccess)
                return no_memory("survivor buffers");
            b.cap_sel = nsel;
        }
    } else if (b.cap_all < n) {
        int rc = grow(b.all_out != nullptr);
        if (rc != TM_OK) return rc;
        if (b.all_out) (void)hipFree(b.all_out);
        b.all_out = nullptr;
        b.cap_all = 0;
        if (hipMalloc((void**)&b.all_out, (size_t)std::max<int64_t>(n, 1) * sizeof(tm_stencil_cost)) != hipSuccess)
            return no_memory("cost buffer");
        b.cap_all = n;
    }
    if (b.cap_seg < nseg + 1) {
        int rc = grow(true);
        if (rc != TM_OK) return rc;
        if (b.seg) (void)hipFree(b.seg);
        b.seg = nullptr;
        b.cap_seg = 0;
        if (hipMalloc((void**)&b.seg, (size_t)(nseg + 1) * 8) != hipSuccess)
            return no_memory("segment buffers");
        b.cap_seg = nseg + 1;
    }
    // segments: copy only when they changed (pinned staging, ordered on s)
    if (b.nseg != nseg || !p->h_seg || std::memcmp(p->h_seg, seg, (size_t)(nseg + 1) * 8) != 0) {
        if (p->up_pending) {
            TM_HIP(hipEventSynchronize(p->up_ev));
            p->up_pending = false;
        }
        if (p->cap_hseg < nseg + 1) {
            if (p->h_seg) (void)hipHostFree(p->h_seg);
            p->h_seg = nullptr;
            if (hipHostMalloc((void**)&p->h_seg, (size_t)(nseg + 1) * 8, hipHostMallocDefault) != hipSuccess)
                return no_memory("segment staging");
            p->cap_hseg = nseg + 1;
        }
        std::memcpy(p->h_seg, seg, (size_t)(nseg + 1) * 8);
        TM_HIP(hipMemcpyAsync(b.seg, p->h_seg, (size_t)(nseg + 1) * 8, hipMemcpyHostToDevice, s));
        TM_HIP(hipEventRecord(p->up_ev, s));
        p->up_pending = true;
    }
    b.nseg = nseg;
    b.k = topk;
    *out = &b;
    return TM_OK;
}

// The best of the candidates chosen in sb (sb->sel), by their exact costs.
hipError_t plan_eval_chosen(tm_plan* p, SearchBufs* sb, int64_t* d_best, tm_stencil_cost* d_best_cost, hipStream_t s) {
    const int64_t nsel = sb->nseg * sb->k;
    const hipError_t e = launch_eval_batch(p->cp.eval, p->d_evals, sb->sub_out, nullptr, nullptr, eval_cus(p->cp.eval), s,
                                           sb->sel, nsel);
    if (e != hipSuccess) return e;
    return launch_select_segments(sb->sub_out, sb->seg, sb->nseg, sb->sel, sb->k, d_best, d_best_cost, s);
}

int plan_exhaustive_search(tm_plan* p, const int64_t* seg, int64_t nseg, int64_t* d_best,
                           tm_stencil_cost* d_best_cost, hipStream_t s) {
    if (!d_best) return set_error(TM_EINVAL, "null output");
    SearchBufs* sb = nullptr;
    int rc = plan_search_prepare(p, seg, nseg, 0, 0, false, &sb, s);
    if (rc != TM_OK) return rc;
    hipError_t e = plan_enqueue(p, -1, sb->all_out, nullptr, s);
    if (e == hipSuccess) p->ran = true;
    if (e == hipSuccess) e = launch_select_segments(sb->all_out, sb->seg, nseg, nullptr, 0, d_best, d_best_cost, s);
    if (e != hipSuccess) return set_error(TM_EDEVICE, "exhaustive search: %s", hipGetErrorString(e));
    return TM_OK;
}

}  // namespace tmk
