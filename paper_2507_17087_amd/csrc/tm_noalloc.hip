// tm_noalloc.hip -- tm_eval_stencil_batch_noalloc: the stencil evaluation of
// tm_eval_stencil_batch for callers that cannot allocate device memory.  Its descriptors
// live in `scratch`, a file-scope device array of TM_NOALLOC_SCRATCH_BYTES held by every
// GPU the library runs on until the process ends.  Host code never uses the array's name as an address (it
// is a host-side stand-in): the device address comes from hipGetSymbolAddress, once
// per device, and only that pointer is passed to the kernels and copies.
#include <hip/hip_runtime.h>

#include <mutex>
#include <vector>

#include "tm_compile.h"
#include "tm_internal.h"
#include "tm_plan.h"

namespace tmk {

static __device__ __align__(256) unsigned char scratch[TM_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
static std::once_flag g_once[kMaxDevices];
static void* g_ptr[kMaxDevices];
static hipError_t g_err[kMaxDevices];

// Device address of this device's copy of `scratch` (looked up on the first call
// on each device, with that device current).
static int scratch_ptr(void** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return set_error(TM_EDEVICE, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return set_error(TM_ENOTSUP, "device %d", dev);
    std::call_once(g_once[dev], [dev]() {
        void* p = nullptr;
        g_err[dev] = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        g_ptr[dev] = g_err[dev] == hipSuccess ? p : nullptr;
    });
    if (g_err[dev] != hipSuccess || !g_ptr[dev])
        return set_error(TM_EDEVICE, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(g_err[dev]));
    *out = g_ptr[dev];
    return TM_OK;
}

// A candidate counts for its compiled descriptor and its table words against
// TM_NOALLOC_SCRATCH_BYTES; the evaluation's descriptor, all that is stored, takes less.
static_assert(sizeof(DevEval) <= sizeof(DevCand), "the evaluation's descriptors fit");

static int64_t up256(int64_t x) { return (x + 255) & ~int64_t(255); }

}  // namespace tmk

using namespace tmk;

extern "C" int tm_eval_stencil_batch_noalloc(const tm_candidate* c, int64_t n, const tm_stencil* st,
                                             tm_stencil_cost* d_out, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    if (!st) return set_error(TM_EINVAL, "null stencil");
    Compiled cp;
    int rc = compile_batch(c, n, st, true, cp);
    if (rc != TM_OK) return rc;
    if (n == 0) return TM_OK;
    if (!d_out) return set_error(TM_EINVAL, "null output");
    // what counts: a header, descriptors, tables, a work counter; what is stored, past the
    // header's place: the evaluation's descriptors
    const int64_t header = up256((int64_t)sizeof(DevHeader));
    const int64_t need = header + up256(n * (int64_t)sizeof(DevCand)) + up256(counted_words(cp) * 4) + 256;
    if (need > (int64_t)TM_NOALLOC_SCRATCH_BYTES)
        return set_error(TM_ECAPACITY, "the batch needs %lld bytes of scratch; the library holds %lld",
                         (long long)need, (long long)TM_NOALLOC_SCRATCH_BYTES);
    rc = refuse_capture(s);
    if (rc != TM_OK) return rc;
    char* base = nullptr;
    rc = scratch_ptr((void**)&base);
    if (rc != TM_OK) return rc;
    layout_eval(cp, 0, false);
    const EvalShape shape{cp.eval.H, cp.eval.node_level, cp.eval.per_item, cp.eval.fill};
    std::vector<DevEval> evals((size_t)n);
    for (int64_t i = 0; i < n; ++i) fill_eval(cp.cands[(size_t)i], shape, &evals[(size_t)i]);
    DevEval* d_evals = reinterpret_cast<DevEval*>(base + header);
    // the descriptors go up from this call's host memory; waiting for the copy keeps it
    // alive until it is done (nothing here allocates pinned staging)
    hipError_t e = hipMemcpyAsync(d_evals, evals.data(), (size_t)n * sizeof(DevEval), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e == hipSuccess) e = launch_eval_batch(cp.eval, d_evals, d_out, nullptr, nullptr, 0, s);
    if (e != hipSuccess) return set_error(TM_EDEVICE, "stencil launch (no allocation): %s", hipGetErrorString(e));
    return TM_OK;
}
