/* A HIP runtime of host memory for tests of the host side without a GPU: allocations that
 * fail on demand, launches that are only counted.  Loaded with RTLD_GLOBAL before the library,
 * so that its calls end here. */
#include <stdlib.h>
#include <string.h>

int fake_fail = 0;      /* device allocations above this many bytes fail (0: none does) */
int fake_launches = 0;  /* kernels launched so far */
int fake_allocs = 0;    /* device allocations so far */
static int last = 0;

static int result(int e) {
    if (e) last = e;
    return e;
}
static int alloc(void** p, size_t n) {
    *p = fake_fail && n > (size_t)fake_fail ? 0 : calloc(1, n ? n : 1);
    return result(*p ? 0 : 2 /* hipErrorOutOfMemory */);
}

int hipGetLastError(void) {
    const int e = last;
    last = 0;
    return e;
}
int hipMalloc(void** p, size_t n) {
    ++fake_allocs;
    return alloc(p, n);
}
int hipHostMalloc(void** p, size_t n, unsigned flags) { return alloc(p, n); }
int hipMallocAsync(void** p, size_t n, void* s) { return alloc(p, n); }
int hipFree(void* p) { free(p); return 0; }
int hipFreeAsync(void* p, void* s) { free(p); return 0; }
int hipHostFree(void* p) { free(p); return 0; }
int hipMemset(void* p, int v, size_t n) { memset(p, v, n); return 0; }
int hipMemsetAsync(void* p, int v, size_t n, void* s) { memset(p, v, n); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int kind) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st) { memcpy(d, s, n); return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { *v = 256; return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipStreamSynchronize(void* s) { return 0; }
int hipStreamIsCapturing(void* s, int* st) { *st = 0; return 0; }
int hipThreadExchangeStreamCaptureMode(int* m) { return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { *e = malloc(1); return 0; }
int hipEventCreate(void** e) { *e = malloc(1); return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { *ms = 1; return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void* e, void* s) { return 0; }
int hipEventSynchronize(void* e) { return 0; }
struct dim3_ { unsigned x, y, z; };
/* the first call of every kernel<<<>>>: counted, and the launch itself skipped */
unsigned __hipPushCallConfiguration(struct dim3_ g, struct dim3_ b, size_t lds, void* s) {
    ++fake_launches;
    return 1;
}
