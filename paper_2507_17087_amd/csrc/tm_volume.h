// tm_volume.h -- launch interface of the matmul tile fetches and the redistribution
// volumes over coordinate groups (tm_volume.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tm_compile.h"
#include "tm_internal.h"

namespace tmk {

// One launch dim of a pair of mappings.  Its joint segments are cut by the change points
// of both mappings' block projections: of block sizes of which one divides another only
// the larger is listed, since its change points include the other's.  M: the least common
// multiple of both mappings' cyclic sizes (DevDim).
struct JointDim {
    int32_t l, M, nseg, G, nblk, ident;
    int32_t s[TM_MAX_MRANK];
    int32_t pad[2];
    double rl, rM, rs, rsum;  // 1/l, 1/M, 1/s[0], 1/(sum of s)
};

struct alignas(16) DevPair {
    DevEval a, b;
    JointDim dim[TM_MAX_LRANK];
    int32_t dim_d, parts, pad[2];  // the dim with the most groups, cut into parts
};
static_assert(sizeof(DevPair) % 16 == 0 && sizeof(DevPair) / 16 <= 256, "staged by 256 threads");

// A pair's workgroups: about this many tuples each.  A pair of one workgroup is counted
// without atomics or cleared output.  Transposes of 512^3 on 128 processors have up to
// 16,384 tuples; on 4,096 processors 273 pairs take 403 us, with four times as many tuples
// a workgroup 693 us.
constexpr int64_t kPairTuples = 16384;
// Up to this many workgroups have 16 waves each: two a CU, whose latency bounds the call where
// a pair has many tuples, and which cost nothing where it has few, since the pairs are then
// read in place from host memory (478 at most).  Beyond, 16 waves still gain on pairs of up to
// 16,384 tuples until about 900 of them, but take twice as long on pairs of 1,024.  Transposes
// on 128 processors, 16 waves and four, us: 108 pairs 16.2 and 26.8, 400 29.9 and 42.2, 512 20.0
// and 25.5, 900 25.4 and 26.0, 1,024 28.4 and 26.3, 2,048 48 and 31; on 32 processors: 108
// 10.6 and 10.6, 400 23.7 and 24.3, 512 11.2 and 7.6, 1,024 19.2 and 7.8, 2,048 35 and 11.
constexpr int64_t kPairWide = 512;
// Most tuples of one group of dim_d (they are indexed in floats, see div_small).
constexpr int64_t kPairRowTuples = int64_t(1) << 20;

// Joint dims, parts and LDS words of candidates a, b (same domain; p->a and p->b are
// filled).  False: not for this kernel (the general one takes it).
bool fill_pair(const CandView& a, const CandView& b, DevPair* p, int32_t* words);
hipError_t launch_pairs(const DevPair* pairs, int64_t n, int32_t parts, int32_t lds_words, int64_t elem_bytes,
                        tm_redist_cost* out, hipStream_t s);

constexpr int32_t kMatmulThreads = 256;

// LDS words of a candidate of launch rank 3; 0: its tables do not fit (the general kernel
// takes it).  A dim has at most as many groups as its projections' sizes multiply to, so a
// candidate has at most as many tuples as owners.
int32_t matmul_words(const DevEval& e);
hipError_t launch_matmul_groups(const DevEval* evals, int64_t n, int32_t lds_words, int64_t tile_bytes,
                                tm_matmul_cost* out, int64_t* per_proc, hipStream_t s);

}  // namespace tmk
