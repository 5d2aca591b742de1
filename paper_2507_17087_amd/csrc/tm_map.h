// tm_map.h -- launch interface of the processor maps (tm_map.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tm_internal.h"

namespace tmk {

// One-wave workgroups writing 4 KB blocks while the owner table is small (many workgroups
// fit a CU; 8 KB blocks are slower: a run with the map of 512^3 points 117.5 us against
// 105.8, a map of 509 x 487 x 521 points 105.1 us against 94.3), else four-wave workgroups writing 16 KB blocks, which stage the table for
// four times the points.
constexpr int32_t kMapNarrowVol = 2048;
constexpr int64_t kMapNarrowBlock = 1024, kMapWideBlock = 4096;  // points
constexpr int64_t kMapMaxGrid = int64_t(1) << 20;                 // more blocks are taken grid-stride

struct MapShape {
    bool narrow;
    int64_t block;
    int grid;
    int32_t base_words, lds_words;
};
// For candidates of volume up to max_vol, max_points points and rows of at least min_row.
MapShape map_shape(int32_t max_vol, int64_t max_points, int64_t min_row);

// Words of a candidate's ids: whole 16-byte pieces.
inline int64_t map_ids_words(int32_t vol) { return (vol + 3) & ~3; }

// Candidate *d_index (or index): its owner table as processor ids, to ids + its offset (and
// with copy its descriptor, to device memory), then its map.
hipError_t launch_map_ids(const DevEval* evals, int64_t n, const int64_t* d_index, int64_t index, int32_t max_vol,
                          int32_t* ids, hipStream_t s, DevEval* copy = nullptr);
hipError_t launch_map(const MapShape& m, const DevEval* evals, int64_t n, const int64_t* d_index, int64_t index,
                      const int32_t* ids, int32_t* out, hipStream_t s);

}  // namespace tmk
