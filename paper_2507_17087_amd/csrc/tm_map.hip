// tm_map.hip -- processor maps: the int32 processor id of every launch point, C order.
//
// The map is written in blocks of consecutive points, four (16 bytes) per store, whatever
// the rows' length: rows that are no multiple of four points cost a few lanes of a wave a
// second lookup where a store spans two rows.  A point's owner is an entry of the
// candidate's owner table (ids, staged in LDS) at the sum of its coordinates'
// contributions: a base per row, and for the last dim, where it is projected by at most
// one block projection of blocks at least four points long, the block of the store's
// first point and the first cell of the next block decide all four.
//
// Bound: HBM writes.  A 512^3 map (537 MB) 79 us and a 509 x 487 x 521 one (517 MB, three of
// four rows not 16-byte aligned) 75.8 us, both 6.8 TB/s, the rate of a plain device fill;
// before, one row a time, the ragged one took 126 us with a 4-byte store per point.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "tm_groups.h"
#include "tm_internal.h"
#include "tm_map.h"

namespace tmk {

// ------------------------------------------------------------------ the owner table

// Processor ids of the candidate's final coordinates (*d_index, or index), written to ids at
// its offset: every candidate of a plan has a place of its own there, so that the maps of two
// of them (on two streams) do not disturb each other, and two of one write the same words.
__global__ __launch_bounds__(256) void k_map_ids(const DevEval* __restrict__ evals, int64_t n,
                                                 const int64_t* __restrict__ d_index, int64_t index,
                                                 int32_t* __restrict__ ids, DevEval* __restrict__ copy) {
    __shared__ DevEval ev;
    const int64_t ci = d_index ? wave_uniform64(*d_index) : index;
    if (ci < 0 || ci >= n) return;  // no candidate selected (empty batch)
    stage_eval(&ev, evals + ci, threadIdx.x);
    __syncthreads();
    if (copy && blockIdx.x == 0) stage_eval(copy, &ev, threadIdx.x);
    const int32_t vol = wave_uniform(ev.vol), per = ((vol + (int)gridDim.x - 1) / (int)gridDim.x + 255) & ~255;
    const int32_t v0 = (int32_t)blockIdx.x * per, v1 = v0 + per < vol ? v0 + per : vol;
    if (v0 < v1) owner_table<true>(ev, ids + wave_uniform64(ev.offset), v0, v1, -1, threadIdx.x, 256);
}

hipError_t launch_map_ids(const DevEval* evals, int64_t n, const int64_t* d_index, int64_t index, int32_t max_vol,
                          int32_t* ids, hipStream_t s, DevEval* copy) {
    const int grid = std::max(1, std::min(16, (max_vol + 1023) / 1024));
    hipLaunchKernelGGL(k_map_ids, dim3(grid), dim3(256), 0, s, evals, n, d_index, index, ids, copy);
    return hipGetLastError();
}

// ------------------------------------------------------------------ the map

typedef const __attribute__((address_space(4))) DevEval* CEval;

// Contribution of coordinate x of launch dim d (the same for all lanes; its fields are
// scalars, and every workgroup of the launch reads the same ones).
__device__ __forceinline__ int32_t coord_of(CEval e, int d, uint32_t x) {
    uint32_t v = 0;
    const int first = e->dim[d].first, nb = e->dim[d].nblk, nc = e->dim[d].ncyc;
    const double rl = e->dim[d].rl;
    for (int j = first; j < first + nb; ++j)
        v += block_index(x, (double)e->pj[j].s, rl) * (uint32_t)e->pj[j].stride;
    for (int j = first + nb; j < first + nb + nc; ++j)
        v += (x - div_wide((double)x, e->pj[j].rs) * (uint32_t)e->pj[j].s) * (uint32_t)e->pj[j].stride;
    return (int32_t)v;
}

template <int NT, int PIECES>
__global__ __launch_bounds__(NT) void k_map(const DevEval* __restrict__ evals, int64_t n,
                                            const int64_t* __restrict__ d_index, int64_t index,
                                            const int32_t* __restrict__ ids, int32_t* __restrict__ out,
                                            int32_t base_words) {
    extern __shared__ __attribute__((aligned(16))) int32_t lds[];  // row bases, then the owner table
    constexpr uint32_t kBlock = NT * PIECES * 4;                    // points
    int32_t* T = lds + base_words;
    const int tid = threadIdx.x;
    const int64_t ci = d_index ? wave_uniform64(*d_index) : index;
    if (ci < 0 || ci >= n) return;  // no candidate selected (empty batch)
    CEval e = (CEval)(evals + ci);
    const int32_t vol = e->vol;
    const int K = e->lrank;
    const int64_t points = e->points;
    ids += e->offset;
    if ((int64_t)blockIdx.x * kBlock >= points) return;  // the grid fits the batch's largest domain
    for (int32_t i = tid * 4; i < vol; i += NT * 4) *reinterpret_cast<i32x4v*>(T + i) = *reinterpret_cast<const i32x4v*>(ids + i);
    const uint32_t L = (uint32_t)e->dim[K - 1].l;
    const double rL = e->dim[K - 1].rl;
    const int64_t rows = points / L;
    const bool aligned = (reinterpret_cast<uintptr_t>(out) & 15) == 0;
    // the last dim's blocks, in floats while (cell x blocks) stays below 2^22 (div_small)
    const int nb = e->dim[K - 1].nblk;
    const uint32_t s = nb ? (uint32_t)e->pj[e->dim[K - 1].first].s : 1u;
    const int32_t st = nb ? e->pj[e->dim[K - 1].first].stride : 0;
    const bool simple = nb <= 1 && e->dim[K - 1].ncyc == 0 && L >= 4 * s && L < (1u << 22) / (s + 1);
    const float sf = (float)s, lf = (float)L, rlf = 1.0f / lf, rsf = 1.0f / sf;
    for (int64_t p0 = (int64_t)blockIdx.x * kBlock; p0 < points; p0 += (int64_t)gridDim.x * kBlock) {
        // the block's first row and cell (exact: p0 < 2^41, half a point from the integers)
        const int64_t row0 = (int64_t)(((double)p0 + 0.5) * rL);
        const uint32_t x0 = (uint32_t)(p0 - row0 * L);
        const uint32_t nrow = (uint32_t)(((uint64_t)x0 + kBlock + 2) / L) + 1;
        if (p0 != (int64_t)blockIdx.x * kBlock) lds_sync(NT / 64);  // the previous block's bases are no longer read
        for (uint32_t i = tid; i < nrow; i += NT) {
            int64_t r = row0 + i < rows ? row0 + i : rows - 1;
            int32_t b = 0;
            for (int d = K - 2; d >= 0; --d) {
                const int64_t q = (int64_t)(((double)r + 0.5) * e->dim[d].rl);
                b += coord_of(e, d, (uint32_t)(r - q * e->dim[d].l));
                r = q;
            }
            lds[i] = b;
        }
        lds_sync(NT / 64);  // table and bases ready
        int32_t* blk = out + p0;
        const int64_t left = points - p0;
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            const uint32_t j = (uint32_t)(tid + i * NT) * 4;
            if (j >= left) break;
            uint32_t o = x0 + j, rl;
            if (L > kBlock) {
                rl = o >= L ? 1u : 0u;
                o -= rl ? L : 0u;
            } else {
                rl = div_small(o, rlf);
                o -= __umul24(rl, L);
            }
            i32x4v id;
            if (simple) {
                const uint32_t a = (uint32_t)(fmaf((float)o, sf, 0.5f) * rlf);
                const uint32_t next = (uint32_t)(fmaf((float)a, lf, lf + sf - 0.5f) * rsf);  // first cell of block a + 1
                const uint32_t here = next - o;
                const int32_t v = lds[rl] + (int32_t)__umul24(a, (uint32_t)st);
                const int32_t t0 = T[v], t1 = T[a + 1 < s ? v + st : v];
                id.x = t0;
                id.y = here > 1 ? t0 : t1;
                id.z = here > 2 ? t0 : t1;
                id.w = here > 3 ? t0 : t1;
                if (o + 3 >= L) {  // the store goes on in the next row's first block
                    const int32_t t2 = T[lds[rl + 1]];
                    id.y = o + 1 >= L ? t2 : id.y;
                    id.z = o + 2 >= L ? t2 : id.z;
                    id.w = t2;
                }
            } else {
                for (int u = 0; u < 4; ++u) {
                    id[u] = T[lds[rl] + coord_of(e, K - 1, o)];
                    if (++o == L) {
                        o = 0;
                        ++rl;
                    }
                }
            }
            if (aligned && j + 4 <= left) {
                *reinterpret_cast<i32x4v*>(blk + j) = id;
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (j + u < left) blk[j + u] = id[u];
            }
        }
    }
}

MapShape map_shape(int32_t max_vol, int64_t max_points, int64_t min_row) {
    MapShape m;
    m.narrow = max_vol <= kMapNarrowVol;
    m.block = m.narrow ? kMapNarrowBlock : kMapWideBlock;
    m.grid = (int)std::max<int64_t>(1, std::min<int64_t>((max_points + m.block - 1) / m.block, kMapMaxGrid));
    m.base_words = (int32_t)((((m.block + 2 + min_row - 1) / min_row + 3) + 3) & ~int64_t(3));
    m.lds_words = m.base_words + ((max_vol + 3) & ~3);
    return m;
}

hipError_t launch_map(const MapShape& m, const DevEval* evals, int64_t n, const int64_t* d_index, int64_t index,
                      const int32_t* ids, int32_t* out, hipStream_t s) {
    const size_t lds = (size_t)m.lds_words * 4;
    if (m.narrow)
        hipLaunchKernelGGL((k_map<64, kMapNarrowBlock / 256>), dim3(m.grid), dim3(64), lds, s, evals, n, d_index, index,
                           ids, out, m.base_words);
    else
        hipLaunchKernelGGL((k_map<256, kMapWideBlock / 1024>), dim3(m.grid), dim3(256), lds, s, evals, n, d_index, index,
                           ids, out, m.base_words);
    return hipGetLastError();
}

}  // namespace tmk
