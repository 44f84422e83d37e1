// key_splits.h -- the share of a workgroup in a row tile whose keys are split,
// and where its partial results go (AttnParams: splits, split_tiles, ...).
#pragma once

#include "kernel_params.h"

namespace attn {
namespace {

// A packed sequence longer than the host was told is computed whole: the
// workspace has no room for its partial rows.
__device__ __forceinline__ bool splittable(const AttnParams& p, int lq, int64_t krow0, int lk)
{
    return !p.cu_q || (lq <= p.max_q && krow0 + lk <= p.total_k);
}

// Narrow the key tiles [lo, hi) of a row tile to those of split `sp`; true when
// the row tile is split. One with no more tiles than a split takes is left to
// the first split, which writes it as if nothing were split. The last split
// takes whatever is left, so every tile has its split.
__device__ __forceinline__ bool split_share(const AttnParams& p, int sp, bool can, int& lo, int& hi)
{
    if (!can || hi - lo <= p.split_tiles) {
        if (sp > 0) lo = hi;
        return false;
    }
    lo += sp * p.split_tiles;
    if (sp < p.splits - 1) hi = min(hi, lo + p.split_tiles);
    return true;
}

// Index of a query row's first partial result; those of its other splits are
// p.part_stride apart. `row`: the row's index in the LSE.
__device__ __forceinline__ int64_t part_index(const AttnParams& p, int64_t row, int64_t krow0, int hq,
                                              int qi)
{
    if (!p.cu_q) return row;
    return (int64_t)fast_div((uint32_t)krow0, p.div_part) * p.part_stride + (int64_t)hq * p.max_q + qi;
}

// What attn_combine is told about a row by its first split; `tiles` is the row
// tile's number of key tiles.
__device__ __forceinline__ void mark_row(const AttnParams& p, int64_t row, bool partial, int64_t part,
                                         int tiles)
{
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef int32_t i32x2 __attribute__((ext_vector_type(2)));
    if (p.cu_q) {
        const int n = partial ? min(p.splits, (tiles + p.split_tiles - 1) / p.split_tiles) : 0;
        *reinterpret_cast<i32x2*>(p.ws_mark + 2 * row) = i32x2{(int32_t)part, n};
    } else if (!partial)
        *reinterpret_cast<f32x4*>(p.ws_ml + 4 * row) = f32x4{0.0f, 0.0f, -1.0f, 0.0f};
}

}  // namespace
}  // namespace attn
