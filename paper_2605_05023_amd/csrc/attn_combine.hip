// attn_combine.hip -- add up the partial results of query rows whose keys were
// split over workgroups (Eq. 1 restated over key ranges): with m the largest
// running max of a row's partials and w_s = 2^(m_s - m),
//   O = sum w_s O_s / sum w_s lo_s,  LSE = (m + log2 sum w_s l_s) ln 2,
// l the fp32 row sum and lo the sum that normalises O (ReLU and Sigmoid: O =
// sum O_s). A partial without keys has m = -inf and l = 0; where a row was not
// split its output is written (kernel_params.h says where the partials are and
// how that is told). One wavefront per row: it takes the rows' scalars one
// split per lane, then walks the splits' O in 16-byte pieces, D / 4 lanes side
// by side. Bound by the latency of its loads: 16 splits are in flight at a time.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernel_params.h"
#include "launch.h"
#include "score_mods.h"

namespace attn {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

constexpr int NT = 256;

template <int D, class OUT, bool PACKED>
__global__ __launch_bounds__(NT) void attn_combine_kernel(AttnParams p)
{
    constexpr int COLS = D / 4, PAR = 64 / COLS;  // pieces of a row, splits side by side
    constexpr int BATCH = 16 / PAR;               // loads in flight per lane
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * (NT / 64) + (threadIdx.x >> 6);
    if (row >= p.ws_rows) return;
    const int64_t per_head = PACKED ? p.total_q : p.seqlen_q;
    const int64_t bh = row / per_head, i = row - bh * per_head;
    const int64_t b = PACKED ? 0 : bh / p.hq, h = bh - b * p.hq;

    // Packed: most rows of an uneven batch are not split, so the row's mark comes
    // first (one more latency, where every row would read 16 pieces). A token of
    // no sequence keeps its output; the limits are for rows that no workgroup
    // computed, whose mark is not written.
    int64_t part = row;
    int n = p.splits;
    if constexpr (PACKED) {
        const i32x2 mark = *reinterpret_cast<const i32x2*>(p.ws_mark + 2 * row);
        const int first = p.cu_q[0], end = p.cu_q[p.batch];
        part = (uint32_t)mark[0];
        n = min(mark[1], p.splits);
        if (i < first || i >= end || n <= 0 || part + (n - 1) * p.part_stride >= p.parts) return;
    }
    // The O pieces of the first BATCH splits are requested beside the scalars
    // that weight them, so a row of few splits waits for memory once (a split
    // that saw no key of the row wrote no O: what is read there is not used).
    const int col = lane % COLS, par = lane / COLS;
    const float* src = p.ws_o + part * D + 4 * col;
    f32x4 x[BATCH];
    auto load = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int s = min(s0 + u * PAR + par, n - 1);
            x[u] = *reinterpret_cast<const f32x4*>(src + s * p.part_stride * D);
        }
    };
    // one split per lane (the launcher keeps them within a wavefront)
    const f32x4 sc = *reinterpret_cast<const f32x4*>(
        p.ws_ml + (part + min(lane, n - 1) * p.part_stride) * 4);
    load(0);
    const bool have = lane < n;
    const float m = have ? sc[0] : -__builtin_inff(), shift = sc[3];
    float l = have ? sc[1] : 0.0f, lo = have ? sc[2] : 0.0f;
    if (__shfl(lo, 0) < 0.0f) return;  // the row was not split and is written
    float m_tot = m;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) m_tot = __builtin_fmaxf(m_tot, __shfl_xor(m_tot, d));
    // (m = -inf with a NaN sum: every score was NaN, which must reach the output)
    // Partials without keys are left out; one whose weight is 0 by underflow is
    // not, so that an infinite O of it gives the NaN of the unsplit call.
    const bool empty = m == -__builtin_inff() && l == 0.0f;
    const float w = empty ? 0.0f : __builtin_amdgcn_exp2f(m - m_tot);
    const uint64_t used = __builtin_amdgcn_ballot_w64(!empty);
    l *= w;
    lo *= w;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        l += __shfl_xor(l, d);
        lo += __shfl_xor(lo, d);
    }
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int s0 = 0; s0 < n; s0 += BATCH * PAR) {
        if (s0 > 0) load(s0);
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int s = s0 + u * PAR + par;
            const float ws = __shfl(w, s & 63);
            if (s < n && (used >> (s & 63) & 1)) acc += x[u] * ws;
        }
    }
#pragma unroll
    for (int d = COLS; d < 64; d <<= 1)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], d);
    if (par == 0) {
        // ReLU, Sigmoid: the partials are shares of O (weight 1 each)
        const float inv = p.norm != kNormSoftmax ? 1.0f
                          : l > 0.0f && lo > 0.0f ? 1.0f / lo
                                                  : l != l ? l : 0.0f;
        OUT* dst = static_cast<OUT*>(p.o) + b * p.so_b + h * p.so_h + i * p.so_s + 4 * col;
        acc *= inv;
        if constexpr (sizeof(OUT) == 2) {
            bf16x4 y;
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = (__bf16)acc[e];
            *reinterpret_cast<bf16x4*>(dst) = y;
        } else {
            *reinterpret_cast<f32x4*>(dst) = acc;
        }
    }
    if (lane == 0 && p.lse && p.norm == kNormSoftmax)
        p.lse[row] = l > 0.0f ? (m_tot + __builtin_log2f(l)) * kLn2 + shift : -__builtin_inff();
}

template <int D, class OUT>
hipError_t launch(const AttnParams& p, hipStream_t stream)
{
    const int64_t blocks = (p.ws_rows + NT / 64 - 1) / (NT / 64);
    if (p.cu_q)
        hipLaunchKernelGGL((attn_combine_kernel<D, OUT, true>), dim3((unsigned)blocks), dim3(NT), 0, stream, p);
    else
        hipLaunchKernelGGL((attn_combine_kernel<D, OUT, false>), dim3((unsigned)blocks), dim3(NT), 0, stream, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_combine(const AttnParams& p, int head_dim, bool bf16, hipStream_t stream)
{
    if (bf16) return head_dim == 128 ? launch<128, __bf16>(p, stream) : launch<64, __bf16>(p, stream);
    return head_dim == 128 ? launch<128, float>(p, stream) : launch<64, float>(p, stream);
}

}  // namespace attn
