// attn_fwd_bf16_decode.hip -- bf16 attention forward for few query rows per kv
// head: decode steps and short verification chunks against a key cache.
//
// With a handful of query rows the work is reading K and V once, so the kernel
// is laid out for memory bandwidth instead of matrix rate:
//  * The query rows of all heads of a kv group share one row tile. Flat row f
//    of a kv group is query f / group of head f % group; a workgroup takes 32
//    consecutive flat rows, so K and V are read once for all the heads that
//    use them (the 32-row blocks of the prefill kernel would hold one valid
//    row per head, and groups of more than four heads would read K and V
//    several times).
//  * The keys of one row tile are split over the four wavefronts of a
//    workgroup (every fourth 32-key tile each) and over workgroups (split_tiles
//    tiles each, the grid's second axis), so that a few sequences still fill
//    the chip. The waves are merged through LDS; the workgroups leave partial
//    results (running max, row sums and O) in the caller's workspace and
//    attn_combine (attn_combine.hip) adds them up. Without a workspace a row
//    tile is not split over workgroups.
//  * Each wavefront streams its own tiles through LDS of its own with direct
//    loads, K of the next tile in flight during the softmax and P V of this
//    one, V during the next K Q^T: no workgroup barrier in the loop, 8 to 16
//    KiB in flight per wave and eight waves per CU.
// Bound by memory: one step of 32 sequences of 256..8192 cached tokens (8 kv
// heads, D = 128, 540 MB of K and V) takes 115 us (4.7 TB/s; a large copy moves
// 4.9) where the prefill kernel took 169; one sequence of 8192 tokens with 128
// query heads 14 us against 111 (it ran 32 workgroups).
// The products, their layouts and the LDS swizzle are those of the prefill
// kernel (bf16_kernel.h) with 32-key tiles; the running max is exact on every
// tile, and O is normalised by the sum of P as rounded to bf16. Closed-form
// masks and softmax only (the launcher's rule); score mods take the exact
// soft-cap form and the two-coefficient bias, as nothing here is bound by
// vector work.
#include "bf16_kernel.h"

namespace attn {
namespace {

constexpr int kRows = 32;  // flat rows per workgroup
constexpr int kBn = 32;    // keys per tile
constexpr int kWaves = 4;

template <int D, int CAP, int BIAS>
__global__ __launch_bounds__(NT, D == 64 ? 4 : 2) void attn_decode_bf16_kernel(AttnParams p)
{
    using T = Traits<D, kBn, CAP, BIAS, kNormSoftmax, false, true>;
    constexpr int ROWS_PER_KB = 1024 / T::ROWB;  // tile rows of one wave's direct load
    constexpr int LW = T::TILE / 1024;           // direct loads per wave and tile
    constexpr int QUADS = 4 * T::DBLK;           // 4-float pieces of a lane's O^T
    // Separate objects for K and V: reads of one must not wait for loads into
    // the other. After the loop they hold the waves' partial O.
    __shared__ __attribute__((aligned(1024))) char lds_k[kWaves * T::TILE];
    __shared__ __attribute__((aligned(1024))) char lds_v[kWaves * T::TILE];
    __shared__ __attribute__((aligned(16))) float ml[kWaves][kRows][4];

    const int tid = threadIdx.x;
    if constexpr (kLdsPoison) {
        for (int i = tid; i < kWaves * T::TILE / 4; i += NT) {
            reinterpret_cast<uint32_t*>(lds_k)[i] = ~0u;
            reinterpret_cast<uint32_t*>(lds_v)[i] = ~0u;
        }
        for (int i = tid; i < (int)(sizeof(ml) / 4); i += NT)
            (&ml[0][0][0])[i] = __builtin_bit_cast(float, ~0u);
        __syncthreads();
    }
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int li = lane & 31, lh = lane >> 5;

    // Work item: (key split, kv group, row tile). The row tiles of a group
    // follow one another and, when the groups are a multiple of eight, on one
    // XCD (ids are dealt round-robin over the 8 XCDs), so that they read its K
    // and V at the same time through one L2.
    const uint32_t ngroups = (uint32_t)(p.batch * p.hkv), nrt = (uint32_t)p.num_q_tiles;
    const uint32_t sp = blockIdx.y, id = blockIdx.x;
    uint32_t g, rt;
    if (ngroups % 8 == 0) {
        const uint32_t k = id >> 3;
        rt = k % nrt;
        g = (id & 7) + 8 * (k / nrt);
    } else {
        rt = id % nrt;
        g = id / nrt;
    }
    const int b = (int)fast_div(g, p.div_hkv), hkv = (int)g - b * p.hkv;
    int lq, lk;
    int64_t qrow0 = 0, krow0 = 0;
    if (p.cu_q) {
        qrow0 = p.cu_q[b];
        lq = p.cu_q[b + 1] - (int)qrow0;
        krow0 = p.cu_k[b];
        lk = p.cu_k[b + 1] - (int)krow0;
    } else {
        lq = p.seqlen_q;
        lk = p.seqlen_k;
    }
    const int f0 = (int)rt * kRows, nflat = lq * p.group;
    if (f0 >= nflat) return;  // whole workgroup
    const int f = min(f0 + li, nflat - 1);
    const bool row_ok = f0 + li < nflat;
    const int qi = (int)fast_div((uint32_t)f, p.div_group), hq = hkv * p.group + (f - qi * p.group);
    auto lse_row = [&](int head, int query) __attribute__((always_inline)) -> int64_t {
        return p.cu_q ? (int64_t)head * p.total_q + qrow0 + query : ((int64_t)b * p.hq + head) * lq + query;
    };

    // Key tiles of the row tile, and this split's share of them.
    const int q0 = (int)fast_div((uint32_t)f0, p.div_group);
    const int q1 = (int)fast_div((uint32_t)min(f0 + kRows, nflat) - 1u, p.div_group);
    const TilePlan gp = plan_tiles(p.band, q0, q1 - q0 + 1, lq, lk, kBn);
    int t_beg = gp.lo, t_end = gp.hi;
    bool partial = false;
    if (p.splits > 1) partial = split_share(p, (int)sp, splittable(p, lq, krow0, lk), t_beg, t_end);

    WaveState<T> ws;
    ws.lh = lh;
    ws.ip = qi + (lk - lq);
    ws.pfx = 0;
    ws.jlo = 1;
    ws.jhi = 0;
    if (row_ok) band_row(p.band, qi, lq, lk, &ws.jlo, &ws.jhi);
    ws.jref = ws.jlo;  // the row's first visible key
    ws.bias_abs = 0.0f;
    ws.bias_lin = 0.0f;
    if constexpr (BIAS != kBiasNone) {
        if (p.slopes) ws.bias_abs = -p.slopes[hq] * p.unit;
        if (p.relpos) ws.bias_lin = p.unit;
    }
    auto lse_shift = [&]() { return ws.bias_lin != 0.0f ? (float)(ws.ip - ws.jref) : 0.0f; };
    if (sp > 0 && t_beg >= t_end) {  // no tiles: an empty partial
        if (partial && !p.cu_q && wave == 0 && lh == 0 && row_ok)
            *reinterpret_cast<f32x4*>(p.ws_ml + (sp * p.part_stride + lse_row(hq, qi)) * 4) =
                f32x4{-__builtin_inff(), 0.0f, 0.0f, lse_shift()};
        return;
    }

    // Q fragment: lane holds its flat row, dims 16t + 8lh .. +7.
    {
        const __bf16* qrow = static_cast<const __bf16*>(p.q) + (int64_t)hq * p.sq_h + 8 * lh +
                             (p.cu_q ? qrow0 + qi : qi) * p.sq_s + (p.cu_q ? 0 : b * p.sq_b);
#pragma unroll
        for (int t = 0; t < T::KSTEPS; ++t) ws.qf[t] = *reinterpret_cast<const bf16x8*>(qrow + 16 * t);
    }
    lds_read_offsets<T>(ws, lane);

    // Direct loads: load i of a tile fills KiB i of the wave's 32-row buffer;
    // lane L writes its bytes 16L.., which hold (row, chunk) with chunk =
    // physical chunk ^ swizzle(row). Tiles past the end read as zero. A slice
    // of one row may have any row stride; the rows past it must not fold onto it.
    const __bf16* kbase = static_cast<const __bf16*>(p.k) + (int64_t)hkv * p.sk_h +
                          (p.cu_q ? krow0 * p.sk_s : b * p.sk_b);
    const __bf16* vbase = static_cast<const __bf16*>(p.v) + (int64_t)hkv * p.sv_h +
                          (p.cu_q ? krow0 * p.sv_s : b * p.sv_b);
    auto slice_bytes = [&](int64_t stride) {
        return lk <= 0 ? 0u : (uint32_t)((((int64_t)lk - 1) * stride + D) * 2);
    };
    const __amdgpu_buffer_rsrc_t krs = make_rsrc(kbase, slice_bytes(p.sk_s));
    const __amdgpu_buffer_rsrc_t vrs = make_rsrc(vbase, slice_bytes(p.sv_s));
    const uint32_t krow = (uint32_t)(lk > 1 ? p.sk_s * 2 : T::ROWB);
    const uint32_t vrow = (uint32_t)(lk > 1 ? p.sv_s * 2 : T::ROWB);
    const int lrow = 16 * lane / T::ROWB, lpc = (16 * lane % T::ROWB) / 16;
    char* kbuf = lds_k + wave * T::TILE;
    char* vbuf = lds_v + wave * T::TILE;
    auto issue = [&](char* buf, __amdgpu_buffer_rsrc_t rs, uint32_t row_bytes, int j0)
                     __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < LW; ++i) {
            const int r = ROWS_PER_KB * i + lrow;  // tile row
            const uint32_t off = (uint32_t)(j0 + r) * row_bytes + 16u * (lpc ^ chunk_swizzle<D>(r));
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)(buf + 1024 * i), 16, off, 0, 0, 0);
        }
    };

#pragma unroll
    for (int d = 0; d < T::DBLK; ++d) ws.oacc[d] = f32x16{};
    float m_run = -__builtin_inff(), l_run = 0.0f, l_o = 0.0f;  // sums: this lane's keys only

    int kt = t_beg + wave;
    issue(kbuf, krs, krow, kt < t_end ? kt * kBn : lk);
    issue(vbuf, vrs, vrow, kt < t_end ? kt * kBn : lk);
    while (kt < t_end) {
        // (not loop-invariant: the compiler would hold the distances of all of a
        // tile's keys from them in registers through the loop, 154 of them at D =
        // 64, which leaves room for three workgroups per CU: 942 groups of 2 heads
        // with ALiBi and one key 8.7 us, 6.9 with four)
        if constexpr (BIAS != kBiasNone) asm volatile("" : "+v"(ws.ip), "+v"(ws.jref));
        const int j0 = kt * kBn, nt = kt + kWaves;
        const int jn = nt < t_end ? nt * kBn : lk;  // past the last tile: rows of zeros
        __builtin_amdgcn_s_waitcnt(vmcnt_only(LW));  // K of this tile has landed (V may not)
        asm volatile("" ::: "memory");
        f32x16 s[1];
        qk_tile<T>(kbuf, ws, s);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // K is read: its buffer is free
        issue(kbuf, krs, krow, jn);

        const bool masked = !(kt >= gp.full_lo && kt < gp.full_hi);
        float mx = masked ? mods_and_max<T, true>(s, p, ws, j0) : mods_and_max<T, false>(s, p, ws, j0);
        // (without score mods s holds raw products and the max is in units)
        const float m_new = __builtin_fmaxf(m_run, mx);
        const float m_use = m_new == -__builtin_inff() ? 0.0f : m_new;
        if (__builtin_amdgcn_ballot_w64(m_new > m_run)) {
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);  // 0 when m_run = -inf
            m_run = m_new;
            l_run *= alpha;
            l_o *= alpha;
#pragma unroll
            for (int d = 0; d < T::DBLK; ++d)
#pragma unroll
                for (int e = 0; e < 16; ++e) ws.oacc[d][e] *= alpha;
        }
        u32x4 pw[1][2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float p0 = norm_value<T>(s[0][8 * u + 2 * q], m_use, p.scale_u);
                const float p1 = norm_value<T>(s[0][8 * u + 2 * q + 1], m_use, p.scale_u);
                pw[0][u][q] = pack_bf16(p0, p1);
                l_run += p0;
                l_run += p1;
                l_o = add_bf16_pair(pw[0][u][q], l_o);
            }
        __builtin_amdgcn_s_waitcnt(vmcnt_only(LW));  // V of this tile has landed (next K may not)
        asm volatile("" ::: "memory");
        pv_tile<T>(vbuf, pw, ws);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // V is read: its buffer is free
        issue(vbuf, vrs, vrow, jn);
        kt = nt;
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_only(0));  // no load may land in the partial results below

    // Merge the four waves: each scales its O to the common running max; wave w
    // adds up pieces w DBLK .. of all of them. A partial with m = -inf saw no
    // key and contributes zeros.
    {
        const float l = pair_sum(l_run), lo = pair_sum(l_o);
        if (lh == 0) *reinterpret_cast<f32x4*>(ml[wave][li]) = f32x4{m_run, l, lo, 0.0f};
    }
    __syncthreads();
    float m_tot = -__builtin_inff(), l_tot = 0.0f, lo_tot = 0.0f;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) m_tot = __builtin_fmaxf(m_tot, ml[k][li][0]);
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
        const float mk = ml[k][li][0];
        const float w = mk == -__builtin_inff() ? 0.0f : __builtin_amdgcn_exp2f(mk - m_tot);
        l_tot += w * ml[k][li][1];
        lo_tot += w * ml[k][li][2];
    }
    // piece i of a wave's partial O, 16 bytes per lane: the first half in its
    // K buffer, the second in its V buffer
    auto piece = [&](int w, int i) __attribute__((always_inline)) -> f32x4* {
        char* buf = i < QUADS / 2 ? lds_k : lds_v;
        return reinterpret_cast<f32x4*>(buf + w * T::TILE + (i % (QUADS / 2)) * 1024) + lane;
    };
    static_assert(QUADS / 2 * 1024 == T::TILE, "the partial O fills the wave's K and V buffers");
    {
        const float w = m_run == -__builtin_inff() ? 0.0f : __builtin_amdgcn_exp2f(m_run - m_tot);
#pragma unroll
        for (int i = 0; i < QUADS; ++i) {
            f32x4 x;
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = ws.oacc[i / 4][4 * (i % 4) + e] * w;
            *piece(wave, i) = x;
        }
    }
    __syncthreads();
    if (!row_ok) return;
    // element e of piece i is head dim 32 (i / 4) + 16 (i % 4 / 2) + 8 lh + 4 (i % 2) + e
    const float inv = l_tot > 0.0f && lo_tot > 0.0f ? 1.0f / lo_tot : 0.0f;
    __bf16* orow = static_cast<__bf16*>(p.o) + (int64_t)hq * p.so_h +
                   (p.cu_q ? qrow0 + qi : qi) * p.so_s + (p.cu_q ? 0 : b * p.so_b);
    const int64_t row = lse_row(hq, qi);
    int64_t part = 0, prt = 0;
    if (p.splits > 1) {
        part = part_index(p, row, krow0, hq, qi);
        prt = part + sp * p.part_stride;
    }
    float* prow = p.ws_o + prt * D;
#pragma unroll
    for (int i0 = 0; i0 < T::DBLK; i0 += 2) {
        const int i = wave * T::DBLK + i0;  // pieces i and i + 1 hold eight consecutive dims
        f32x4 x[2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
            x[h] = (*piece(0, i + h) + *piece(1, i + h)) + (*piece(2, i + h) + *piece(3, i + h));
        const int dim = 32 * (i / 4) + 16 * (i % 4 / 2) + 8 * lh;
        if (partial) {
            *reinterpret_cast<f32x4*>(prow + dim) = x[0];
            *reinterpret_cast<f32x4*>(prow + dim + 4) = x[1];
        } else {
            u32x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                o[e] = pack_bf16(x[e / 2][2 * (e % 2)] * inv, x[e / 2][2 * (e % 2) + 1] * inv);
            *reinterpret_cast<u32x4*>(orow + dim) = o;
        }
    }
    if (wave == 0 && lh == 0) {
        if (partial) *reinterpret_cast<f32x4*>(p.ws_ml + prt * 4) = f32x4{m_tot, l_tot, lo_tot, lse_shift()};
        if (p.splits > 1 && sp == 0) mark_row(p, row, partial, part, gp.hi - gp.lo);
        if (!partial && p.lse)
            p.lse[row] = l_tot > 0.0f ? (m_tot + __builtin_log2f(l_tot)) * kLn2 + lse_shift()
                                      : -__builtin_inff();
    }
}

template <int D, int CAP, int BIAS>
hipError_t launch(const AttnParams& p, hipStream_t stream)
{
    hipLaunchKernelGGL((attn_decode_bf16_kernel<D, CAP, BIAS>), dim3((unsigned)p.grid, (unsigned)p.splits), dim3(NT),
                       0, stream, p);
    return hipGetLastError();
}

template <int D>
hipError_t launch_d(const AttnParams& p, hipStream_t stream)
{
    const bool bias = p.slopes != nullptr || p.relpos != 0;
    if (p.softcap > 0.0f)
        return bias ? launch<D, kCapExact, kBiasGeneral>(p, stream)
                    : launch<D, kCapExact, kBiasNone>(p, stream);
    return bias ? launch<D, kCapOff, kBiasGeneral>(p, stream) : launch<D, kCapOff, kBiasNone>(p, stream);
}

}  // namespace

int decode_rows() { return kRows; }
int decode_keys() { return kBn; }

hipError_t launch_bf16_decode(const AttnParams& p, int head_dim, hipStream_t stream)
{
    return head_dim == 128 ? launch_d<128>(p, stream) : launch_d<64>(p, stream);
}

}  // namespace attn
