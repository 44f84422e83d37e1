// attn_fwd_f32.hip -- fused attention forward for fp32 inputs on gfx950.
//
// Both products run on the fp32 matrix instruction v_mfma_f32_32x32x2_f32:
// fp32 operands, products and sums, as vector FMAs would give, at the fp32
// matrix rate (157 TFLOP/s nominal; a large library product reaches 153 here),
// where vector FMAs without packed instructions stop at half of that and the
// LDS broadcasts that feed them at an eighth.
//
// A wavefront owns 32 query rows of one query head and walks key tiles of 32.
//  * Scores are computed transposed, S^T = K Q^T, so a lane owns one query row
//    (lane % 32) and 16 of the 32 keys: the row max and sum are per-lane
//    reductions and one exchange with lane ^ 32.
//  * The contraction order over the head dim is free, so lane half h takes the
//    dims 8c + 4h .. 8c + 4h + 3 of chunk c: one 16-byte load of K (global) and
//    one of Q (LDS, stored in this fragment order) feed four products.
//  * The accumulator of half h holds keys (r & 3) + 8 (r >> 2) + 4 h in
//    register r, which is the B operand of O^T = V^T P^T as it stands when the
//    A operand takes the same key: each half loads that key's V row.
//  * Row i of the 32-row block d of O^T is head dim (D / 32) i + d, so one
//    16-byte (D = 64: 8-byte) load of V feeds all blocks and an output row is
//    stored in 16-byte (8-byte) pieces.
//  * K and V go straight from memory to registers, each tile's K while the
//    previous tile's P V products run and its V while its own K Q^T products
//    run: the products of a tile take 64 D clocks of a SIMD, longer than the
//    loads, and nothing waits at a barrier.
// The four wavefronts of a workgroup take the same 32 rows and every fourth
// key tile each (wave w tiles lo + w, lo + w + 4, ...); their partial results
// (running max, sum and O per row) are merged through LDS. Bound by the matrix
// cores and, at up to a few thousand rows, by how evenly the rows' keys fill
// the chip, so the work items are kept small: 128-row workgroups (one 32-row
// block and all keys per wave) measured 4 % faster only for 2 x 16 heads of
// 4096 rows without a mask (2090 against 2184 us) and slower elsewhere (2 x 16
// causal heads of 1000 rows at D = 128: 1.4 times the time), and sum longer
// chains (relative error 1.3e-6 against 7.1e-7). The vector-FMA kernel before
// took 410 us (20 TFLOP/s) there, this one 91. The score modifications, the masks with tile skipping, the base-2 online softmax
// and the ReLU / Sigmoid normalisations are the same as in the bf16 kernel (Eq.
// 1 and 2 of Section 2.2, Appendix A). On the general mask path each lane
// derives its row's visible keys (row_vis.h) and the wave visits the tiles
// that some row of it sees.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "key_splits.h"
#include "kernel_params.h"
#include "launch.h"
#include "row_vis.h"
#include "score_mods.h"

namespace attn {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int NW = 4;      // wavefronts, each with a share of the key tiles
constexpr int NT = 64 * NW;
constexpr int BM = 32;     // query rows per workgroup (every wavefront the same ones)
constexpr int BN = 32;     // keys per tile

__device__ __forceinline__ int wave_min(int x)
{
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) x = min(x, __shfl_xor(x, o));
    return x;
}

__device__ __forceinline__ int wave_max(int x)
{
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) x = max(x, __shfl_xor(x, o));
    return x;
}

// Lanes l and l ^ 32 hold the two halves of the same query row.
__device__ __forceinline__ float pair_max(float x)
{
    auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x),
                                              __builtin_bit_cast(uint32_t, x), false, false);
    return __builtin_fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]),
                           __builtin_bit_cast(float, (uint32_t)r[1]));
}

__device__ __forceinline__ float pair_sum(float x)
{
    auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x),
                                              __builtin_bit_cast(uint32_t, x), false, false);
    return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}

// Buffer descriptor of one (sequence, head) slice: rows past its end read as zero.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t slice_rsrc(const float* base, int rows, int64_t stride,
                                                             int d)
{
    const uint32_t bytes = rows <= 0 ? 0u : (uint32_t)((((int64_t)rows - 1) * stride + d) * 4);
    // dword3 0x00020000: 32-bit untyped data format, no swizzle (gfx9 family)
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), (short)0, (int)bytes, 0x00020000);
}

// (the bounds keep two workgroups per CU at D = 128 and three at D = 64, where
// unseen_values below would otherwise take the registers of one)
template <int D, bool SOFTCAP, int BIAS, int NORM, bool GEN>
__global__ __launch_bounds__(NT, D == 64 ? 3 : 2) void attn_fwd_f32_kernel(AttnParams p)
{
    constexpr bool SOFTMAX = NORM == kNormSoftmax;
    constexpr bool MODS = SOFTCAP || BIAS != kBiasNone;
    constexpr int QC = D / 8;    // 16-byte chunks of Q and K per lane
    constexpr int DB = D / 32;   // 32-row blocks of O^T
    typedef float vrow_t __attribute__((ext_vector_type(DB)));
    // Q fragments [chunk][lane], then (after the key loop) the waves' partial O
    // [wave][register][lane]
    constexpr int WAVE_BYTES = BM * D * 4;
    __shared__ __attribute__((aligned(16))) char lds[NW * WAVE_BYTES];
    __shared__ float ml[NW][BM][2];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int li = lane & 31, lh = lane >> 5;
    if constexpr (kLdsPoison) {
        for (int i = tid; i < (int)(sizeof(lds) / 4); i += NT) reinterpret_cast<uint32_t*>(lds)[i] = ~0u;
        for (int i = tid; i < (int)(sizeof(ml) / 4); i += NT)
            (&ml[0][0][0])[i] = __builtin_bit_cast(float, ~0u);
        __syncthreads();
    }
    // Work item: (sequence, query head, query tile), longest tiles first. With
    // map_mode 1 the query heads of a kv group go to one XCD (ids are dealt
    // round-robin over the 8 XCDs) and read its K/V through one L2.
    int b, hq, qt;
    const uint32_t sp = blockIdx.z;  // key split
    {
        const uint32_t w = blockIdx.y * gridDim.x + blockIdx.x, nbh = (uint32_t)(p.batch * p.hq);
        if (w >= (uint32_t)p.grid) return;
        const int t = (int)(w / nbh), r = (int)(w - (uint32_t)t * nbh);
        if (p.map_mode == 1) {
            const int x = r & 7, k = r >> 3, gpx = (p.batch * p.hkv) >> 3;
            const int h = k / gpx, g = x + 8 * (k - h * gpx);  // head in group, kv group
            b = g / p.hkv;
            hq = (g - b * p.hkv) * p.group + h;
        } else {
            b = r / p.hq;
            hq = r - b * p.hq;
        }
        qt = p.q_order ? t : p.num_q_tiles - 1 - t;
    }

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
    const int q0 = qt * BM;
    if (q0 >= lq) return;  // whole workgroup
    const int hkv = hq / p.group;
    const float* qb = static_cast<const float*>(p.q);
    const float* kb = static_cast<const float*>(p.k);
    const float* vb = static_cast<const float*>(p.v);
    float* ob = static_cast<float*>(p.o);
    int64_t ooff;
    if (p.cu_q) {
        qb += qrow0 * p.sq_s + (int64_t)hq * p.sq_h;
        kb += krow0 * p.sk_s + (int64_t)hkv * p.sk_h;
        vb += krow0 * p.sv_s + (int64_t)hkv * p.sv_h;
        ooff = qrow0 * p.so_s + (int64_t)hq * p.so_h;
    } else {
        qb += (int64_t)b * p.sq_b + (int64_t)hq * p.sq_h;
        kb += (int64_t)b * p.sk_b + (int64_t)hkv * p.sk_h;
        vb += (int64_t)b * p.sv_b + (int64_t)hkv * p.sv_h;
        ooff = (int64_t)b * p.so_b + (int64_t)hq * p.so_h;
    }
    const int qi = q0 + li;

    // Visible keys of this lane's row, the key tiles this wave may visit, and
    // the tiles every row sees whole.
    const int32_t* gtok = p.gtok ? p.gtok + (int64_t)b * p.gtok_stride : nullptr;
    const int32_t* seg = p.seg ? p.seg + (int64_t)b * p.seg_stride : nullptr;
    RowVis rv = {0, 1, 0};
    int t_lo, t_hi;
    TilePlan gp = {0, 0, 0, 0};
    int pmin = 0, lomax = 0, himin = 0;  // GEN: bounds of the fully visible tiles
    if constexpr (GEN) {
        if (qi < lq)
            rv = gtok ? row_vis_listed(p.band, gtok, p.num_global, qi, lq, lk)
                      : row_visibility(p.mask_kind, p.band, p.num_global, seg, p.num_seg,
                                       p.query_start, qi, lq, lk);
        const bool band = rv.jlo <= rv.jhi, any = rv.pfx > 0 || band;
        const int first = any ? (rv.pfx > 0 ? 0 : rv.jlo) : 0x3fffffff;
        const int last = any ? (band ? rv.jhi : rv.pfx - 1) : -1;
        t_lo = __builtin_amdgcn_readfirstlane(wave_min(first)) / BN;
        t_hi = __builtin_amdgcn_readfirstlane(wave_max(last));
        t_hi = t_hi < 0 ? t_lo : t_hi / BN + 1;
        const bool row = qi < lq;  // rows past the end take no part
        pmin = __builtin_amdgcn_readfirstlane(wave_min(row ? rv.pfx : 0x3fffffff));
        lomax = __builtin_amdgcn_readfirstlane(wave_max(row ? (band ? rv.jlo : 0x3fffffff) : 0));
        himin = __builtin_amdgcn_readfirstlane(wave_min(row ? (band ? rv.jhi : -1) : 0x3fffffff));
    } else {
        if (qi < lq) band_row(p.band, qi, lq, lk, &rv.jlo, &rv.jhi);
        gp = plan_tiles(p.band, q0, BM, lq, lk, BN);
        t_lo = gp.lo;
        t_hi = gp.hi;
    }
    // This split's share of the tiles.
    const int64_t row = p.cu_q ? (int64_t)hq * p.total_q + qrow0 + qi
                               : ((int64_t)b * p.hq + hq) * lq + qi;  // index of its LSE
    bool partial = false;
    const int tiles = t_hi - t_lo;
    if (p.splits > 1) {
        partial = split_share(p, (int)sp, splittable(p, lq, krow0, lk), t_lo, t_hi);
        if (sp > 0 && t_lo >= t_hi) {  // no tiles: an empty partial
            if (partial && !p.cu_q && wave == 0 && lh == 0 && qi < lq)
                *reinterpret_cast<f32x4*>(p.ws_ml + (sp * p.part_stride + row) * 4) =
                    f32x4{-__builtin_inff(), 0.0f, 0.0f, 0.0f};
            return;
        }
    }
    auto full_tile = [&](int kt) __attribute__((always_inline)) -> bool {
        if constexpr (GEN) {
            const int j0 = kt * BN;
            return j0 + BN <= pmin || (lomax <= j0 && j0 + BN - 1 <= himin);
        }
        return kt >= gp.full_lo && kt < gp.full_hi;
    };
    // this wave's next tile, from kt on, that some row sees
    auto next_tile = [&](int kt) __attribute__((always_inline)) -> int {
        if constexpr (GEN) {
            while (kt < t_hi) {
                const int j0 = kt * BN;
                const bool hit = (rv.jlo <= rv.jhi && rv.jhi >= j0 && rv.jlo <= j0 + BN - 1) || j0 < rv.pfx;
                if (__builtin_amdgcn_ballot_w64(hit)) break;
                kt += NW;
            }
        }
        return kt;
    };

    // K and V rows: 32-bit byte offsets inside the slice. A slice of at most
    // one row may have any row stride; the rows past it must not fold onto it.
    const __amdgpu_buffer_rsrc_t krs = slice_rsrc(kb, lk, p.sk_s, D);
    const __amdgpu_buffer_rsrc_t vrs = slice_rsrc(vb, lk, p.sv_s, D);
    const uint32_t krow = (uint32_t)(lk > 1 ? p.sk_s * 4 : D * 4);
    const uint32_t vrow = (uint32_t)(lk > 1 ? p.sv_s * 4 : D * 4);
    f32x4 kf[QC];
    vrow_t vf[16];
    // 16-byte chunk c of this lane's K row at byte offset `off`; V row of the
    // key of accumulator register r at position key(i), i its index in the tile
    auto load_k = [&](uint32_t off, int c) __attribute__((always_inline)) {
        kf[c] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(krs, off + 32 * c, 0, 0));
    };
    auto load_v = [&](auto key, int r) __attribute__((always_inline)) {
        const uint32_t off = (uint32_t)key((r & 3) + 8 * (r >> 2) + 4 * lh) * vrow + DB * 4 * li;
        if constexpr (DB == 4)
            vf[r] = __builtin_bit_cast(vrow_t, __builtin_amdgcn_raw_buffer_load_b128(vrs, off, 0, 0));
        else
            vf[r] = __builtin_bit_cast(vrow_t, __builtin_amdgcn_raw_buffer_load_b64(vrs, off, 0, 0));
    };
    auto k_offset = [&](int key) __attribute__((always_inline)) -> uint32_t {
        return (uint32_t)key * krow + 16 * lh;
    };

    int kt = next_tile(t_lo + wave);
    if (kt < t_hi) {
        const uint32_t off = k_offset(kt * BN + li);
#pragma unroll
        for (int c = 0; c < QC; ++c) load_k(off, c);
    }

    // Q rows into LDS in fragment order, the four waves sharing the work; rows
    // past the end are zero.
    f32x4* qs = reinterpret_cast<f32x4*>(lds) + lane;
    {
        const __amdgpu_buffer_rsrc_t qrs = slice_rsrc(qb, lq, p.sq_s, D);
        const uint32_t off = qi < lq ? (uint32_t)((int64_t)qi * p.sq_s * 4) + 16 * lh : 0xffff0000u;
#pragma unroll
        for (int i = 0; i < QC / NW; ++i) {
            const int c = wave * (QC / NW) + i;
            qs[c * 64] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(qrs, off + 32 * c, 0, 0));
        }
    }

    const int ip = qi + (lk - lq);
    // relative-position reference (see score_u): first visible key for softmax
    int jref = SOFTMAX ? (rv.pfx > 0 ? 0 : rv.jlo) : ip;
    if (GEN && SOFTMAX && gtok) {  // the smallest visible key may be one of G
        int jr = rv.jlo <= rv.jhi ? rv.jlo : 0x7fffffff;
        if (p.num_global > 0 && gtok[0] < lk) jr = min(jr, gtok[0]);
        jref = jr == 0x7fffffff ? 0 : jr;
    }
    float bias_abs = 0.0f, bias_lin = 0.0f;
    if constexpr (BIAS == kBiasAlibi || BIAS == kBiasGeneral)
        if (p.slopes) bias_abs = -p.slopes[hq] * p.unit;
    if constexpr (BIAS == kBiasRelPos || BIAS == kBiasGeneral)
        if (p.relpos) bias_lin = p.unit;
    f32x16 o[DB];
#pragma unroll
    for (int d = 0; d < DB; ++d) o[d] = f32x16{};
    float m_run = -__builtin_inff(), l_run = 0.0f;  // l: this lane's keys only
    __syncthreads();

    // S^T = K Q^T of the tile in kf, loading the tile's V rows: half of them
    // ahead of the products, the others as the K chunks are used up, which
    // keeps the registers of both within two wavefronts per SIMD.
    auto scores = [&](auto key) __attribute__((always_inline)) -> f32x16 {
        f32x16 s = {};
#pragma unroll
        for (int r = 0; r < 8; ++r) load_v(key, r);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < QC; ++c) {
            const f32x4 q = qs[c * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[c][e], q[e], s, 0, 0, 0);
            if (c < 8) load_v(key, 8 + c);
            __builtin_amdgcn_sched_barrier(0);
        }
        return s;
    };
    // Score mods and mask. The key of register r sits at position jpos(i) and is
    // visible iff vis(i), i its index in the tile.
    auto modify = [&](f32x16& s, auto jpos, auto vis) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int i = (r & 3) + 8 * (r >> 2) + 4 * lh;
            float x = MODS ? score_u<SOFTCAP, BIAS>(s[r], p.scale_u, p.softcap_pre, p.softcap_post_u,
                                                    bias_abs, bias_lin, ip, jref, jpos(i))
                           : s[r] * p.scale_u;
            if (!vis(i)) x = -__builtin_inff();
            s[r] = x;
        }
    };
    // Online softmax (or activation): scores to P.
    auto normalise = [&](f32x16& s) __attribute__((always_inline)) {
        if constexpr (SOFTMAX) {
            float mx = s[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) mx = __builtin_fmaxf(mx, s[r]);
            // A row that has seen no key yet (m_run = -inf) and sees none of
            // this tile either keeps m = -inf with O and l at 0: the
            // exponentials take 0 in place of the max, where
            // exp2(-inf - (-inf)) would be NaN.
            const float m_new = __builtin_fmaxf(m_run, pair_max(mx));
            const float m_use = m_new == -__builtin_inff() ? 0.0f : m_new;
            if (__builtin_amdgcn_ballot_w64(m_new > m_run)) {
                const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);  // 0 when m_run = -inf
                m_run = m_new;
                l_run *= alpha;
#pragma unroll
                for (int d = 0; d < DB; ++d)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[d][r] *= alpha;
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                s[r] = __builtin_amdgcn_exp2f(s[r] - m_use);
                l_run += s[r];
            }
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = activation<NORM>(s[r]);  // the 1/L comes at the end
        }
    };
    // O^T += V^T P^T of the tile in vf, loading the next tile's K (`koff`: its
    // rows' byte offset; past the slice's end the loads return zeros) likewise.
    auto accumulate = [&](const f32x16& pr, uint32_t koff) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < QC / 2; ++c) load_k(koff, c);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
#pragma unroll
            for (int d = 0; d < DB; ++d)
                o[d] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[r][d], pr[r], o[d], 0, 0, 0);
            if (r < QC / 2) load_k(koff, QC / 2 + r);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // A key that a row does not see has P = 0, which an infinite or NaN value
    // would turn into NaN: where the tile in vf holds such values they are set
    // to zero, and the rows that see them get them here, one key at a time
    // (P = 0 times infinity stays NaN). Only partly visible tiles are checked
    // (every row sees the others whole), 64 multiplies beside 8192 clocks of
    // products: 2 x 16 causal heads of 1000 rows take 91 us with it, 92 without.
    auto unseen_values = [&](const f32x16& pr, auto key, auto vis) __attribute__((always_inline)) {
        auto finite = [](float x) { return __builtin_fabsf(x) < __builtin_inff(); };
        vrow_t z = {};
#pragma unroll
        for (int r = 0; r < 16; ++r) z += vf[r] * 0.0f;
        bool odd = false;
#pragma unroll
        for (int d = 0; d < DB; ++d) odd = odd || z[d] != z[d];
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(odd) == 0, 1)) return;
        uint32_t seen = 0, zero = 0;  // bit i: the row sees key i of the tile, and P = 0 there
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int i = (r & 3) + 8 * (r >> 2);
            const bool v = vis(i + 4 * lh);
            seen |= (uint32_t)v << i;
            zero |= (uint32_t)(v && pr[r] == 0.0f) << i;
#pragma unroll
            for (int d = 0; d < DB; ++d) vf[r][d] = finite(vf[r][d]) ? vf[r][d] : 0.0f;
        }
        seen <<= 4 * lh;
        zero <<= 4 * lh;
        seen |= __shfl_xor(seen, 32);
        zero |= __shfl_xor(zero, 32);
#pragma unroll 1
        for (int i = 0; i < BN; ++i) {
            const bool has = seen >> i & 1, nil = zero >> i & 1;
            const uint32_t off = (uint32_t)key(i) * vrow + DB * 16 * lh;
#pragma unroll
            for (int r = 0; r < 16; ++r) {  // O^T's rows of this lane: head dims DB (..) + d
                const uint32_t at = off + DB * 4 * ((r & 3) + 8 * (r >> 2));
                vrow_t x;
                if constexpr (DB == 4)
                    x = __builtin_bit_cast(vrow_t, __builtin_amdgcn_raw_buffer_load_b128(vrs, at, 0, 0));
                else
                    x = __builtin_bit_cast(vrow_t, __builtin_amdgcn_raw_buffer_load_b64(vrs, at, 0, 0));
#pragma unroll
                for (int d = 0; d < DB; ++d)
                    if (has && !finite(x[d])) o[d][r] += nil ? __builtin_nanf("") : x[d];
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    constexpr uint32_t kPastEnd = 0xffff0000u;  // beyond every slice (all are below 2 GiB)

    while (kt < t_hi) {
        const int j0 = kt * BN, nt = next_tile(kt + NW);
        auto pos = [&](int i) { return j0 + i; };
        auto vis = [&](int i) { return row_sees(rv, j0 + i); };
        f32x16 s = scores(pos);
        const bool full = full_tile(kt);
        if (full)
            modify(s, pos, [](int) { return true; });
        else
            modify(s, pos, vis);
        normalise(s);
        if (!full) unseen_values(s, pos, vis);
        __builtin_amdgcn_sched_barrier(0);
        accumulate(s, nt < t_hi ? k_offset(nt * BN + li) : kPastEnd);
        kt = nt;
    }
    // A listed global set (global sliding window): its keys outside the row's
    // band, BN list entries per tile, the waves taking turns.
    if (GEN && gtok) {
        const int ng = p.num_global;
        for (int g0 = wave * BN; g0 < ng; g0 += NW * BN) {
            auto key = [&](int i) { return g0 + i < ng ? min(gtok[g0 + i], lk) : lk; };
            const uint32_t off = k_offset(key(li));
#pragma unroll
            for (int c = 0; c < QC; ++c) load_k(off, c);
            f32x16 s = scores(key);
            auto vis = [&](int i) {
                const int kj = key(i);
                return qi < lq && kj < lk && !(kj >= rv.jlo && kj <= rv.jhi);
            };
            modify(s, key, vis);
            normalise(s);
            unseen_values(s, key, vis);
            accumulate(s, kPastEnd);
        }
    }

    // Merge the four partial results: every wave scales its O to the common
    // running max, and wave w adds up registers 4w .. 4w + 3 of all of them. A
    // partial with m = -inf saw no key and contributes zeros.
    float l_tot = pair_sum(l_run), m_tot = -__builtin_inff();
    vrow_t* part = reinterpret_cast<vrow_t*>(lds) + lane;
    if constexpr (SOFTMAX) {
        if (lh == 0) {
            ml[wave][li][0] = m_run;
            ml[wave][li][1] = l_tot;
        }
    }
    __syncthreads();  // also: every wave is done with Q
    float w = 1.0f;
    if constexpr (SOFTMAX) {
#pragma unroll
        for (int k = 0; k < NW; ++k) m_tot = __builtin_fmaxf(m_tot, ml[k][li][0]);
        l_tot = 0.0f;
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const float mk = ml[k][li][0];
            // (a NaN sum beside m = -inf, every score NaN, must reach l_tot)
            l_tot += ml[k][li][1] * (mk == -__builtin_inff() ? 0.0f : __builtin_amdgcn_exp2f(mk - m_tot));
        }
        w = m_run == -__builtin_inff() ? 0.0f : __builtin_amdgcn_exp2f(m_run - m_tot);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        vrow_t x;
#pragma unroll
        for (int d = 0; d < DB; ++d) x[d] = o[d][r] * w;
        part[(wave * 16 + r) * 64] = x;
    }
    __syncthreads();
    if (qi >= lq) return;
    float inv;
    if constexpr (SOFTMAX)
        inv = l_tot > 0.0f ? 1.0f / l_tot : 0.0f;
    else
        inv = lk > 0 ? 1.0f / (float)lk : 0.0f;
    float* dst = ob + ooff + (int64_t)qi * p.so_s + DB * (8 * wave + 4 * lh);
    const int64_t first = part_index(p, row, krow0, hq, qi), prt = first + sp * p.part_stride;
    if (partial) {  // unnormalised O (ReLU, Sigmoid: the share of O)
        dst = p.ws_o + prt * D + DB * (8 * wave + 4 * lh);
        if (SOFTMAX) inv = 1.0f;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {  // register 4 wave + e: row 8 wave + 4 lh + e of each block
        const int r = 4 * wave + e;
        const vrow_t x = (part[r * 64] + part[(16 + r) * 64]) + (part[(32 + r) * 64] + part[(48 + r) * 64]);
        *reinterpret_cast<vrow_t*>(dst + DB * e) = x * inv;
    }
    if (p.splits > 1 && wave == 0 && lh == 0) {
        if (partial)
            *reinterpret_cast<f32x4*>(p.ws_ml + prt * 4) =
                SOFTMAX ? f32x4{m_tot, l_tot, l_tot, bias_lin != 0.0f ? (float)(ip - jref) : 0.0f}
                        : f32x4{0.0f, 1.0f, 1.0f, 0.0f};
        if (sp == 0) mark_row(p, row, partial, first, tiles);
    }
    if (SOFTMAX && !partial && p.lse && wave == 0 && lh == 0) {
        float lse = -__builtin_inff();
        if (l_tot > 0.0f) {
            lse = (m_tot + __builtin_log2f(l_tot)) * kLn2;
            if (bias_lin != 0.0f) lse += (float)(ip - jref);
        }
        p.lse[row] = lse;
    }
}

template <int D, bool SOFTCAP, int BIAS, int NORM, bool GEN>
hipError_t launch(const AttnParams& p, hipStream_t stream)
{
    // rows of 2^22 workgroups: a grid dimension holds less than 2^32 threads
    const uint32_t blocks = (uint32_t)p.grid, gx = blocks < (1u << 22) ? blocks : 1u << 22;
    hipLaunchKernelGGL((attn_fwd_f32_kernel<D, SOFTCAP, BIAS, NORM, GEN>),
                       dim3(gx, (blocks - 1) / gx + 1, (unsigned)p.splits), dim3(NT), 0, stream, p);
    return hipGetLastError();
}

template <int D, bool SOFTCAP>
hipError_t launch_d(const AttnParams& p, hipStream_t stream)
{
    const bool closed = p.mask_kind >= 0 && p.mask_kind <= 3;  // band masks of plan.h
    const bool al = p.slopes != nullptr, rp = p.relpos != 0;
    if (p.norm == kNormSoftmax && closed && !(al && rp)) {
        if (al) return launch<D, SOFTCAP, kBiasAlibi, kNormSoftmax, false>(p, stream);
        if (rp) return launch<D, SOFTCAP, kBiasRelPos, kNormSoftmax, false>(p, stream);
        return launch<D, SOFTCAP, kBiasNone, kNormSoftmax, false>(p, stream);
    }
    const bool bias = al || rp;
    if (p.norm == kNormRelu)
        return bias ? launch<D, SOFTCAP, kBiasGeneral, kNormRelu, true>(p, stream)
                    : launch<D, SOFTCAP, kBiasNone, kNormRelu, true>(p, stream);
    if (p.norm == kNormSigmoid)
        return bias ? launch<D, SOFTCAP, kBiasGeneral, kNormSigmoid, true>(p, stream)
                    : launch<D, SOFTCAP, kBiasNone, kNormSigmoid, true>(p, stream);
    return bias ? launch<D, SOFTCAP, kBiasGeneral, kNormSoftmax, true>(p, stream)
                : launch<D, SOFTCAP, kBiasNone, kNormSoftmax, true>(p, stream);
}

}  // namespace

int f32_block_m() { return BM; }
int f32_block_n() { return BN; }

hipError_t launch_f32(const AttnParams& p, int head_dim, hipStream_t stream)
{
    const bool sc = p.softcap > 0.0f;
    if (head_dim == 128) return sc ? launch_d<128, true>(p, stream) : launch_d<128, false>(p, stream);
    return sc ? launch_d<64, true>(p, stream) : launch_d<64, false>(p, stream);
}

}  // namespace attn
