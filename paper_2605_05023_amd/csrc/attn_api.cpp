// attn_api.cpp -- C ABI of libattn.so: validation, planning and dispatch.
//
// Every check runs on the host before the first HIP call, so a rejected call
// has no side effect and the error paths are testable without a GPU. Only
// ATTN_FLAG_VALIDATE reads device memory (the cu_seqlens, segment and global
// position arrays, copied to the host) before the launch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <vector>

#include "../../include/attn.h"
#include "kernel_params.h"
#include "launch.h"
#include "row_vis.h"
#include "softcap_poly.h"

namespace {

// The most key splits of a row tile (attn_combine takes one per lane).
constexpr int64_t kMaxSplits = 64;
// Flat query rows (query heads of a kv group x queries) that the decode kernel
// may take: up to 64, and up to 128 while there are at most 256 kv groups.
constexpr int64_t kDecodeFlatRows = 64, kDecodeFlatRowsFew = 128, kDecodeFewGroups = 256;

bool aligned16(const void* ptr) { return (reinterpret_cast<uintptr_t>(ptr) & 15u) == 0; }

// Resolve one tensor's strides (0 = contiguous default) and check them.
// Returns ATTN_OK or an error code.
int resolve_strides(int varlen, int64_t heads, int64_t seqlen, int64_t d, int64_t elt_align,
                    int64_t in_b, int64_t in_h, int64_t in_s, int64_t* out_b, int64_t* out_h,
                    int64_t* out_s)
{
    int64_t b, h, s;
    if (varlen) {
        // [T, H, D]: token stride H*D, head stride D
        b = 0;
        h = in_h ? in_h : d;
        s = in_s ? in_s : heads * d;
    } else {
        // [B, H, S, D]
        s = in_s ? in_s : d;
        h = in_h ? in_h : seqlen * d;
        b = in_b ? in_b : heads * seqlen * d;
    }
    if (h < 0 || s < 0 || b < 0) return ATTN_ERR_BAD_SHAPE;
    if (s < d && seqlen > 1) return ATTN_ERR_BAD_SHAPE;  // rows would overlap
    if ((h % elt_align) || (s % elt_align) || (b % elt_align)) return ATTN_ERR_ALIGNMENT;
    *out_b = b;
    *out_h = h;
    *out_s = s;
    return ATTN_OK;
}

// The kernels address one (sequence, head) slice with 32-bit byte offsets.
bool slice_fits(int64_t rows, int64_t stride_s, int64_t d, int64_t elt_bytes, int64_t pad_rows)
{
    if (rows <= 0) return true;
    int64_t bytes = ((rows + pad_rows) * stride_s + d) * elt_bytes;
    return bytes < (int64_t(1) << 31);
}

// Do the D-element rows of an output with these sizes and strides stay
// disjoint? Ordered by stride, every dimension must step past the whole extent
// of the ones inside it (sufficient, and what every ordinary layout meets);
// dimensions of size one are ignored. Overlapping output rows would make the
// result depend on which workgroup writes last.
bool rows_disjoint(int64_t d, int n, const int64_t* size, const int64_t* stride)
{
    int64_t sz[3], st[3];
    int m = 0;
    for (int i = 0; i < n; ++i)
        if (size[i] > 1) {
            sz[m] = size[i];
            st[m] = stride[i];
            ++m;
        }
    for (int a = 0; a < m; ++a)  // insertion sort by stride
        for (int b = a; b > 0 && st[b] < st[b - 1]; --b) {
            int64_t t = st[b]; st[b] = st[b - 1]; st[b - 1] = t;
            t = sz[b]; sz[b] = sz[b - 1]; sz[b - 1] = t;
        }
    int64_t extent = d;  // elements covered by one row
    for (int a = 0; a < m; ++a) {
        if (st[a] < extent) return false;
        extent = st[a] * (sz[a] - 1) + extent;
    }
    return true;
}

// Host copy of a device int32 array, on `stream` (ATTN_FLAG_VALIDATE only).
bool fetch_i32(const int32_t* dev, int64_t n, hipStream_t stream, std::vector<int32_t>* out)
{
    out->assign((size_t)n, 0);
    if (n == 0) return true;
    if (hipMemcpyAsync(out->data(), dev, (size_t)n * sizeof(int32_t), hipMemcpyDeviceToHost,
                       stream) != hipSuccess)
        return false;
    return hipStreamSynchronize(stream) == hipSuccess;
}

bool strictly_increasing_nonneg(const std::vector<int32_t>& a)
{
    for (size_t i = 0; i < a.size(); ++i)
        if (a[i] < 0 || (i > 0 && a[i] <= a[i - 1])) return false;
    return true;
}

// ATTN_FLAG_VALIDATE: check the device-side preconditions on the host.
int validate_device_inputs(const attn_variant_desc& d, bool varlen, bool segments, bool glist)
{
    hipStream_t stream = static_cast<hipStream_t>(d.stream);
    std::vector<int32_t> a;
    if (varlen) {
        const int32_t* cus[2] = {d.cu_seqlens_q, d.cu_seqlens_k};
        const int64_t total[2] = {d.total_q, d.total_k};
        const int64_t maxlen[2] = {d.max_seqlen_q, d.max_seqlen_k};
        for (int t = 0; t < 2; ++t) {
            if (!fetch_i32(cus[t], (int64_t)d.batch + 1, stream, &a)) return ATTN_ERR_LAUNCH;
            if (a[0] != 0 || a[(size_t)d.batch] != total[t]) return ATTN_ERR_BAD_SHAPE;
            for (int32_t s = 0; s < d.batch; ++s) {
                const int64_t len = (int64_t)a[(size_t)s + 1] - a[(size_t)s];
                if (len < 0 || len > maxlen[t]) return ATTN_ERR_BAD_SHAPE;
            }
        }
    }
    // one array, or one per sequence (a stride apart)
    auto check_arrays = [&](const int32_t* base, int64_t n, int64_t stride) {
        const int64_t copies = stride > 0 ? d.batch : 1;
        for (int64_t s = 0; s < copies; ++s) {
            if (!fetch_i32(base + s * stride, n, stream, &a)) return ATTN_ERR_LAUNCH;
            if (!strictly_increasing_nonneg(a)) return ATTN_ERR_BAD_VARIANT;
        }
        return ATTN_OK;
    };
    int rc = ATTN_OK;
    if (segments) rc = check_arrays(d.segment_starts, d.num_segments, d.segment_stride);
    if (rc == ATTN_OK && glist) rc = check_arrays(d.global_tokens, d.num_global, d.global_stride);
    return rc;
}

// ATTN_FLAG_LOG: the kernel variant and launch plan of one call, on stderr
// (the variant follows the dispatch of launch_bf16 / launch_f32).
void log_plan(const attn_variant_desc& d, const AttnParams& p)
{
    static const char* masks[] = {"none", "causal", "sliding_window", "prefix_lm",
                                  "global_sliding_window", "share_question", "causal_blockwise"};
    static const char* norms[] = {"softmax", "relu", "sigmoid"};
    const bool closed = d.mask_kind >= ATTN_MASK_NONE && d.mask_kind <= ATTN_MASK_PREFIX_LM;
    const bool both = p.slopes && p.relpos;
    const char* path = p.decode ? "decode"
                       : p.gtok ? "general, listed global set"
                       : (d.norm_kind != ATTN_NORM_SOFTMAX || !closed || both) ? "general"
                       : p.band.wl >= 0 ? "closed-form band with a left bound"
                                        : "closed-form band, running max checked through the row sums";
    const char* cap = d.softcap <= 0.0f                          ? "off"
                      : d.softcap <= 256.0f && p.cap_zmax >= 0.0f ? "short form, polynomial where in range"
                      : d.softcap <= 256.0f                       ? "short form"
                                                                  : "exact";
    const char* order = p.map_mode == 1 ? "kv groups per XCD" : "natural";
    std::fprintf(stderr,
                 "attn_fwd: %s D=%d B=%d Hq=%d Hkv=%d %s mask=%s norm=%s alibi=%d relpos=%d "
                 "softcap=%g (%s) | %s kernel, grid %d, %d rows x %d heads per workgroup, "
                 "order %s, chunk %d%s, global-row items %d, key splits %d\n",
                 d.dtype == ATTN_BF16 ? "bf16" : "fp32", d.head_dim, d.batch, d.num_q_heads,
                 d.num_kv_heads, p.cu_q ? "varlen" : "fixed-length", masks[d.mask_kind],
                 norms[d.norm_kind], p.slopes != nullptr, p.relpos, (double)d.softcap, cap,
                 d.dtype == ATTN_BF16 ? path : "fp32", p.grid, p.wg_rows, p.hp, order, p.chunk,
                 p.compact ? ", packed grid" : "", p.glob_items, p.splits);
}

}  // namespace

static_assert(ATTN_MAX_SEGMENTS == kMaxGlobalList, "LDS staging of the listed global set");

extern "C" int attn_abi_version(void) { return ATTN_ABI_VERSION; }

extern "C" const char* attn_status_string(int status)
{
    switch (status) {
    case ATTN_OK: return "ok";
    case ATTN_ERR_NULL_PTR: return "a required pointer is NULL";
    case ATTN_ERR_BAD_SHAPE: return "non-positive or inconsistent sizes or strides";
    case ATTN_ERR_BAD_VARIANT: return "bad mask or norm kind, window, scale, soft-cap, prefix or segments";
    case ATTN_ERR_ALIGNMENT: return "pointer or stride not 16-byte aligned";
    case ATTN_ERR_UNSUPPORTED: return "head_dim, dtype or size outside the compiled set";
    case ATTN_ERR_ABI: return "attn_variant_desc.struct_size does not match the library";
    case ATTN_ERR_LAUNCH: return "the HIP kernel launch failed";
    default: return "unknown status";
    }
}

// The band (plan.h) of the closed-form mask kinds; for the global sliding
// window it is the window part.
static KeyBand band_of(const attn_variant_desc* d)
{
    KeyBand b = {-1, -1, 0};
    switch (d->mask_kind) {
    case ATTN_MASK_CAUSAL: b.wr = 0; break;
    case ATTN_MASK_PREFIX_LM:
        b.wr = 0;
        b.pl = d->prefix_len;
        break;
    case ATTN_MASK_SLIDING_WINDOW:
    case ATTN_MASK_GLOBAL_SLIDING_WINDOW:
        b.wl = d->window_left < 0 ? -1 : d->window_left;
        b.wr = d->window_right < 0 ? -1 : d->window_right;
        break;
    default: break;
    }
    return b;
}

static bool closed_form_mask(int kind)
{
    return kind == ATTN_MASK_NONE || kind == ATTN_MASK_CAUSAL ||
           kind == ATTN_MASK_SLIDING_WINDOW || kind == ATTN_MASK_PREFIX_LM;
}

static bool segment_mask(int kind)
{
    return kind == ATTN_MASK_SHARE_QUESTION || kind == ATTN_MASK_CAUSAL_BLOCKWISE;
}

static int check_variant(const attn_variant_desc* d)
{
    if (d->mask_kind < ATTN_MASK_NONE || d->mask_kind > ATTN_MASK_CAUSAL_BLOCKWISE)
        return ATTN_ERR_BAD_VARIANT;
    if ((d->mask_kind == ATTN_MASK_SLIDING_WINDOW ||
         d->mask_kind == ATTN_MASK_GLOBAL_SLIDING_WINDOW) &&
        (d->window_left < -1 || d->window_right < -1))
        return ATTN_ERR_BAD_VARIANT;
    if (d->mask_kind == ATTN_MASK_PREFIX_LM && d->prefix_len < 0) return ATTN_ERR_BAD_VARIANT;
    if (d->mask_kind == ATTN_MASK_GLOBAL_SLIDING_WINDOW && d->num_global < 0)
        return ATTN_ERR_BAD_VARIANT;
    if (segment_mask(d->mask_kind) &&
        (d->num_segments < 1 || d->num_segments > ATTN_MAX_SEGMENTS || d->query_start < 0))
        return ATTN_ERR_BAD_VARIANT;
    if (d->norm_kind < ATTN_NORM_SOFTMAX || d->norm_kind > ATTN_NORM_SIGMOID)
        return ATTN_ERR_BAD_VARIANT;
    if (d->relative_position != 0 && d->relative_position != 1) return ATTN_ERR_BAD_VARIANT;
    if (!std::isfinite(d->scale) || !(d->scale > 0.0f)) return ATTN_ERR_BAD_VARIANT;
    if (!std::isfinite(d->softcap) || d->softcap < 0.0f) return ATTN_ERR_BAD_VARIANT;
    // the kernels scale the dot product by 2 log2(e) scale / C: it must be finite
    if (d->softcap > 0.0f && !std::isfinite(d->scale / d->softcap * (float)(2.0 * 1.4426950408889634)))
        return ATTN_ERR_BAD_VARIANT;
    if (d->mask_kind == ATTN_MASK_GLOBAL_SLIDING_WINDOW && d->global_tokens &&
        d->num_global > ATTN_MAX_SEGMENTS)
        return ATTN_ERR_BAD_VARIANT;
    if (d->flags & ~(ATTN_FLAG_VALIDATE | ATTN_FLAG_LOG)) return ATTN_ERR_BAD_VARIANT;
    // per-sequence layouts: whole arrays a stride apart
    if (d->segment_stride < 0 || d->global_stride < 0) return ATTN_ERR_BAD_VARIANT;
    if (segment_mask(d->mask_kind) && d->segment_stride > 0 &&
        d->segment_stride < d->num_segments)
        return ATTN_ERR_BAD_VARIANT;
    if (d->mask_kind == ATTN_MASK_GLOBAL_SLIDING_WINDOW && d->global_tokens &&
        d->global_stride > 0 && d->global_stride < d->num_global)
        return ATTN_ERR_BAD_VARIANT;
    return ATTN_OK;
}

extern "C" int attn_plan_tiles(const attn_variant_desc* desc, int32_t q0, int32_t rows,
                               int32_t lq, int32_t lk, int32_t block_n, int32_t out[4])
{
    if (!desc || !out) return ATTN_ERR_NULL_PTR;
    if (desc->struct_size != sizeof(attn_variant_desc)) return ATTN_ERR_ABI;
    int rc = check_variant(desc);
    if (rc != ATTN_OK) return rc;
    if (!closed_form_mask(desc->mask_kind)) return ATTN_ERR_UNSUPPORTED;
    if (block_n <= 0 || lq < 0 || lk < 0 || rows < 0 || q0 < 0) return ATTN_ERR_BAD_SHAPE;
    TilePlan p = plan_tiles(band_of(desc), q0, rows, lq, lk, block_n);
    out[0] = p.lo;
    out[1] = p.full_lo;
    out[2] = p.full_hi;
    out[3] = p.hi;
    return ATTN_OK;
}

extern "C" int attn_row_range(const attn_variant_desc* desc, const int32_t* segment_starts,
                              int32_t i, int32_t lq, int32_t lk, int32_t out[3])
{
    if (!desc || !out) return ATTN_ERR_NULL_PTR;
    if (desc->struct_size != sizeof(attn_variant_desc)) return ATTN_ERR_ABI;
    int rc = check_variant(desc);
    if (rc != ATTN_OK) return rc;
    if (segment_mask(desc->mask_kind) && !segment_starts) return ATTN_ERR_NULL_PTR;
    // a listed global set is not a prefix plus a band
    if (desc->mask_kind == ATTN_MASK_GLOBAL_SLIDING_WINDOW && desc->global_tokens &&
        desc->num_global > 0)
        return ATTN_ERR_UNSUPPORTED;
    if (i < 0 || i >= lq || lk < 0) return ATTN_ERR_BAD_SHAPE;
    const int32_t* seg = segment_mask(desc->mask_kind) ? segment_starts : nullptr;
    const int32_t nseg = seg ? desc->num_segments : 0;
    RowVis r = row_visibility(desc->mask_kind, band_of(desc), desc->num_global, seg, nseg,
                              desc->query_start, i, lq, lk);
    out[0] = r.pfx;
    out[1] = r.jlo;
    out[2] = r.jhi;
    return ATTN_OK;
}

namespace {

// Sizes of a call derived from its descriptor.
struct CallShape {
    int64_t max_q, max_k;   // longest query and key length
    int64_t q_tiles, blocks;
    int hp, block_m;
};

// Check everything but the pointers and resolve the strides (p.s*_*).
int check_shape(const attn_variant_desc& d, AttnParams& p, CallShape* c)
{
    if (d.dtype != ATTN_BF16 && d.dtype != ATTN_FP32) return ATTN_ERR_UNSUPPORTED;
    if (d.head_dim != 64 && d.head_dim != 128) return ATTN_ERR_UNSUPPORTED;
    if (d.batch < 0 || d.num_q_heads <= 0 || d.num_kv_heads <= 0) return ATTN_ERR_BAD_SHAPE;
    if (d.num_q_heads % d.num_kv_heads != 0) return ATTN_ERR_BAD_SHAPE;
    int rc = check_variant(&d);
    if (rc != ATTN_OK) return rc;
    const int varlen = d.cu_seqlens_q != nullptr;
    if (varlen && !d.cu_seqlens_k) return ATTN_ERR_NULL_PTR;
    if (!varlen && d.cu_seqlens_k) return ATTN_ERR_BAD_SHAPE;
    int64_t max_q, max_k;
    if (varlen) {
        if (d.max_seqlen_q < 0 || d.max_seqlen_k < 0 || d.total_q < 0 || d.total_k < 0)
            return ATTN_ERR_BAD_SHAPE;
        if (d.total_q > INT32_MAX || d.total_k > INT32_MAX) return ATTN_ERR_UNSUPPORTED;
        max_q = d.max_seqlen_q;
        max_k = d.max_seqlen_k;
    } else {
        if (d.seqlen_q < 0 || d.seqlen_k < 0) return ATTN_ERR_BAD_SHAPE;
        max_q = d.seqlen_q;
        max_k = d.seqlen_k;
    }
    const int64_t elt = d.dtype == ATTN_BF16 ? 2 : 4;
    const int64_t align = 16 / elt;
    const int64_t D = d.head_dim;
    rc = resolve_strides(varlen, d.num_q_heads, max_q, D, align, d.stride_q_b, d.stride_q_h,
                         d.stride_q_s, &p.sq_b, &p.sq_h, &p.sq_s);
    if (rc == ATTN_OK)
        rc = resolve_strides(varlen, d.num_kv_heads, max_k, D, align, d.stride_k_b, d.stride_k_h,
                             d.stride_k_s, &p.sk_b, &p.sk_h, &p.sk_s);
    if (rc == ATTN_OK)
        rc = resolve_strides(varlen, d.num_kv_heads, max_k, D, align, d.stride_v_b, d.stride_v_h,
                             d.stride_v_s, &p.sv_b, &p.sv_h, &p.sv_s);
    if (rc == ATTN_OK)
        rc = resolve_strides(varlen, d.num_q_heads, max_q, D, align, d.stride_o_b, d.stride_o_h,
                             d.stride_o_s, &p.so_b, &p.so_h, &p.so_s);
    if (rc != ATTN_OK) return rc;
    // 32-bit offsets inside one slice, with one tile of padding past the end.
    if (!slice_fits(max_q, p.sq_s, D, elt, 128) || !slice_fits(max_k, p.sk_s, D, elt, 128) ||
        !slice_fits(max_k, p.sv_s, D, elt, 128) || !slice_fits(max_q, p.so_s, D, elt, 128))
        return ATTN_ERR_UNSUPPORTED;

    // bf16: the query heads of one kv group share a workgroup, up to four of
    // them (one 32-row block each), so every K/V tile in LDS serves all of
    // them and the workgroup's 128 (head, row) pairs span only 32 positions,
    // which leaves fewer partially visible tiles at the mask edges.
    const int group = d.num_q_heads / d.num_kv_heads;
    int hp = d.dtype != ATTN_BF16 ? 1 : group % 4 == 0 ? 4 : group % 2 == 0 ? 2 : 1;
    if (d.sched_heads_per_wg != 0) {  // tuning override: 1, 2 or 4 dividing the group
        const int h = d.sched_heads_per_wg;
        if ((h != 1 && h != 2 && h != 4) || group % h != 0 || (d.dtype != ATTN_BF16 && h != 1))
            return ATTN_ERR_BAD_VARIANT;
        hp = h;
    }
    if (d.sched_order < 0 || d.sched_order > 2) return ATTN_ERR_BAD_VARIANT;
    if (d.sched_order == 2 && ((int64_t)d.batch * d.num_kv_heads) % 8 != 0)
        return ATTN_ERR_BAD_VARIANT;
    if (d.sched_chunk < 0 || (d.sched_chunk > 0 && d.sched_order == 1))
        return ATTN_ERR_BAD_VARIANT;
    const int block_m = d.dtype == ATTN_BF16 ? attn::bf16_block_m() / hp : attn::f32_block_m();
    // a multiple of hp: the hp query tiles of one 128-row span are issued
    // together (their K/V reads then meet in the L2)
    const int64_t q_tiles = (max_q + hp * block_m - 1) / (hp * block_m) * hp;
    const int64_t blocks = q_tiles * (d.num_q_heads / hp) * (int64_t)d.batch;
    // (the fp32 kernel numbers its workgroups with 32 unsigned bits)
    if (blocks > (d.dtype == ATTN_BF16 ? (int64_t)INT32_MAX : (int64_t)UINT32_MAX))
        return ATTN_ERR_UNSUPPORTED;
    if (blocks > 0 && (int64_t)d.batch * d.num_q_heads > INT32_MAX) return ATTN_ERR_UNSUPPORTED;
    c->max_q = max_q;
    c->max_k = max_k;
    c->q_tiles = q_tiles;
    c->blocks = blocks;
    c->hp = hp;
    c->block_m = block_m;
    return ATTN_OK;
}

// The pointer checks of a call that has something to compute.
int check_pointers(const attn_variant_desc& d, const AttnParams& p, const CallShape& c, const void* q,
                   const void* k, const void* v, const void* out, const float* lse)
{
    const int64_t D = d.head_dim;
    const int varlen = d.cu_seqlens_q != nullptr;
    if (!q || !k || !v || !out) return ATTN_ERR_NULL_PTR;
    if (segment_mask(d.mask_kind) && !d.segment_starts) return ATTN_ERR_NULL_PTR;
    {
        // output rows must not overlap (input rows may)
        const int64_t osize[3] = {varlen ? d.total_q : (int64_t)d.batch, d.num_q_heads,
                                  varlen ? 1 : c.max_q};
        const int64_t ostride[3] = {varlen ? p.so_s : p.so_b, p.so_h, p.so_s};
        if (!rows_disjoint(D, 3, osize, ostride)) return ATTN_ERR_BAD_SHAPE;
    }
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out))
        return ATTN_ERR_ALIGNMENT;
    if ((reinterpret_cast<uintptr_t>(lse) & 3u) != 0) return ATTN_ERR_ALIGNMENT;

    return ATTN_OK;
}

// Keys that a row tile spanning `span` of max_q query positions can see, at
// most (rows of leading global positions, which see all of them, apart). With a
// left bound wl query i sees lq - i + wl keys at most, whatever the right one is.
int64_t max_keys(const AttnParams& p, int64_t max_q, int64_t max_k, int64_t span)
{
    if (p.band.wl < 0) return max_k;
    int64_t seen = (int64_t)p.band.wl + max_q;
    if (p.band.wr >= 0 && p.band.wr + span < max_q) seen = (int64_t)p.band.wl + p.band.wr + span;
    return seen < max_k ? seen : max_k;
}

// Key tiles of `bn` keys that `keys` consecutive keys can touch, at most: those
// of a window start anywhere in a tile.
int64_t key_tiles(int64_t keys, int64_t max_k, int64_t bn)
{
    return keys < max_k ? keys / bn + 2 : (keys + bn - 1) / bn;
}

// Does the decode kernel take the call rather than the prefill kernel, which
// would launch `blocks` workgroups? `units` row tiles of 32 flat rows against
// `keys` keys. Graph-timed on both over 1..128 queries, groups of 1..8 heads,
// 4..8192 kv groups and 16..3000 keys:
//  * One 64-key tile of the prefill kernel (up to 64 keys): the decode kernel's
//    merge of four waves costs 0.5-0.9 us (one head of 16..64 rows and keys 4.8
//    against 5.6 us) and with more row tiles than prefill workgroups up to twice
//    the time (1517 heads of 48 rows 18.5 against 37). It wins where the prefill
//    kernel launches twice the workgroups, most of them empty (172 groups of 8
//    heads x 1 query 12.1 against 4.6), and at D = 64 on large grids (6096
//    heads x 16 queries 44 against 28).
//  * Beyond, it wins where its row tiles leave no CU without one (16 groups of
//    100 rows and 200 keys 8.4 against 7.3, 64 groups of 128 rows and 6000 keys
//    110 against 68) or are no more than the prefill workgroups (128 groups of
//    4 x 32 rows and 4000 keys 102 against 85; 256 groups of 8 heads x 8 rows
//    and 1000 keys 100 against 28). With more row tiles it reads K and V more
//    often (227 heads of 128 rows and keys 8.1 against 17); where the groups of an XCD share
//    its L2, long key ranges still pay: 384 keys and more at D = 64, up to two
//    row tiles a CU (256 heads of 48 rows and 3000 keys 40 against 32), 2048 at
//    D = 128 while the prefill kernel fills half the CUs at most (128 heads of
//    128 rows and 3000 keys 48 against 44, 1024 keys 20 against 20; 256 heads
//    of 64 rows and 8192 keys 183 against 203).
//  * D = 128 and up to 192 keys on a full chip: one wave's tile each is too
//    little work for the merge (2048 heads of 32 rows and 128 keys 31 against
//    35) unless prefill workgroups stay empty.
bool decode_pays(int64_t D, int64_t keys, int64_t blocks, int64_t units, int64_t groups, int hp)
{
    if (keys <= 64) return (blocks > 256 && blocks >= 2 * units) ||
                           (D == 64 && blocks > 512 && blocks >= units);
    if (units <= 256) return true;
    if (units > blocks)
        return groups % 8 == 0 &&
               (D == 64 ? keys >= 384 && (units <= 512 || 2 * units <= 3 * blocks)
                        : keys >= 2048 && groups <= 128);
    return D == 64 || keys > 192 || blocks >= 2 * units || hp == 4;
}

int64_t workspace_need(const AttnParams& p, int64_t D)
{
    if (p.splits <= 1) return 0;
    return p.parts * (D + 4) * 4 + (p.cu_q ? p.ws_rows * 8 : 0);
}

// Largest workspace of a call that moves `io` bytes of inputs and outputs.
// Calls of even lengths need 35 MB at most (a split is made where there are
// fewer workgroups than CUs); an uneven packed batch with many query rows could
// ask for any amount, and coarser splits serve it nearly as well.
int64_t workspace_limit(int64_t io) { return io / 4 > (int64_t)64 << 20 ? io / 4 : (int64_t)64 << 20; }

// Split row tiles of up to max_tiles tiles of `bn` keys every `per` tiles, or
// more where the partial results would take more than `limit` bytes. (A packed
// batch without rows has nothing to combine.)
void set_splits(AttnParams& p, int64_t D, int64_t bn, int64_t max_tiles, int64_t per, int64_t limit)
{
    for (; p.ws_rows > 0 && per < max_tiles; per *= 2) {
        p.splits = (int32_t)((max_tiles + per - 1) / per);
        p.split_tiles = (int32_t)per;
        p.part_stride = p.ws_rows;
        p.parts = p.splits * p.ws_rows;
        if (p.cu_q) {
            const int64_t half = per * bn / 2;
            p.part_stride = (int64_t)p.hq * p.max_q;
            p.parts = p.total_k / half * p.part_stride;
            p.div_part = make_fastdiv((uint32_t)half);
        }
        if (p.parts > 0 && p.parts <= INT32_MAX && workspace_need(p, D) <= limit) return;
    }
    p.splits = 1;
    p.split_tiles = 1 << 30;
}

// Key splits of the decode kernel for `units` row tiles (of `groups` kv groups)
// of max_tiles key tiles at most and avg_tiles on average. Up to 512 keys stay
// whole (300 keys: 6.7 us whole, 9.0 split). Beyond, a split takes at least an
// eighth of the tiles, up to 512 keys (1000 keys, one sequence: 9.4 us in eight
// splits, 11.6 in two; 8192 keys: 13.7 us in splits of 512, 14.4 of 256, 16.1 of
// 1024). Sequences of one length share the chip evenly when there is one
// workgroup per CU; packed ones of uneven length are cut into eight times as
// many pieces, so that the longest do not outlast the rest (32 of 256..8192
// keys: 138 us with 256 pieces aimed at, 119 with 1024, 116 with 2048).
// The split is made when it saves more than it costs. Four tiles (a round of the
// waves) take a workgroup 0.78 us (D = 64: 0.6), all K and V together at least
// their bytes at 7 TB/s (half the CUs alone draw a tenth less), a workgroup's
// dispatch 4.5 ns (those of short rows' empty splits too), and the longest row
// tile of an uneven batch half its time beyond that; a split adds 2.5 us for its second launch and the partial
// rows at 2.5 TB/s. Over 444 split calls this chose the faster side but for 8 %
// at most; without it 143 of them were slower split (192 groups of 4 x 16 rows
// and 101..576 keys 23.1 us against 8.8 whole, 128 groups of 1000 keys 26.9
// against 22.9).
void split_decode(AttnParams& p, int64_t D, bool packed, int64_t groups, int64_t units,
                  int64_t max_tiles, int64_t avg_tiles, int64_t limit)
{
    if (max_tiles <= 16) return;
    const int64_t pieces = packed ? 2048 : 256;
    if (avg_tiles > max_tiles) avg_tiles = max_tiles;
    int64_t per = (units * avg_tiles + pieces - 1) / pieces;
    int64_t least = max_tiles / 8 < 16 ? max_tiles / 8 : 16;
    const int64_t floor_splits = (max_tiles + kMaxSplits - 1) / kMaxSplits;
    if (least < floor_splits) least = floor_splits;
    if (per < least) per = least;
    per = (per + 3) / 4 * 4;  // whole rounds of the four waves
    const int64_t splits = (max_tiles + per - 1) / per;
    if (splits <= 1) return;
    const double stream = (double)(groups * avg_tiles * attn::decode_keys()) * (double)D * 4.0 / 7e6;
    auto run = [&](int64_t tiles, int64_t cuts) {
        const double own = (double)((tiles + 3) / 4) * (D == 128 ? 0.78 : 0.6);
        const double all = cuts == 1 && units <= 128 ? 1.1 * stream : stream;
        const double dispatch = (double)(units * cuts) * 0.0045;
        return std::max({own, all, dispatch}) + (packed ? 0.5 * own : 0.0);
    };
    const int64_t usual = std::min(avg_tiles / per + 1, splits);
    const double cost = 2.5 + (double)(p.ws_rows * usual) * (double)(D + 4) * 8.0 / 2.5e6;
    if (run(max_tiles, 1) - run(per, splits) < cost) return;
    set_splits(p, D, attn::decode_keys(), max_tiles, per, limit);
}

// Key splits of the prefill and fp32 kernels for `items` workgroups with rows,
// max_tiles key tiles at most and avg_tiles on average, for calls whose
// workgroups do not fill the chip: pieces for one workgroup per CU, at least
// `least` tiles each. A workgroup alone on its CU takes tile_us per tile, so a
// split shortens the longest by saved us; against that stand the second launch
// and the writing and reading of the partial rows (about 2.5 TB/s), and it is
// made when it saves a third more than it costs. 32 heads of 256 queries and
// 8192 keys (64 workgroups): 115 us whole, 51 in 4 splits; 8 heads of 512
// queries, 4096 keys, D = 64: 44 and 19; 16 heads of 2048 causal rows (256
// workgroups): 37 whole, 50 in splits of 16 tiles. fp32, 8 heads, one query,
// 4000 keys: 142 and 26. The segments of an index mask are not known here: 17 of
// 106 share-question calls, whose rows see few of the keys, lost up to 20 % to
// their second launch, the others won up to 85 %; taking two or three even shares
// of the keys as what a row sees lost as many of either.
void split_underfilled(AttnParams& p, int64_t D, int64_t bn, int64_t items, int64_t max_tiles,
                       int64_t avg_tiles, int64_t least, double tile_us, int64_t limit)
{
    if (avg_tiles > max_tiles) avg_tiles = max_tiles;
    if (avg_tiles < 1) return;
    int64_t per = (items * avg_tiles + 255) / 256;
    const int64_t floor_splits = (max_tiles + kMaxSplits - 1) / kMaxSplits;
    if (per < floor_splits) per = floor_splits;
    per = (per + least - 1) / least * least;
    const int64_t splits = (max_tiles + per - 1) / per;
    if (splits <= 1) return;
    int64_t usual = avg_tiles / per + 1;  // splits of the usual row
    if (usual > splits) usual = splits;
    const double saved = (double)(max_tiles - per) * tile_us;
    const double cost = 5.0 + (double)(p.ws_rows * usual) * (double)(D + 4) * 8.0 / 2.5e6;
    if (saved < 1.33 * cost) return;
    set_splits(p, D, bn, max_tiles, per, limit);
}

// Everything the kernels take but the data pointers: schedule and score
// constants. Needs check_shape's results.
int plan_launch(const attn_variant_desc& d, AttnParams& p, const CallShape& c)
{
    const int varlen = d.cu_seqlens_q != nullptr;
    const int64_t D = d.head_dim, elt = d.dtype == ATTN_BF16 ? 2 : 4;
    const int64_t max_q = c.max_q, q_tiles = c.q_tiles, blocks = c.blocks;
    const int hp = c.hp, block_m = c.block_m, group = d.num_q_heads / d.num_kv_heads;
    p.slopes = d.alibi_slopes;
    p.cu_q = d.cu_seqlens_q;
    p.cu_k = d.cu_seqlens_k;
    p.batch = d.batch;
    p.hq = d.num_q_heads;
    p.hkv = d.num_kv_heads;
    p.group = group;
    p.hp = hp;
    p.hp_shift = hp == 4 ? 2 : hp == 2 ? 1 : 0;
    p.wg_rows = block_m;
    p.seqlen_q = d.seqlen_q;
    p.seqlen_k = d.seqlen_k;
    p.num_q_tiles = (int32_t)q_tiles;
    p.total_q = varlen ? d.total_q : 0;
    p.band = band_of(&d);
    p.mask_kind = d.mask_kind;
    p.num_global = d.num_global;
    p.seg = segment_mask(d.mask_kind) ? d.segment_starts : nullptr;
    p.num_seg = segment_mask(d.mask_kind) ? d.num_segments : 0;
    p.seg_stride = segment_mask(d.mask_kind) ? d.segment_stride : 0;
    p.query_start = d.query_start;
    p.norm = d.norm_kind;
    p.relpos = d.relative_position;
    // softmax runs in base 2; the other normalisations need natural scores
    p.unit = d.norm_kind == ATTN_NORM_SOFTMAX ? 1.4426950408889634f : 1.0f;
    p.scale = d.scale;
    p.scale_u = d.scale * p.unit;
    p.softcap = d.softcap;
    p.softcap_pre = d.softcap > 0.0f ? d.scale / d.softcap : 0.0f;
    p.softcap_pre2 = p.softcap_pre * (float)(2.0 * 1.4426950408889634);
    p.softcap_post_u = d.softcap * p.unit;
    {
        // Soft-cap as dot (b0 + z (b1 + z b2)), z = dot^2 (softcap_poly.h):
        // the widest tabulated range |y| <= R, y = (scale / C) dot, whose
        // error bound C' R rel stays within kCapPolyMaxErr; the polynomial
        // holds while dot^2 <= (R / s)^2.
        p.cap_zmax = -1.0f;  // no polynomial (kernels take the exact form)
        if (d.softcap > 0.0f) {
            const double sc = (double)d.scale / d.softcap, cu = (double)p.softcap_post_u;
            int f = 0;
            while (f + 1 < kCapPolyFitCount &&
                   cu * kCapPolyFits[f].r * kCapPolyFits[f].rel > kCapPolyMaxErr)
                ++f;
            const CapPolyFit& fit = kCapPolyFits[f];
            bool normal = cu * fit.r * fit.rel <= kCapPolyMaxErr;
            double sk = sc;
            for (int c = 0; c < 3; ++c) {
                p.cap_poly[c] = (float)(cu * sk * fit.a[c]);
                normal = normal && std::fabs(p.cap_poly[c]) >= 1.1754943508222875e-38;
                sk *= sc * sc;
            }
            const double zmax = (double)fit.r * fit.r / (sc * sc);
            if (normal) p.cap_zmax = zmax < 3.0e38 ? (float)zmax : 3.0e38f;
        }
    }
    // Longest tiles first: the last query tiles under causal-like masks, the
    // first ones when global rows (which see every key) sit at the start.
    p.q_order = d.mask_kind == ATTN_MASK_GLOBAL_SLIDING_WINDOW && d.num_global > 0 ? 1 : 0;
    // Keep each kv-head group on one XCD when the groups divide evenly. The
    // longest-first order over all groups balances best and is kept while
    // the K/V of all groups fill at most half of the 256 MB Infinity Cache;
    // beyond that (measured: 537 MB of K/V 1.39x and 254 MB 1.03x faster
    // chunked) the groups of an XCD are walked in chunks holding at least one
    // round of its workgroup slots (32 CUs x 2), so the live K/V stays cached.
    // Not for masks where a few query tiles of each group see many times the
    // keys of the rest (the global rows of the global sliding window, the
    // rows after the question of causal blockwise): a chunk's long tiles
    // would start only with their chunk and end after everything else
    // (measured unchunked at 268 MB of K/V: 1.25x and 1.03x faster).
    // Without a mask every query tile of a group reads all of its K/V at the
    // same pace, so the groups are chunked as soon as the K/V of all groups
    // an XCD holds exceed its 4 MB L2 (ALiBi + soft-cap, 8 x 16 heads of 4096
    // keys at D = 64: L2-fabric bytes 8.6x -> 1.13x the algorithmic ones,
    // 1.04x faster).
    p.map_mode = ((int64_t)d.batch * d.num_kv_heads) % 8 == 0 ? 1 : 0;
    if (d.sched_order != 0) p.map_mode = d.sched_order == 2 ? 1 : 0;
    if (d.sched_chunk > 0 && p.map_mode != 1) return ATTN_ERR_BAD_VARIANT;
    // Size of the packed grid of a bf16 variable-length batch walked one kv
    // group at a time per XCD (see below), or -1 where it cannot apply. An
    // XCD's groups hold at most ceil(hkv / 8) kv heads of any one sequence,
    // so their query tiles (128 / hp rows) number at most
    // ceil(hkv / 8) * total_q * hp / 128 + (groups per XCD).
    int64_t packed = -1;
    if (d.dtype == ATTN_BF16 && varlen && p.map_mode == 1) {
        const int64_t groups_per_xcd = ((int64_t)d.batch * d.num_kv_heads) / 8;
        const int64_t per_seq = (d.num_kv_heads + 7) / 8;
        packed = 8 * (per_seq * d.total_q * hp / 128 + groups_per_xcd) * (group / hp);
    }
    {
        const int64_t groups_per_xcd = ((int64_t)d.batch * d.num_kv_heads) / 8;
        const int64_t kv_tokens = varlen ? d.total_k : (int64_t)d.batch * d.seqlen_k;
        const int64_t kv_bytes = kv_tokens * d.num_kv_heads * D * elt * 2;
        const int64_t per_group = (int64_t)(p.group / hp) * q_tiles;  // workgroups of a kv group
        int64_t chunk = groups_per_xcd;
        const bool few_long = d.mask_kind == ATTN_MASK_GLOBAL_SLIDING_WINDOW ||
                              d.mask_kind == ATTN_MASK_CAUSAL_BLOCKWISE;
        const int64_t groups = (int64_t)d.batch * d.num_kv_heads;
        const bool l2_spill = d.mask_kind == ATTN_MASK_NONE && groups > 0 &&
                              kv_bytes / groups * groups_per_xcd > (int64_t)4 << 20;
        if ((kv_bytes > (int64_t)128 << 20 || l2_spill) && !few_long)
            chunk = (64 + per_group - 1) / per_group;
        // A packed batch whose padded grid would be mostly workgroups past
        // their sequence's end (lengths far below the longest) walks its
        // groups one at a time for the packed grid, whatever its K/V size:
        // each empty workgroup still costs a dispatch and a decode (511
        // sequences of 1-64 tokens beside one of 8192: 1.05M -> 22k
        // workgroups, 1.96x faster; uniform length mixes within 2 %).
        if (packed >= 0 && !few_long && 2 * packed < blocks) chunk = 1;
        if (chunk > groups_per_xcd) chunk = groups_per_xcd;
        p.chunk = (int32_t)(chunk > 0 ? chunk : 1);
    }
    if (d.sched_chunk > 0) {  // tuning override: kv groups per chunk
        const int64_t groups_per_xcd = ((int64_t)d.batch * d.num_kv_heads) / 8;
        if (d.sched_chunk > groups_per_xcd) return ATTN_ERR_BAD_VARIANT;
        p.chunk = d.sched_chunk;
    }
    // Divisors of the workgroup-id decode (all >= 1; blocks <= INT32_MAX
    // bounds every dividend).
    const int hsets = d.num_q_heads / hp, gsets = group / hp;
    p.div_bh = make_fastdiv((uint32_t)(d.batch * hsets));
    p.div_hq = make_fastdiv((uint32_t)hsets);
    p.div_group = make_fastdiv((uint32_t)gsets);
    p.div_hkv = make_fastdiv((uint32_t)d.num_kv_heads);
    p.div_chunk_items = p.div_chunk_full = p.div_chunk_last = make_fastdiv(1);
    p.last_chunk = 0;
    if (p.map_mode == 1) {
        const int64_t groups_per_xcd = ((int64_t)d.batch * d.num_kv_heads) / 8;
        const int64_t last = (groups_per_xcd + p.chunk - 1) / p.chunk - 1;
        const int64_t last_groups = groups_per_xcd - last * p.chunk;
        p.div_chunk_items = make_fastdiv((uint32_t)((int64_t)p.chunk * gsets * q_tiles));
        p.div_chunk_full = make_fastdiv((uint32_t)(p.chunk * gsets));
        p.div_chunk_last = make_fastdiv((uint32_t)(last_groups * gsets));
        p.last_chunk = (int32_t)last;
    }
    // bf16 variable-length batch walked one kv group at a time per XCD: a
    // packed grid of only the query spans each sequence has, when smaller.
    p.grid = (int32_t)(uint32_t)blocks;
    p.compact = 0;
    p.groups_per_xcd = 0;
    p.items_per_tile = gsets;
    if (packed >= 0 && p.chunk == 1 && packed < blocks) {
        p.compact = 1;
        p.groups_per_xcd = (int32_t)(((int64_t)d.batch * d.num_kv_heads) / 8);
        p.grid = (int32_t)packed;
    }
    const bool glist = d.mask_kind == ATTN_MASK_GLOBAL_SLIDING_WINDOW && d.global_tokens &&
                       d.num_global > 0;
    p.gtok = glist ? d.global_tokens : nullptr;
    p.gtok_stride = glist ? d.global_stride : 0;
    p.glob_items = 0;
    p.glob_chunks = 1;
    if (glist && d.dtype == ATTN_BF16) {
        p.glob_chunks = (int32_t)((d.num_global + block_m - 1) / block_m);
        const int64_t items = (int64_t)d.batch * hsets * p.glob_chunks;
        if ((int64_t)p.grid + items > INT32_MAX) return ATTN_ERR_UNSUPPORTED;
        p.glob_items = (int32_t)items;
        p.grid += p.glob_items;
    }
    // Third workgroup per CU for D = 64 (where compiled: no score mods, no left
    // bound) on long sequences and grids of about three rounds and more: 4 x 16
    // heads of 3000 causal rows 99 -> 90 us, 4096 165 -> 153, 2 x 16 x 8000
    // without a mask 555 -> 528 (36 shapes: 10 % faster to 1 % slower); below, its spills at start-up and the uneven
    // last round cost more (4 x 16 x 1000 18.6 against 20.2, 32 x 16 x 500 41.7
    // against 43.6, packed lengths of 100..3000 182 against 183).
    p.wide = D == 64 && p.grid >= 1500 && (varlen ? d.total_k / d.batch : d.seqlen_k) >= 2560;
    p.decode = 0;
    p.splits = 1;
    p.split_tiles = 1 << 30;
    p.ws_rows = varlen ? (int64_t)d.num_q_heads * d.total_q
                       : (int64_t)d.batch * d.num_q_heads * d.seqlen_q;
    p.max_q = (int32_t)max_q;
    p.total_k = varlen ? d.total_k : 0;
    const int64_t keys = varlen ? d.total_k : (int64_t)d.batch * d.seqlen_k;
    const int64_t limit = workspace_limit((p.ws_rows + keys * d.num_kv_heads) * 2 * D * elt);
    // Few query rows per kv head: the decode kernel (schedule overrides keep
    // the prefill kernel that they describe).
    const int64_t groups = (int64_t)d.batch * d.num_kv_heads;
    const int64_t flat = max_q * group, rt = (flat + attn::decode_rows() - 1) / attn::decode_rows();
    const bool scheduled = d.sched_heads_per_wg || d.sched_order || d.sched_chunk;
    const int64_t tile_keys = max_keys(p, max_q, c.max_k, max_q);
    if (d.dtype == ATTN_BF16 && d.norm_kind == ATTN_NORM_SOFTMAX && closed_form_mask(d.mask_kind) &&
        !scheduled && groups * rt <= (1 << 20) &&
        flat <= (groups <= kDecodeFewGroups ? kDecodeFlatRowsFew : kDecodeFlatRows) &&
        decode_pays(D, tile_keys, blocks, groups * rt, groups, hp)) {
        p.decode = 1;
        p.num_q_tiles = (int32_t)rt;
        p.div_group = make_fastdiv((uint32_t)group);
        const int64_t bn = attn::decode_keys();
        const int64_t avg_k = varlen ? d.total_k / d.batch : d.seqlen_k;
        split_decode(p, D, varlen, groups, groups * rt, key_tiles(tile_keys, c.max_k, bn),
                     (avg_k + bn - 1) / bn, limit);
        p.grid = (int32_t)(groups * rt);
    } else if (!scheduled && !p.gtok) {
        const bool bf16 = d.dtype == ATTN_BF16;
        const int64_t bn = bf16 ? attn::bf16_block_n() : attn::f32_block_n();
        const int64_t usual_q = varlen ? d.total_q / d.batch : d.seqlen_q;
        const int64_t usual_k = varlen ? d.total_k / d.batch : d.seqlen_k;
        const int64_t items =
            groups * (group / hp) * ((usual_q + block_m - 1) / block_m);
        const int64_t tiles = key_tiles(max_keys(p, max_q, c.max_k, block_m), c.max_k, bn);
        // causal-like masks: the average row sees usual_k - usual_q / 2 keys
        const int64_t seen = d.mask_kind == ATTN_MASK_NONE ? usual_k : usual_k - usual_q / 2;
        const double tile_us = (D == 128 ? 0.85 : 0.5) * (bf16 ? 1.0 : 1.2);
        split_underfilled(p, D, bn, items, tiles, (seen + bn - 1) / bn, bf16 ? 8 : 4, tile_us, limit);
    }
    return ATTN_OK;
}

}  // namespace

extern "C" int64_t attn_workspace_bytes(const attn_variant_desc* desc)
{
    if (!desc) return ATTN_ERR_NULL_PTR;
    if (desc->struct_size != sizeof(attn_variant_desc)) return ATTN_ERR_ABI;
    AttnParams p = {};
    CallShape c;
    int rc = check_shape(*desc, p, &c);
    if (rc == ATTN_OK && c.blocks == 0) return 0;
    if (rc == ATTN_OK) rc = plan_launch(*desc, p, c);
    return rc == ATTN_OK ? workspace_need(p, desc->head_dim) : rc;
}

extern "C" int attn_fwd(const void* q, const void* k, const void* v, void* out, float* lse,
                        const attn_variant_desc* desc)
{
    return attn_fwd_ws(q, k, v, out, lse, desc, nullptr, 0);
}

extern "C" int attn_fwd_ws(const void* q, const void* k, const void* v, void* out, float* lse,
                           const attn_variant_desc* desc, void* workspace, int64_t workspace_bytes)
{
    if (!desc) return ATTN_ERR_NULL_PTR;
    if (desc->struct_size != sizeof(attn_variant_desc)) return ATTN_ERR_ABI;
    const attn_variant_desc& d = *desc;
    AttnParams p = {};
    CallShape c;
    int rc = check_shape(d, p, &c);
    if (rc != ATTN_OK) return rc;
    if (c.blocks == 0) return ATTN_OK;  // nothing to compute
    rc = check_pointers(d, p, c, q, k, v, out, lse);
    if (rc == ATTN_OK && !aligned16(workspace)) rc = ATTN_ERR_ALIGNMENT;
    if (rc == ATTN_OK) rc = plan_launch(d, p, c);
    if (rc != ATTN_OK) return rc;
    p.q = q;
    p.k = k;
    p.v = v;
    p.o = out;
    p.lse = lse;
    const int64_t need = workspace_need(p, d.head_dim);
    // One workgroup per row tile without a workspace. The decode kernel still
    // gains on the prefill kernel then: 8 groups of 4 heads, one query and 8192
    // keys 111 -> 52 us, 8 heads of 600 keys 12.3 -> 8.5 (251 shapes: 0.10-0.77 of
    // its time).
    if (need > 0 && (!workspace || workspace_bytes < need)) {
        p.splits = 1;
        p.split_tiles = 1 << 30;
    } else if (need > 0) {
        p.ws_o = static_cast<float*>(workspace);
        p.ws_ml = p.ws_o + p.parts * d.head_dim;
        p.ws_mark = reinterpret_cast<int32_t*>(p.ws_ml + p.parts * 4);
    }
    if (d.flags & ATTN_FLAG_VALIDATE) {
        rc = validate_device_inputs(d, p.cu_q != nullptr, p.seg != nullptr, p.gtok != nullptr);
        if (rc != ATTN_OK) return rc;
    }
    hipStream_t stream = static_cast<hipStream_t>(d.stream);
    if (d.flags & ATTN_FLAG_LOG) log_plan(d, p);
    hipError_t err = p.decode                ? attn::launch_bf16_decode(p, d.head_dim, stream)
                     : d.dtype == ATTN_BF16 ? attn::launch_bf16(p, d.head_dim, stream)
                                            : attn::launch_f32(p, d.head_dim, stream);
    if (err == hipSuccess && p.splits > 1)
        err = attn::launch_combine(p, d.head_dim, d.dtype == ATTN_BF16, stream);
    if (err != hipSuccess && (d.flags & ATTN_FLAG_LOG))
        std::fprintf(stderr, "attn_fwd: launch failed: %s\n", hipGetErrorString(err));
    return err == hipSuccess ? ATTN_OK : ATTN_ERR_LAUNCH;
}
