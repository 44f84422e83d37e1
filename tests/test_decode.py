"""The decode kernel (few query rows per kv head) and its key splits.

The row tile holds 32 flat rows (query heads of a kv group x queries), the
waves take every fourth 32-key tile, and longer key ranges are split over
workgroups when a workspace is given, so the cases sit around 32 flat rows,
32 and 128 keys, and one and several splits with a ragged last one. Each runs
with the workspace that `fwd` allocates and without one (attn_fwd); both are
compared with the fp64 oracle, element by element at the bars of the other
parity tests and row by row against the row's own norm, and with each other at
twice the rounding of bf16 outputs. The launch plan must name the decode kernel
for the cases of more than 64 keys, and for the last ones, whose few keys stand
against many row tiles; those with keys for more than one split must have a
workspace.
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2605_05023_amd as attn
from gpu_util import LSE_TOL, O_TOL, ROW_TOL, gpu_available, log, row_error
from paper_2605_05023_amd import _abi
from paper_2605_05023_amd.build import LIB_POISON
from paper_2605_05023_amd.workloads import (MASK_CAUSAL, MASK_NAMES, MASK_NONE, MASK_PREFIX_LM,
                                            MASK_SLIDING_WINDOW, alibi_slopes)

# (D, group, hkv, [(lq, lk)] (packed when they differ), mask, options)
CASES = [
    (128, 1, 1, [(1, 1)], MASK_NONE, {}),
    (64, 8, 2, [(1, 31)] * 2, MASK_CAUSAL, {}),
    (128, 31, 1, [(1, 129)], MASK_CAUSAL, dict(alibi=True)),
    (64, 32, 1, [(1, 513)], MASK_CAUSAL, dict(softcap=30.0)),
    (128, 33, 1, [(1, 545)], MASK_CAUSAL, dict(relpos=True)),
    (128, 3, 2, [(21, 700)] * 2, MASK_CAUSAL, {}),
    (64, 4, 2, [(32, 33)], MASK_CAUSAL, {}),
    (128, 1, 8, [(128, 1100)], MASK_CAUSAL, {}),
    (128, 4, 2, [(5, 3)], MASK_CAUSAL, {}),  # rows that see no key
    (128, 4, 2, [(2, 2000)] * 3, MASK_SLIDING_WINDOW, dict(window=(700, 3))),
    (64, 4, 2, [(3, 1500)], MASK_SLIDING_WINDOW, dict(window=(40, 0), softcap=400.0)),
    (128, 16, 1, [(2, 4001)], MASK_PREFIX_LM, dict(prefix_len=3999, alibi=True, relpos=True,
                                                   softcap=50.0)),
    (128, 4, 2, [(1, 1), (4, 3000), (0, 50), (2, 0), (3, 700), (1, 512), (0, 0)], MASK_CAUSAL, {}),
    (64, 2, 4, [(1, 600), (1, 5), (1, 2500), (1, 64)], MASK_NONE, dict(alibi=True)),
    # one long sequence first, amid and last among many short ones
    (128, 4, 2, [(1, 9000)] + [(1, 7 + 5 * i) for i in range(40)], MASK_CAUSAL, {}),
    (128, 4, 2, [(2, 9 + i) for i in range(25)] + [(4, 8100)] + [(1, 400 + i) for i in range(9)],
     MASK_CAUSAL, dict(softcap=30.0)),
    (64, 3, 2, [(1, 20 + i) for i in range(30)] + [(3, 7003)], MASK_NONE, {}),
    # a key cache stored token-major: the head stride is smaller than the row stride
    (128, 4, 2, [(3, 1300)] * 2, MASK_CAUSAL, dict(token_major=True)),
    (64, 8, 3, [(1, 77)] * 3, MASK_CAUSAL, dict(token_major=True)),
    # one 64-key tile of the prefill kernel: the decode kernel takes large grids
    (64, 8, 16, [(1, 31)] * 12, MASK_CAUSAL, dict(many=True)),
    (128, 4, 32, [(5, 3)] * 8, MASK_CAUSAL, dict(many=True)),  # rows that see no key
    (64, 1, 64, [(33, 64)] * 20, MASK_CAUSAL, {}),  # more row tiles than prefill workgroups
]


def _inputs(c):
    D, group, hkv, lens, mask, opt = c
    g = torch.Generator().manual_seed(sum(a * 31 + b for a, b in lens) + D + group)
    packed = len(set(lens)) > 1
    lq, lk = [a for a, _ in lens], [b for _, b in lens]
    hq = hkv * group
    qs = (sum(lq), hq, D) if packed else (len(lens), hq, lq[0], D)
    ks = (sum(lk), hkv, D) if packed else (len(lens), hkv, lk[0], D)
    q, k, v = (torch.randn(s, generator=g).to(torch.bfloat16) for s in (qs, ks, ks))
    if opt.get("token_major"):
        k, v = (t.transpose(1, 2).contiguous().transpose(1, 2) for t in (k, v))
    kw = dict(mask=MASK_NAMES[mask], softcap=opt.get("softcap", 0.0),
              relative_position=opt.get("relpos", False), prefix_len=opt.get("prefix_len", 0))
    okw = dict(mask=mask, softcap=opt.get("softcap", 0.0), relpos=opt.get("relpos", False),
               prefix_len=opt.get("prefix_len", 0))
    if "window" in opt:
        kw["window"] = opt["window"]
        okw.update(window_left=opt["window"][0], window_right=opt["window"][1])
    if opt.get("alibi"):
        kw["alibi_slopes"] = alibi_slopes(hq).cuda()
        okw["slopes"] = alibi_slopes(hq)
    if packed:
        cuq, cuk = (torch.tensor([0] + list(np.cumsum(x)), dtype=torch.int32) for x in (lq, lk))
        kw.update(cu_seqlens_q=cuq.cuda(), cu_seqlens_k=cuk.cuda(), max_seqlen_q=max(lq),
                  max_seqlen_k=max(lk))
        okw.update(cu_seqlens_q=cuq, cu_seqlens_k=cuk)
    return q, k, v, packed, kw, okw


def _call(lib, q, k, v, packed, kw, workspace):
    out = torch.empty_like(q)
    lse = torch.empty(attn.lse_shape(q, packed), dtype=torch.float32, device=q.device)
    d = attn.make_desc(q, k, v, out, **kw)
    n = lib.attn_workspace_bytes(ctypes.byref(d)) if workspace else 0
    ws = torch.full((max(n, 16),), 255, dtype=torch.uint8, device=q.device)  # NaN
    st = lib.attn_fwd_ws(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), lse.data_ptr(),
                         ctypes.byref(d), ws.data_ptr() if n else None, n)
    assert st == 0
    return out, lse


def _check(o, lse, o_ref, lse_ref, what):
    og = o.float().cpu().numpy().astype(np.float64)
    lg = lse.cpu().numpy().astype(np.float64)
    assert np.isfinite(og).all()
    assert np.array_equal(np.isinf(lg), np.isinf(lse_ref)), what
    fin = np.isfinite(lse_ref)
    o_err = float(np.abs(og - o_ref).max()) if og.size else 0.0
    l_err = float(np.abs(lg[fin] - lse_ref[fin]).max()) if fin.any() else 0.0
    r_err = row_error(og, o_ref)
    log(f"  {what}: max|dO| = {o_err:.3e}, rows {r_err:.3e}, max|dLSE| = {l_err:.3e}")
    assert o_err <= O_TOL["bf16"] and r_err <= ROW_TOL["bf16"] and l_err <= LSE_TOL, what


@pytest.mark.parametrize("i", range(len(CASES)))
@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
def test_decode_parity(i, capfd):
    c = CASES[i]
    log(f"[decode] {c}")
    q, k, v, packed, kw, okw = _inputs(c)
    qg, kg, vg = q.cuda(), k.cuda(), v.cuda()
    attn.fwd(qg, kg, vg, log=True, **kw)
    seen = max(min(b, sum(c[5].get("window", (b, 0))) + a) for a, b in c[3])  # keys of a row tile
    assert ("| decode kernel" in capfd.readouterr().err) == (seen > 64 or c[5].get("many", False))
    need = attn.load().attn_workspace_bytes(
        ctypes.byref(attn.make_desc(qg, kg, vg, torch.empty_like(qg), **kw)))
    assert (need > 0) == (seen > 513), "split or whole"
    o, lse = attn.fwd(qg, kg, vg, **kw)
    o1, lse1 = _call(attn.load(), qg, kg, vg, packed, kw, False)
    torch.cuda.synchronize()
    o_ref, lse_ref = oracle.attention(q, k, v, scale=c[0] ** -0.5, **okw)
    _check(o, lse, o_ref, lse_ref, "with workspace")
    _check(o1, lse1, o_ref, lse_ref, "without")
    # P is rounded against another running max: two roundings of 2^-8 each
    assert float((o.float() - o1.float()).abs().max()) <= 2 * 2 ** -8 * float(np.abs(o_ref).max())
    assert row_error(o.float().cpu().numpy(), o1.float().cpu().numpy()) <= ROW_TOL["bf16"]


@pytest.mark.parametrize("d,group,b,lq,lk,decode", [
    (64, 1, 32, 48, 384, True), (64, 1, 32, 48, 383, False),    # two row tiles a CU
    (128, 1, 16, 97, 2048, True), (128, 1, 16, 97, 2047, False),  # half the CUs
    (128, 1, 8, 100, 200, True), (128, 1, 9, 128, 200, False),  # a row tile for every CU
    (64, 2, 17, 1, 33, True), (64, 2, 16, 1, 33, False),        # one 64-key tile
    (128, 1, 33, 32, 193, True), (128, 1, 33, 32, 192, False),  # a tile for every wave
])
@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
def test_route(d, group, b, lq, lk, decode, capfd):
    """Both sides of the rules that choose the kernel, against the prefill kernel
    (a schedule override keeps it), with a window that starts inside a tile."""
    g = torch.Generator(device="cuda").manual_seed(lk)
    q, k, v = (torch.randn(b, h, n, d, generator=g, device="cuda").to(torch.bfloat16)
               for h, n in ((8 * group, lq), (8, lk), (8, lk)))
    attn.fwd(q, k, v, causal=True, log=True)
    assert ("| decode kernel" in capfd.readouterr().err) == decode
    for kw in (dict(causal=True), dict(window=(lk - 7, 3))):
        o, lse = attn.fwd(q, k, v, **kw)
        o1, lse1 = attn.fwd(q, k, v, order="natural", **kw)
        torch.cuda.synchronize()
        assert row_error(o.float().cpu().numpy(), o1.float().cpu().numpy()) <= ROW_TOL["bf16"]
        assert float((lse - lse1).abs().max()) <= LSE_TOL


@pytest.mark.parametrize("i", [0, 5, 9, 12, 13])
@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
def test_poisoned_lds_and_workspace_change_nothing(i):
    q, k, v, packed, kw, _ = _inputs(CASES[i])
    a = (q.cuda(), k.cuda(), v.cuda(), packed, kw, True)
    o, lse = _call(attn.load(), *a)
    o1, lse1 = _call(_abi.load(LIB_POISON), *a)
    torch.cuda.synchronize()
    assert torch.isfinite(o.float()).all()
    assert torch.equal(o, o1) and torch.equal(lse, lse1)


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
@pytest.mark.parametrize("lq,told", [(3, 2), (40, 32)])
def test_sequence_with_more_rows_than_told_stays_in_the_workspace(lq, told):
    """max_seqlen_q below a sequence's length: the rows that the grid covers are
    right, and no partial result lands past the workspace (a guard behind it)."""
    g = torch.Generator().manual_seed(lq)
    q = torch.randn(1 + lq, 8, 128, generator=g).to(torch.bfloat16).cuda()
    k, v = (torch.randn(12000, 2, 128, generator=g).to(torch.bfloat16).cuda() for _ in range(2))
    cu = [torch.tensor(x, dtype=torch.int32, device="cuda") for x in ([0, 1, 1 + lq], [0, 6000, 12000])]
    kw = dict(mask="none", cu_seqlens_q=cu[0], cu_seqlens_k=cu[1], max_seqlen_q=told, max_seqlen_k=6000)
    out = torch.zeros_like(q)
    d = attn.make_desc(q, k, v, out, **kw)
    n = attn.load().attn_workspace_bytes(ctypes.byref(d))
    assert n > 0
    ws = torch.full((n + (1 << 22),), 255, dtype=torch.uint8, device="cuda")
    assert attn.load().attn_fwd_ws(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), None,
                                   ctypes.byref(d), ws.data_ptr(), n) == 0
    kw["max_seqlen_q"] = lq
    want, _ = attn.fwd(q, k, v, **kw)
    torch.cuda.synchronize()
    assert (ws[n:] == 255).all()
    rows = 1 + told
    # another split of the keys, two bf16 roundings of |O| < 0.25
    assert float((out[:rows].float() - want[:rows].float()).abs().max()) <= 2.0 ** -9


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
def test_nan_query_row_stays_nan():
    """A NaN query gives NaN outputs for its row alone, split or not."""
    g = torch.Generator().manual_seed(1)
    q = torch.randn(1, 4, 2, 128, generator=g).to(torch.bfloat16)
    q[0, 1, 0, 5] = float("nan")
    k, v = (torch.randn(1, 1, 3000, 128, generator=g).to(torch.bfloat16).cuda() for _ in range(2))
    o, _ = attn.fwd(q.cuda(), k, v, causal=True)
    torch.cuda.synchronize()
    nan = torch.isnan(o.float()).cpu()
    assert nan[0, 1, 0].all() and int(nan.sum()) == 128


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
def test_split_call_in_a_graph():
    """A captured split call gives the eager result on every replay."""
    g = torch.Generator().manual_seed(2)
    q = torch.randn(1, 32, 1, 128, generator=g).to(torch.bfloat16).cuda()
    k, v = (torch.randn(1, 8, 6000, 128, generator=g).to(torch.bfloat16).cuda() for _ in range(2))
    want, want_lse = attn.fwd(q, k, v)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        o, lse = attn.fwd(q, k, v)
    for _ in range(3):
        o.zero_()
        graph.replay()
        attn.fwd(q[:, :8].contiguous(), k[:, :2].contiguous(), v[:, :2].contiguous())
        torch.cuda.synchronize()
        assert torch.equal(o, want) and torch.equal(lse, want_lse)


# ---- the ABI of the workspace (no GPU: rejected before any HIP call) --------

def _desc(**kw):
    d = _abi.AttnVariantDesc.new()
    d.dtype, d.batch, d.num_q_heads, d.num_kv_heads, d.head_dim = _abi.ATTN_BF16, 1, 32, 8, 128
    d.scale, d.mask_kind, d.seqlen_q, d.seqlen_k = 0.1, _abi.ATTN_MASK_CAUSAL, 1, 8192
    for k, v in kw.items():
        setattr(d, k, v)
    return d


def test_workspace_bytes():
    lib = attn.load()
    need = lib.attn_workspace_bytes(ctypes.byref(_desc()))
    assert need > 0 and need % (32 * (128 + 4) * 4) == 0  # splits x rows x (D + 4) floats
    assert lib.attn_workspace_bytes(ctypes.byref(_desc(seqlen_k=64))) == 0
    assert lib.attn_workspace_bytes(ctypes.byref(_desc(batch=0))) == 0
    assert lib.attn_workspace_bytes(None) == _abi.STATUS_CODE["ATTN_ERR_NULL_PTR"]
    assert lib.attn_workspace_bytes(ctypes.byref(_desc(struct_size=8))) == \
        _abi.STATUS_CODE["ATTN_ERR_ABI"]
    assert lib.attn_workspace_bytes(ctypes.byref(_desc(num_kv_heads=5))) == \
        _abi.STATUS_CODE["ATTN_ERR_BAD_SHAPE"]
    assert lib.attn_workspace_bytes(ctypes.byref(_desc(sched_order=3))) == \
        _abi.STATUS_CODE["ATTN_ERR_BAD_VARIANT"]


def _packed_desc(hq, hkv, lens, **kw):
    """A packed descriptor (dummy device arrays: only sizes are looked at)."""
    return _desc(num_q_heads=hq, num_kv_heads=hkv, seqlen_q=0, seqlen_k=0, cu_seqlens_q=16,
                 cu_seqlens_k=16, batch=len(lens), total_q=sum(a for a, _ in lens),
                 total_k=sum(b for _, b in lens), max_seqlen_q=max(a for a, _ in lens),
                 max_seqlen_k=max(b for _, b in lens), **kw)


@pytest.mark.parametrize("hq,hkv,lens,kw", [
    (128, 8, [(1, 384)] * 511 + [(1, 131072)], {}),
    (32, 8, [(1, 384)] * 511 + [(1, 131072)], {}),
    (128, 8, [(1, 750)] * 255 + [(1, 65536)], {}),
    (32, 8, [(1, 84)] * 2047 + [(1, 32768)], {}),
    (8, 8, [(100, 100)] * 299 + [(100, 60000)], {}),
    (8, 1, [(150, 150)] * 499 + [(4000, 30000)], {}),
    (8, 8, [(64, 64)] * 299 + [(64, 20000)], dict(dtype=_abi.ATTN_FP32)),
    (8, 2, [(64, 64)] * 199 + [(8192, 8192)], dict(dtype=_abi.ATTN_FP32)),
])
def test_workspace_of_an_uneven_batch_is_bounded(hq, hkv, lens, kw):
    """One long sequence among many short ones: the workspace follows the rows
    that can be split, not every row times the longest one's splits (the first
    case asked for 2.2 GB). A quarter of the inputs and outputs, or 64 MiB."""
    need = attn.load().attn_workspace_bytes(ctypes.byref(_packed_desc(hq, hkv, lens, **kw)))
    elt = 4 if kw else 2
    io = 2 * 128 * elt * (hq * sum(a for a, _ in lens) + hkv * sum(b for _, b in lens))
    assert 0 <= need <= max(64 << 20, io // 4)


@pytest.mark.parametrize("kw,split", [
    (dict(batch=1), True),
    (dict(batch=64, seqlen_k=1000), False),  # 512 groups: the chip is full
    (dict(batch=16, num_q_heads=8, seqlen_k=1000), False),
    (dict(batch=1, num_q_heads=8, seqlen_q=128, seqlen_k=3000), True),
    # a left bound alone leaves few keys to a decode step
    (dict(mask_kind=_abi.ATTN_MASK_SLIDING_WINDOW, window_left=30, window_right=-1), False),
    (dict(mask_kind=_abi.ATTN_MASK_SLIDING_WINDOW, window_left=3000, window_right=-1), True),
])
def test_a_split_is_made_where_it_saves_more_than_it_costs(kw, split):
    assert (attn.load().attn_workspace_bytes(ctypes.byref(_desc(**kw))) > 0) == split


@pytest.mark.parametrize("hq,hkv,lens", [(64, 16, [(16, 101)] * 11 + [(16, 576)]),
                                         (8, 8, [(37, 144)] * 8 + [(37, 1166)] * 8)])
def test_rows_too_many_to_split(hq, hkv, lens):
    """Uneven packed chunks whose partial rows would take longer than the rest."""
    assert attn.load().attn_workspace_bytes(ctypes.byref(_packed_desc(hq, hkv, lens, head_dim=64))) == 0


def test_misaligned_workspace_is_refused():
    lib, P = attn.load(), 0x10000  # dummy device pointers, never dereferenced
    d = _desc()
    st = lib.attn_fwd_ws(P, P, P, P, None, ctypes.byref(d), P + 8, 1 << 30)
    assert st == _abi.STATUS_CODE["ATTN_ERR_ALIGNMENT"]
