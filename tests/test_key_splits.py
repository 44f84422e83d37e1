"""Key splits of the prefill and fp32 kernels.

Calls whose workgroups would not fill the chip leave partial results in the
workspace. The cases cover rows written whole beside split ones (causal rows
with few keys, a packed sequence with a short cache), splits that hold no tile
of a row, ragged last splits, every normalisation, the general mask path, the
relative position's LSE shift and fp32. Each must really be split
(attn_workspace_bytes > 0), is run on a workspace full of NaN, and is compared
with the fp64 oracle, element by element at the bars of the other parity tests
and row by row against the row's own norm.
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
from paper_2605_05023_amd.workloads import (MASK_CAUSAL, MASK_CAUSAL_BLOCKWISE, MASK_GLOBAL_WINDOW,
                                            MASK_NAMES, MASK_NONE, MASK_PREFIX_LM, MASK_SHARE_QUESTION,
                                            MASK_SLIDING_WINDOW, alibi_slopes)

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

# (dtype, D, hq, hkv, [(lq, lk)] (packed when they differ), mask, options)
CASES = [
    ("bf16", 128, 2, 2, [(150, 4000)], MASK_CAUSAL, {}),
    ("bf16", 128, 2, 2, [(2500, 2500)], MASK_CAUSAL, {}),
    ("bf16", 64, 4, 4, [(200, 3001)], MASK_NONE, dict(alibi=True, softcap=50.0)),
    ("bf16", 64, 3, 1, [(130, 3000)], MASK_CAUSAL, dict(relpos=True)),
    ("bf16", 128, 8, 2, [(60, 3000), (200, 210), (1, 5000), (0, 40), (129, 0)], MASK_CAUSAL, {}),
    ("bf16", 128, 4, 1, [(140, 4100)], MASK_SLIDING_WINDOW, dict(window=(3000, -1))),
    ("bf16", 128, 2, 2, [(300, 3100)], MASK_CAUSAL, dict(norm="sigmoid")),
    ("bf16", 64, 2, 2, [(300, 5100)], MASK_CAUSAL, dict(norm="relu", softcap=400.0)),
    ("bf16", 128, 2, 2, [(2600, 2600)], MASK_SHARE_QUESTION, dict(seg=[900, 1500, 2300])),
    ("bf16", 64, 2, 2, [(400, 5000)], MASK_CAUSAL_BLOCKWISE, dict(seg=[1000, 4700], query_start=4900,
                                                                alibi=True, relpos=True)),
    ("fp32", 128, 2, 2, [(1, 1500)], MASK_CAUSAL, dict(relpos=True)),
    ("fp32", 64, 4, 2, [(70, 2001)], MASK_SLIDING_WINDOW, dict(window=(1500, 0), alibi=True)),
    ("fp32", 128, 2, 1, [(600, 600)], MASK_CAUSAL, dict(norm="sigmoid")),
    ("fp32", 64, 2, 2, [(33, 1600), (64, 64), (5, 900), (3, 0)], MASK_SHARE_QUESTION,
     dict(seg=[500, 1000])),
    # one long sequence among short ones: only its rows have room in the workspace
    ("bf16", 128, 2, 2, [(20, 90)] * 12 + [(130, 6000)] + [(40, 41)] * 3, MASK_CAUSAL, {}),
    ("fp32", 64, 2, 2, [(65, 2500)] + [(9, 30)] * 10, MASK_CAUSAL, dict(norm="relu")),
    # ALiBi without a soft-cap (its descending run of keys) across split boundaries
    ("bf16", 128, 2, 2, [(150, 4000)], MASK_CAUSAL, dict(alibi=True)),
    ("bf16", 64, 2, 2, [(2500, 2500)], MASK_CAUSAL, dict(alibi=True)),
    # a prefix that ends inside a split, and leading global rows, which see every
    # key where the other rows see their window
    ("bf16", 128, 2, 2, [(300, 4000)], MASK_PREFIX_LM, dict(prefix_len=1500)),
    ("fp32", 64, 2, 2, [(100, 1500)], MASK_PREFIX_LM, dict(prefix_len=1450)),
    ("bf16", 128, 1, 1, [(2000, 2000)], MASK_GLOBAL_WINDOW, dict(window=(1500, 0), num_global=40)),
    ("bf16", 64, 1, 1, [(2600, 2600)], MASK_GLOBAL_WINDOW, dict(window=(1900, 90), num_global=3,
                                                               norm="sigmoid")),
    ("fp32", 128, 1, 1, [(900, 900)], MASK_GLOBAL_WINDOW, dict(window=(600, 0), num_global=33)),
]
NORMS = {"softmax": 0, "relu": 1, "sigmoid": 2}


def _token_ids(starts, n):
    return [sum(pos >= s for s in starts) - 1 for pos in range(n)]


def _call(lib, q, k, v, packed, kw, softmax):
    out = torch.empty_like(q)
    lse = torch.empty(attn.lse_shape(q, packed), dtype=torch.float32, device=q.device) \
        if softmax else None
    d = attn.make_desc(q, k, v, out, **kw)
    n = lib.attn_workspace_bytes(ctypes.byref(d))
    assert n > 0, "the case is not split"
    ws = torch.full((n,), 255, dtype=torch.uint8, device=q.device)  # NaN
    st = lib.attn_fwd_ws(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(),
                         lse.data_ptr() if softmax else None, ctypes.byref(d), ws.data_ptr(), n)
    assert st == 0
    return out, lse


@pytest.mark.parametrize("i", range(len(CASES)))
def test_split_parity(i):
    dtype, D, hq, hkv, lens, mask, opt = CASES[i]
    log(f"[key splits] {CASES[i]}")
    g = torch.Generator().manual_seed(77 + i)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    packed = len(set(lens)) > 1
    lq, lk = [a for a, _ in lens], [b for _, b in lens]
    qs = (sum(lq), hq, D) if packed else (len(lens), hq, lq[0], D)
    ks = (sum(lk), hkv, D) if packed else (len(lens), hkv, lk[0], D)
    q, k, v = (torch.randn(s, generator=g).to(tdt) for s in (qs, ks, ks))
    norm = opt.get("norm", "softmax")
    kw = dict(mask=MASK_NAMES[mask], softcap=opt.get("softcap", 0.0), norm=norm,
              relative_position=opt.get("relpos", False), query_start=opt.get("query_start", 0),
              prefix_len=opt.get("prefix_len", 0), num_global=opt.get("num_global", 0))
    okw = dict(mask=mask, softcap=opt.get("softcap", 0.0), norm=NORMS[norm],
               relpos=opt.get("relpos", False), query_start=opt.get("query_start", 0),
               prefix_len=opt.get("prefix_len", 0))
    if "num_global" in opt:
        okw["global_tokens"] = list(range(opt["num_global"]))
    if "window" in opt:
        kw["window"] = opt["window"]
        okw.update(window_left=opt["window"][0], window_right=opt["window"][1])
    if opt.get("alibi"):
        kw["alibi_slopes"] = alibi_slopes(hq).cuda()
        okw["slopes"] = alibi_slopes(hq)
    if "seg" in opt:
        kw["segment_starts"] = torch.tensor(opt["seg"], dtype=torch.int32, device="cuda")
        okw["token_ids"] = _token_ids(opt["seg"], max(lk))
    if packed:
        cuq, cuk = (torch.tensor([0] + list(np.cumsum(x)), dtype=torch.int32) for x in (lq, lk))
        kw.update(cu_seqlens_q=cuq.cuda(), cu_seqlens_k=cuk.cuda(), max_seqlen_q=max(lq),
                  max_seqlen_k=max(lk))
        okw.update(cu_seqlens_q=cuq, cu_seqlens_k=cuk)
    a = (q.cuda(), k.cuda(), v.cuda(), packed, kw, norm == "softmax")
    o, lse = _call(attn.load(), *a)
    o1, lse1 = _call(_abi.load(LIB_POISON), *a)
    torch.cuda.synchronize()
    assert torch.equal(o, o1), "output differs with poisoned LDS"
    o_ref, lse_ref = oracle.attention(q, k, v, scale=D ** -0.5, **okw)
    og = o.float().cpu().numpy().astype(np.float64)
    assert np.isfinite(og).all()
    o_err, tol = float(np.abs(og - o_ref).max()), O_TOL[dtype]
    if norm != "softmax":
        tol *= float(np.abs(o_ref).max())
    r_err = row_error(og, o_ref)
    log(f"  max|dO| = {o_err:.3e} (tol {tol:.1e}), rows {r_err:.3e} (tol {ROW_TOL[dtype]:.1e})")
    assert o_err <= tol and r_err <= ROW_TOL[dtype]
    if norm == "softmax":
        lg = lse.cpu().numpy().astype(np.float64)
        assert np.array_equal(np.isinf(lg), np.isinf(lse_ref))
        fin = np.isfinite(lse_ref)
        assert float(np.abs(lg[fin] - lse_ref[fin]).max()) <= LSE_TOL


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("what", ["nan query", "nan key", "inf value"])
def test_nan_and_inf_as_without_a_split(what, dtype):
    """NaN queries and keys, and an infinite value in a split whose weight
    underflows, give the NaN that the unsplit call gives."""
    g = torch.Generator().manual_seed(8)
    q, k, v = (torch.randn(1, 2, n, 64, generator=g).to(dtype).cuda() for n in (140, 4000, 4000))
    if what == "nan query":
        q[0, 1, 7, 3] = float("nan")
    elif what == "nan key":
        k[0, 1, 2100, 3] = float("nan")
    else:  # scores of the first half 800 below the others
        q[:] = 1.0
        k[:, :, :2000] = -100.0
        k[:, :, 2000:] = 0.0
        v[0, 1, 5, 9] = float("inf")
    kw = dict(mask="none")
    o, _ = _call(attn.load(), q, k, v, False, kw, True)
    out, lse = torch.empty_like(q), torch.empty(attn.lse_shape(q, False), device="cuda")
    d = attn.make_desc(q, k, v, out, **kw)
    assert attn.load().attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(),
                                lse.data_ptr(), ctypes.byref(d)) == 0
    torch.cuda.synchronize()
    assert torch.isnan(out).any()
    assert torch.equal(torch.isnan(o), torch.isnan(out))


@pytest.mark.parametrize("dtype,lq", [("bf16", 1), ("bf16", 150), ("fp32", 40)])
def test_rows_of_no_sequence_stay_as_they_are(dtype, lq):
    """A packed call writes the rows of its sequences: tokens before the first
    and past the last one keep what out and lse held."""
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator().manual_seed(lq)
    hq, lk, pre, post = 2, 4000, 5, 3
    q = torch.randn(pre + lq + post, hq, 128, generator=g).to(tdt).cuda()
    k, v = (torch.randn(lk, hq, 128, generator=g).to(tdt).cuda() for _ in range(2))
    cu = [torch.tensor(x, dtype=torch.int32, device="cuda") for x in ([pre, pre + lq], [0, lk])]
    kw = dict(causal=True, cu_seqlens_q=cu[0], cu_seqlens_k=cu[1], max_seqlen_q=lq, max_seqlen_k=lk)
    out, lse = torch.full_like(q, 7.0), torch.full((hq, q.shape[0]), 7.0, device="cuda")
    d = attn.make_desc(q, k, v, out, **kw)
    assert attn.load().attn_workspace_bytes(ctypes.byref(d)) > 0
    attn.fwd(q, k, v, out=out, lse=lse, **kw)
    kw["cu_seqlens_q"] = torch.tensor([0, lq], dtype=torch.int32, device="cuda")
    want, lse_want = attn.fwd(q[pre:pre + lq].contiguous(), k, v, **kw)
    torch.cuda.synchronize()
    assert torch.equal(out[pre:pre + lq], want) and torch.equal(lse[:, pre:pre + lq], lse_want)
    for s in (slice(0, pre), slice(pre + lq, None)):
        assert (out[s] == 7.0).all() and (lse[:, s] == 7.0).all()


def test_two_streams_share_nothing():
    """Split calls on two streams, interleaved: each gets the output of the
    same call run alone (every call has a workspace of its own)."""
    g = torch.Generator().manual_seed(5)
    x = [[torch.randn(1, 4, n, 128, generator=g).to(torch.bfloat16).cuda() for n in (150, 4000, 4000)]
         for _ in range(2)]
    want = [attn.fwd(*t, causal=True) for t in x]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in x]
    got = [[], []]
    for _ in range(4):
        for s, t, r in zip(streams, x, got):
            with torch.cuda.stream(s):
                r.append(attn.fwd(*t, causal=True))
    torch.cuda.synchronize()
    for w, r in zip(want, got):
        for o, lse in r:
            assert torch.equal(o, w[0]) and torch.equal(lse, w[1])


@pytest.mark.parametrize("mask,lk", [(MASK_NONE, 2560), (MASK_CAUSAL, 2561), (MASK_CAUSAL, 2559)])
def test_third_workgroup_per_cu(mask, lk):
    """D = 64 on both sides of the rule (2560 keys, 1500 workgroups) that gives a
    CU a third workgroup; sampled rows against the oracle."""
    lq, h = 385, 512  # 4 query tiles, the last one with one row
    g = torch.Generator(device="cuda").manual_seed(lk)
    q, k, v = (torch.randn(1, h, n, 64, generator=g, device="cuda").to(torch.bfloat16)
               for n in (lq, lk, lk))
    o, lse = attn.fwd(q, k, v, mask=MASK_NAMES[mask])
    torch.cuda.synchronize()
    for head in (0, 255, 511):
        one = [t[:, head:head + 1].cpu() for t in (q, k, v)]
        o_ref, lse_ref = oracle.attention(*one, scale=0.125, mask=mask)
        assert float(np.abs(o[:, head:head + 1].float().cpu().numpy() - o_ref).max()) <= O_TOL["bf16"]
        assert float(np.abs(lse[:, head:head + 1].cpu().numpy() - lse_ref).max()) <= LSE_TOL
