"""The fp32 kernel at the edges of its tiles.

A workgroup takes 32 query rows and its four waves every fourth 32-key tile,
so the lengths here sit around 32 (row blocks, key tiles) and 128 (one tile
per wave): waves without a tile, a last tile with one key, a last block with
one row, fewer keys than queries. Every output element is compared with the
fp64 oracle. Tolerance: O is a convex combination of V rows, |V| < 6 for these
draws; the score error (D products and lk exponentials in fp32, 2^-24 each)
moves it by less than 1e-5, so 2e-5 leaves a factor of two.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import gpu_available, log
from paper_2605_05023_amd import fwd
from paper_2605_05023_amd.workloads import (MASK_CAUSAL, MASK_NAMES, MASK_NONE, MASK_SHARE_QUESTION,
                                            MASK_SLIDING_WINDOW)

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]
TOL = 2e-5
CASES = [(d, lq, lk, mask)
         for d, lq, lk in [(64, 1, 1), (128, 31, 33), (64, 32, 32), (128, 33, 31), (64, 33, 127),
                           (128, 32, 128), (64, 65, 129), (128, 97, 161), (128, 1, 640)]
         for mask in (MASK_NONE, MASK_CAUSAL, MASK_SLIDING_WINDOW, MASK_SHARE_QUESTION)]


def _token_ids(starts, n):
    return [sum(pos >= s for s in starts) - 1 for pos in range(n)]


@pytest.mark.parametrize("d,lq,lk,mask", CASES)
def test_tile_edges(d, lq, lk, mask):
    log(f"[f32 tiles] D={d} lq={lq} lk={lk} mask={MASK_NAMES[mask]}")
    g = torch.Generator().manual_seed(1000 * lq + lk + d)
    q = torch.randn(2, 4, lq, d, generator=g)
    # token-major K and V: the head stride is smaller than the row stride
    k, v = (torch.randn(2, lk, 2, d, generator=g).transpose(1, 2) for _ in range(2))
    kw, okw = {}, {}
    if mask == MASK_SLIDING_WINDOW:
        kw["window"] = (40, 3)
        okw.update(window_left=40, window_right=3)
    if mask == MASK_SHARE_QUESTION:
        seg = [lk // 3, lk // 3 + 1 + lk // 4]
        kw["segment_starts"] = torch.tensor(seg, dtype=torch.int32, device="cuda")
        okw["token_ids"] = _token_ids(seg, lk)
    o, lse = fwd(q.cuda(), k.cuda(), v.cuda(), mask=MASK_NAMES[mask], **kw)
    torch.cuda.synchronize()
    o_ref, lse_ref = oracle.attention(q, k, v, scale=d ** -0.5, mask=mask, **okw)
    lg = lse.cpu().numpy().astype(np.float64)
    assert np.array_equal(np.isinf(lg), np.isinf(lse_ref))
    fin = np.isfinite(lse_ref)
    assert np.abs(o.cpu().numpy() - o_ref).max() <= TOL
    assert not fin.any() or np.abs(lg[fin] - lse_ref[fin]).max() <= TOL


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("what", ["causal", "window", "prefix_lm", "share_question", "listed global",
                                  "relu", "sigmoid split", "gathered past the band"])
def test_values_of_unseen_keys_stay_out(what, d):
    """Infinite and NaN values reach the rows that see their key, and no other
    row of the 32-row block: those are bit for bit what zeros in their place
    give (a product with P = 0 would make them NaN)."""
    lq, lk = (150, 1700) if what == "sigmoid split" else (97, 161)
    g = torch.Generator().manual_seed(d + len(what))
    q = torch.randn(1, 2, lq, d, generator=g)
    k, v = (torch.randn(1, 1, lk, d, generator=g) for _ in range(2))
    bad = {lk - 1: float("inf"), lk - 30: float("nan"), lk - 70: float("-inf"), 3: float("inf"),
           70: float("nan")}
    dims = {j: (7 * n + 1) % d for n, j in enumerate(bad)}
    v_bad, v_zero = v.clone(), v.clone()
    for j, x in bad.items():
        v_bad[0, 0, j, dims[j]], v_zero[0, 0, j, dims[j]] = x, 0.0
    v_bad[0, 0, 3, dims[lk - 30]], v_zero[0, 0, 3, dims[lk - 30]] = float("-inf"), 0.0
    i, j = np.arange(lq)[:, None] + (lk - lq), np.arange(lk)[None, :]
    causal, kw = j <= i, dict(causal=True)
    seen = causal
    if what == "window":
        seen, kw = (i - j <= 40) & (j - i <= 3), dict(window=(40, 3))
    elif what == "prefix_lm":
        seen, kw = causal | (j < 50), dict(mask="prefix_lm", prefix_len=50)
    elif what == "share_question":
        starts = np.array([20, 90, 130])
        seg = lambda t: np.searchsorted(starts, t, side="right")
        seen = causal & ((seg(j) == 0) | (seg(i) == seg(j)))
        kw = dict(mask="share_question", segment_starts=torch.tensor(starts, dtype=torch.int32).cuda())
    elif what in ("listed global", "gathered past the band"):
        tok = [3, 70, 100] if what == "listed global" else [5, lk - 30, lk - 1]
        w = (40, 3) if what == "listed global" else (10, 0)
        seen = ((i - j <= w[0]) & (j - i <= w[1])) | np.isin(i, tok) | np.isin(j, tok)
        kw = dict(mask="global_sliding_window", window=w,
                  global_tokens=torch.tensor(tok, dtype=torch.int32).cuda())
    elif what != "causal":
        kw["norm"] = what.split()[0]
    got, want = (fwd(q.cuda(), k.cuda(), x.cuda(), return_lse=False, **kw).cpu() for x in (v_bad, v_zero))
    hit = np.zeros((lq, d), bool)
    for key in bad:
        hit[seen[:, key], dims[key]] = True
    hit[seen[:, 3], dims[lk - 30]] = True
    hit = torch.from_numpy(hit).expand(1, 2, -1, -1)
    assert hit.any() and not hit.all()
    assert torch.equal(got[~hit], want[~hit])
    assert not torch.isfinite(got[hit]).any()
    if what == "causal":  # one infinite key seen: its infinity; none of these rows sees two
        only = hit.clone()
        only[..., [x for n, x in dims.items() if n != lk - 1]] = False
        assert torch.isinf(got[only]).all() and (got[only] > 0).all()


@pytest.mark.parametrize("d", [64, 128])
def test_one_key_of_small_row_stride(d):
    """A single key row may have any row stride; the rows past it stay zero."""
    g = torch.Generator().manual_seed(d)
    q = torch.randn(1, 2, 5, d, generator=g).cuda()
    kv = torch.randn(2, 2, d, generator=g).cuda()
    kv[1, 1, 3] = float("inf")  # a row read twice would turn 0 * inf into NaN
    k, v = (kv[i].as_strided((1, 2, 1, d), (2 * d, d, 4, 1)) for i in range(2))
    o, lse = fwd(q, k, v)
    torch.cuda.synchronize()
    assert torch.equal(o, v.expand(1, 2, 5, d))
    want = (q * k).double().sum(-1) * d ** -0.5
    assert (lse.double() - want).abs().max() <= TOL
