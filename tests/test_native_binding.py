"""The native argument marshalling against the Python path it stands in for:
the same descriptor (the launch plan printed by the log flag apart, which only
the Python path takes), the same outputs bit for bit, and the same refusals.
"""
import ctypes
import subprocess
import threading

import pytest
import torch

import paper_2605_05023_amd as attn
from gpu_util import gpu_available, log
from paper_2605_05023_amd.workloads import alibi_slopes

gpu = pytest.mark.gpu
needs_gpu = pytest.mark.skipif(not gpu_available(), reason="needs a GPU")


def _x(*shape, dtype=torch.bfloat16, seed=0):
    g = torch.Generator().manual_seed(seed + sum(shape))
    return torch.randn(*shape, generator=g).to(dtype).cuda()


_ARGS = dict(causal=False, window=None, alibi_slopes=None, softcap=0.0, scale=None, cu_seqlens_q=None,
             cu_seqlens_k=None, max_seqlen_q=None, max_seqlen_k=None, out=None, lse=None, return_lse=True,
             mask=None, prefix_len=0, num_global=0, global_tokens=None, segment_starts=None, query_start=0,
             relative_position=False, norm="softmax")


def _native(*x, **kw):
    """The call as the native path makes it; it must not be left to the Python path."""
    assert not set(kw) - set(_ARGS)
    res = attn._load_native().fwd(*x, *{**_ARGS, **kw}.values())
    assert res is not NotImplemented
    return res


def _i32(v):
    return torch.tensor(v, dtype=torch.int32, device="cuda")


def _cases():
    q, k, v = _x(2, 8, 70, 64), _x(2, 2, 90, 64), _x(2, 2, 90, 64, seed=1)
    pq, pk, pv = _x(130, 4, 128), _x(200, 2, 128), _x(200, 2, 128, seed=1)
    cu = dict(cu_seqlens_q=_i32([0, 30, 130]), cu_seqlens_k=_i32([0, 80, 200]), max_seqlen_q=100,
              max_seqlen_k=120)
    f = torch.float32
    bshd = [t.transpose(1, 2) for t in (_x(1, 50, 4, 64), _x(1, 50, 4, 64), _x(1, 50, 4, 64, seed=1))]
    out, lse = torch.empty_like(q), torch.empty(2, 8, 70, device="cuda")
    return [
        ((q, k, v), {}),
        ((q, k, v), dict(causal=True, return_lse=False)),
        ((q, k, v), dict(causal=True, out=out, lse=lse)),
        ((q, k, v), dict(window=(20, 3), scale=0.2, softcap=30)),
        ((q, k, v), dict(mask="prefix_lm", prefix_len=11, alibi_slopes=alibi_slopes(8).cuda())),
        ((q, k, v), dict(mask=4, window=(9, 9), num_global=3, relative_position=True)),
        ((q, k, v), dict(mask="global_sliding_window", window=(9, -1), global_tokens=_i32([1, 40, 77]))),
        ((q, k, v), dict(mask="share_question", segment_starts=_i32([[20, 50], [30, 60]]))),
        ((q, k, v), dict(mask="causal_blockwise", segment_starts=_i32([20, 50]), query_start=60,
                         norm="relu")),
        ((q, k, v), dict(causal=True, norm=2)),
        (tuple(bshd), dict(causal=True)),
        ((_x(1, 2, 40, 64, dtype=f), _x(1, 2, 40, 64, dtype=f), _x(1, 2, 40, 64, dtype=f, seed=1)), {}),
        ((pq, pk, pv), dict(causal=True, **cu)),
        ((q[:, :, :1], k, v), dict(causal=True)),
    ]


@gpu
@needs_gpu
def test_same_outputs_as_the_python_path():
    for i, (x, kw) in enumerate(_cases()):
        log(f"[native binding] case {i} {sorted(kw)}")
        got = _native(*x, **kw)
        got = [t.clone() for t in (got if isinstance(got, tuple) else (got,))]
        want = attn.fwd(*x, **kw, validate=True)  # taken by the Python path
        want = want if isinstance(want, tuple) else (want,)
        torch.cuda.synchronize()
        assert len(got) == len(want)
        for a, b in zip(got, want):
            assert a.shape == b.shape and a.stride() == b.stride() and torch.equal(a, b)


@gpu
@needs_gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_expanded_inputs_match_their_copies(dtype):
    """An expanded axis (stride 0) of q, k or v, which the descriptor cannot
    express: the same outputs as with the copies; an expanded output is refused."""
    x = dict(dtype=dtype)
    q, k, v = _x(3, 4, 40, 64, **x), _x(3, 2, 90, 64, **x), _x(3, 2, 90, 64, seed=1, **x)
    pq, pk, pv = _x(50, 4, 64, **x), _x(50, 1, 64, **x), _x(50, 1, 64, seed=1, **x)
    cu = dict(cu_seqlens_q=_i32([0, 20, 50]), max_seqlen_q=30, max_seqlen_k=30)
    for (a, b, c), kw in [
        ((q, k[:1].expand(3, -1, -1, -1), v[:1].expand(3, -1, -1, -1)), {}),
        ((q, k[:, :1].expand(-1, 4, -1, -1), v[:, 1:].expand(-1, 4, -1, -1)), {}),
        ((q, k, v[:, :, :1].expand(-1, -1, 90, -1)), {}),
        ((q[:1, :1].expand(3, 4, -1, -1), k, v), {}),
        ((pq, pk.expand(-1, 2, -1), pv.expand(-1, 2, -1)), cu),
    ]:
        want = attn.fwd(*(t.contiguous() for t in (a, b, c)), causal=True, **kw)
        got = attn.fwd(a, b, c, causal=True, **kw)
        torch.cuda.synchronize()
        assert all(torch.equal(g, w) for g, w in zip(got, want))
    with pytest.raises(ValueError, match="expanded"):
        attn.fwd(q, k, v, out=torch.empty_like(q[:, :1]).expand(-1, 4, -1, -1))


@gpu
@needs_gpu
def test_given_outputs_come_back():
    q, k, v = _x(1, 2, 20, 64), _x(1, 2, 20, 64), _x(1, 2, 20, 64, seed=1)
    out, lse = torch.empty_like(q), torch.empty(1, 2, 20, device="cuda")
    o, l = attn.fwd(q, k, v, out=out, lse=lse)
    assert o is out and l is lse
    assert attn.fwd(q, k, v, out=out, lse=lse, return_lse=False) is out


@gpu
@needs_gpu
@pytest.mark.parametrize("path", ["native", "python"])
def test_no_memory_for_a_workspace(path):
    """A call whose keys would be split, with no room for the 17 MB workspace, is
    computed without the split (outputs of bf16: rounding steps apart)."""
    torch.cuda.synchronize()
    torch.cuda.empty_cache()  # segments of their own, with no room left in them
    q, k, v = _x(1, 32, 512, 128), _x(1, 32, 8192, 128), _x(1, 32, 8192, 128, seed=1)
    call = _native if path == "native" else lambda *x, **kw: attn.fwd(*x, validate=True, **kw)
    want, lse_want = attn.fwd(q, k, v)
    out, lse = torch.empty_like(q), torch.empty(1, 32, 512, device="cuda")
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    torch.cuda.set_per_process_memory_fraction(1e-6)
    try:
        with pytest.raises(torch.OutOfMemoryError):
            torch.empty(17 << 20, dtype=torch.uint8, device="cuda")
        torch.cuda.reset_peak_memory_stats()
        held = torch.cuda.memory_allocated()
        call(q, k, v, out=out, lse=lse)
        assert torch.cuda.max_memory_allocated() == held  # no workspace
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    torch.cuda.synchronize()
    # |O| < 0.25 here, where neighbouring bf16 values are 2^-10 apart at most
    assert float((out.float() - want.float()).abs().max()) <= 2.0 ** -9
    assert float((lse - lse_want).abs().max()) <= 1e-4


@gpu
@needs_gpu
def test_refusals_are_those_of_the_python_path():
    q, k, v = _x(1, 4, 20, 64), _x(1, 2, 20, 64), _x(1, 2, 20, 64, seed=1)
    for err, x, kw in [
        (TypeError, (q, k.float(), v), {}),
        (ValueError, (q, k, v[:, :, :19]), {}),
        (ValueError, (q.transpose(2, 3), k, v), {}),
        (ValueError, (q, k, v), dict(alibi_slopes=torch.ones(3, device="cuda"))),
        (TypeError, (q, k, v), dict(alibi_slopes=torch.ones(4))),
        (TypeError, (q, k, v), dict(lse=torch.empty(1, 4, 20))),
        (ValueError, (q, k, v), dict(out=torch.empty_like(q)[:, :, :5])),
        (KeyError, (q, k, v), dict(mask="diagonal")),
        (ValueError, (q[0].transpose(0, 1), k[0].transpose(0, 1), v[0].transpose(0, 1)),
         dict(cu_seqlens_q=_i32([0, 20]))),
        (attn.AttnError, (q, k, v), dict(window=(-2, 0))),
        (attn.AttnError, (q, k, v), dict(scale=-1.0)),
        (attn.AttnError, (_x(1, 3, 20, 64), k, v), {}),
        (ValueError, (q.cpu(), k.cpu(), v.cpu()), {}),
    ]:
        with pytest.raises(err):
            attn.fwd(*x, **kw)


@gpu
@needs_gpu
def test_subclasses_and_modes_take_the_python_path():
    class Sub(torch.Tensor):
        pass

    q, k, v = _x(1, 2, 20, 64), _x(1, 2, 20, 64), _x(1, 2, 20, 64, seed=1)
    args = (False, None, None, 0.0, None, None, None, None, None, None, None, True, None, 0, 0, None,
            None, 0, False, "softmax")
    native = attn._load_native()
    assert native.fwd(q, k, v, *args) is not NotImplemented
    assert native.fwd(q.as_subclass(Sub), k, v, *args) is NotImplemented
    with torch.utils._python_dispatch.TorchDispatchMode():
        assert native.fwd(q, k, v, *args) is NotImplemented
    o = torch.empty(20, 64)
    assert torch.func.vmap(lambda t: o if native.fwd(t, t, t, *args) is NotImplemented else t[0, 0])(
        torch.stack([q, q])).shape == (2, 20, 64)


@gpu
@needs_gpu
def test_other_threads_run_during_a_call(tmp_path):
    """The native path gives up the interpreter lock for the call into the
    library: in its place a function that waits (3 s at most) until another
    Python thread has seen it start."""
    src = tmp_path / "wait.c"
    src.write_text("""
        #include <time.h>
        volatile int started, answered, in_time;
        int wait_fwd(void *q, void *k, void *v, void *o, float *l, void *d, void *w, long long n)
        {
            struct timespec a, b;
            clock_gettime(CLOCK_MONOTONIC, &a);
            started = 1;
            do clock_gettime(CLOCK_MONOTONIC, &b);
            while (!answered && b.tv_sec - a.tv_sec < 3);
            in_time = answered;
            return 0;
        }
        long long no_bytes(void *d) { return 0; }
        """)
    so = tmp_path / "wait.so"
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    started, answered = (ctypes.c_int.in_dll(lib, n) for n in ("started", "answered"))
    done = threading.Event()

    def answer():
        while not started.value and not done.is_set():
            done.wait(0.001)
        if not done.is_set():
            answered.value = 1

    native = attn._load_native()
    q, k, v = _x(1, 2, 20, 64), _x(1, 2, 20, 64), _x(1, 2, 20, 64, seed=1)
    native.bind(ctypes.cast(lib.wait_fwd, ctypes.c_void_p).value,
                ctypes.cast(lib.no_bytes, ctypes.c_void_p).value)
    t = threading.Thread(target=answer)
    try:
        t.start()
        attn.fwd(q, k, v)
    finally:
        done.set()
        t.join()
        attn._load_native()
    assert ctypes.c_int.in_dll(lib, "in_time").value == 1


@gpu
@needs_gpu
def test_a_failed_launch_is_raised_once():
    """ATTN_ERR_LAUNCH comes back as AttnError from the call that got it; the
    call is not repeated through the Python path."""
    native = attn._load_native()
    q, k, v = _x(1, 2, 20, 64), _x(1, 2, 20, 64), _x(1, 2, 20, 64, seed=1)
    calls = []
    failing = ctypes.CFUNCTYPE(ctypes.c_int, *[ctypes.c_void_p] * 7, ctypes.c_int64)(
        lambda *a: calls.append(1) or -7)
    native.bind(ctypes.cast(failing, ctypes.c_void_p).value,
                ctypes.cast(attn.load().attn_workspace_bytes, ctypes.c_void_p).value)
    try:
        with pytest.raises(attn.AttnError) as e:
            attn.fwd(q, k, v)
    finally:
        attn._load_native()
    assert e.value.status == -7 and len(calls) == 1
    o, _ = attn.fwd(q, k, v)
    torch.cuda.synchronize()
    assert torch.isfinite(o.float()).all()
