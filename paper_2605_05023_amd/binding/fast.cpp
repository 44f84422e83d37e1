// fast.cpp -- native argument marshalling of paper_2605_05023_amd.fwd.
//
// The Python binding spent 15 us of host time per call outside the library
// (descriptor fields one by one through ctypes, shape checks, allocations),
// more than the kernels of a short prompt or a decode step take. This module
// makes the same checks on the tensors themselves, fills the descriptor,
// allocates out, lse and the workspace, and calls the C ABI. Host time a call
// 19.4 -> 6.1 us with one launch (the launch itself takes 4), 23.4 -> 9.9 with
// a key split; 1 x 32/8 heads x 333 tokens 18.3 -> 9.7 us a call (now the
// kernel's time).
//
// It only takes calls that need nothing else: plain device tensors, checked
// arguments of the expected types, no schedule override, no validation or log.
// Everything it does not take (anything it would have to report as an error
// included) returns NotImplemented before any work, and the Python path of
// fwd, which raises the errors, runs instead. A launch that fails is raised
// here: the call is not made a second time. No arithmetic is done here.
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <Python.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cmath>

#include "../../include/attn.h"

namespace {

using fwd_ws_t = int (*)(const void*, const void*, const void*, void*, float*, const attn_variant_desc*,
                         void*, int64_t);
using ws_bytes_t = int64_t (*)(const attn_variant_desc*);
fwd_ws_t g_fwd_ws = nullptr;
ws_bytes_t g_ws_bytes = nullptr;

// A plain device tensor: no subclass, no functional transform, no lazy bit.
bool plain(PyObject* o, at::Tensor* t)
{
    if (!THPVariable_CheckExact(o)) return false;
    *t = THPVariable_Unpack(o);
    if (!t->defined() || !t->is_cuda() || t->layout() != at::kStrided) return false;
    using c10::DispatchKey;
    const c10::DispatchKeySet odd({DispatchKey::Python, DispatchKey::Functionalize, DispatchKey::Conjugate,
                                   DispatchKey::Negative, DispatchKey::ZeroTensor,
                                   DispatchKey::FuncTorchBatched, DispatchKey::FuncTorchGradWrapper});
    return !t->key_set().has_any(odd);
}

// An axis of more than one entry with stride 0 (an expanded tensor): the
// descriptor takes a stride of 0 for the contiguous default.
bool broadcast(const at::Tensor& t)
{
    for (int64_t i = 0; i < t.dim(); ++i)
        if (t.stride(i) == 0 && t.size(i) > 1) return true;
    return false;
}

bool as_int(PyObject* o, int64_t* v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    *v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}

bool as_i32(PyObject* o, int32_t* v)
{
    int64_t x;
    if (!as_int(o, &x) || x < INT32_MIN || x > INT32_MAX) return false;
    *v = (int32_t)x;
    return true;
}

bool as_float(PyObject* o, float* v)
{
    if (PyFloat_CheckExact(o)) {
        *v = (float)PyFloat_AS_DOUBLE(o);
        return true;
    }
    int32_t i;
    if (!as_i32(o, &i)) return false;
    *v = (float)i;
    return true;
}

bool is(PyObject* o, const char* s) { return PyUnicode_CompareWithASCIIString(o, s) == 0; }

// The value of a name in `names`, or of an exact int.
bool as_kind(PyObject* o, const char* const* names, int n, int32_t* v)
{
    if (PyUnicode_CheckExact(o)) {
        for (int i = 0; i < n; ++i)
            if (is(o, names[i])) {
                *v = i;
                return true;
            }
        return false;
    }
    return as_i32(o, v);
}

const char* const kMasks[] = {"none", "causal", "sliding_window", "prefix_lm",
                              "global_sliding_window", "share_question", "causal_blockwise"};
const char* const kNorms[] = {"softmax", "relu", "sigmoid"};

// An index-mask layout: [n], or one row per sequence.
bool layout_array(const at::Tensor& t, const at::Tensor& q, int64_t nseq, int64_t* n, int64_t* stride)
{
    if (t.scalar_type() != at::kInt || t.device() != q.device()) return false;
    *stride = 0;
    if (t.dim() == 1) {
        *n = t.numel();
        return t.is_contiguous();
    }
    if (t.dim() != 2 || t.size(0) != nseq) return false;
    *n = t.size(1);
    if (*n > 0) {
        if (t.stride(1) != 1 || t.stride(0) < *n) return false;
        *stride = t.stride(0);
    }
    return true;
}

struct NoGil {
    PyThreadState* state = PyEval_SaveThread();
    ~NoGil() { PyEval_RestoreThread(state); }
};

enum Arg {
    kQ, kK, kV, kCausal, kWindow, kSlopes, kSoftcap, kScale, kCuQ, kCuK, kMaxQ, kMaxK, kOut, kLse,
    kReturnLse, kMask, kPrefix, kNumGlobal, kGlobalTokens, kSegments, kQueryStart, kRelPos, kNorm,
    kArgs
};

// True with the outputs and the library's status set when the call was made;
// false when the Python path has to take it.
bool call(PyObject* const* a, at::Tensor* out, at::Tensor* lse, bool* with_lse, int* status)
{
    at::Tensor q, k, v;
    if (!plain(a[kQ], &q) || !plain(a[kK], &k) || !plain(a[kV], &v)) return false;
    if (at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set())
        return false;
    attn_variant_desc d = {};
    d.struct_size = sizeof(d);
    const auto dt = q.scalar_type();
    if (dt != at::kBFloat16 && dt != at::kFloat) return false;
    d.dtype = dt == at::kBFloat16 ? ATTN_BF16 : ATTN_FP32;
    if (k.scalar_type() != dt || v.scalar_type() != dt) return false;
    const bool varlen = a[kCuQ] != Py_None;
    const int64_t rank = varlen ? 3 : 4;
    for (const at::Tensor* t : {&q, &k, &v})
        if (t->dim() != rank || t->device() != q.device() || t->stride(rank - 1) != 1 || broadcast(*t))
            return false;
    if (k.sizes() != v.sizes() || k.size(rank - 1) != q.size(rank - 1)) return false;
    if (!varlen && k.size(0) != q.size(0)) return false;
    for (const at::Tensor* t : {&q, &k})
        for (int64_t i = 0; i < rank; ++i)
            if (t->size(i) > INT32_MAX) return false;
    const int64_t D = q.size(rank - 1), hq = q.size(1);
    d.head_dim = (int32_t)D;

    const int causal = PyObject_IsTrue(a[kCausal]), want_lse = PyObject_IsTrue(a[kReturnLse]);
    const int relpos = PyObject_IsTrue(a[kRelPos]);
    if (causal < 0 || want_lse < 0 || relpos < 0) {
        PyErr_Clear();
        return false;
    }
    if (a[kScale] == Py_None)
        d.scale = (float)(1.0 / std::sqrt((double)D));
    else if (!as_float(a[kScale], &d.scale))
        return false;
    d.window_left = d.window_right = -1;
    if (a[kWindow] != Py_None) {
        if (!PyTuple_CheckExact(a[kWindow]) || PyTuple_GET_SIZE(a[kWindow]) < 2 ||
            !as_i32(PyTuple_GET_ITEM(a[kWindow], 0), &d.window_left) ||
            !as_i32(PyTuple_GET_ITEM(a[kWindow], 1), &d.window_right))
            return false;
    }
    if (a[kMask] != Py_None) {
        if (!as_kind(a[kMask], kMasks, 7, &d.mask_kind)) return false;
    } else {
        d.mask_kind = a[kWindow] != Py_None ? ATTN_MASK_SLIDING_WINDOW
                      : causal             ? ATTN_MASK_CAUSAL
                                           : ATTN_MASK_NONE;
    }
    if (!as_i32(a[kPrefix], &d.prefix_len) || !as_i32(a[kNumGlobal], &d.num_global) ||
        !as_i32(a[kQueryStart], &d.query_start) || !as_float(a[kSoftcap], &d.softcap) ||
        !as_kind(a[kNorm], kNorms, 3, &d.norm_kind))
        return false;
    d.relative_position = relpos;
    const bool softmax = d.norm_kind == ATTN_NORM_SOFTMAX;

    at::Tensor cuq, cuk, slopes, seg, glob;
    int64_t nseq = q.size(0), n;
    if (varlen) {
        if (!plain(a[kCuQ], &cuq)) return false;
        if (a[kCuK] == Py_None)
            cuk = cuq;
        else if (!plain(a[kCuK], &cuk))
            return false;
        for (const at::Tensor* t : {&cuq, &cuk})
            if (t->scalar_type() != at::kInt || t->device() != q.device() || t->dim() != 1 ||
                !t->is_contiguous())
                return false;
        if (cuq.numel() != cuk.numel() || cuq.numel() < 1) return false;
        if (!as_i32(a[kMaxQ], &d.max_seqlen_q) || !as_i32(a[kMaxK], &d.max_seqlen_k)) return false;
        nseq = cuq.numel() - 1;
        if (nseq > INT32_MAX) return false;
        d.cu_seqlens_q = cuq.const_data_ptr<int32_t>();
        d.cu_seqlens_k = cuk.const_data_ptr<int32_t>();
        d.total_q = q.size(0);
        d.total_k = k.size(0);
    } else {
        if (a[kCuK] != Py_None) return false;
        d.seqlen_q = (int32_t)q.size(2);
        d.seqlen_k = (int32_t)k.size(2);
    }
    d.batch = (int32_t)nseq;
    d.num_q_heads = (int32_t)hq;
    d.num_kv_heads = (int32_t)k.size(1);
    if (a[kSlopes] != Py_None) {
        if (!plain(a[kSlopes], &slopes) || slopes.scalar_type() != at::kFloat ||
            slopes.device() != q.device() || !slopes.is_contiguous() || slopes.numel() != hq)
            return false;
        d.alibi_slopes = slopes.const_data_ptr<float>();
    }
    if (a[kSegments] != Py_None) {
        if (!plain(a[kSegments], &seg) || !layout_array(seg, q, nseq, &n, &d.segment_stride) ||
            n > INT32_MAX)
            return false;
        d.num_segments = (int32_t)n;
        d.segment_starts = seg.const_data_ptr<int32_t>();
    }
    if (a[kGlobalTokens] != Py_None) {
        if (!plain(a[kGlobalTokens], &glob) || !layout_array(glob, q, nseq, &n, &d.global_stride) ||
            n > INT32_MAX || (d.num_global != 0 && d.num_global != n))
            return false;
        d.num_global = (int32_t)n;
        d.global_tokens = n ? glob.const_data_ptr<int32_t>() : nullptr;
    }

    if (a[kOut] != Py_None && (!plain(a[kOut], out) || out->scalar_type() != dt ||
                               out->sizes() != q.sizes() || out->device() != q.device()))
        return false;
    *with_lse = softmax && want_lse;
    const at::DimVector shape = varlen ? at::DimVector{hq, q.size(0)}
                                       : at::DimVector{q.size(0), hq, q.size(2)};
    if (softmax && a[kLse] != Py_None &&
        (!plain(a[kLse], lse) || lse->scalar_type() != at::kFloat || !lse->is_contiguous() ||
         lse->device() != q.device() || lse->sizes() != at::IntArrayRef(shape)))
        return false;

    // From here on no Python object is touched: other threads run meanwhile (an
    // allocation or a launch can wait for the GPU).
    const NoGil nogil;
    // outputs and workspace (kernel outputs take no part in autograd)
    at::AutoDispatchBelowADInplaceOrView below;
    if (!out->defined()) *out = at::empty_like(q);
    if (out->stride(rank - 1) != 1 || broadcast(*out)) return false;
    if (*with_lse && !lse->defined()) *lse = at::empty(shape, q.options().dtype(at::kFloat));
    const int64_t sb = varlen ? -1 : 0, ss = varlen ? 0 : 2;  // axes of the batch and token strides
    auto strides = [&](const at::Tensor& t, int64_t* b, int64_t* h, int64_t* s) {
        if (sb >= 0) *b = t.stride(sb);
        *h = t.stride(1);
        *s = t.stride(ss);
    };
    strides(q, &d.stride_q_b, &d.stride_q_h, &d.stride_q_s);
    strides(k, &d.stride_k_b, &d.stride_k_h, &d.stride_k_s);
    strides(v, &d.stride_v_b, &d.stride_v_h, &d.stride_v_s);
    strides(*out, &d.stride_o_b, &d.stride_o_h, &d.stride_o_s);
    d.stream = c10::hip::getCurrentHIPStream(q.device().index()).stream();
    const int64_t bytes = g_ws_bytes(&d);
    if (bytes < 0) return false;
    at::Tensor ws;
    if (bytes > 0) {
        try {
            ws = at::empty({bytes}, q.options().dtype(at::kByte));
        } catch (const c10::OutOfMemoryError&) {
            // No room for a workspace: the call is computed without the split. The
            // allocator frees its cached blocks before it gives up, which waits for
            // the GPU: a process at its memory limit pays that on every such call.
        }
    }
    *status = g_fwd_ws(q.const_data_ptr(), k.const_data_ptr(), v.const_data_ptr(),
                       out->mutable_data_ptr(),
                       lse->defined() ? lse->mutable_data_ptr<float>() : nullptr, &d,
                       ws.defined() ? ws.mutable_data_ptr() : nullptr, ws.defined() ? bytes : 0);
    // every other status is a refusal of the arguments, before any launch
    return *status == ATTN_OK || *status == ATTN_ERR_LAUNCH;
}

PyObject* py_fwd(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (n != kArgs) {
        PyErr_Format(PyExc_TypeError, "fwd takes %d arguments, got %zd", (int)kArgs, n);
        return nullptr;
    }
    try {
        at::Tensor out, lse;
        bool with_lse = false;
        int status = ATTN_OK;
        if (!g_fwd_ws || !call(a, &out, &lse, &with_lse, &status)) Py_RETURN_NOTIMPLEMENTED;
        if (status != ATTN_OK) {  // raises AttnError
            PyObject* abi = PyImport_ImportModule("paper_2605_05023_amd._abi");
            PyObject* none = abi ? PyObject_CallMethod(abi, "check", "i", status) : nullptr;
            Py_XDECREF(abi);
            return none;
        }
        PyObject* o = a[kOut] == Py_None ? THPVariable_Wrap(out) : Py_NewRef(a[kOut]);
        if (!o || !with_lse) return o;
        PyObject* l = a[kLse] == Py_None ? THPVariable_Wrap(lse) : Py_NewRef(a[kLse]);
        if (!l) {
            Py_DECREF(o);
            return nullptr;
        }
        PyObject* r = PyTuple_Pack(2, o, l);
        Py_DECREF(o);
        Py_DECREF(l);
        return r;
    } catch (const std::exception&) {
        // (out of memory, a device error): the Python path reports it
        PyErr_Clear();
        Py_RETURN_NOTIMPLEMENTED;
    }
}

// bind(address of attn_fwd_ws, address of attn_workspace_bytes)
PyObject* py_bind(PyObject*, PyObject* args)
{
    unsigned long long f, w;
    if (!PyArg_ParseTuple(args, "KK", &f, &w)) return nullptr;
    g_fwd_ws = reinterpret_cast<fwd_ws_t>((uintptr_t)f);
    g_ws_bytes = reinterpret_cast<ws_bytes_t>((uintptr_t)w);
    Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"fwd", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_fwd)), METH_FASTCALL,
     "The attention forward, or NotImplemented where the Python path has to take the call."},
    {"bind", py_bind, METH_VARARGS, "Set the entry points of libattn.so."},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_fast", nullptr, -1, kMethods, nullptr, nullptr, nullptr,
                       nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fast() { return PyModule_Create(&kModule); }
