// CPython marshalling of the package's entry points: torch tensors to the C
// ABI's pointers and strides, outputs and workspaces from torch's allocator,
// the current stream.  Host time bounds the smallest calls (a committed unit:
// 3 us of kernel behind 10 us of ctypes marshalling), so the common case runs
// here: device tensors, (host, device) pairs of int32 arrays.  Anything else
// (another type, a wrong shape or dtype) returns None before anything is
// enqueued, and the Python code, which states the checks and
// raises their errors, takes the call.  Python objects are read first; the
// allocations and the C ABI call (validation, planning, launches, which block
// on a full hardware queue) run without the GIL, as through ctypes.
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>

#include <algorithm>
#include <cmath>

#include "../../include/ws_attn.h"

namespace {

// C ABI functions, by address (the package loads the library and hands its
// addresses over, so both speak to the same one)
struct Abi {
    decltype(&ws_kv_append) kv_append;
    decltype(&ws_kv_append_varlen) kv_append_varlen;
    decltype(&ws_block_causal_attn_fwd) fwd;
    decltype(&ws_block_causal_attn_fwd_text) fwd_text;
    decltype(&ws_block_causal_attn_fwd_varlen) fwd_varlen;
    decltype(&ws_block_causal_attn_fwd_noalloc) fwd_noalloc;
    decltype(&ws_block_causal_prefill) prefill;
    decltype(&ws_block_causal_prefill_text) prefill_text;
    decltype(&ws_block_causal_prefill_bwd) bwd;
    decltype(&ws_workspace_bytes) workspace_bytes;
    decltype(&ws_step_workspace_bytes_varlen) workspace_bytes_varlen;
} abi;

PyObject *cache_class;   // PagedCache

PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 1 + (Py_ssize_t)(sizeof(Abi) / sizeof(void *))) {
        PyErr_SetString(PyExc_TypeError, "the cache class and one address per ABI function");
        return nullptr;
    }
    for (Py_ssize_t i = 1; i < n; ++i) {
        void *p = PyLong_AsVoidPtr(args[i]);
        if (PyErr_Occurred()) return nullptr;
        ((void **)&abi)[i - 1] = p;
    }
    Py_INCREF(args[0]);
    Py_XSETREF(cache_class, args[0]);
    Py_RETURN_NONE;
}

// A plain torch.Tensor (no subclass: those may hold no memory), else nullptr
const at::Tensor *tensor(PyObject *o) {
    if ((PyObject *)Py_TYPE(o) != THPVariableClass) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.defined() && t.layout() == at::kStrided && t.has_storage() ? &t : nullptr;
}

bool shaped(const at::Tensor &t, std::initializer_list<int64_t> shape) { return t.sizes() == at::IntArrayRef(shape); }

// descriptor of a [B][L][H][d] device tensor with a contiguous last dim
bool token_tensor(const at::Tensor *t, std::initializer_list<int64_t> shape, ws_tensor4 &d) {
    if (!t || !t->is_cuda() || !shaped(*t, shape) || t->stride(3) != 1) return false;
    const auto dt = t->scalar_type();
    if (dt != at::kBFloat16 && dt != at::kFloat) return false;
    d = ws_tensor4{t->data_ptr(), dt == at::kBFloat16 ? WS_DTYPE_BF16 : WS_DTYPE_F32, t->stride(0), t->stride(1),
                   t->stride(2)};
    return true;
}

struct Ints {
    const int32_t *host = nullptr, *dev = nullptr;
    const at::Tensor *h = nullptr;
};

// a (host, device) pair of int32 arrays of the given shape (packed: any shape
// of that many contiguous elements); None gives null pointers (so an empty
// array, whose pointers are null too, is declined)
bool int_pair(PyObject *o, std::initializer_list<int64_t> shape, bool packed, Ints &x) {
    if (o == Py_None) return true;
    if (!PyTuple_CheckExact(o) || PyTuple_GET_SIZE(o) != 2) return false;
    const at::Tensor *t[2] = {tensor(PyTuple_GET_ITEM(o, 0)), tensor(PyTuple_GET_ITEM(o, 1))};
    int64_t numel = 1;
    for (int64_t n : shape) numel *= n;
    if (numel == 0) return false;
    for (const at::Tensor *p : t) {
        if (!p || p->scalar_type() != at::kInt) return false;
        if (packed ? (p->numel() != numel || !p->is_contiguous()) : !shaped(*p, shape)) return false;
    }
    if (!t[0]->is_cpu() || !t[1]->is_cuda()) return false;
    x.host = (const int32_t *)t[0]->data_ptr();
    x.dev = (const int32_t *)t[1]->data_ptr();
    x.h = t[0];
    return true;
}

// Runs its scope without the GIL.
struct NoGil {
    PyThreadState *state = PyEval_SaveThread();
    ~NoGil() { PyEval_RestoreThread(state); }
};

PyObject *names[7];   // attribute names of PagedCache, in the order below

// The paged cache's descriptor, with its table checked for `batch` rows.  The
// cache's tensors are held: without the GIL another thread may replace them.
struct Paged : ws_paged_kv {
    at::Tensor hold[4];
};
bool paged(PyObject *cache, int64_t batch, Paged &d) {
    // (another class may have a descriptor of its own: desc())
    if ((PyObject *)Py_TYPE(cache) != cache_class) return false;
    PyObject *v[7] = {};
    bool ok = true;
    for (int i = 0; i < 7 && ok; ++i) ok = (v[i] = PyObject_GetAttr(cache, names[i])) != nullptr;
    if (!ok) PyErr_Clear();
    const at::Tensor *k = nullptr, *vp = nullptr, *th = nullptr, *td = nullptr;
    if (ok) {
        k = tensor(v[0]);
        vp = tensor(v[1]);
        th = tensor(v[2]);
        td = tensor(v[3]);
        ok = k && vp && th && td && th->dim() == 2 && th->size(0) >= batch && td->sizes() == th->sizes() &&
             PyLong_CheckExact(v[4]) && PyLong_CheckExact(v[5]) && PyLong_CheckExact(v[6]);
    }
    if (ok) {
        static_cast<ws_paged_kv &>(d) = ws_paged_kv{k->data_ptr(), vp->data_ptr(), (const int32_t *)td->data_ptr(), (const int32_t *)th->data_ptr(),
                        (int32_t)PyLong_AsLong(v[4]), WS_PAGE_SIZE, (int32_t)th->size(1), (int32_t)PyLong_AsLong(v[5]),
                        (int32_t)PyLong_AsLong(v[6])};
        d.hold[0] = *k, d.hold[1] = *vp, d.hold[2] = *th, d.hold[3] = *td;
    }
    for (PyObject *o : v) Py_XDECREF(o);
    return ok;
}

void *stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

// scale: None (1 / sqrt(d)) or a float
bool scale_of(PyObject *o, int64_t d, float &s) {
    if (o == Py_None) {
        s = (float)(1.0 / std::sqrt((double)d));
        return true;
    }
    if (!PyFloat_CheckExact(o)) return false;
    s = (float)PyFloat_AS_DOUBLE(o);
    return true;
}

// The caller's output of the given shape, or, for None, undefined
bool given(PyObject *o, std::initializer_list<int64_t> shape, at::Tensor &t) {
    if (o == Py_None) return true;
    const at::Tensor *p = tensor(o);
    if (!p || !p->is_cuda() || !shaped(*p, shape)) return false;
    t = *p;
    return true;
}

// A new output of the given shape where the caller gave none
void allocate(at::Tensor &t, std::initializer_list<int64_t> shape, at::ScalarType type, const at::Tensor &like) {
    if (!t.defined()) t = at::empty(at::IntArrayRef(shape), like.options().dtype(type));
}

bool flag(PyObject *o, bool &b) {
    if (o != Py_True && o != Py_False) return false;
    b = o == Py_True;
    return true;
}

at::ScalarType dtype_of(PyObject *o) {
    return THPDtype_Check(o) ? ((THPDtype *)o)->scalar_type : at::kDouble;
}

// (status, tensors...), None for an undefined one
PyObject *result(int rc, std::initializer_list<at::Tensor> out) {
    THPObjectPtr r(PyTuple_New(1 + (Py_ssize_t)out.size()));
    if (!r) return nullptr;
    PyObject *s = PyLong_FromLong(rc);
    if (!s) return nullptr;
    PyTuple_SET_ITEM(r.get(), 0, s);
    Py_ssize_t i = 1;
    for (const at::Tensor &t : out) {
        PyObject *o = t.defined() ? THPVariable_Wrap(t) : (Py_INCREF(Py_None), Py_None);
        if (!o) return nullptr;
        PyTuple_SET_ITEM(r.get(), i++, o);
    }
    return r.release();
}

// append(cache, lens, k_new, v_new, new_lens) -> status, or None
PyObject *append(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 5) Py_RETURN_NONE;
    const at::Tensor *k = tensor(a[2]);
    if (!k || k->dim() != 4) Py_RETURN_NONE;
    const int64_t B = k->size(0), L = k->size(1);
    Paged kv{};
    ws_tensor4 kd, vd;
    Ints lens, nl;
    if (!paged(a[0], B, kv) || !token_tensor(k, {B, L, kv.num_kv_heads, kv.head_dim}, kd) ||
        !token_tensor(tensor(a[3]), {B, L, kv.num_kv_heads, kv.head_dim}, vd) || a[1] == Py_None ||
        !int_pair(a[1], {B}, false, lens) || !int_pair(a[4], {B}, true, nl))
        Py_RETURN_NONE;
    int rc;
    {
        NoGil free;
        rc = nl.host ? abi.kv_append_varlen(&kv, B, lens.host, lens.dev, nl.host, nl.dev, L, kd, vd, stream())
                     : abi.kv_append(&kv, B, lens.host, lens.dev, L, kd, vd, stream());
    }
    return PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

// step(q, k_new, v_new, cache, lens, scale, fuse_append, out, out_dtype,
//      want_lse, lse, workspace, text_starts, new_lens, noalloc)
//   -> (status, out, lse), or None
PyObject *step(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 15) Py_RETURN_NONE;
    const at::Tensor *q = tensor(a[0]);
    if (!q || q->dim() != 4) Py_RETURN_NONE;
    const int64_t B = q->size(0), L = q->size(1), H = q->size(2), D = q->size(3);
    if (B == 0 || L == 0) Py_RETURN_NONE;
    Paged kv{};
    ws_tensor4 qd, kd, vd, od;
    Ints lens, text, nl;
    bool fuse, want_lse, noalloc;
    float scale;
    if (!flag(a[6], fuse) || !flag(a[9], want_lse) || !flag(a[14], noalloc) || !paged(a[3], B, kv) || kv.head_dim != D ||
        !token_tensor(q, {B, L, H, D}, qd) || !token_tensor(tensor(a[1]), {B, L, kv.num_kv_heads, D}, kd) ||
        !token_tensor(tensor(a[2]), {B, L, kv.num_kv_heads, D}, vd) || a[4] == Py_None ||
        !int_pair(a[4], {B}, false, lens) || !scale_of(a[5], D, scale) || !int_pair(a[12], {B}, true, text) ||
        !int_pair(a[13], {B}, true, nl))
        Py_RETURN_NONE;
    const at::ScalarType type = a[7] == Py_None ? dtype_of(a[8]) : at::kBFloat16;
    if (type != at::kBFloat16 && type != at::kFloat) Py_RETURN_NONE;
    const at::Tensor *wsp = a[11] == Py_None ? nullptr : tensor(a[11]);
    if (a[11] != Py_None && !wsp) Py_RETURN_NONE;
    at::Tensor out, lse, own;
    const bool with_lse = want_lse || a[10] != Py_None;
    if (!given(a[7], {B, L, H, D}, out) || (out.defined() && !token_tensor(&out, {B, L, H, D}, od)) ||
        !given(a[10], {B, H, L}, lse))
        Py_RETURN_NONE;
    const int flags = fuse ? WS_FUSE_APPEND : 0;
    int rc;
    {
        NoGil free;
        allocate(out, {B, L, H, D}, type, *q);
        token_tensor(&out, {B, L, H, D}, od);
        if (with_lse) allocate(lse, {B, H, L}, at::kFloat, *q);
        float *lp = lse.defined() ? (float *)lse.data_ptr() : nullptr;
        void *wp = nullptr;
        size_t wn = 0;
        if (wsp) {
            wp = wsp->data_ptr();
            wn = wsp->numel();
        } else if (!noalloc) {
            int32_t most = 0;
            for (int64_t b = 0; b < B; ++b) most = std::max(most, lens.host[b * lens.h->stride(0)]);
            wn = nl.host ? abi.workspace_bytes_varlen(B, H, kv.num_kv_heads, L, lens.host, nl.host)
                         : abi.workspace_bytes(WS_OP_STEP, B, H, kv.num_kv_heads, L, (int32_t)std::min<int64_t>(most + L, INT32_MAX));
            if (wn) {
                own = at::empty({(int64_t)wn}, q->options().dtype(at::kByte));
                wp = own.data_ptr();
            }
        }
        if (noalloc)
            rc = abi.fwd_noalloc(qd, kd, vd, &kv, lens.host, lens.dev, B, L, H, scale, flags, od, lp, stream());
        else if (nl.host)
            rc = abi.fwd_varlen(qd, kd, vd, &kv, lens.host, lens.dev, nl.host, nl.dev, text.host, text.dev, B, L, H, scale,
                                flags, od, lp, wp, wn, stream());
        else if (text.host)
            rc = abi.fwd_text(qd, kd, vd, &kv, lens.host, lens.dev, text.host, text.dev, B, L, H, scale, flags, od, lp, wp,
                              wn, stream());
        else
            rc = abi.fwd(qd, kd, vd, &kv, lens.host, lens.dev, B, L, H, scale, flags, od, lp, wp, wn, stream());
    }
    return result(rc, {out, lse});
    END_HANDLE_TH_ERRORS
}

// prefill(q, k, v, offsets, scale, cache, num_kv_heads, out, out_dtype,
//         want_lse, lse, text_starts) -> (status, out, lse), or None
PyObject *prefill(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 12) Py_RETURN_NONE;
    const at::Tensor *q = tensor(a[0]);
    if (!q || q->dim() != 4) Py_RETURN_NONE;
    const int64_t B = q->size(0), L = q->size(1), H = q->size(2), D = q->size(3);
    const bool contiguous = a[1] != Py_None;
    if (contiguous != (a[2] != Py_None)) Py_RETURN_NONE;
    Paged kv{};
    ws_tensor4 qd, kd{nullptr, WS_DTYPE_BF16, 0, 0, 0}, vd = kd, od;
    Ints off, text;
    bool want_lse;
    float scale;
    int64_t hkv = 0;
    if (!flag(a[9], want_lse) || !token_tensor(q, {B, L, H, D}, qd) || !scale_of(a[4], D, scale)) Py_RETURN_NONE;
    if (contiguous) {
        const at::Tensor *k = tensor(a[1]);
        if (!k || k->dim() != 4) Py_RETURN_NONE;
        hkv = k->size(2);
        if (!token_tensor(k, {B, L, hkv, D}, kd) || !token_tensor(tensor(a[2]), {B, L, hkv, D}, vd)) Py_RETURN_NONE;
    }
    if (a[5] != Py_None) {
        if (!paged(a[5], contiguous ? 0 : B, kv)) Py_RETURN_NONE;
    } else if (!contiguous) {
        Py_RETURN_NONE;
    }
    if (!contiguous) {
        hkv = kv.num_kv_heads;
        if (a[6] != Py_None) {
            if (!PyLong_CheckExact(a[6])) Py_RETURN_NONE;
            hkv = PyLong_AsLong(a[6]);
        }
    }
    if (!PyTuple_CheckExact(a[3]) || PyTuple_GET_SIZE(a[3]) != 2) Py_RETURN_NONE;
    const at::Tensor *oh = tensor(PyTuple_GET_ITEM(a[3], 0));
    if (!oh || oh->dim() != 2) Py_RETURN_NONE;
    const int64_t nb = oh->size(1) - 1;
    if (nb < 0 || !int_pair(a[3], {B, nb + 1}, false, off) || !int_pair(a[11], {B, nb}, true, text)) Py_RETURN_NONE;
    const at::ScalarType type = a[7] == Py_None ? dtype_of(a[8]) : at::kBFloat16;
    if (type != at::kBFloat16 && type != at::kFloat) Py_RETURN_NONE;
    at::Tensor out, lse;
    const bool with_lse = want_lse || a[10] != Py_None;
    if (!given(a[7], {B, L, H, D}, out) || (out.defined() && !token_tensor(&out, {B, L, H, D}, od)) ||
        !given(a[10], {B, H, L}, lse))
        Py_RETURN_NONE;
    const ws_paged_kv *kvp = a[5] != Py_None ? &kv : nullptr;
    int rc;
    {
        NoGil free;
        allocate(out, {B, L, H, D}, type, *q);
        token_tensor(&out, {B, L, H, D}, od);
        if (with_lse) allocate(lse, {B, H, L}, at::kFloat, *q);
        float *lp = lse.defined() ? (float *)lse.data_ptr() : nullptr;
        rc = text.host ? abi.prefill_text(qd, kd, vd, kvp, off.host, off.dev, text.host, text.dev, B, L, nb, H, hkv, D, scale,
                                          od, lp, stream())
                       : abi.prefill(qd, kd, vd, kvp, off.host, off.dev, B, L, nb, H, hkv, D, scale, od, lp, stream());
    }
    return result(rc, {out, lse});
    END_HANDLE_TH_ERRORS
}

// prefill_bwd(q, k, v, o, dout, lse, offsets, scale, text_starts, dq, dk, dv,
//             workspace) -> (status, dq, dk, dv), or None
PyObject *prefill_bwd(PyObject *, PyObject *const *a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 13) Py_RETURN_NONE;
    const at::Tensor *q = tensor(a[0]), *k = tensor(a[1]), *lse = tensor(a[5]);
    if (!q || q->dim() != 4 || !k || k->dim() != 4 || !lse) Py_RETURN_NONE;
    const int64_t B = q->size(0), L = q->size(1), H = q->size(2), D = q->size(3), hkv = k->size(2);
    if (B == 0 || L == 0) Py_RETURN_NONE;
    ws_tensor4 qd, kd, vd, od, dd, dqd, dkd, dvd;
    Ints off, text;
    float scale;
    if (!token_tensor(q, {B, L, H, D}, qd) || !token_tensor(k, {B, L, hkv, D}, kd) ||
        !token_tensor(tensor(a[2]), {B, L, hkv, D}, vd) || !token_tensor(tensor(a[3]), {B, L, H, D}, od) ||
        !token_tensor(tensor(a[4]), {B, L, H, D}, dd) || !lse->is_cuda() || !shaped(*lse, {B, H, L}) ||
        !scale_of(a[7], D, scale) || !PyTuple_CheckExact(a[6]) || PyTuple_GET_SIZE(a[6]) != 2)
        Py_RETURN_NONE;
    const at::Tensor *oh = tensor(PyTuple_GET_ITEM(a[6], 0));
    if (!oh || oh->dim() != 2) Py_RETURN_NONE;
    const int64_t nb = oh->size(1) - 1;
    if (nb < 0 || !int_pair(a[6], {B, nb + 1}, false, off) || !int_pair(a[8], {B, nb}, true, text)) Py_RETURN_NONE;
    const at::Tensor *wsp = a[12] == Py_None ? nullptr : tensor(a[12]);
    if (a[12] != Py_None && !wsp) Py_RETURN_NONE;
    at::Tensor dq, dk, dv, own;
    if (!given(a[9], {B, L, H, D}, dq) || (dq.defined() && !token_tensor(&dq, {B, L, H, D}, dqd)) ||
        !given(a[10], {B, L, hkv, D}, dk) || (dk.defined() && !token_tensor(&dk, {B, L, hkv, D}, dkd)) ||
        !given(a[11], {B, L, hkv, D}, dv) || (dv.defined() && !token_tensor(&dv, {B, L, hkv, D}, dvd)))
        Py_RETURN_NONE;
    int rc = -1;
    {
        NoGil free;
        const size_t need = wsp ? 0 : abi.workspace_bytes(WS_OP_PREFILL_BWD, B, H, hkv, L, L);
        if (wsp || need) {
            allocate(dq, {B, L, H, D}, at::kFloat, *q);
            allocate(dk, {B, L, hkv, D}, at::kFloat, *q);
            allocate(dv, {B, L, hkv, D}, at::kFloat, *q);
            token_tensor(&dq, {B, L, H, D}, dqd);
            token_tensor(&dk, {B, L, hkv, D}, dkd);
            token_tensor(&dv, {B, L, hkv, D}, dvd);
            if (!wsp) {
                own = at::empty({(int64_t)need}, q->options().dtype(at::kByte));
                wsp = &own;
            }
            rc = abi.bwd(qd, kd, vd, od, dd, (const float *)lse->data_ptr(), off.host, off.dev, text.host, text.dev, B, L, nb,
                         H, hkv, D, scale, dqd, dkd, dvd, wsp->data_ptr(), wsp->numel(), stream());
        }
    }
    if (rc < 0) Py_RETURN_NONE;   // (the Python code names the mistake)
    return result(rc, {dq, dk, dv});
    END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"bind", (PyCFunction)(void (*)())bind, METH_FASTCALL, "the cache class, then the C ABI's addresses in Abi's order"},
    {"append", (PyCFunction)(void (*)())append, METH_FASTCALL, nullptr},
    {"step", (PyCFunction)(void (*)())step, METH_FASTCALL, nullptr},
    {"prefill", (PyCFunction)(void (*)())prefill, METH_FASTCALL, nullptr},
    {"prefill_bwd", (PyCFunction)(void (*)())prefill_bwd, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_wsbinding", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__wsbinding() {
    const char *n[7] = {"k_pool", "v_pool", "page_table_host", "page_table", "num_pages", "num_kv_heads", "head_dim"};
    for (int i = 0; i < 7; ++i)
        if (!(names[i] = PyUnicode_InternFromString(n[i]))) return nullptr;
    return PyModule_Create(&module);
}
