// fastcall.cpp -- the torch-tensor calls of the Python binding (fbl.py) in
// native code: argument marshalling only, the work is behind the C ABI.
//
// Why: a call through ctypes spends 10 .. 16 us in Python -- building 4 to 9
// layout descriptors, device and dtype checks, 12 to 25 argument conversions --
// and the small calls are bound by it.  Read straight from the tensors the same
// takes under 1 us beside the launches.  Host time of a pass, before and after:
// forward + backward in two launches 29 -> 6.2 us, in four 34 -> 10.4, three
// projection products 31 -> 8.5, a LoRA adapter's six 62 -> 17 (its step 64 ->
// 26 us: now the kernels').
//
// Every function takes all arguments of its namesake by position and either
// does the whole call and returns its result, or does nothing and returns None:
// then the caller runs its own general path, which makes every check and raises
// every error.  So only plain calls are handled here -- exact torch.Tensor (or
// Parameter) arguments in strided device memory on the current device without
// wrapper or lazy-view state, plain Python numbers, the current stream -- and
// an error status of the C ABI (nothing enqueued) also goes back to the caller.
// Nothing is cached.
#include <ATen/ATen.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <c10/hip/HIPFunctions.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <cmath>

#include "../../include/fbl.h"

#define FBL_STR2(x) #x
#define FBL_STR(x) FBL_STR2(x)
#define FBL_PYTHON FBL_STR(PY_MAJOR_VERSION) "." FBL_STR(PY_MINOR_VERSION)

namespace {

using at::Tensor;

// ------------------------------------------------------------ plain arguments
// A tensor whose memory is what its sizes and strides say: no subclass, no
// functional, batching or grad-tracking wrapper, no conjugate or negative view.
const Tensor* plain(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const Tensor& t = THPVariable_Unpack(o);
    static const uint64_t allowed = (c10::DispatchKeySet(c10::DispatchKey::Dense) |
                                     c10::DispatchKeySet(c10::BackendComponent::CUDABit) |
                                     c10::DispatchKeySet(c10::DispatchKey::AutogradFunctionality) |
                                     c10::DispatchKeySet(c10::DispatchKey::ADInplaceOrView) |
                                     c10::DispatchKeySet(c10::DispatchKey::AutocastCUDA))
                                        .raw_repr();
    if (!t.defined() || !t.is_cuda() || (t.key_set().raw_repr() & ~allowed)) return nullptr;
    return &t;
}

// The call's arguments, read one after the other; `ok` falls at the first that is not plain.
struct Args {
    PyObject* const* a;
    bool ok = true;
    int device = -1;  // of the first tensor; all others must be on it
    const Tensor* tensor(int i) {
        const Tensor* t = ok ? plain(a[i]) : nullptr;
        if (!t) return ok = false, nullptr;
        const int d = t->device().index();
        if (device < 0) device = d;
        if (d != device) ok = false;
        return t;
    }
    const Tensor* tensor_or_none(int i) { return a[i] == Py_None ? nullptr : tensor(i); }
    int64_t integer(int i) {
        int overflow = 0;
        if (!ok || !PyLong_CheckExact(a[i])) return ok = false, 0;
        const long long v = PyLong_AsLongLongAndOverflow(a[i], &overflow);
        if (overflow || v < INT32_MIN || v > INT32_MAX) ok = false;
        return v;
    }
    bool flag(int i) {
        if (a[i] != Py_True && a[i] != Py_False) ok = false;
        return a[i] == Py_True;
    }
    // softmax scale: None is 1 / sqrt(D)
    float scale(int i, int64_t D) {
        if (a[i] == Py_None) return (float)(1.0 / std::sqrt((double)D));
        if (!PyFloat_CheckExact(a[i])) return ok = false, 0.f;
        return (float)PyFloat_AS_DOUBLE(a[i]);
    }
    void no_stream(int i) {
        if (a[i] != Py_None) ok = false;
    }
    bool ready() const { return ok && device >= 0 && (int)c10::hip::current_device() == device; }
    void* stream() const {
        return (void*)c10::hip::getCurrentHIPStreamMasqueradingAsCUDA((c10::DeviceIndex)device).stream();
    }
};

int dtype_code(const Tensor& t) {
    return t.scalar_type() == at::kBFloat16 ? FBL_BF16 : t.scalar_type() == at::kFloat ? FBL_F32 : -1;
}

// Descriptor of a token-major [B, S, H*D] tensor.
bool layout(const Tensor* t, int64_t H, fbl_layout* l) {
    if (!t || t->dim() != 3 || H <= 0 || t->size(2) % H || t->stride(2) != 1 || dtype_code(*t) < 0) return false;
    const int64_t B = t->size(0);
    return fbl_layout_desc(l, dtype_code(*t), B, t->size(1), H, t->size(2) / H, t->stride(1), B > 1 ? t->stride(0) : 0,
                           0) == FBL_OK;
}

// Descriptors and addresses of Q, K, V in a packed [B, S, (Hq + 2 Hkv) D] tensor.
struct Packed {
    fbl_layout q, k, v;
    char *pq, *pk, *pv;
    bool set(const Tensor* t, int64_t Hq, int64_t Hkv) {
        if (!t || t->dim() != 3 || Hq <= 0 || Hkv <= 0 || t->stride(2) != 1 || t->stride(1) != t->size(2) ||
            t->size(2) % (Hq + 2 * Hkv) || dtype_code(*t) < 0)
            return false;
        int64_t ko = 0, vo = 0;
        if (fbl_layout_packed_qkv(&q, &k, &v, &ko, &vo, dtype_code(*t), t->size(0), t->size(1), Hq, Hkv,
                                  t->size(2) / (Hq + 2 * Hkv), t->size(0) > 1 ? t->stride(0) : 0, 0) != FBL_OK)
            return false;
        pq = static_cast<char*>(t->data_ptr());
        pk = pq + ko * (int64_t)t->element_size();
        pv = pq + vo * (int64_t)t->element_size();
        return true;
    }
};

bool kv_len_fits(const Tensor* t, int64_t B) {
    return !t || (t->scalar_type() == at::kInt && t->dim() == 1 && (t->numel() <= 1 || t->stride(0) == 1) &&
                  t->numel() >= B);
}
bool lse_fits(const Tensor* t, int64_t B, int64_t Hq, int64_t S) {
    return !t || (t->scalar_type() == at::kFloat && t->dim() == 3 && t->size(0) == B && t->size(1) == Hq &&
                  t->size(2) == S && t->is_contiguous());
}
fbl_mask mask_of(bool causal, const Tensor* kv_len) {
    fbl_mask m{};
    m.kind = (causal ? FBL_MASK_CAUSAL : 0u) | (kv_len ? FBL_MASK_KEY_PADDING : 0u);
    m.kv_len = kv_len ? static_cast<const int32_t*>(kv_len->data_ptr()) : nullptr;
    return m;
}

// The library call without the interpreter lock (no tensor is read in it).
template <typename F>
fbl_status unlocked(F&& f) {
    PyThreadState* save = PyEval_SaveThread();
    const fbl_status st = f();
    PyEval_RestoreThread(save);
    return st;
}

// Result objects: the caller's own where it gave one, else the new tensor.
PyObject* object_of(PyObject* given, const Tensor& made) {
    if (given != Py_None) return Py_NewRef(given);
    return THPVariable_Wrap(made);
}
template <int N>
PyObject* tuple_of(PyObject* const (&x)[N]) {
    PyObject* t = PyTuple_New(N);
    bool bad = !t;
    for (PyObject* o : x) bad = bad || !o;
    for (int i = 0; i < N; ++i)
        if (!bad) PyTuple_SET_ITEM(t, i, x[i]);
        else Py_XDECREF(x[i]);
    if (bad) Py_CLEAR(t);
    return t;
}

Tensor empty(at::IntArrayRef size, at::ScalarType type, const Tensor& like) {
    return at::empty(size, at::TensorOptions().dtype(type).device(like.device()));
}

// ---------------------------------------------------------------------- calls
// attn_fwd(q, k, v, Hq, Hkv, scale, causal, kv_len, out, lse, stream, tile)
PyObject* attn_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 12) Py_RETURN_NONE;
    Args g{a};
    const Tensor *q = g.tensor(0), *k = g.tensor(1), *v = g.tensor(2);
    const int64_t Hq = g.integer(3), Hkv = g.integer(4);
    const bool causal = g.flag(6);
    const Tensor *kv_len = g.tensor_or_none(7), *out = g.tensor_or_none(8), *lse = g.tensor_or_none(9);
    g.no_stream(10);
    const int64_t tile = g.integer(11);
    fbl_layout lq, lk, lv, lo;
    if (!g.ready() || !layout(q, Hq, &lq) || !layout(k, Hkv, &lk) || !layout(v, Hkv, &lv)) Py_RETURN_NONE;
    const float scale = g.scale(5, lq.D);
    if (!g.ok || !kv_len_fits(kv_len, lq.B) || !lse_fits(lse, lq.B, Hq, lq.S)) Py_RETURN_NONE;
    Tensor made_o, made_lse;
    if (!out) made_o = empty(q->sizes(), q->scalar_type(), *q), out = &made_o;
    if (!lse) made_lse = empty({lq.B, Hq, lq.S}, at::kFloat, *q), lse = &made_lse;
    if (!layout(out, Hq, &lo)) Py_RETURN_NONE;
    const fbl_mask m = mask_of(causal, kv_len);
    void *s = g.stream(), *pq = q->data_ptr(), *pk = k->data_ptr(), *pv = v->data_ptr(), *po = out->data_ptr();
    float* pl = static_cast<float*>(lse->data_ptr());
    const fbl_status st = unlocked([&] {
        return fbl_attn_fwd_tiled(&lq, pq, &lk, pk, &lv, pv, &lo, po, pl, scale, m, (int32_t)tile, s);
    });
    if (st != FBL_OK) Py_RETURN_NONE;
    return tuple_of<2>({object_of(a[8], made_o), object_of(a[9], made_lse)});
    END_HANDLE_TH_ERRORS
}

// attn_bwd(q, k, v, o, do, lse, Hq, Hkv, scale, causal, kv_len, dq, dk, dv, workspace, stream, phases, kv_tile, dq_tile)
PyObject* attn_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 19) Py_RETURN_NONE;
    Args g{a};
    const Tensor *q = g.tensor(0), *k = g.tensor(1), *v = g.tensor(2), *o = g.tensor(3), *dO = g.tensor(4);
    const Tensor* lse = g.tensor(5);
    const int64_t Hq = g.integer(6), Hkv = g.integer(7);
    const bool causal = g.flag(9);
    const Tensor *kv_len = g.tensor_or_none(10), *dq = g.tensor_or_none(11), *dk = g.tensor_or_none(12);
    const Tensor *dv = g.tensor_or_none(13), *ws = g.tensor_or_none(14);
    g.no_stream(15);
    const int64_t phases = g.integer(16), kv_tile = g.integer(17), dq_tile = g.integer(18);
    fbl_layout lq, lk, lv, lo, ldo, ldq, ldk, ldv;
    if (!g.ready() || phases < 0 || !layout(q, Hq, &lq) || !layout(k, Hkv, &lk) || !layout(v, Hkv, &lv) ||
        !layout(o, Hq, &lo) || !layout(dO, Hq, &ldo))
        Py_RETURN_NONE;
    const float scale = g.scale(8, lq.D);
    if (!g.ok || !kv_len_fits(kv_len, lq.B) || !lse_fits(lse, lq.B, Hq, lq.S) || (ws && !ws->is_contiguous()))
        Py_RETURN_NONE;
    Tensor made_q, made_k, made_v, made_ws;
    if (!dq) made_q = empty(q->sizes(), q->scalar_type(), *q), dq = &made_q;
    if (!dk) made_k = empty(k->sizes(), k->scalar_type(), *q), dk = &made_k;
    if (!dv) made_v = empty(v->sizes(), v->scalar_type(), *q), dv = &made_v;
    if (!ws) {
        size_t need = 0;
        if (fbl_attn_bwd_workspace(&lq, &lk, &need) != FBL_OK) Py_RETURN_NONE;
        made_ws = empty({(int64_t)need}, at::kByte, *q), ws = &made_ws;
    }
    if (!layout(dq, Hq, &ldq) || !layout(dk, Hkv, &ldk) || !layout(dv, Hkv, &ldv)) Py_RETURN_NONE;
    const fbl_mask m = mask_of(causal, kv_len);
    void *s = g.stream(), *pq = q->data_ptr(), *pk = k->data_ptr(), *pv = v->data_ptr(), *po = o->data_ptr();
    void *pg = dO->data_ptr(), *pdq = dq->data_ptr(), *pdk = dk->data_ptr(), *pdv = dv->data_ptr();
    void* pw = ws->data_ptr();
    const float* pl = static_cast<const float*>(lse->data_ptr());
    const size_t ws_bytes = (size_t)(ws->numel() * ws->element_size());
    const fbl_status st = unlocked([&] {
        return fbl_attn_bwd_tiled((uint32_t)phases, &lq, pq, &lk, pk, &lv, pv, &lo, po, &ldo, pg, pl, scale, m, &ldq,
                                  pdq, &ldk, pdk, &ldv, pdv, pw, ws_bytes, (int32_t)kv_tile, (int32_t)dq_tile, s);
    });
    if (st != FBL_OK) Py_RETURN_NONE;
    return tuple_of<3>({object_of(a[11], made_q), object_of(a[12], made_k), object_of(a[13], made_v)});
    END_HANDLE_TH_ERRORS
}

// attn_fwd_packed(qkv, Hq, Hkv, scale, causal, kv_len, out, lse, stream)
PyObject* attn_fwd_packed(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 9) Py_RETURN_NONE;
    Args g{a};
    const Tensor* qkv = g.tensor(0);
    const int64_t Hq = g.integer(1), Hkv = g.integer(2);
    const bool causal = g.flag(4);
    const Tensor *kv_len = g.tensor_or_none(5), *out = g.tensor_or_none(6), *lse = g.tensor_or_none(7);
    g.no_stream(8);
    Packed p;
    fbl_layout lo;
    if (!g.ready() || !p.set(qkv, Hq, Hkv)) Py_RETURN_NONE;
    const float scale = g.scale(3, p.q.D);
    if (!g.ok || !kv_len_fits(kv_len, p.q.B) || !lse_fits(lse, p.q.B, Hq, p.q.S)) Py_RETURN_NONE;
    Tensor made_o, made_lse;
    if (!out) made_o = empty({p.q.B, p.q.S, Hq * p.q.D}, qkv->scalar_type(), *qkv), out = &made_o;
    if (!lse) made_lse = empty({p.q.B, Hq, p.q.S}, at::kFloat, *qkv), lse = &made_lse;
    if (!layout(out, Hq, &lo)) Py_RETURN_NONE;
    const fbl_mask m = mask_of(causal, kv_len);
    void *s = g.stream(), *po = out->data_ptr();
    float* pl = static_cast<float*>(lse->data_ptr());
    const fbl_status st = unlocked(
        [&] { return fbl_attn_fwd(&p.q, p.pq, &p.k, p.pk, &p.v, p.pv, &lo, po, pl, scale, m, s); });
    if (st != FBL_OK) Py_RETURN_NONE;
    return tuple_of<2>({object_of(a[6], made_o), object_of(a[7], made_lse)});
    END_HANDLE_TH_ERRORS
}

// attn_bwd_packed(qkv, o, do, lse, Hq, Hkv, scale, causal, kv_len, dqkv, workspace, stream)
PyObject* attn_bwd_packed(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 12) Py_RETURN_NONE;
    Args g{a};
    const Tensor *qkv = g.tensor(0), *o = g.tensor(1), *dO = g.tensor(2), *lse = g.tensor(3);
    const int64_t Hq = g.integer(4), Hkv = g.integer(5);
    const bool causal = g.flag(7);
    const Tensor *kv_len = g.tensor_or_none(8), *dqkv = g.tensor_or_none(9), *ws = g.tensor_or_none(10);
    g.no_stream(11);
    Packed p, d;
    fbl_layout lo, ldo;
    if (!g.ready() || !p.set(qkv, Hq, Hkv) || !layout(o, Hq, &lo) || !layout(dO, Hq, &ldo)) Py_RETURN_NONE;
    const float scale = g.scale(6, p.q.D);
    if (!g.ok || !kv_len_fits(kv_len, p.q.B) || !lse_fits(lse, p.q.B, Hq, p.q.S) || (ws && !ws->is_contiguous()))
        Py_RETURN_NONE;
    Tensor made_d, made_ws;
    if (!dqkv) made_d = empty(qkv->sizes(), qkv->scalar_type(), *qkv), dqkv = &made_d;
    if (dqkv->sizes() != qkv->sizes() || dqkv->strides() != qkv->strides() ||
        dqkv->scalar_type() != qkv->scalar_type() || !d.set(dqkv, Hq, Hkv))
        Py_RETURN_NONE;
    if (!ws) {
        size_t need = 0;
        if (fbl_attn_bwd_workspace(&p.q, &p.k, &need) != FBL_OK) Py_RETURN_NONE;
        made_ws = empty({(int64_t)need}, at::kByte, *qkv), ws = &made_ws;
    }
    const fbl_mask m = mask_of(causal, kv_len);
    void *s = g.stream(), *po = o->data_ptr(), *pg = dO->data_ptr(), *pw = ws->data_ptr();
    const float* pl = static_cast<const float*>(lse->data_ptr());
    const size_t ws_bytes = (size_t)(ws->numel() * ws->element_size());
    const fbl_status st = unlocked([&] {
        return fbl_attn_bwd(&p.q, p.pq, &p.k, p.pk, &p.v, p.pv, &lo, po, &ldo, pg, pl, scale, m, &p.q, d.pq, &p.k, d.pk,
                            &p.v, d.pv, pw, ws_bytes, s);
    });
    if (st != FBL_OK) Py_RETURN_NONE;
    return object_of(a[9], made_d);
    END_HANDLE_TH_ERRORS
}

// proj(op, a, b, out, tile, stream)
PyObject* proj(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 6) Py_RETURN_NONE;
    Args g{a};
    const int64_t op = g.integer(0);
    const Tensor *x = g.tensor(1), *y = g.tensor(2), *out = g.tensor_or_none(3);
    const int64_t tile = g.integer(4);
    g.no_stream(5);
    const auto rows = [](const Tensor* t) { return t->dim() == 2 && t->stride(1) == 1; };
    if (!g.ready() || op < 0 || op > FBL_PROJ_BWD_WEIGHT || !rows(x) || !rows(y) || (out && !rows(out))) Py_RETURN_NONE;
    const int dt = dtype_code(*x);
    if (dt < 0 || y->scalar_type() != x->scalar_type() || (out && out->scalar_type() != x->scalar_type()))
        Py_RETURN_NONE;
    const int64_t M = x->size(0);
    const int64_t K = op == FBL_PROJ_BWD_DATA ? y->size(0) : x->size(1);
    const int64_t N = op == FBL_PROJ_BWD_DATA ? x->size(1) : y->size(1);
    // the extent that both operands state, and the result's shape: the library checks neither
    const int64_t orows = op == FBL_PROJ_BWD_WEIGHT ? K : M, ocols = op == FBL_PROJ_BWD_DATA ? K : N;
    if (op == FBL_PROJ_FWD ? y->size(0) != K : op == FBL_PROJ_BWD_DATA ? y->size(1) != N : y->size(0) != M)
        Py_RETURN_NONE;
    if (out && (out->size(0) != orows || out->size(1) != ocols)) Py_RETURN_NONE;
    Tensor made;
    if (!out) {
        made = empty({orows, ocols}, x->scalar_type(), *x);
        out = &made;
    }
    void *s = g.stream(), *px = x->data_ptr(), *py = y->data_ptr(), *pc = out->data_ptr();
    const int64_t lda = x->stride(0), ldb = y->stride(0), ldc = out->stride(0);
    const fbl_status st = unlocked([&] {
        return fbl_proj_dt((uint32_t)op, dt, M, K, N, px, lda, py, ldb, pc, ldc, (int32_t)tile, s);
    });
    if (st != FBL_OK) Py_RETURN_NONE;
    return object_of(a[3], made);
    END_HANDLE_TH_ERRORS
}

PyMethodDef kMethods[] = {
    {"attn_fwd", (PyCFunction)(void (*)())attn_fwd, METH_FASTCALL, nullptr},
    {"attn_bwd", (PyCFunction)(void (*)())attn_bwd, METH_FASTCALL, nullptr},
    {"attn_fwd_packed", (PyCFunction)(void (*)())attn_fwd_packed, METH_FASTCALL, nullptr},
    {"attn_bwd_packed", (PyCFunction)(void (*)())attn_bwd_packed, METH_FASTCALL, nullptr},
    {"proj", (PyCFunction)(void (*)())proj, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the torch and Python versions, for the binding to compare before it
// makes a call here (their headers' struct layouts are compiled in).
PyMODINIT_FUNC PyInit__fastcall(void) {
    PyObject* m = PyModule_Create(&kModule);
    PyObject* v = m ? Py_BuildValue("(ss)", TORCH_VERSION, FBL_PYTHON) : nullptr;
    if (v && PyModule_AddObject(m, "built_for", v) == 0) return m;
    Py_XDECREF(v);
    Py_XDECREF(m);
    return nullptr;
}
