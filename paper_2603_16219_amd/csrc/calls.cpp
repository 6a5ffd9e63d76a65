// The binding's wrappers on arguments that need nothing done to them, in native code: the checks, the outputs and the call of the
// library.  In Python those took most of a small call: 9.9 us of host time beside the launch for 64 sampled rows (half of it the three
// allocations, 1.3 us each) where this takes 5.6, 14.7 beside the launches for the two calls of the split (now 5.8), 14.6 for a block with
// log-prob rows (7.8).  Since the host no longer is what rows without drafts wait for, they are shaped for the GPU's time here: 64 of
// V = 151936 13.0 -> 9.6 us a call, in two launches instead of one; the split of 4 rows fp32, V = 50257 18.9 -> 16.3.
//
// Every function returns the wrapper's result, an integer (the library's status, not 0), or None for arguments that it leaves
// to the wrapper: whatever has to be converted, copied or refused, and what is no plain GPU tensor.  No device code here.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "specsteer.h"
#include "unbound.h"

namespace {

// The library that the binding has loaded.
struct Library {
    decltype(&specsteer_workspace_bytes) workspace_bytes;
    decltype(&specsteer_verify_block_unbound) verify_block;
    decltype(&specsteer_cloud_topk) cloud_topk;
    decltype(&specsteer_edge_resample) edge_resample;
} lib;
PyObject* current_raw_stream = nullptr;  // of a device index

// A plain tensor of its own memory on a GPU, or NULL.
const at::Tensor* gpu_tensor(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return t.is_cuda() && t.has_storage() && t.layout() == at::kStrided ? &t : nullptr;
}

// The same, contiguous, of this type on this device.
const at::Tensor* ready(PyObject* o, at::ScalarType type, const at::Tensor& like) {
    const at::Tensor* t = gpu_tensor(o);
    return t && t->scalar_type() == type && t->device() == like.device() && t->is_contiguous() ? t : nullptr;
}

bool same_form(const at::Tensor& a, const at::Tensor& b) {
    return a.scalar_type() == b.scalar_type() && a.device() == b.device() && a.sizes() == b.sizes() && a.strides() == b.strides();
}

// Logits [B, k_max + 1, V], or rows [B, V], of a type the library takes, the vocabulary contiguous and no row twice.
bool describe(const at::Tensor& t, ss_params& p) {
    const bool rows = t.dim() == 2;
    if (!rows && t.dim() != 3) return false;
    if (t.scalar_type() != at::kFloat && t.scalar_type() != at::kBFloat16) return false;
    const int64_t B = t.size(0), k1 = rows ? 1 : t.size(1), V = t.size(-1);
    if (B < 1 || B > INT32_MAX || k1 < 1 || k1 > INT32_MAX || V < 1 || V > INT32_MAX || t.stride(-1) != 1) return false;
    const int64_t sb = B > 1 ? t.stride(0) : 0, st = k1 > 1 ? t.stride(1) : 0;
    if ((B > 1 && sb == 0) || (k1 > 1 && st == 0)) return false;
    p.batch = (int32_t)B;
    p.k_max = (int32_t)k1 - 1;
    p.vocab = (int32_t)V;
    p.dtype = t.scalar_type() == at::kFloat ? SS_F32 : SS_BF16;
    p.stride_b = sb;
    p.stride_t = st;
    p.lambda = 0.5f;
    p.beta = p.temperature = 1.f;
    p.flags = 0;
    return true;
}

bool number(PyObject* o, float& v) {
    if (!PyFloat_CheckExact(o) && !PyLong_CheckExact(o)) return false;
    const double x = PyFloat_AsDouble(o);
    if (x == -1.0 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    v = (float)x;
    return true;
}

bool truth(PyObject* o, bool& v) {
    if (!PyBool_Check(o)) return false;
    v = o == Py_True;
    return true;
}

// torch's current stream on the tensor's device; false with a Python error set.
bool stream_of(const at::Tensor& t, void*& s) {
    PyObject* index = PyLong_FromLong(t.get_device());
    PyObject* handle = index ? PyObject_CallOneArg(current_raw_stream, index) : nullptr;
    Py_XDECREF(index);
    if (!handle) return false;
    s = PyLong_AsVoidPtr(handle);
    Py_DECREF(handle);
    return !PyErr_Occurred();
}

// Without the interpreter's lock, as a call through ctypes is.
template <typename F>
ss_status unlocked(F call) {
    PyThreadState* const saved = PyEval_SaveThread();
    const ss_status rc = call();
    PyEval_RestoreThread(saved);
    return rc;
}

at::Tensor make(const at::Tensor& like, at::IntArrayRef size, at::ScalarType type) { return at::empty(size, like.options().dtype(type).requires_grad(false)); }

// A dict entry; None for an undefined tensor.
bool put(PyObject* dict, const char* key, const at::Tensor& t) {
    PyObject* v = t.defined() ? THPVariable_Wrap(t) : Py_NewRef(Py_None);
    const bool ok = v && PyDict_SetItemString(dict, key, v) == 0;
    Py_XDECREF(v);
    return ok;
}

template <typename T>
T* ptr(const at::Tensor& t) { return t.defined() ? static_cast<T*>(t.data_ptr()) : nullptr; }

// verify_block(G, S_ctx, S_noctx, draft, uniforms, lam, beta, temperature, draft_len, want_recovery_logprobs, want_draft_logprobs,
//              workspace, greedy, full_rows)
PyObject* verify_block(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 14) Py_RETURN_NONE;
    const at::Tensor *G = gpu_tensor(a[0]), *Sp = gpu_tensor(a[1]), *Sm = gpu_tensor(a[2]);
    ss_params p;
    bool rec, dlp, greedy, full;
    if (!G || !Sp || !Sm || G->dim() != 3 || !same_form(*G, *Sp) || !same_form(*G, *Sm) || !describe(*G, p)) Py_RETURN_NONE;
    const at::Tensor *draft = ready(a[3], at::kInt, *G), *un = ready(a[4], at::kFloat, *G);
    const at::Tensor *len = a[8] == Py_None ? nullptr : ready(a[8], at::kInt, *G), *given = a[11] == Py_None ? nullptr : gpu_tensor(a[11]);
    if (!draft || !un || (!len && a[8] != Py_None) || (!given && a[11] != Py_None)) Py_RETURN_NONE;
    if (!number(a[5], p.lambda) || !number(a[6], p.beta) || !number(a[7], p.temperature)) Py_RETURN_NONE;
    if (!truth(a[9], rec) || !truth(a[10], dlp) || !truth(a[12], greedy) || !truth(a[13], full)) Py_RETURN_NONE;
    const int64_t B = p.batch, K = p.k_max;
    if (draft->dim() != 2 || draft->size(0) != B || draft->size(1) != K || un->dim() != 2 || un->size(0) != B || un->size(1) != K + 1) Py_RETURN_NONE;
    if (len && (len->dim() != 1 || len->size(0) != B)) Py_RETURN_NONE;
    if (given && (!given->is_contiguous() || given->device() != G->device())) Py_RETURN_NONE;
    p.flags = (greedy ? SS_FLAG_GREEDY : 0u) | (full ? SS_FLAG_FULL_ROWS : 0u);
    const size_t need = lib.workspace_bytes(&p);
    const at::Tensor ws = given ? *given : make(*G, {(int64_t)(need > 256 ? need : 256)}, at::kByte);
    const at::Tensor acc = make(*G, {B}, at::kInt), tok = make(*G, {B}, at::kInt), lp = make(*G, {B}, at::kFloat);
    const at::Tensor rows = rec ? make(*G, {B, p.vocab}, at::kFloat) : at::Tensor(), drafts = dlp ? make(*G, {B, K, 2}, at::kFloat) : at::Tensor();
    void* stream;
    if (!stream_of(*G, stream)) return nullptr;
    const void *g = G->data_ptr(), *sp = Sp->data_ptr(), *sm = Sm->data_ptr();
    const int32_t *d = K > 0 ? ptr<int32_t>(*draft) : nullptr, *l = len ? ptr<int32_t>(*len) : nullptr;
    const float* u = ptr<float>(*un);
    const size_t bytes = ws.nbytes();
    int32_t *o_acc = ptr<int32_t>(acc), *o_tok = ptr<int32_t>(tok);
    float *o_lp = ptr<float>(lp), *o_rows = ptr<float>(rows), *o_drafts = ptr<float>(drafts);
    void* const w = ws.data_ptr();
    const ss_status rc = unlocked([&] { return lib.verify_block(g, sp, sm, d, l, u, &p, o_acc, o_tok, o_lp, o_rows, o_drafts, w, bytes, stream); });
    if (rc != SS_OK) return PyLong_FromLong(rc);
    PyObject* out = PyDict_New();
    if (out && put(out, "accepted_len", acc) && put(out, "next_token", tok) && put(out, "next_token_logprob", lp) &&
        put(out, "recovery_logprobs", rows) && put(out, "draft_logprobs", drafts))
        return out;
    Py_XDECREF(out);
    return nullptr;
    END_HANDLE_TH_ERRORS
}

// steer_rows(G, S_ctx, S_noctx, uniforms, beta, temperature, greedy, want_logprobs)
PyObject* steer_rows(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 8) Py_RETURN_NONE;
    const at::Tensor *G = gpu_tensor(a[0]), *Sp = gpu_tensor(a[1]), *Sm = gpu_tensor(a[2]);
    ss_params p;
    bool greedy, want;
    if (!G || !Sp || !Sm || G->dim() != 2 || !same_form(*G, *Sp) || !same_form(*G, *Sm) || !describe(*G, p)) Py_RETURN_NONE;
    const at::Tensor* un = ready(a[3], at::kFloat, *G);
    if (!un || un->numel() != p.batch) Py_RETURN_NONE;
    if (!number(a[4], p.beta) || !number(a[5], p.temperature) || !truth(a[6], greedy) || !truth(a[7], want)) Py_RETURN_NONE;
    p.flags = greedy ? SS_FLAG_GREEDY : 0u;
    // one allocation for the workspace and, behind it, the accepted lengths (all 0) that nobody asked for
    const int64_t B = p.batch, got = (int64_t)lib.workspace_bytes(&p), need = ((got > 256 ? got : 256) + 255) / 256 * 256;
    const at::Tensor ws = make(*G, {need + 4 * B}, at::kByte), tok = make(*G, {B}, at::kInt), lp = make(*G, {B}, at::kFloat);
    const at::Tensor rows = want ? make(*G, {B, p.vocab}, at::kFloat) : at::Tensor();
    void* stream;
    if (!stream_of(*G, stream)) return nullptr;
    const void *g = G->data_ptr(), *sp = Sp->data_ptr(), *sm = Sm->data_ptr();
    const float* u = ptr<float>(*un);
    char* const w = ptr<char>(ws);
    int32_t* const o_tok = ptr<int32_t>(tok);
    float *o_lp = ptr<float>(lp), *o_rows = ptr<float>(rows);
    const ss_status rc = unlocked([&] {
        return lib.verify_block(g, sp, sm, nullptr, nullptr, u, &p, reinterpret_cast<int32_t*>(w + need), o_tok, o_lp, o_rows, nullptr, w, (size_t)need, stream);
    });
    if (rc != SS_OK) return PyLong_FromLong(rc);
    PyObject* out = PyDict_New();
    if (out && put(out, "token", tok) && put(out, "token_logprob", lp) && put(out, "logprobs", rows)) return out;
    Py_XDECREF(out);
    return nullptr;
    END_HANDLE_TH_ERRORS
}

// cloud_topk(G, S_noctx, row, beta, topk)
PyObject* cloud_topk(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 5) Py_RETURN_NONE;
    const at::Tensor *G = gpu_tensor(a[0]), *Sm = gpu_tensor(a[1]);
    ss_params p;
    if (!G || !Sm || G->dim() != 3 || !same_form(*G, *Sm) || !describe(*G, p)) Py_RETURN_NONE;
    const at::Tensor* row = ready(a[2], at::kInt, *G);
    if (!row || row->dim() != 1 || row->size(0) != p.batch || !number(a[3], p.beta) || !PyLong_CheckExact(a[4])) Py_RETURN_NONE;
    int overflow = 0;
    const long topk = PyLong_AsLongAndOverflow(a[4], &overflow);
    if (overflow || topk < 1 || topk > SS_MAX_TOPK) Py_RETURN_NONE;
    const at::Tensor idx = make(*G, {p.batch, topk}, at::kInt), val = make(*G, {p.batch, topk}, at::kFloat);
    void* stream;
    if (!stream_of(*G, stream)) return nullptr;
    const void *g = G->data_ptr(), *sm = Sm->data_ptr();
    const int32_t* r = ptr<int32_t>(*row);
    int32_t* const o_idx = ptr<int32_t>(idx);
    float* const o_val = ptr<float>(val);
    const ss_status rc = unlocked([&] { return lib.cloud_topk(g, sm, r, &p, (int32_t)topk, o_idx, o_val, stream); });
    if (rc != SS_OK) return PyLong_FromLong(rc);
    PyObject *i = THPVariable_Wrap(idx), *v = i ? THPVariable_Wrap(val) : nullptr, *out = v ? PyTuple_Pack(2, i, v) : nullptr;
    Py_XDECREF(i);
    Py_XDECREF(v);
    return out;
    END_HANDLE_TH_ERRORS
}

// edge_resample(index, value, S_ctx, row, uniform, beta, temperature, greedy)
PyObject* edge_resample(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 8) Py_RETURN_NONE;
    const at::Tensor* Sp = gpu_tensor(a[2]);
    ss_params p;
    bool greedy;
    if (!Sp || Sp->dim() != 3 || !describe(*Sp, p)) Py_RETURN_NONE;
    const at::Tensor *idx = ready(a[0], at::kInt, *Sp), *val = ready(a[1], at::kFloat, *Sp), *row = ready(a[3], at::kInt, *Sp);
    const at::Tensor* un = a[4] == Py_None ? nullptr : ready(a[4], at::kFloat, *Sp);
    if (!idx || !val || !row || (!un && a[4] != Py_None) || !number(a[5], p.beta) || !number(a[6], p.temperature) || !truth(a[7], greedy)) Py_RETURN_NONE;
    const int64_t B = p.batch;
    if (idx->dim() != 2 || idx->size(0) != B || idx->sizes() != val->sizes() || idx->size(1) < 1 || idx->size(1) > SS_MAX_TOPK) Py_RETURN_NONE;
    if (row->dim() != 1 || row->size(0) != B || (!un && !greedy) || (un && !greedy && (un->dim() != 1 || un->size(0) != B))) Py_RETURN_NONE;
    p.flags = greedy ? SS_FLAG_GREEDY : 0u;
    const at::Tensor tok = make(*Sp, {B}, at::kInt), lp = make(*Sp, {B}, at::kFloat);
    void* stream;
    if (!stream_of(*Sp, stream)) return nullptr;
    const int32_t *i = ptr<int32_t>(*idx), *r = ptr<int32_t>(*row);
    const float *v = ptr<float>(*val), *u = un ? ptr<float>(*un) : nullptr;
    const void* sp = Sp->data_ptr();
    const int32_t topk = (int32_t)idx->size(1);
    int32_t* const o_tok = ptr<int32_t>(tok);
    float* const o_lp = ptr<float>(lp);
    const ss_status rc = unlocked([&] { return lib.edge_resample(i, v, sp, r, u, &p, topk, o_tok, o_lp, stream); });
    if (rc != SS_OK) return PyLong_FromLong(rc);
    PyObject* out = PyDict_New();
    if (out && put(out, "next_token", tok) && put(out, "next_token_logprob", lp)) return out;
    Py_XDECREF(out);
    return nullptr;
    END_HANDLE_TH_ERRORS
}

// use(workspace_bytes, verify_block_unbound, cloud_topk, edge_resample, current_raw_stream): the library's functions by their addresses,
// and what gives torch's current stream on a device
PyObject* use(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 5) return PyErr_Format(PyExc_TypeError, "five arguments");
    void* f[4];
    for (int i = 0; i < 4; ++i) {
        f[i] = PyLong_AsVoidPtr(a[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    lib.workspace_bytes = reinterpret_cast<decltype(lib.workspace_bytes)>(f[0]);
    lib.verify_block = reinterpret_cast<decltype(lib.verify_block)>(f[1]);
    lib.cloud_topk = reinterpret_cast<decltype(lib.cloud_topk)>(f[2]);
    lib.edge_resample = reinterpret_cast<decltype(lib.edge_resample)>(f[3]);
    Py_INCREF(a[4]);
    Py_XSETREF(current_raw_stream, a[4]);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"use", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(use)), METH_FASTCALL, nullptr},
    {"verify_block", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(verify_block)), METH_FASTCALL, nullptr},
    {"steer_rows", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(steer_rows)), METH_FASTCALL, nullptr},
    {"cloud_topk", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(cloud_topk)), METH_FASTCALL, nullptr},
    {"edge_resample", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(edge_resample)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void) { return PyModule_Create(&module); }
