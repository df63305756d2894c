// The short calls of binding.py in native code.  Calls of a few microseconds of GPU time were bound by the host, and up to half of
// that was Python taking tensors apart (us of host time a call, its launches of 2.65 each included, in Python / here):  greedy and sampling
// acceptance 8.2 / 5.35, scores of one small layer 12.3 / 8.5, selection and gather 14.45 / 8.0, attention of a ragged batch 14.5 / 9.7.
//
// Every function here takes the arguments of its namesake in binding.py by position and serves the plain call: tensors of torch's
// own types in the memory of a GPU, numbers of Python's and NumPy's types, arguments that fit together.  It returns that function's
// result, or the C function's status if that is not 0, or None for anything else, which it leaves to the general code in binding.py:
// what is refused there, and how, is decided in one place.  Leaving a call costs 0.1 us (an exception for it, 2.4).
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/headeronly/version.h>

#include <algorithm>
#include <optional>

#include "specvlm.h"

namespace {

decltype(&specvlm_accept) c_accept;
decltype(&specvlm_accept_workspace_bytes) c_accept_bytes;
decltype(&specvlm_score) c_score;
decltype(&specvlm_score_workspace_bytes) c_score_bytes;
decltype(&specvlm_select) c_select;
decltype(&specvlm_top_p_count) c_top_p_count;
decltype(&specvlm_gather_kv) c_gather_kv;
decltype(&specvlm_decode_attn) c_decode_attn;
decltype(&specvlm_tree_attn) c_tree_attn;
decltype(&specvlm_decode_attn_workspace_bytes) c_attn_bytes;

// A call's arguments.  What reads one that is not plain clears `plain` and gets nothing; a function looks at it before it uses what it read.
struct Args {
    PyObject* const* o;
    bool plain = true;

    bool none(int i) const { return o[i] == Py_None; }
    const at::Tensor* tensor(int i)
    {
        if (THPVariable_CheckExact(o[i])) {
            const at::Tensor& t = THPVariable_Unpack(o[i]);
            // (wrappers of transforms and of tensors without memory have keys of their own, or no storage)
            if (t.is_cuda() && t.has_storage() && t.layout() == at::kStrided && !t.key_set().has(c10::DispatchKey::Python) &&
                !t.key_set().has_any(c10::DispatchKeySet({c10::DispatchKey::Functionalize, c10::DispatchKey::FuncTorchBatched,
                                                          c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Conjugate,
                                                          c10::DispatchKey::Negative, c10::DispatchKey::ZeroTensor})))
                return &t;
        }
        plain = false;
        return nullptr;
    }
    const at::Tensor* tensor(int i, int dims)
    {
        const at::Tensor* const t = tensor(i);
        if (!t || t->dim() == dims) return t;
        plain = false;
        return nullptr;
    }
    void* ptr(int i)                     // (null for None)
    {
        const at::Tensor* const t = none(i) ? nullptr : tensor(i);
        return t ? t->data_ptr() : nullptr;
    }
    void* contiguous(int i)
    {
        const at::Tensor* const t = none(i) ? nullptr : tensor(i);
        if (!t) return nullptr;
        if (!t->is_contiguous()) plain = false;
        return t->data_ptr();
    }
    bool number_like(int i)              // (a tensor has the same conversions, and waits for the GPU in them)
    {
        if (!PyBool_Check(o[i]) && !PyObject_TypeCheck(o[i], reinterpret_cast<PyTypeObject*>(THPVariableClass))) return true;
        plain = false;
        return false;
    }
    int number(int i)                    // (what does not fit the C function's int is left to ctypes)
    {
        int64_t v = 0;
        if (PyLong_CheckExact(o[i])) {
            v = PyLong_AsLongLong(o[i]);
        } else if (number_like(i)) {
            PyObject* const n = PyNumber_Index(o[i]);
            v = n ? PyLong_AsLongLong(n) : -1;
            Py_XDECREF(n);
        }
        if (v == -1 && PyErr_Occurred()) { PyErr_Clear(); plain = false; return 0; }
        return as_int(v);
    }
    double real(int i)
    {
        if (PyFloat_Check(o[i])) return PyFloat_AS_DOUBLE(o[i]);
        if (!PyBool_Check(o[i]) && !number_like(i)) return 0.;
        const double v = PyFloat_AsDouble(o[i]);
        if (v == -1. && PyErr_Occurred()) { PyErr_Clear(); plain = false; }
        return v;
    }
    bool truth(int i)
    {
        if (o[i] == Py_True || o[i] == Py_False || o[i] == Py_None) return o[i] == Py_True;
        if (PyLong_CheckExact(o[i])) return PyObject_IsTrue(o[i]) == 1;
        plain = false;
        return false;
    }
    int as_int(int64_t v)
    {
        if (v != (int)v) plain = false;
        return (int)v;
    }
};

// The tensor a call was given, or a new one; keeps a new one alive for the length of the call.
struct Out {
    PyObject* given = nullptr;
    std::optional<at::Tensor> made;
    void* at = nullptr;

    template <class F> Out(Args& a, int i, F&& make)
    {
        if (!a.none(i)) { given = a.o[i]; at = a.ptr(i); }
        else if (a.plain) { made = make(); at = made->data_ptr(); }
    }
    const at::Tensor& tensor() const { return given ? THPVariable_Unpack(given) : *made; }
    PyObject* result() const { return given ? Py_NewRef(given) : THPVariable_Wrap(*made); }
};

at::Tensor make(at::IntArrayRef shape, at::ScalarType type, const at::Tensor& like) { return at::empty(shape, like.options().dtype(type)); }

struct Workspace {
    std::optional<at::Tensor> made;
    void* at = nullptr;
    size_t bytes = 0;

    template <class F> Workspace(Args& a, int i, const at::Tensor& like, F&& need)
    {
        if (!a.plain) return;
        if (a.none(i)) made = make({std::max<int64_t>((int64_t)need(), 256)}, at::kByte, like);
        const at::Tensor* const t = made ? &*made : a.tensor(i);
        if (t) { at = t->data_ptr(); bytes = (size_t)t->numel(); }
    }
};

// The C function on torch's current stream, without the interpreter's lock.
template <class F, class... A> int call(F f, A... a)
{
    void* const stream = c10::hip::getCurrentHIPStream().stream();
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = f(a..., stream);
    Py_END_ALLOW_THREADS
    return status;
}

PyObject* pair(PyObject* a, PyObject* b)
{
    PyObject* t = a && b ? PyTuple_New(2) : nullptr;
    if (!t) { Py_XDECREF(a); Py_XDECREF(b); return nullptr; }
    PyTuple_SET_ITEM(t, 0, a);
    PyTuple_SET_ITEM(t, 1, b);
    return t;
}

// (null without an error: the call is left)
PyObject* accept(Args& a)                // target, tokens, draft, uniforms, temperature, workspace, n_accepted, out_tokens
{
    const at::Tensor* const target = a.tensor(0, 3);
    if (!target) return nullptr;
    const int64_t batch = target->size(0), g1 = target->size(1), vocab = target->size(2);
    void* const logits = a.contiguous(0);
    void* const tokens = a.contiguous(1);
    void* const draft = a.contiguous(2);
    void* const uniforms = a.contiguous(3);
    const float temperature = (float)a.real(4);
    const int b = a.as_int(batch), gamma = a.as_int(g1 - 1), v = a.as_int(vocab);
    if (!a.plain || !tokens) return nullptr;
    const Out n_accepted(a, 6, [&] { return make({batch}, at::kInt, *target); });
    const Out out_tokens(a, 7, [&] { return make({batch, g1}, at::kInt, *target); });
    const Workspace ws(a, 5, *target, [&] { return c_accept_bytes(b, gamma, v, !a.none(3)); });
    if (!a.plain) return nullptr;
    const int status = call(c_accept, (const float*)logits, (const float*)draft, (const int32_t*)tokens, (const float*)uniforms, b, gamma, v,
                            temperature, (int32_t*)n_accepted.at, (int32_t*)out_tokens.at, ws.at, ws.bytes);
    if (status) return PyLong_FromLong(status);
    return pair(n_accepted.result(), out_tokens.result());
}

// q_text, k_cache, video_start, n_video, text_pos0, softmax_scale, norm_mode, row_lse, beta, scores, workspace
PyObject* score(Args& a)
{
    const at::Tensor *const q = a.tensor(0, 3), *const k = a.tensor(1, 3);
    if (!a.plain || q->stride(2) != 1 || k->stride(2) != 1) return nullptr;
    const int n_text = a.as_int(q->size(0)), hq = a.as_int(q->size(1)), d = a.as_int(q->size(2)), n_keys = a.as_int(k->size(0)), hkv = a.as_int(k->size(1));
    const int video_start = a.number(2), n_video = a.number(3), text_pos0 = a.number(4), norm_mode = a.number(6);
    const float scale = (float)a.real(5);
    const double beta = a.real(8);           // (one that 32 bits take for 0 needs scores too)
    const float* const row_lse = (const float*)a.ptr(7);
    if (!a.plain || (a.none(9) && beta != 0.)) return nullptr;
    const Out scores(a, 9, [&] { return make({n_video}, at::kFloat, *q); });
    const Workspace ws(a, 10, *q, [&] { return c_score_bytes(1, n_text, n_keys, n_video, hq, hkv, d, !a.none(7)); });
    if (!a.plain) return nullptr;
    const int status = call(c_score, q->data_ptr(), q->stride(0), q->stride(1), k->data_ptr(), k->stride(0), k->stride(1), (const int32_t*)nullptr,
                            (const int32_t*)nullptr, (const int32_t*)nullptr, 1, n_text, n_keys, video_start, n_video, text_pos0, hq, hkv, d, scale,
                            norm_mode, row_lse, (float)beta, (float*)scores.at, ws.at, ws.bytes);
    return status ? PyLong_FromLong(status) : scores.result();
}

PyObject* select(Args& a)                // scores, k_top, keep_budget, total_keep, cu_video, cu_keep, max_n_video, want_flags, keep_idx
{
    const at::Tensor *const scores = a.tensor(0), *const k_top = a.tensor(1);
    if (!a.plain || (a.none(6) && !a.none(4))) return nullptr;
    const int batch = a.as_int(k_top->numel()), total = a.number(3), longest = a.none(6) ? a.as_int(scores->numel()) : a.number(6);
    const bool want_flags = a.truth(7);
    void* const budget = a.ptr(2);
    void* const cu_video = a.ptr(4);
    void* const cu_keep = a.ptr(5);
    const Out keep_idx(a, 8, [&] { return make({total}, at::kInt, *scores); });
    if (!a.plain) return nullptr;
    std::optional<at::Tensor> flags;
    if (want_flags) flags = make({total}, at::kByte, *scores);
    const int status = call(c_select, (const float*)scores->data_ptr(), (const int32_t*)cu_video, (const int32_t*)k_top->data_ptr(),
                            (const int32_t*)budget, (const int32_t*)cu_keep, batch, longest, total, (int32_t*)keep_idx.at,
                            (uint8_t*)(flags ? flags->data_ptr() : nullptr), (int32_t*)nullptr, (void*)nullptr, (size_t)0);
    if (status) return PyLong_FromLong(status);
    return pair(keep_idx.result(), flags ? THPVariable_Wrap(*flags) : Py_NewRef(Py_None));
}

PyObject* top_p_count(Args& a)           // scores, lam, cu_video, max_n_video, max_count, count
{
    const at::Tensor* const scores = a.tensor(0);
    const at::Tensor* const cu = a.none(2) ? nullptr : a.tensor(2);
    if (!a.plain || (a.none(3) && cu)) return nullptr;
    const float lam = (float)a.real(1);
    const int64_t batch = cu ? cu->numel() - 1 : 1;
    const int b = a.as_int(batch), longest = a.none(3) ? a.as_int(scores->numel()) : a.number(3);
    void* const most = a.ptr(4);
    const Out count(a, 5, [&] { return make({batch}, at::kInt, *scores); });
    if (!a.plain) return nullptr;
    const int status = call(c_top_p_count, (const float*)scores->data_ptr(), (const int32_t*)(cu ? cu->data_ptr() : nullptr), b, longest, lam,
                            (const int32_t*)most, (int32_t*)count.at, (void*)nullptr, (size_t)0);
    return status ? PyLong_FromLong(status) : count.result();
}

PyObject* gather_kv(Args& a)             // k_src, v_src, video_start, n_video, keep_idx, k_dst, v_dst, cu_keys, cu_video, cu_keep
{
    const at::Tensor *const k = a.tensor(0, 4), *const keep = a.tensor(4);
    const at::Tensor *const v = a.none(1) ? nullptr : a.tensor(1), *const cu_keys = a.none(7) ? nullptr : a.tensor(7);
    if (!a.plain || k->stride(3) != 1 || (v && v->strides() != k->strides())) return nullptr;
    const int video_start = a.number(2), n_video = a.number(3);
    const int layers = a.as_int(k->size(0)), n_keys = a.as_int(k->size(1)), hkv = a.as_int(k->size(2)), d = a.as_int(k->size(3));
    const int n_keep = a.as_int(keep->numel()), batch = cu_keys ? a.as_int(cu_keys->numel() - 1) : 1;
    void* const cu_video = a.ptr(8);
    void* const cu_keep = a.ptr(9);
    const Out k_dst(a, 5, [&] { return at::empty({layers, (int64_t)n_keys - n_video + n_keep, hkv, d}, k->options()); });
    if (!a.plain || k_dst.tensor().dim() != 4) return nullptr;
    const at::Tensor& kd = k_dst.tensor();
    std::optional<Out> v_dst;
    if (v || !a.none(6)) v_dst.emplace(a, 6, [&] { return at::empty_like(kd); });
    if (!a.plain || (v_dst && v_dst->tensor().strides() != kd.strides())) return nullptr;
    const int status = call(c_gather_kv, k->data_ptr(), v ? v->data_ptr() : nullptr, k->stride(0), k->stride(1), k->stride(2), k_dst.at,
                            v_dst ? v_dst->at : nullptr, kd.stride(0), kd.stride(1), kd.stride(2), layers, n_keys, video_start, n_video,
                            (const int32_t*)keep->data_ptr(), n_keep, (const int32_t*)(cu_keys ? cu_keys->data_ptr() : nullptr),
                            (const int32_t*)cu_video, (const int32_t*)cu_keep, batch, (int32_t*)nullptr, hkv, d);
    if (status) return PyLong_FromLong(status);
    return pair(k_dst.result(), v_dst ? v_dst->result() : Py_NewRef(Py_None));
}

// q, k, v, softmax_scale, cu_q, cu_kv, max_q_len, max_kv_len, out, want_lse, num_splits, workspace, ancestor_mask
PyObject* decode_attn(Args& a)
{
    const at::Tensor *const q = a.tensor(0, 3), *const k = a.tensor(1, 3), *const v = a.tensor(2);
    const at::Tensor* const cu = a.none(4) ? nullptr : a.tensor(4);
    if (!a.plain || q->stride(2) != 1 || k->stride(2) != 1 || v->strides() != k->strides()) return nullptr;
    const int64_t tq = q->size(0), hq = q->size(1);
    const int h = a.as_int(hq), hkv = a.as_int(k->size(1)), d = a.as_int(q->size(2));
    const int batch = cu ? a.as_int(cu->numel() - 1) : 1;
    const int q_len = cu ? a.number(6) : a.as_int(tq), kv_len = cu ? a.number(7) : a.as_int(k->size(0));
    const float scale = (float)a.real(3);
    const bool want_lse = a.truth(9);
    const int splits = a.number(10);
    const int32_t* const cu_q = (const int32_t*)(cu ? cu->data_ptr() : nullptr);
    const int32_t* const cu_kv = (const int32_t*)a.ptr(5);
    const uint64_t* const mask = (const uint64_t*)a.ptr(12);
    const Out out(a, 8, [&] { return at::empty_like(*q); });
    if (!a.plain || out.tensor().strides() != q->strides()) return nullptr;
    std::optional<at::Tensor> lse;
    if (want_lse) lse = make({tq, hq}, at::kFloat, *q);
    const Workspace ws(a, 11, *q, [&] { return c_attn_bytes(batch, q_len, kv_len, h, hkv, d, splits); });
    if (!a.plain) return nullptr;
    float* const lse_at = lse ? (float*)lse->data_ptr() : nullptr;
    const int status =
        !a.none(12) ? call(c_tree_attn, q->data_ptr(), q->stride(0), q->stride(1), k->data_ptr(), v->data_ptr(), k->stride(0), k->stride(1), cu_q, cu_kv,
                           batch, q_len, kv_len, h, hkv, d, scale, mask, out.at, lse_at, splits, ws.at, ws.bytes)
                    : call(c_decode_attn, q->data_ptr(), q->stride(0), q->stride(1), k->data_ptr(), v->data_ptr(), k->stride(0), k->stride(1), cu_q, cu_kv,
                           batch, q_len, kv_len, h, hkv, d, scale, out.at, lse_at, splits, ws.at, ws.bytes);
    if (status) return PyLong_FromLong(status);
    return want_lse ? pair(out.result(), THPVariable_Wrap(*lse)) : out.result();
}

template <PyObject* (*F)(Args&), Py_ssize_t N>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (n != N) { PyErr_SetString(PyExc_TypeError, "wrong number of arguments"); return nullptr; }
    // nothing has been launched where torch throws: what it refuses (an allocation, a tensor without memory) the general code
    // meets again and reports
    try {
        if (!at::impl::torch_function_mode_enabled()) {
            Args a{args};
            PyObject* const got = F(a);
            if (got || PyErr_Occurred()) return got;
        }
    } catch (const std::exception&) {
        PyErr_Clear();
    }
    Py_RETURN_NONE;
}

// The functions that are called here, by the names under which connect() is handed their addresses.
struct { const char* name; void** at; } const functions[] = {
    {"specvlm_accept", (void**)&c_accept}, {"specvlm_accept_workspace_bytes", (void**)&c_accept_bytes}, {"specvlm_score", (void**)&c_score},
    {"specvlm_score_workspace_bytes", (void**)&c_score_bytes}, {"specvlm_select", (void**)&c_select}, {"specvlm_top_p_count", (void**)&c_top_p_count},
    {"specvlm_gather_kv", (void**)&c_gather_kv}, {"specvlm_decode_attn", (void**)&c_decode_attn}, {"specvlm_tree_attn", (void**)&c_tree_attn},
    {"specvlm_decode_attn_workspace_bytes", (void**)&c_attn_bytes}};

// connect(version, address of every function by its name), once, before any call: the version is the library's, which has to be the one whose
// header this was compiled with.
PyObject* connect(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (n != 2 || !PyLong_Check(args[0]) || !PyDict_Check(args[1])) { PyErr_SetString(PyExc_TypeError, "a version and a dict of addresses"); return nullptr; }
    if (PyLong_AsLong(args[0]) != SPECVLM_VERSION) {
        PyErr_Clear();
        return PyErr_Format(PyExc_ImportError, "compiled for version %d of the library, which is %S", SPECVLM_VERSION, args[0]);
    }
    constexpr size_t N = sizeof(functions) / sizeof(functions[0]);
    void* at[N];
    for (size_t i = 0; i < N; ++i) {
        PyObject* const address = PyDict_GetItemString(args[1], functions[i].name);
        at[i] = address ? PyLong_AsVoidPtr(address) : nullptr;
        if (!at[i]) { if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, functions[i].name); return nullptr; }
    }
    for (size_t i = 0; i < N; ++i) *functions[i].at = at[i];
    Py_RETURN_NONE;
}

#define SPECVLM_CALL(name, n) {#name, (PyCFunction)(void (*)())entry<name, n>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"connect", (PyCFunction)(void (*)())connect, METH_FASTCALL, nullptr},
    SPECVLM_CALL(accept, 8), SPECVLM_CALL(score, 11), SPECVLM_CALL(select, 9), SPECVLM_CALL(top_p_count, 6), SPECVLM_CALL(gather_kv, 10),
    SPECVLM_CALL(decode_attn, 13),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject* PyInit__calls()
{
    PyObject* const m = PyModule_Create(&module);
    if (!m) return nullptr;
    PyObject* const names = PyTuple_New(sizeof(functions) / sizeof(functions[0]));
    for (Py_ssize_t i = 0; names && i < PyTuple_GET_SIZE(names); ++i) PyTuple_SET_ITEM(names, i, PyUnicode_FromString(functions[i].name));
    if (!names || PyErr_Occurred() || PyModule_AddObjectRef(m, "functions", names) || PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION)) {
        Py_XDECREF(names);
        Py_DECREF(m);
        return nullptr;
    }
    Py_DECREF(names);
    return m;
}
