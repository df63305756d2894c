// The short calls of binding.py in native code.  Calls of a few microseconds of GPU time were bound by the host, and up to half of
// that was Python taking tensors apart (us of host time a call, its launches of 2.65 each included, in Python / here):  greedy and sampling
// acceptance 8.2 / 5.35, scores of one small layer 12.3 / 8.5, selection and gather 14.45 / 8.0, attention of a ragged batch 14.5 / 9.7.
//
// Every function here takes the arguments of its namesake in binding.py by position and serves the plain call: tensors of torch's
// own type in the memory of a GPU, numbers of Python's own types, arguments that fit together.  It returns that function's result, or
// the C function's status if that is not 0, or None for anything else, which it leaves to the general code in binding.py: what is
// refused there, and how, is decided in one place.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>

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

struct NotPlain {};                      // the call is left to the general code

struct Arg {
    PyObject* o;

    bool none() const { return o == Py_None; }
    const at::Tensor& tensor() const
    {
        if (Py_TYPE(o) != reinterpret_cast<PyTypeObject*>(THPVariableClass)) throw NotPlain();
        const at::Tensor& t = THPVariable_Unpack(o);
        // (wrappers of transforms and of tensors without memory have keys of their own, or no storage)
        if (!t.is_cuda() || !t.has_storage() || t.layout() != at::kStrided || t.key_set().has(c10::DispatchKey::Python) ||
            t.key_set().has_any(c10::DispatchKeySet({c10::DispatchKey::Functionalize, c10::DispatchKey::FuncTorchBatched,
                                                     c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Conjugate,
                                                     c10::DispatchKey::Negative, c10::DispatchKey::ZeroTensor})))
            throw NotPlain();
        return t;
    }
    void* ptr() const { return none() ? nullptr : tensor().data_ptr(); }
    void* contiguous() const
    {
        if (none()) return nullptr;
        const at::Tensor& t = tensor();
        if (!t.is_contiguous()) throw NotPlain();
        return t.data_ptr();
    }
    int64_t integer() const
    {
        if (!PyLong_CheckExact(o)) throw NotPlain();
        const int64_t v = PyLong_AsLongLong(o);
        if (v == -1 && PyErr_Occurred()) { PyErr_Clear(); throw NotPlain(); }
        return v;
    }
    int number() const                   // (what does not fit the C function's int is left to ctypes)
    {
        const int64_t v = integer();
        if (v != (int)v) throw NotPlain();
        return (int)v;
    }
    double real() const
    {
        if (PyFloat_CheckExact(o)) return PyFloat_AS_DOUBLE(o);
        return (double)integer();
    }
    bool truth() const
    {
        if (o != Py_True && o != Py_False) throw NotPlain();
        return o == Py_True;
    }
};

int as_int(int64_t v)
{
    if (v != (int)v) throw NotPlain();
    return (int)v;
}

// The tensor a call was given, or a new one; keeps a new one alive for the length of the call.
struct Out {
    PyObject* given = nullptr;
    std::optional<at::Tensor> made;
    void* at = nullptr;

    template <class F> Out(Arg a, F&& make)
    {
        if (!a.none()) { given = a.o; at = a.ptr(); }
        else { made = make(); at = made->data_ptr(); }
    }
    PyObject* result() const { return given ? Py_NewRef(given) : THPVariable_Wrap(*made); }
};

at::Tensor make(at::IntArrayRef shape, at::ScalarType type, const at::Tensor& like) { return at::empty(shape, like.options().dtype(type)); }

struct Workspace {
    std::optional<at::Tensor> made;
    void* at;
    size_t bytes;

    template <class F> Workspace(Arg a, const at::Tensor& like, F&& need)
    {
        if (a.none()) made = make({std::max<int64_t>((int64_t)need(), 256)}, at::kByte, like);
        const at::Tensor& t = a.none() ? *made : a.tensor();
        at = t.data_ptr();
        bytes = (size_t)t.numel();
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

PyObject* accept(const Arg* a)           // target, tokens, draft, uniforms, temperature, workspace, n_accepted, out_tokens
{
    const at::Tensor& target = a[0].tensor();
    if (target.dim() != 3) throw NotPlain();
    const int64_t batch = target.size(0), g1 = target.size(1), vocab = target.size(2);
    void* const logits = a[0].contiguous();
    void* const tokens = a[1].contiguous();
    void* const draft = a[2].contiguous();
    void* const uniforms = a[3].contiguous();
    const float temperature = (float)a[4].real();
    const int b = as_int(batch), gamma = as_int(g1 - 1), v = as_int(vocab);
    if (!tokens) throw NotPlain();
    const Out n_accepted(a[6], [&] { return make({batch}, at::kInt, target); });
    const Out out_tokens(a[7], [&] { return make({batch, g1}, at::kInt, target); });
    const Workspace ws(a[5], target, [&] { return c_accept_bytes(b, gamma, v, !a[3].none()); });
    const int status = call(c_accept, (const float*)logits, (const float*)draft, (const int32_t*)tokens, (const float*)uniforms, b, gamma, v,
                            temperature, (int32_t*)n_accepted.at, (int32_t*)out_tokens.at, ws.at, ws.bytes);
    if (status) return PyLong_FromLong(status);
    return pair(n_accepted.result(), out_tokens.result());
}

// q_text, k_cache, video_start, n_video, text_pos0, softmax_scale, norm_mode, row_lse, beta, scores, workspace
PyObject* score(const Arg* a)
{
    const at::Tensor &q = a[0].tensor(), &k = a[1].tensor();
    if (q.dim() != 3 || k.dim() != 3 || q.stride(2) != 1 || k.stride(2) != 1) throw NotPlain();
    const int n_text = as_int(q.size(0)), hq = as_int(q.size(1)), d = as_int(q.size(2)), n_keys = as_int(k.size(0)), hkv = as_int(k.size(1));
    const int video_start = a[2].number(), n_video = a[3].number(), text_pos0 = a[4].number(), norm_mode = a[6].number();
    const float scale = (float)a[5].real();
    const double beta = a[8].real();         // (one that 32 bits take for 0 needs scores too)
    const float* const row_lse = (const float*)a[7].ptr();
    if (a[9].none() && beta != 0.) throw NotPlain();
    const Out scores(a[9], [&] { return make({n_video}, at::kFloat, q); });
    const Workspace ws(a[10], q, [&] { return c_score_bytes(1, n_text, n_keys, n_video, hq, hkv, d, !a[7].none()); });
    const int status = call(c_score, q.data_ptr(), q.stride(0), q.stride(1), k.data_ptr(), k.stride(0), k.stride(1), (const int32_t*)nullptr,
                            (const int32_t*)nullptr, (const int32_t*)nullptr, 1, n_text, n_keys, video_start, n_video, text_pos0, hq, hkv, d, scale,
                            norm_mode, row_lse, (float)beta, (float*)scores.at, ws.at, ws.bytes);
    return status ? PyLong_FromLong(status) : scores.result();
}

PyObject* select(const Arg* a)           // scores, k_top, keep_budget, total_keep, cu_video, cu_keep, max_n_video, want_flags, keep_idx
{
    const at::Tensor &scores = a[0].tensor(), &k_top = a[1].tensor();
    const int batch = as_int(k_top.numel()), total = a[3].number();
    if (a[6].none() && !a[4].none()) throw NotPlain();
    const int longest = a[6].none() ? as_int(scores.numel()) : a[6].number();
    const bool want_flags = a[7].truth();
    void* const budget = a[2].ptr();
    void* const cu_video = a[4].ptr();
    void* const cu_keep = a[5].ptr();
    const Out keep_idx(a[8], [&] { return make({total}, at::kInt, scores); });
    std::optional<at::Tensor> flags;
    if (want_flags) flags = make({total}, at::kByte, scores);
    const int status = call(c_select, (const float*)scores.data_ptr(), (const int32_t*)cu_video, (const int32_t*)k_top.data_ptr(),
                            (const int32_t*)budget, (const int32_t*)cu_keep, batch, longest, total, (int32_t*)keep_idx.at,
                            (uint8_t*)(flags ? flags->data_ptr() : nullptr), (int32_t*)nullptr, (void*)nullptr, (size_t)0);
    if (status) return PyLong_FromLong(status);
    return pair(keep_idx.result(), flags ? THPVariable_Wrap(*flags) : Py_NewRef(Py_None));
}

PyObject* top_p_count(const Arg* a)      // scores, lam, cu_video, max_n_video, max_count, count
{
    const at::Tensor& scores = a[0].tensor();
    const float lam = (float)a[1].real();
    if (a[3].none() && !a[2].none()) throw NotPlain();
    const int64_t batch = a[2].none() ? 1 : a[2].tensor().numel() - 1;
    const int b = as_int(batch), longest = a[3].none() ? as_int(scores.numel()) : a[3].number();
    void* const cu_video = a[2].ptr();
    void* const most = a[4].ptr();
    const Out count(a[5], [&] { return make({batch}, at::kInt, scores); });
    const int status = call(c_top_p_count, (const float*)scores.data_ptr(), (const int32_t*)cu_video, b, longest, lam, (const int32_t*)most,
                            (int32_t*)count.at, (void*)nullptr, (size_t)0);
    return status ? PyLong_FromLong(status) : count.result();
}

PyObject* gather_kv(const Arg* a)        // k_src, v_src, video_start, n_video, keep_idx, k_dst, v_dst, cu_keys, cu_video, cu_keep
{
    const at::Tensor& k = a[0].tensor();
    if (k.dim() != 4 || k.stride(3) != 1 || a[1].none()) throw NotPlain();
    const at::Tensor &v = a[1].tensor(), &keep = a[4].tensor();
    const int video_start = a[2].number(), n_video = a[3].number();
    const int layers = as_int(k.size(0)), n_keys = as_int(k.size(1)), hkv = as_int(k.size(2)), d = as_int(k.size(3)), n_keep = as_int(keep.numel());
    const int batch = a[7].none() ? 1 : as_int(a[7].tensor().numel() - 1);
    // (the destinations of a call that names neither or both)
    if (a[5].none() != a[6].none() || v.strides() != k.strides()) throw NotPlain();
    const Out k_dst(a[5], [&] { return at::empty({layers, (int64_t)n_keys - n_video + n_keep, hkv, d}, k.options()); });
    const at::Tensor& kd = a[5].none() ? *k_dst.made : a[5].tensor();
    const Out v_dst(a[6], [&] { return at::empty_like(kd); });
    const at::Tensor& vd = a[6].none() ? *v_dst.made : a[6].tensor();
    if (kd.dim() != 4 || vd.strides() != kd.strides()) throw NotPlain();
    void* const cu_keys = a[7].ptr();
    void* const cu_video = a[8].ptr();
    void* const cu_keep = a[9].ptr();
    const int status = call(c_gather_kv, k.data_ptr(), v.data_ptr(), k.stride(0), k.stride(1), k.stride(2), k_dst.at, v_dst.at, kd.stride(0),
                            kd.stride(1), kd.stride(2), layers, n_keys, video_start, n_video, (const int32_t*)keep.data_ptr(), n_keep,
                            (const int32_t*)cu_keys, (const int32_t*)cu_video, (const int32_t*)cu_keep, batch, (int32_t*)nullptr, hkv, d);
    if (status) return PyLong_FromLong(status);
    return pair(k_dst.result(), v_dst.result());
}

// q, k, v, softmax_scale, cu_q, cu_kv, max_q_len, max_kv_len, out, want_lse, num_splits, workspace, ancestor_mask
PyObject* decode_attn(const Arg* a)
{
    const at::Tensor &q = a[0].tensor(), &k = a[1].tensor(), &v = a[2].tensor();
    if (q.dim() != 3 || k.dim() != 3 || q.stride(2) != 1 || k.stride(2) != 1 || v.strides() != k.strides()) throw NotPlain();
    const int64_t tq = q.size(0), hq = q.size(1);
    const int h = as_int(hq), hkv = as_int(k.size(1)), d = as_int(q.size(2));
    int batch = 1, q_len = 0, kv_len = 0;
    if (a[4].none()) {
        q_len = as_int(tq); kv_len = as_int(k.size(0));
    } else {
        batch = as_int(a[4].tensor().numel() - 1); q_len = a[6].number(); kv_len = a[7].number();
    }
    const float scale = (float)a[3].real();
    const bool want_lse = a[9].truth();
    const int splits = a[10].number();
    void* const cu_q = a[4].ptr();
    void* const cu_kv = a[5].ptr();
    void* const mask = a[12].ptr();
    if (!a[8].none() && a[8].tensor().strides() != q.strides()) throw NotPlain();
    const Out out(a[8], [&] { return at::empty_like(q); });
    if (a[8].none() && out.made->strides() != q.strides()) throw NotPlain();
    std::optional<at::Tensor> lse;
    if (want_lse) lse = make({tq, hq}, at::kFloat, q);
    const Workspace ws(a[11], q, [&] { return c_attn_bytes(batch, q_len, kv_len, h, hkv, d, splits); });
    float* const lse_at = lse ? (float*)lse->data_ptr() : nullptr;
    const int status =
        !a[12].none() ? call(c_tree_attn, q.data_ptr(), q.stride(0), q.stride(1), k.data_ptr(), v.data_ptr(), k.stride(0), k.stride(1), (const int32_t*)cu_q,
                             (const int32_t*)cu_kv, batch, q_len, kv_len, h, hkv, d, scale, (const uint64_t*)mask, out.at, lse_at, splits, ws.at, ws.bytes)
                      : call(c_decode_attn, q.data_ptr(), q.stride(0), q.stride(1), k.data_ptr(), v.data_ptr(), k.stride(0), k.stride(1), (const int32_t*)cu_q,
                             (const int32_t*)cu_kv, batch, q_len, kv_len, h, hkv, d, scale, out.at, lse_at, splits, ws.at, ws.bytes);
    if (status) return PyLong_FromLong(status);
    return want_lse ? pair(out.result(), THPVariable_Wrap(*lse)) : out.result();
}

template <PyObject* (*F)(const Arg*), Py_ssize_t N>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (n != N) { PyErr_SetString(PyExc_TypeError, "wrong number of arguments"); return nullptr; }
    Arg a[N];
    for (Py_ssize_t i = 0; i < N; ++i) a[i].o = args[i];
    // nothing has been launched where one of these is thrown: what torch refuses (an allocation, a tensor without memory) the general code
    // meets again and reports
    try {
        if (!at::impl::torch_function_mode_enabled()) return F(a);
    } catch (const NotPlain&) {
    } catch (const std::exception&) {
    }
    PyErr_Clear();
    Py_RETURN_NONE;
}

PyObject* connect(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    void** const to[] = {(void**)&c_accept, (void**)&c_accept_bytes, (void**)&c_score, (void**)&c_score_bytes, (void**)&c_select,
                         (void**)&c_top_p_count, (void**)&c_gather_kv, (void**)&c_decode_attn, (void**)&c_tree_attn, (void**)&c_attn_bytes};
    if (n != (Py_ssize_t)(sizeof(to) / sizeof(to[0]))) { PyErr_SetString(PyExc_TypeError, "wrong number of addresses"); return nullptr; }
    void* at[sizeof(to) / sizeof(to[0])];
    for (Py_ssize_t i = 0; i < n; ++i) {
        at[i] = PyLong_AsVoidPtr(args[i]);
        if (!at[i]) { if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "no address"); return nullptr; }
    }
    for (Py_ssize_t i = 0; i < n; ++i) *to[i] = at[i];
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

extern "C" __attribute__((visibility("default"))) PyObject* PyInit__calls() { return PyModule_Create(&module); }
