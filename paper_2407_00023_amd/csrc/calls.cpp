// Python module _calls: the three calls of the hot path and the admission of a request, taking torch tensors.
//
// Argument marshalling only, in native code because a step of a small batch (a few requests being decoded) takes the
// GPU some tens of microseconds: through ctypes the three calls cost the host 38 us (checks, pointer objects, 3 us per
// look-up of the current stream), which the GPU then waits for; here the same checks take 1 us and what is left is the
// runtime's kernel launches.  Every function checks its tensors and forwards to the C entry point of the same name.
#include <Python.h>
#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>
#include <vector>

#include "../../include/prefixattn.h"

namespace {

PyObject* g_error_class = nullptr;  // PrefixAttnError(code, where)

// Arguments of one call by position or by name.  Returns false with a Python exception set.
template <int N>
bool parse_args(const char* fn, const char* const (&names)[N], int n_positional, int n_required, PyObject* const* args,
                Py_ssize_t nargs, PyObject* kwnames, PyObject* (&out)[N]) {
    for (int i = 0; i < N; ++i) out[i] = nullptr;
    if (nargs > n_positional) {
        PyErr_Format(PyExc_TypeError, "%s() takes %d positional arguments but %zd were given", fn, n_positional, nargs);
        return false;
    }
    for (Py_ssize_t i = 0; i < nargs; ++i) out[i] = args[i];
    const Py_ssize_t nkw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    for (Py_ssize_t k = 0; k < nkw; ++k) {
        PyObject* name = PyTuple_GET_ITEM(kwnames, k);
        const char* text = PyUnicode_AsUTF8(name);
        int at = -1;
        for (int i = 0; text && i < N && at < 0; ++i)
            if (std::strcmp(text, names[i]) == 0) at = i;
        if (at < 0) {
            PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", fn, name);
            return false;
        }
        if (out[at]) {
            PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%U'", fn, name);
            return false;
        }
        out[at] = args[nargs + k];
    }
    for (int i = 0; i < N; ++i) {
        const bool required = i < n_required || (i >= n_positional && (std::strcmp(names[i], "page_size") == 0 ||
                              std::strcmp(names[i], "num_slots") == 0 || std::strcmp(names[i], "max_kv_len") == 0));
        if (required && !out[i]) {
            PyErr_Format(PyExc_TypeError, "%s() missing required argument '%s'", fn, names[i]);
            return false;
        }
        if (out[i] == Py_None) out[i] = nullptr;
    }
    return true;
}

// The tensor behind a Python object; nullptr with a TypeError set if it is none.
const at::Tensor* tensor_of(PyObject* o, const char* name) {
    if (!o || !THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s must be a torch tensor", name);
        return nullptr;
    }
    return &THPVariable_Unpack(o);
}

bool device_int32(const at::Tensor& t, const char* name) {
    if (t.scalar_type() == at::kInt && t.is_cuda() && t.is_contiguous()) return true;
    PyErr_Format(PyExc_TypeError, "%s must be a contiguous int32 CUDA tensor", name);
    return false;
}

// None: torch's current stream; a torch stream object; or the raw handle as an integer.
bool stream_of(PyObject* o, void** out) {
    if (!o) {
        *out = static_cast<void*>(c10::hip::getCurrentHIPStream().stream());
        return true;
    }
    PyObject* raw = PyObject_HasAttrString(o, "cuda_stream") ? PyObject_GetAttrString(o, "cuda_stream") : PyNumber_Long(o);
    if (!raw) return false;
    *out = reinterpret_cast<void*>(static_cast<uintptr_t>(PyLong_AsUnsignedLongLongMask(raw)));
    Py_DECREF(raw);
    return !PyErr_Occurred();
}

// While one is alive, tensors are allocated for the call's stream instead of torch's current one: the caching allocator hands a
// block that is free on a stream to that stream's next tensors, and the kernels that use it are on the call's.  A tensor that is
// given to the caller is also marked as used on the current stream, where the caller will read it.
struct AllocateOn {
    const c10::hip::HIPStream before;
    bool other = false;
    AllocateOn(void* stream, const at::Tensor& like) : before(c10::hip::getCurrentHIPStream(like.device().index())) {
        hipStream_t s = static_cast<hipStream_t>(stream);
        if (s == hipStreamLegacy) s = nullptr;  // (two names of the default stream)
        other = before.stream() != s;
        if (other) c10::hip::setCurrentHIPStream(c10::hip::getStreamFromExternal(s, like.device().index()));
    }
    ~AllocateOn() { if (other) c10::hip::setCurrentHIPStream(before); }
    at::Tensor given(at::Tensor t) const {
        if (other) t.record_stream(c10::Stream(c10::Stream::UNSAFE, t.device(), before.id()));
        return t;
    }
    AllocateOn(const AllocateOn&) = delete;
    AllocateOn& operator=(const AllocateOn&) = delete;
};

// The interpreter's lock is given up while the library launches (other threads run on while a launch waits for a full queue).
struct WithoutGil {
    PyThreadState* const state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

PyObject* raise_code(int rc, const char* where) {
    PyObject* e = PyObject_CallFunction(g_error_class, "is", rc, where);
    if (e) {
        PyErr_SetObject(g_error_class, e);
        Py_DECREF(e);
    }
    return nullptr;
}

bool int_of(PyObject* o, long long* out) {
    if (!o) {
        PyErr_SetString(PyExc_TypeError, "page_size, num_slots and max_kv_len must be integers");
        return false;
    }
    *out = PyLong_AsLongLong(o);
    return !(*out == -1 && PyErr_Occurred());
}

// The library's dtype value of bf16 / fp32 tensors, kv8: the pool in its fp8 form.
bool dtype_of(const at::Tensor& t, PyObject* kv8, int* out) {
    const int on = kv8 ? PyObject_IsTrue(kv8) : 0;
    if (on < 0) return false;
    if (t.scalar_type() == at::kBFloat16) *out = on ? PA_BF16_KV8 : PA_BF16;
    else if (on) {
        PyErr_SetString(PyExc_TypeError, "the fp8 KV pool goes with bfloat16 tensors");
        return false;
    } else if (t.scalar_type() == at::kFloat) *out = PA_F32;
    else {
        PyErr_SetString(PyExc_TypeError, "tensors must be float32 or bfloat16");
        return false;
    }
    return true;
}

bool pool_large_enough(const at::Tensor& pool, long long num_slots, int Hkv, int D, int dtype, long long page_size) {
    const size_t need = pa_kv_pool_bytes(num_slots, Hkv, D, dtype, static_cast<int>(page_size));
    if (need == 0) PyErr_SetString(PyExc_ValueError, "pa_kv_pool_bytes: invalid arguments");
    else if (pool.nbytes() < need) PyErr_SetString(PyExc_ValueError, "kv_pool smaller than pa_kv_pool_bytes");
    return need != 0 && pool.nbytes() >= need;
}

#define CALLS_TRY try {
#define CALLS_CATCH                                       \
    }                                                     \
    catch (const std::exception& e) {                     \
        PyErr_SetString(PyExc_RuntimeError, e.what());    \
        return nullptr;                                   \
    }

// The tree of a Python Tree object; false with an exception set if it is none.
bool tree_of(PyObject* o, pa_tree** out) {
    PyObject* holder = o ? PyObject_GetAttrString(o, "_h") : nullptr;  // (ctypes.c_void_p of the tree)
    if (!holder) {
        if (!o) PyErr_SetString(PyExc_TypeError, "tree must be a Tree");
        return false;
    }
    PyObject* value = holder == Py_None ? Py_NewRef(holder) : PyObject_GetAttrString(holder, "value");
    Py_DECREF(holder);
    if (!value) return false;
    *out = value == Py_None ? nullptr : static_cast<pa_tree*>(PyLong_AsVoidPtr(value));
    Py_DECREF(value);
    return !PyErr_Occurred();
}

// match_prefixes(tree, tokens, offsets, prefix_len=None, slot_idx=None, stream=None); `tree` is the handle's address here
PyObject* match_prefixes(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    static const char* const names[] = {"tree", "tokens", "offsets", "prefix_len", "slot_idx", "stream"};
    PyObject* a[6];
    if (!parse_args("match_prefixes", names, 6, 3, args, nargs, kwnames, a)) return nullptr;
    CALLS_TRY
    pa_tree* tree = nullptr;
    if (!tree_of(a[0], &tree)) return nullptr;
    const at::Tensor *tokens = tensor_of(a[1], "tokens"), *offsets = tokens ? tensor_of(a[2], "offsets") : nullptr;
    if (!offsets || !device_int32(*tokens, "tokens") || !device_int32(*offsets, "offsets")) return nullptr;
    const int64_t B = offsets->numel() - 1;
    void* stream = nullptr;
    if (!stream_of(a[5], &stream)) return nullptr;
    at::Tensor made_len, made_slots;
    const at::Tensor *len = nullptr, *slots = nullptr;
    if (!a[3] || !a[4]) {
        const AllocateOn streams(stream, *tokens);
        if (!a[3]) len = &(made_len = streams.given(at::empty({B}, tokens->options())));
        if (!a[4]) slots = &(made_slots = streams.given(at::empty_like(*tokens)));
    }
    if (a[3]) len = tensor_of(a[3], "prefix_len");
    if (!len) return nullptr;
    if (a[4]) slots = tensor_of(a[4], "slot_idx");
    if (!slots || !device_int32(*len, "prefix_len") || !device_int32(*slots, "slot_idx")) return nullptr;
    if (len->numel() < B || slots->numel() < tokens->numel()) {
        PyErr_SetString(PyExc_ValueError, "output tensors too small");
        return nullptr;
    }
    int rc = PA_OK;
    {
        const WithoutGil released;
        rc = pa_match_prefixes(tree, static_cast<const int32_t*>(tokens->const_data_ptr()),
                               static_cast<const int32_t*>(offsets->const_data_ptr()), static_cast<int>(B),
                               static_cast<int32_t*>(len->data_ptr()), static_cast<int32_t*>(slots->data_ptr()), stream);
    }
    if (rc != PA_OK) return raise_code(rc, "pa_match_prefixes");
    PyObject* l = a[3] ? Py_NewRef(a[3]) : THPVariable_Wrap(made_len);
    PyObject* s = a[4] ? Py_NewRef(a[4]) : THPVariable_Wrap(made_slots);
    PyObject* both = l && s ? PyTuple_Pack(2, l, s) : nullptr;
    Py_XDECREF(l);
    Py_XDECREF(s);
    return both;
    CALLS_CATCH
}

// extend_attention(q_ext, k_ext, v_ext, kv_pool, slot_idx, slot_offsets, prefix_len, ext_len, ext_offsets, scale, *,
//                  page_size, num_slots, max_kv_len, out=None, workspace=None, stream=None, kv8=False)
PyObject* extend_attention(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    static const char* const names[] = {"q_ext", "k_ext", "v_ext", "kv_pool", "slot_idx", "slot_offsets", "prefix_len",
                                        "ext_len", "ext_offsets", "scale", "page_size", "num_slots", "max_kv_len", "out",
                                        "workspace", "stream", "kv8"};
    PyObject* a[17];
    if (!parse_args("extend_attention", names, 10, 10, args, nargs, kwnames, a)) return nullptr;
    CALLS_TRY
    const at::Tensor* t[9];
    for (int i = 0; i < 9; ++i)
        if (!(t[i] = tensor_of(a[i], names[i]))) return nullptr;
    const at::Tensor &q = *t[0], &k = *t[1], &v = *t[2], &pool = *t[3];
    int dtype = 0;
    if (!dtype_of(q, a[16], &dtype)) return nullptr;
    for (int i = 0; i < 3; ++i)
        if (!t[i]->is_cuda() || !t[i]->is_contiguous() || t[i]->scalar_type() != q.scalar_type()) {
            PyErr_Format(PyExc_TypeError, "%s must be a contiguous CUDA tensor of dtype %s", names[i], c10::toString(q.scalar_type()));
            return nullptr;
        }
    if (q.dim() != 3 || k.dim() != 3 || v.dim() != 3 || k.size(0) != q.size(0) || k.size(2) != q.size(2) || v.sizes() != k.sizes()) {
        PyErr_SetString(PyExc_ValueError, "k_ext / v_ext shape mismatch");
        return nullptr;
    }
    const int64_t T = q.size(0);
    const int Hq = static_cast<int>(q.size(1)), Hkv = static_cast<int>(k.size(1)), D = static_cast<int>(q.size(2));
    for (int i = 4; i < 9; ++i)
        if (!device_int32(*t[i], names[i])) return nullptr;
    const int64_t B = t[6]->numel();
    if (t[5]->numel() != B + 1 || t[8]->numel() != B + 1 || t[7]->numel() != B) {
        PyErr_SetString(PyExc_ValueError, "per-request arrays disagree on B");
        return nullptr;
    }
    if (!a[9]) {
        PyErr_SetString(PyExc_TypeError, "scale must be a number");
        return nullptr;
    }
    const double scale = PyFloat_AsDouble(a[9]);
    if (scale == -1.0 && PyErr_Occurred()) return nullptr;
    long long page_size = 0, num_slots = 0, max_kv_len = 0;
    if (!int_of(a[10], &page_size) || !int_of(a[11], &num_slots) || !int_of(a[12], &max_kv_len)) return nullptr;
    if (!pool_large_enough(pool, num_slots, Hkv, D, dtype, page_size)) return nullptr;
    void* stream = nullptr;
    if (!stream_of(a[15], &stream)) return nullptr;
    at::Tensor made_out, made_ws;
    const at::Tensor *out = nullptr, *ws = nullptr;
    if (a[13]) {
        if (!(out = tensor_of(a[13], "out"))) return nullptr;
        if (out->sizes() != q.sizes() || out->scalar_type() != q.scalar_type() || !out->is_contiguous() || !out->is_cuda()) {
            PyErr_SetString(PyExc_ValueError, "bad out tensor");
            return nullptr;
        }
    }
    const size_t need = pa_extend_workspace_bytes(static_cast<int>(B), T, max_kv_len, Hq, Hkv, D, dtype);
    if (need == 0) {
        PyErr_SetString(PyExc_ValueError, "pa_extend_workspace_bytes: invalid arguments");
        return nullptr;
    }
    if (a[14] && !(ws = tensor_of(a[14], "workspace"))) return nullptr;
    if (!out || !ws) {
        const AllocateOn streams(stream, q);
        if (!out) out = &(made_out = streams.given(at::empty_like(q)));
        if (!ws) ws = &(made_ws = at::empty({static_cast<int64_t>(need)}, q.options().dtype(at::kByte)));
    }
    auto i32 = [&](int i) { return static_cast<const int32_t*>(t[i]->const_data_ptr()); };
    int rc = PA_OK;
    {
        const WithoutGil released;
        rc = pa_extend_attention(q.const_data_ptr(), k.const_data_ptr(), v.const_data_ptr(), pool.const_data_ptr(), i32(4),
                                 i32(5), i32(6), i32(7), i32(8), static_cast<int>(B), T, max_kv_len, Hq, Hkv, D,
                                 static_cast<int>(page_size), num_slots, dtype, static_cast<float>(scale),
                                 out->data_ptr(), ws->data_ptr(), ws->nbytes(), stream);
    }
    if (rc != PA_OK) return raise_code(rc, "pa_extend_attention");
    return a[13] ? Py_NewRef(a[13]) : THPVariable_Wrap(made_out);
    CALLS_CATCH
}

// append_kv(kv_pool, new_slots, k_ext, v_ext, *, page_size, num_slots, stream=None, kv8=False)
PyObject* append_kv(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    static const char* const names[] = {"kv_pool", "new_slots", "k_ext", "v_ext", "page_size", "num_slots", "stream", "kv8"};
    PyObject* a[8];
    if (!parse_args("append_kv", names, 4, 4, args, nargs, kwnames, a)) return nullptr;
    CALLS_TRY
    const at::Tensor* t[4];
    for (int i = 0; i < 4; ++i)
        if (!(t[i] = tensor_of(a[i], names[i]))) return nullptr;
    const at::Tensor &pool = *t[0], &slots = *t[1], &k = *t[2], &v = *t[3];
    if (!device_int32(slots, "new_slots")) return nullptr;
    if (k.dim() != 3 || slots.numel() != k.size(0) || v.sizes() != k.sizes() || v.scalar_type() != k.scalar_type()) {
        PyErr_SetString(PyExc_ValueError, "append_kv: shape mismatch");
        return nullptr;
    }
    if (!k.is_cuda() || !v.is_cuda() || !k.is_contiguous() || !v.is_contiguous()) {
        PyErr_SetString(PyExc_TypeError, "k_ext / v_ext must be contiguous CUDA tensors");
        return nullptr;
    }
    int dtype = 0;
    long long page_size = 0, num_slots = 0;
    if (!dtype_of(k, a[7], &dtype) || !int_of(a[4], &page_size) || !int_of(a[5], &num_slots)) return nullptr;
    const int Hkv = static_cast<int>(k.size(1)), D = static_cast<int>(k.size(2));
    if (!pool_large_enough(pool, num_slots, Hkv, D, dtype, page_size)) return nullptr;
    void* stream = nullptr;
    if (!stream_of(a[6], &stream)) return nullptr;
    int rc = PA_OK;
    {
        const WithoutGil released;
        rc = pa_append_kv(pool.data_ptr(), static_cast<const int32_t*>(slots.const_data_ptr()), k.const_data_ptr(),
                          v.const_data_ptr(), k.size(0), Hkv, D, static_cast<int>(page_size), num_slots, dtype, stream);
    }
    if (rc != PA_OK) return raise_code(rc, "pa_append_kv");
    Py_RETURN_NONE;
    CALLS_CATCH
}

// tree_admit(tree, tokens, now) -> (n_cached, new_slots, handle), or None where tokens is no contiguous int32 vector in host
// memory or now no Python integer: nothing is done then, and the caller converts tokens or goes through ctypes, which takes (and
// refuses) all other types.  Native because a serving loop makes this call once per request: marshalled through ctypes and torch
// it took 6.4 us for 2 us of work.
PyObject* tree_admit(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    if (nargs != 3) {
        PyErr_SetString(PyExc_TypeError, "tree_admit() takes 3 arguments");
        return nullptr;
    }
    CALLS_TRY
    if (!THPVariable_Check(args[1])) Py_RETURN_NONE;
    const at::Tensor& tokens = THPVariable_Unpack(args[1]);
    if (tokens.scalar_type() != at::kInt || !tokens.is_cpu() || tokens.dim() != 1 || !tokens.is_contiguous() || tokens.numel() > INT32_MAX) Py_RETURN_NONE;
    if (!PyLong_Check(args[2])) Py_RETURN_NONE;
    const int64_t now = static_cast<int64_t>(PyLong_AsUnsignedLongLongMask(args[2]));
    pa_tree* tree = nullptr;
    if (PyErr_Occurred() || !tree_of(args[0], &tree)) return nullptr;
    const int32_t n = static_cast<int32_t>(tokens.numel());
    int32_t cached = 0;
    int64_t handle = 0;
    std::vector<int32_t> slots(static_cast<size_t>(n) + 1);
    int rc = PA_OK;
    {
        const WithoutGil released;
        rc = pa_tree_admit(tree, static_cast<const int32_t*>(tokens.const_data_ptr()), n, now, slots.data(), &cached, &handle);
    }
    if (rc != PA_OK) return raise_code(rc, "pa_tree_admit");
    at::Tensor fresh = at::empty({n - cached}, tokens.options());
    if (n > cached) std::memcpy(fresh.mutable_data_ptr(), slots.data() + cached, sizeof(int32_t) * static_cast<size_t>(n - cached));
    return Py_BuildValue("iNL", static_cast<int>(cached), THPVariable_Wrap(std::move(fresh)), static_cast<long long>(handle));
    CALLS_CATCH
}

// setup(PrefixAttnError): the exception class that error codes are raised as
PyObject* setup(PyObject*, PyObject* cls) {
    Py_INCREF(cls);
    Py_XSETREF(g_error_class, cls);
    Py_RETURN_NONE;
}

#define PA_FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL | METH_KEYWORDS
PyMethodDef g_methods[] = {
    {"match_prefixes", PA_FAST(match_prefixes),
     "match_prefixes($module, /, tree, tokens, offsets, prefix_len=None, slot_idx=None, stream=None)\n--\n\n"
     "-> (prefix_len int32 [B], slot_idx int32 like tokens).  Asynchronous on the stream."},
    {"extend_attention", PA_FAST(extend_attention),
     "extend_attention($module, /, q_ext, k_ext, v_ext, kv_pool, slot_idx, slot_offsets, prefix_len, ext_len, ext_offsets, "
     "scale, *, page_size, num_slots, max_kv_len, out=None, workspace=None, stream=None, kv8=False)\n--\n\n"
     "q_ext [T,Hq,D], k_ext/v_ext [T,Hkv,D] -> out [T,Hq,D].  Asynchronous on the stream."},
    {"append_kv", PA_FAST(append_kv),
     "append_kv($module, /, kv_pool, new_slots, k_ext, v_ext, *, page_size, num_slots, stream=None, kv8=False)\n--\n\n"
     "pool[new_slots[t]] = (k_ext[t], v_ext[t]).  Asynchronous on the stream."},
    {"tree_admit", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(tree_admit)), METH_FASTCALL,
     "tree_admit($module, tree, tokens, now, /)\n--\n\n-> (n_cached, new_slots, handle), or None if tokens or now is of another type than the usual one."},
    {"setup", setup, METH_O, "setup($module, error_class, /)\n--\n\nThe exception class error codes are raised as."},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_calls", "The hot-path calls of libprefixattn on torch tensors.", -1, g_methods,
                        nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() { return PyModule_Create(&g_module); }
