// The library's per-step calls for Python (module _sdp_native): the C functions of sdp.h, with tensors where they take
// device pointers.  A call checks every tensor (contiguous, on the GPU, of the expected type; TypeError otherwise) and
// passes its address; integers pass as they are.  The GIL is released around the call.  Returns the status.
//
// Through ctypes a worker's MLP forward or backward costs the host about 9 us, most of it in marshalling 20 arguments,
// which is more than the fp32 kernels of a small step take on the GPU (four workers of 256 tokens, 10 calls and 18 launches:
// 139 us a step then, 101 this way).
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include "sdp.h"

namespace {

// A pointer parameter: its name in messages and what it points to: 'a' the type given by the call's dtype argument,
// 'i' int32, 'f' float32, in capitals where None stands for a null pointer; 0 for parameters passed as they are
// (integers, workspace and stream addresses).
struct Param {
    const char* name = nullptr;
    char kind = 0;
};

bool type_error(const Param& p, c10::ScalarType t) {
    const char* n = t == c10::kFloat ? "torch.float32" : t == c10::kBFloat16 ? "torch.bfloat16" : "torch.int32";
    PyErr_Format(PyExc_TypeError, "%s: expected a contiguous %s tensor on the GPU", p.name, n);
    return false;
}

template <class A>
bool take(PyObject* o, const Param& p, c10::ScalarType act, A& out) {
    if constexpr (std::is_pointer_v<A>) {
        if (p.kind == 0) {
            out = (A)PyLong_AsVoidPtr(o);
            return !PyErr_Occurred();
        }
        const bool optional = p.kind == 'A' || p.kind == 'I';
        if (optional && o == Py_None) {
            out = nullptr;
            return true;
        }
        const c10::ScalarType want = p.kind == 'f' ? c10::kFloat : p.kind == 'i' || p.kind == 'I' ? c10::kInt : act;
        if (!THPVariable_Check(o)) return type_error(p, want);
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.is_cuda() || !t.is_contiguous() || t.scalar_type() != want) return type_error(p, want);
        out = (A)t.data_ptr();
        return true;
    } else if constexpr (std::is_unsigned_v<A>) {
        out = (A)PyLong_AsUnsignedLongLong(o);
        return !PyErr_Occurred();
    } else {
        const long long v = PyLong_AsLongLong(o);
        if (v == -1 && PyErr_Occurred()) return false;
        if (v != (long long)(A)v) {
            PyErr_SetString(PyExc_OverflowError, "integer argument out of range");
            return false;
        }
        out = (A)v;
        return true;
    }
}

template <class... A, size_t... I>
PyObject* call(int (*fn)(A...), const Param* params, int dtype_at, PyObject* const* args, Py_ssize_t n, std::index_sequence<I...>) {
    if (n != (Py_ssize_t)sizeof...(A)) {
        PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", (Py_ssize_t)sizeof...(A), n);
        return nullptr;
    }
    const long dtype = PyLong_AsLong(args[dtype_at]);
    if (dtype == -1 && PyErr_Occurred()) return nullptr;
    const c10::ScalarType act = dtype == SDP_F32 ? c10::kFloat : c10::kBFloat16;
    std::tuple<A...> v;
    int rc = 0;
    try {
        if (!(take(args[I], params[I], act, std::get<I>(v)) && ...)) return nullptr;
    } catch (const std::exception& e) { // a tensor without storage
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
    Py_BEGIN_ALLOW_THREADS
    rc = std::apply(fn, v);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

#define SDP_ENTRY(py, fn, dtype_at, ...)                                                                     \
    const Param py##_params[] = {__VA_ARGS__};                                                               \
    template <class... A>                                                                                    \
    PyObject* py##_call(int (*f)(A...), PyObject* const* args, Py_ssize_t n) {                               \
        static_assert(sizeof(py##_params) / sizeof(Param) == sizeof...(A), "one entry per parameter");       \
        return call(f, py##_params, dtype_at, args, n, std::index_sequence_for<A...>{});                     \
    }                                                                                                        \
    PyObject* py(PyObject*, PyObject* const* args, Py_ssize_t n) { return py##_call(&fn, args, n); }

SDP_ENTRY(mlp_fwd, sdp_masked_mlp_fwd, 1, {}, {}, {}, {}, {}, {}, {"X", 'a'}, {"W1", 'a'}, {"W3", 'a'}, {"W2T", 'a'},
          {"idx_k", 'I'}, {"Y", 'a'}, {"G_save", 'a'}, {"U_save", 'a'}, {}, {}, {})
SDP_ENTRY(mlp_bwd, sdp_masked_mlp_bwd, 1, {}, {}, {}, {}, {}, {}, {"X", 'a'}, {"dY", 'a'}, {"W1", 'a'}, {"W3", 'a'},
          {"W2T", 'a'}, {"idx_k", 'i'}, {"G_save", 'a'}, {"U_save", 'a'}, {"dX", 'a'}, {"dW1", 'a'}, {"dW3", 'a'}, {"dW2T", 'a'},
          {}, {}, {}, {})
SDP_ENTRY(attn_fwd, sdp_masked_attn_fwd, 1, {}, {}, {}, {}, {}, {}, {}, {}, {"X", 'a'}, {"Wqkv", 'a'}, {"WoT", 'a'},
          {"head_idx_k", 'I'}, {"Y", 'a'}, {"QKV_save", 'a'}, {"O_save", 'a'}, {"LSE_save", 'f'}, {}, {}, {})
SDP_ENTRY(attn_bwd, sdp_masked_attn_bwd, 1, {}, {}, {}, {}, {}, {}, {}, {}, {"X", 'a'}, {"dY", 'a'}, {"Wqkv", 'a'},
          {"WoT", 'a'}, {"head_idx_k", 'i'}, {"QKV_save", 'a'}, {"O_save", 'a'}, {"LSE_save", 'f'}, {"dX", 'a'}, {"dWqkv", 'a'},
          {"dWoT", 'a'}, {}, {}, {}, {})
SDP_ENTRY(block_fwd, sdp_block_fwd, 2, {}, {}, {}, {}, {}, {}, {}, {}, {}, {"X", 'a'}, {"Wqkv", 'a'}, {"WoT", 'a'},
          {"W1", 'a'}, {"W3", 'a'}, {"W2T", 'a'}, {"Y", 'a'}, {"Hm_save", 'a'}, {"QKV_save", 'a'}, {"O_save", 'a'},
          {"LSE_save", 'f'}, {"G_save", 'a'}, {"U_save", 'a'}, {}, {}, {})
SDP_ENTRY(block_bwd, sdp_block_bwd, 3, {}, {}, {}, {}, {}, {}, {}, {}, {}, {}, {"X", 'a'}, {"dY", 'a'}, {"Wqkv", 'a'},
          {"WoT", 'a'}, {"W1", 'a'}, {"W3", 'a'}, {"W2T", 'a'}, {"Hm_save", 'a'}, {"QKV_save", 'a'}, {"O_save", 'a'},
          {"LSE_save", 'f'}, {"G_save", 'a'}, {"U_save", 'a'}, {"dX", 'a'}, {"dW", 'A'}, {"dW", 'A'}, {"dW", 'A'}, {"dW", 'A'},
          {"dW", 'A'}, {}, {}, {})

#define SDP_METHOD(py) {#py, (PyCFunction)(void (*)(void))py, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {SDP_METHOD(mlp_fwd),   SDP_METHOD(mlp_bwd),   SDP_METHOD(attn_fwd), SDP_METHOD(attn_bwd),
                         SDP_METHOD(block_fwd), SDP_METHOD(block_bwd), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_sdp_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__sdp_native() {
    PyObject* m = PyModule_Create(&module);
    // the C++ interface of one torch build: binding.py compares
    if (m && PyModule_AddStringConstant(m, "torch_version", SDP_TORCH_VERSION) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
