// The marshalling of binding.py's calls on the hot path, natively: exact Python ints, bf16 device tensors, mode names and the current stream
// to the arguments of the C entry points.  Whatever else a caller may pass (a tensor subclass other than a parameter, a raw address, a stream object, a numpy integer, a tensor
// that is refused) is answered with None, and binding.py takes its general path, which raises what there is to raise.
//
// What it is for: the launch itself takes 2.8 us on the host, the same marshalling in Python and ctypes takes 2.6 more, 0.25 of it per
// tensor and 0.37 for the stream; a product of less than 6 us on the GPU is bound by it.  The three products of a layer of 256 tokens, 512 -> 512:
// 18.6 us the general way, 12.7 here; of 1024 tokens, 512 -> 2048, where the kernels take 6 us each, 17.9 and 17.6.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <cstdint>
#include <exception>

namespace {

typedef int (*gemm_t)(int64_t, int64_t, int64_t, int, const void*, const void*, void*, int, void*);
typedef int (*tuned_t)(int, int64_t, int64_t, int64_t, const void*, const void*, void*, const void*, void*, size_t, int, void*, int*);
typedef int (*transpose_t)(int64_t, int64_t, const void*, void*, void*);

bool integer(PyObject* o, int64_t* v) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    *v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}

bool small_integer(PyObject* o, int* v) {
    int64_t x;
    if (!integer(o, &x) || x < INT_MIN || x > INT_MAX) return false;
    *v = (int)x;
    return true;
}

template <class F>
bool address(PyObject* o, F* f) {
    int64_t x;
    if (!integer(o, &x) || x == 0) return false;
    *f = reinterpret_cast<F>(x);
    return true;
}

// one of `names`, or a number
bool choice(PyObject* o, const char* const (&names)[3], int* v) {
    if (!PyUnicode_CheckExact(o)) return small_integer(o, v);
    for (int i = 0; i < 3; ++i)
        if (PyUnicode_CompareWithASCIIString(o, names[i]) == 0) {
            *v = i;
            return true;
        }
    return false;
}
const char* const kModes[3] = {"NN", "NT", "TN"};
const char* const kOps[3] = {"fwd", "bwd_data", "bwd_weight"};

bool tensor(PyObject* o, void** p) {
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || t.scalar_type() != at::kBFloat16 || !t.is_cuda() || !t.is_contiguous()) return false;
    *p = t.data_ptr();
    return true;
}

bool current_or_handle(PyObject* o, void** s) {
    if (o == Py_None) {
        *s = c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    int64_t x;
    if (!integer(o, &x)) return false;
    *s = reinterpret_cast<void*>(x);
    return true;
}

// Whether the arguments are all of the kinds above.  What the tensors and torch throw about them goes the general way too, and is thrown again there.
template <class F>
bool taken(F&& f) {
    try {
        return f();
    } catch (...) {
        PyErr_Clear();
        return false;
    }
}

// As ctypes does: other threads run while the call may wait for room in the queue.
struct OthersRun {
    PyThreadState* const state = PyEval_SaveThread();
    ~OthersRun() { PyEval_RestoreThread(state); }
};

// The call itself.  It has run, whatever comes out of it: never the general way a second time.
template <class F>
PyObject* status(F&& f) {
    int rc;
    try {
        OthersRun others;
        rc = f();
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
    return PyLong_FromLong(rc);
}

// (entry point, M, N, K, layout, first, second, out, fp32_accumulate, stream) -> status
PyObject* gemm(PyObject*, PyObject* const* v, Py_ssize_t n) {
    gemm_t f;
    int64_t M, N, K;
    int layout, fp32;
    void *a, *b, *c, *s;
    if (!taken([&] {
            return n == 10 && address(v[0], &f) && integer(v[1], &M) && integer(v[2], &N) && integer(v[3], &K) && choice(v[4], kModes, &layout) &&
                   tensor(v[5], &a) && tensor(v[6], &b) && tensor(v[7], &c) && small_integer(v[8], &fp32) && current_or_handle(v[9], &s);
        }))
        Py_RETURN_NONE;
    return status([&] { return f(M, N, K, layout, a, b, c, fp32, s); });
}

// (entry point, op, M, N, K, first, second, out, second_restored or None, fp32_accumulate, stream) -> the mode that ran, or a status below 0.
// Without scratch memory.
PyObject* tuned(PyObject*, PyObject* const* v, Py_ssize_t n) {
    tuned_t f;
    int64_t M, N, K;
    int op, fp32;
    void *a, *b, *c, *restored = nullptr, *s;
    if (!taken([&] {
            return n == 11 && address(v[0], &f) && choice(v[1], kOps, &op) && integer(v[2], &M) && integer(v[3], &N) && integer(v[4], &K) && tensor(v[5], &a) &&
                   tensor(v[6], &b) && tensor(v[7], &c) && (v[8] == Py_None || tensor(v[8], &restored)) && small_integer(v[9], &fp32) &&
                   current_or_handle(v[10], &s);
        }))
        Py_RETURN_NONE;
    return status([&] {
        int used = -1;
        const int rc = f(op, M, N, K, a, b, c, restored, nullptr, 0, fp32, s, &used);
        return rc == 0 ? used : rc;
    });
}

// (entry point, rows, cols, src, dst, stream) -> status
PyObject* transpose(PyObject*, PyObject* const* v, Py_ssize_t n) {
    transpose_t f;
    int64_t rows, cols;
    void *src, *dst, *s;
    if (!taken([&] {
            return n == 6 && address(v[0], &f) && integer(v[1], &rows) && integer(v[2], &cols) && tensor(v[3], &src) && tensor(v[4], &dst) &&
                   current_or_handle(v[5], &s);
        }))
        Py_RETURN_NONE;
    return status([&] { return f(rows, cols, src, dst, s); });
}

template <class F>
PyCFunction fast(F* f) { return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)); }
PyMethodDef kMethods[] = {{"gemm", fast(gemm), METH_FASTCALL, nullptr},
                          {"tuned", fast(tuned), METH_FASTCALL, nullptr},
                          {"transpose", fast(transpose), METH_FASTCALL, nullptr},
                          {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "axonn_marshal", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_axonn_marshal() {
    PyObject* const m = PyModule_Create(&kModule);
    // torch's classes are read by the layout that they had here
    if (m && PyModule_AddStringConstant(m, "torch_version", AXONN_TORCH_VERSION) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
