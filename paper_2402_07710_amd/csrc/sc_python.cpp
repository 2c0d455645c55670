// CPython front of the calls a layer makes every frame: takes torch tensors, checks them, hands
// pointers and sizes to libsc's C functions and returns their status.  Argument marshalling only.
//
// A layer on a small cloud is three launches of 4-5 us of GPU time each, so the host's part of a call
// decides its pace.  The same marshalling in Python over ctypes costs 8.4-9.2 us per call (the current
// stream 2.7, seven to eight tensors 0.35 each, the ctypes conversion 0.8, the launch itself ~4); here
// everything but the launch is well under half a microsecond.
//
// The C functions are the ones of the library that binding.py has loaded: it passes their addresses
// to bind(), so both always use the same libsc.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "sc.h"

namespace {

struct Lib {
    decltype(&sc_hash_build) hash_build;
    decltype(&sc_hash_rebuild) hash_rebuild;
    decltype(&sc_kmap_build) kmap_build;
    decltype(&sc_kmap_build_noalloc) kmap_build_noalloc;
    decltype(&sc_kmap_transpose) kmap_transpose;
    decltype(&sc_conv_fwd) conv_fwd;
    decltype(&sc_conv_fwd_packed) conv_fwd_packed;
    decltype(&sc_conv_up_fwd) conv_up_fwd;
    decltype(&sc_conv_fwd_grid) conv_fwd_grid;
    decltype(&sc_grid_build) grid_build;
    decltype(&sc_kmap_build_grid) kmap_build_grid;
} lib;

struct PyFailure {};      // a Python exception is set

[[noreturn]] void fail(PyObject* kind, const char* what) {
    PyErr_SetString(kind, what);
    throw PyFailure{};
}

const at::Tensor& tensor(PyObject* o) {
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "tensor expected");
    return THPVariable_Unpack(o);
}
// device pointer of a tensor argument; null for None
void* ptr(PyObject* o) {
    if (o == Py_None) return nullptr;
    const at::Tensor& t = tensor(o);
    if (!t.is_cuda()) fail(PyExc_ValueError, "device tensor expected");
    if (!t.is_contiguous()) fail(PyExc_ValueError, "contiguous tensor expected");
    return t.data_ptr();
}
size_t nbytes(PyObject* o) { return o == Py_None ? 0 : tensor(o).nbytes(); }
int64_t size(PyObject* o, int dim) {
    const at::Tensor& t = tensor(o);
    if (dim >= t.dim()) fail(PyExc_IndexError, "tensor has too few dimensions");
    return t.size(dim);
}
int dtype(PyObject* o) {
    switch (tensor(o).scalar_type()) {
        case at::kFloat: return SC_F32;
        case at::kHalf: return SC_F16;
        case at::kBFloat16: return SC_BF16;
        default: fail(PyExc_KeyError, "dtype must be float32, float16 or bfloat16");
    }
}
long long integer(PyObject* o) {
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw PyFailure{};
    return v;
}
int small_int(PyObject* o) {
    const long long v = integer(o);
    if (v < INT32_MIN || v > INT32_MAX) fail(PyExc_OverflowError, "integer out of range");
    return (int)v;
}
uint32_t epoch32(PyObject* o) {
    const long long v = integer(o);
    if (v < 0 || v > (long long)UINT32_MAX) fail(PyExc_OverflowError, "epoch out of range");
    return (uint32_t)v;
}
struct Dims {
    int32_t B, X, Y, Z;
};
Dims dims(PyObject* o) {
    PyObject* seq = PySequence_Fast(o, "dims must be (B, X, Y, Z)");
    if (seq == nullptr) throw PyFailure{};
    Dims d{};
    try {
        if (PySequence_Fast_GET_SIZE(seq) != 4) fail(PyExc_TypeError, "dims must be (B, X, Y, Z)");
        int32_t* v[4] = {&d.B, &d.X, &d.Y, &d.Z};
        for (int i = 0; i < 4; ++i) *v[i] = small_int(PySequence_Fast_GET_ITEM(seq, i));
    } catch (...) {
        Py_DECREF(seq);
        throw;
    }
    Py_DECREF(seq);
    return d;
}
// None: torch's current stream; a torch stream; or the stream itself as an integer
void* stream(PyObject* o) {
    if (o == Py_None) return (void*)c10::hip::getCurrentHIPStream().stream();
    if (PyLong_Check(o)) {
        void* p = PyLong_AsVoidPtr(o);
        if (p == nullptr && PyErr_Occurred()) throw PyFailure{};
        return p;
    }
    PyObject* raw = PyObject_GetAttrString(o, "cuda_stream");
    if (raw == nullptr) throw PyFailure{};
    void* p = PyLong_AsVoidPtr(raw);
    Py_DECREF(raw);
    if (p == nullptr && PyErr_Occurred()) throw PyFailure{};
    return p;
}
// [rows, channels] and no other number of dimensions: a row's channels are contiguous
void check_matrix(PyObject* o, const char* what) {
    if (tensor(o).dim() != 2) fail(PyExc_ValueError, what);
}
bool same_dtype(PyObject* a, PyObject* b) { return tensor(a).scalar_type() == tensor(b).scalar_type(); }
// weight must be [K^3, C_in, C_out] in the feature type
bool weight_fits(PyObject* weight, PyObject* feat, int K, int64_t C_in, int64_t C_out) {
    const at::Tensor& w = tensor(weight);
    return w.dim() == 3 && w.size(0) == (int64_t)K * K * K && w.size(1) == C_in && w.size(2) == C_out && same_dtype(weight, feat);
}

using Args = PyObject* const*;

// The library's call with the interpreter lock released: a launch may block (full queue, first load of a code
// object) and other Python threads go on meanwhile.  The arguments have been read under the lock, and the
// caller's frame holds the tensors they point into.
template <class F, class... A>
int unlocked(F function, A... arguments) {
    PyThreadState* const thread = PyEval_SaveThread();
    const int rc = function(arguments...);
    PyEval_RestoreThread(thread);
    return rc;
}

int hash_build(Args a) {                 // coords, table, counts, stream
    return unlocked(lib.hash_build, (const int32_t*)ptr(a[0]), size(a[0], 0), ptr(a[1]), nbytes(a[1]), (sc_counts*)ptr(a[2]), stream(a[3]));
}
int hash_rebuild(Args a) {               // coords, table, epoch, counts, stream
    return unlocked(lib.hash_rebuild, (const int32_t*)ptr(a[0]), size(a[0], 0), ptr(a[1]), nbytes(a[1]), small_int(a[2]), (sc_counts*)ptr(a[3]),
                            stream(a[4]));
}
int kmap_build(Args a) {                 // coords, table, K, stride, mode, out_coords, kmap, scratch, counts, stream
    return unlocked(lib.kmap_build, (const int32_t*)ptr(a[0]), size(a[0], 0), ptr(a[1]), small_int(a[2]), small_int(a[3]), small_int(a[4]),
                          (int32_t*)ptr(a[5]), ptr(a[6]), nbytes(a[6]), ptr(a[7]), nbytes(a[7]), (sc_counts*)ptr(a[8]), stream(a[9]));
}
int kmap_build_noalloc(Args a) {         // coords, table, K, stride, mode, out_coords, kmap, counts, stream
    return unlocked(lib.kmap_build_noalloc, (const int32_t*)ptr(a[0]), size(a[0], 0), ptr(a[1]), small_int(a[2]), small_int(a[3]), small_int(a[4]),
                                  (int32_t*)ptr(a[5]), ptr(a[6]), nbytes(a[6]), (sc_counts*)ptr(a[7]), stream(a[8]));
}
int kmap_transpose(Args a) {             // kmap, n, K, stride, counts, kmap_inv, stream
    return unlocked(lib.kmap_transpose, ptr(a[0]), integer(a[1]), small_int(a[2]), small_int(a[3]), (const sc_counts*)ptr(a[4]), ptr(a[5]),
                              nbytes(a[5]), stream(a[6]));
}
int grid_build(Args a) {                 // coords, grid, dims, epoch, counts, stream
    const Dims d = dims(a[2]);
    return unlocked(lib.grid_build, (const int32_t*)ptr(a[0]), size(a[0], 0), ptr(a[1]), nbytes(a[1]), d.B, d.X, d.Y, d.Z, epoch32(a[3]),
                          (sc_counts*)ptr(a[4]), stream(a[5]));
}
int kmap_build_grid(Args a) {            // coords, grid, dims, epoch, K, kmap, counts, stream
    const Dims d = dims(a[2]);
    return unlocked(lib.kmap_build_grid, (const int32_t*)ptr(a[0]), size(a[0], 0), ptr(a[1]), nbytes(a[1]), d.B, d.X, d.Y, d.Z, epoch32(a[3]),
                               small_int(a[4]), ptr(a[5]), nbytes(a[5]), (sc_counts*)ptr(a[6]), stream(a[7]));
}
int conv_fwd(Args a) {                   // feat_in, n_map, weight, feat_out, kmap, counts, K, stride, mode, workspace, stream
    const int K = small_int(a[6]);
    check_matrix(a[0], "feat_in must be [rows, C_in]");
    check_matrix(a[3], "feat_out must be [rows, C_out]");
    const int64_t n_in = size(a[0], 0), C_in = size(a[0], 1), n_out_cap = size(a[3], 0), C_out = size(a[3], 1);
    if (!weight_fits(a[2], a[0], K, C_in, C_out)) fail(PyExc_ValueError, "weight must be [K^3, C_in, C_out] in the feature dtype");
    return unlocked(lib.conv_fwd, ptr(a[0]), a[1] == Py_None ? n_in : integer(a[1]), ptr(a[2]), ptr(a[3]), n_out_cap, ptr(a[4]), nbytes(a[4]),
                        (const sc_counts*)ptr(a[5]), K, small_int(a[7]), small_int(a[8]), (int)C_in, (int)C_out, dtype(a[0]), dtype(a[3]),
                        ptr(a[9]), nbytes(a[9]), stream(a[10]));
}
int conv_fwd_packed(Args a) {            // feat_in, n_map, packed, C_out, feat_out, kmap, counts, K, stride, mode, stream
    check_matrix(a[0], "feat_in must be [rows, C_in]");
    check_matrix(a[4], "feat_out must be [rows, C_out]");
    const int64_t n_in = size(a[0], 0), C_in = size(a[0], 1), n_out_cap = size(a[4], 0), C_out = integer(a[3]);
    if (size(a[4], 1) != C_out) fail(PyExc_ValueError, "feat_out must have C_out columns");
    return unlocked(lib.conv_fwd_packed, ptr(a[0]), a[1] == Py_None ? n_in : integer(a[1]), ptr(a[2]), ptr(a[4]), n_out_cap, ptr(a[5]),
                               nbytes(a[5]), (const sc_counts*)ptr(a[6]), small_int(a[7]), small_int(a[8]), small_int(a[9]), (int)C_in,
                               (int)C_out, dtype(a[0]), dtype(a[4]), stream(a[10]));
}
int conv_up_fwd(Args a) {                // feat_coarse, n_map, weight, feat_fine, kmap, counts, K, stream
    const int K = small_int(a[6]);
    const int64_t n_map = integer(a[1]), C_in = size(a[2], 1), C_out = size(a[2], 2);
    if (!weight_fits(a[2], a[0], K, C_in, C_out) || tensor(a[0]).dim() != 2 || size(a[0], 1) != C_in || tensor(a[3]).dim() != 2 || size(a[3], 0) != n_map ||
        size(a[3], 1) != C_out)
        return SC_EINVAL;
    return unlocked(lib.conv_up_fwd, ptr(a[0]), n_map, ptr(a[2]), ptr(a[3]), ptr(a[4]), nbytes(a[4]), (const sc_counts*)ptr(a[5]), K, (int)C_in,
                           (int)C_out, dtype(a[0]), dtype(a[3]), stream(a[7]));
}
int conv_fwd_grid(Args a) {              // feat_in, coords, grid, dims, epoch, weight, feat_out, K, workspace, stream
    const Dims d = dims(a[3]);
    return unlocked(lib.conv_fwd_grid, ptr(a[0]), (const int32_t*)ptr(a[1]), size(a[1], 0), ptr(a[2]), nbytes(a[2]), d.B, d.X, d.Y, d.Z,
                             epoch32(a[4]), ptr(a[5]), ptr(a[6]), small_int(a[7]), (int)size(a[5], 1), (int)size(a[5], 2), dtype(a[0]),
                             dtype(a[6]), ptr(a[8]), nbytes(a[8]), stream(a[9]));
}

template <int (*F)(Args), int N>
PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    if (nargs != N) {
        PyErr_Format(PyExc_TypeError, "%d arguments expected, %zd given", N, nargs);
        return nullptr;
    }
    try {
        return PyLong_FromLong(F(args));
    } catch (const PyFailure&) {
        return nullptr;
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// the addresses of the C functions, in the order of Lib's members
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    void* addr[sizeof(Lib) / sizeof(void*)];
    if (nargs != (Py_ssize_t)(sizeof(Lib) / sizeof(void*))) {
        PyErr_SetString(PyExc_TypeError, "one address per function expected");
        return nullptr;
    }
    for (Py_ssize_t i = 0; i < nargs; ++i) {
        addr[i] = PyLong_AsVoidPtr(args[i]);
        if (addr[i] == nullptr) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null function address");
            return nullptr;
        }
    }
    memcpy(&lib, addr, sizeof lib);
    Py_RETURN_NONE;
}

#define SC_METHOD(name, nargs) {#name, (PyCFunction)(void (*)(void))call<name, nargs>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"bind", (PyCFunction)(void (*)(void))bind, METH_FASTCALL, nullptr},
    SC_METHOD(hash_build, 4),
    SC_METHOD(hash_rebuild, 5),
    SC_METHOD(kmap_build, 10),
    SC_METHOD(kmap_build_noalloc, 9),
    SC_METHOD(kmap_transpose, 7),
    SC_METHOD(grid_build, 6),
    SC_METHOD(kmap_build_grid, 8),
    SC_METHOD(conv_fwd, 11),
    SC_METHOD(conv_fwd_packed, 11),
    SC_METHOD(conv_up_fwd, 8),
    SC_METHOD(conv_fwd_grid, 10),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "argument marshalling for libsc's calls", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
