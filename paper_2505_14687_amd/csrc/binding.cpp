// The binding's calls in native code: an ordinary call (device tensors of a supported type, plain integers, the
// current or a given stream) is checked, its result allocated and the library entered without Python in between.  Of
// about 14 us a call took the host in Python, 8 went into attribute reads, comparisons and argument conversion.
//
// Every function returns what the call returns, or an int (the library's status where that is not GRAT_OK),
// or None: not an ordinary call, nothing has been done.  The caller then goes the long way in Python, which is where
// everything that is refused is refused, with its message.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/device_lazy_init.h>

#include "grat.h"

namespace {

struct Library {   // entry points of libgrat.so, as the loader has found them
    decltype(&grat_block_list_shape) list_shape;
    decltype(&grat_build_block_lists) build_lists;
    decltype(&grat_attention_fwd) attention;
    decltype(&grat_attention_global_fwd) attention_global;
    decltype(&grat_attention_packed_fwd) attention_packed;
    decltype(&grat_dense_attention_fwd) dense;
} g_lib;

// set_library(addresses): in the order above
PyObject* set_library(PyObject*, PyObject* args) {
    unsigned long long a[6];
    if (!PyArg_ParseTuple(args, "KKKKKK", a, a + 1, a + 2, a + 3, a + 4, a + 5)) return nullptr;
    g_lib = {(decltype(g_lib.list_shape))a[0],       (decltype(g_lib.build_lists))a[1],
             (decltype(g_lib.attention))a[2],        (decltype(g_lib.attention_global))a[3],
             (decltype(g_lib.attention_packed))a[4], (decltype(g_lib.dense))a[5]};
    Py_RETURN_NONE;
}

struct Unusual {};   // thrown where a call is not an ordinary one

void need(bool ok) {
    if (!ok) throw Unusual{};
}

// A plain dense tensor: no subclass, no wrapper of a transform, no lazy negation or conjugation.
const at::Tensor& tensor_of(PyObject* o) {
    need(THPVariable_CheckExact(o));
    const at::Tensor& t = THPVariable_Unpack(o);
    need(t.defined() && t.layout() == at::kStrided && t.has_storage());
    using K = c10::DispatchKey;
    const c10::DispatchKeySet keys = t.key_set();
    for (const K k : {K::Python, K::PythonTLSSnapshot, K::FuncTorchBatched, K::FuncTorchGradWrapper, K::Functionalize,
                      K::Negative, K::Conjugate, K::ZeroTensor})
        need(!keys.has(k));
    return t;
}

int64_t int_of(PyObject* o) {
    need(PyLong_CheckExact(o));
    int overflow = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
    need(overflow == 0 && v >= INT32_MIN && v <= INT32_MAX);
    return v;
}

int32_t bool_of(PyObject* o) {   // bool() as Python has it, of the kinds that cannot run code of their own
    need(PyBool_Check(o) || PyLong_CheckExact(o));
    return PyObject_IsTrue(o) ? 1 : 0;
}

float scale_of(PyObject* o) {
    need(PyFloat_CheckExact(o) || PyLong_CheckExact(o));
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) {
        PyErr_Clear();
        throw Unusual{};
    }
    return (float)v;
}

struct Extents {   // of a grid, a group or a radius
    int32_t n = 0, v[3];
    explicit Extents(PyObject* o) {
        const bool list = PyList_CheckExact(o);
        need(list || PyTuple_Check(o));
        n = (int32_t)(list ? PyList_GET_SIZE(o) : PyTuple_GET_SIZE(o));
        need(n >= 1 && n <= 3);
        for (int i = 0; i < n; ++i) v[i] = (int32_t)int_of(list ? PyList_GET_ITEM(o, i) : PyTuple_GET_ITEM(o, i));
    }
};

// The device is set up as it is ahead of every tensor that Python makes there, and nothing is done in a forked child.
hipStream_t stream_of(PyObject* o) {
    need(!torch::utils::is_device_in_bad_fork(at::kCUDA));
    torch::utils::device_lazy_init(at::kCUDA);
    if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
    PyObject* p = PyObject_GetAttrString(o, "cuda_stream");
    const bool ok = p && PyLong_Check(p);
    const unsigned long long v = ok ? PyLong_AsUnsignedLongLong(p) : 0;
    Py_XDECREF(p);
    if (!ok || PyErr_Occurred()) {
        PyErr_Clear();
        throw Unusual{};
    }
    return (hipStream_t)(uintptr_t)v;
}

grat_dtype dtype_of(const at::Tensor& t) {
    switch (t.scalar_type()) {
        case at::kBFloat16: return GRAT_BF16;
        case at::kHalf: return GRAT_F16;
        case at::kFloat: return GRAT_F32;
        default: throw Unusual{};
    }
}

void check_like(const at::Tensor& q, const at::Tensor& t) {
    need(t.sizes() == q.sizes() && t.strides() == q.strides() && t.scalar_type() == q.scalar_type() && t.device() == q.device());
}

struct Lists {
    const at::Tensor &count, &index;
    Lists(PyObject* c, PyObject* i, const Extents& grid, const Extents& group, const at::Tensor& q)
        : count(tensor_of(c)), index(tensor_of(i)) {
        need(grid.n == group.n);
        int64_t groups = 1;
        for (int k = 0; k < grid.n; ++k) {
            need(grid.v[k] >= 1 && group.v[k] >= 1 && groups < INT32_MAX);
            groups *= ((int64_t)grid.v[k] + group.v[k] - 1) / group.v[k];
        }
        for (const at::Tensor* t : {&count, &index})
            need(t->scalar_type() == at::kInt && t->is_contiguous() && t->device() == q.device());
        need(count.dim() == 1 && count.numel() == groups);
        need(index.dim() == 2 && index.size(0) == groups && index.size(1) >= 1 && index.size(1) <= INT32_MAX);
    }
    const int32_t* c() const { return (const int32_t*)count.data_ptr(); }
    const int32_t* i() const { return (const int32_t*)index.data_ptr(); }
    int32_t max_kv() const { return (int32_t)index.size(1); }
};

void check_sequence(int64_t rows, const Extents& grid, int64_t n_global) {
    __int128 n = 1;
    for (int k = 0; k < grid.n; ++k) n *= grid.v[k];
    need(n_global >= 0 && (__int128)rows == n + n_global);
}

template <typename F>
grat_status without_gil(F&& f) {
    PyThreadState* s = PyEval_SaveThread();
    const grat_status st = f();
    PyEval_RestoreThread(s);
    return st;
}

PyObject* result(grat_status st, PyObject* given, const at::Tensor& o) {
    if (st != GRAT_OK) return PyLong_FromLong((long)st);
    if (given != Py_None) {
        Py_INCREF(given);
        return given;
    }
    return THPVariable_Wrap(o);
}

// Runs f(), which returns a new reference; None where the call is not an ordinary one (or something went wrong before
// the library was entered: the long way then meets the same and reports it).
template <typename F>
PyObject* ordinary(Py_ssize_t have, Py_ssize_t want, F&& f) {
    if (have != want) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    try {
        need(!at::impl::torch_function_mode_enabled() && !c10::impl::TorchDispatchModeTLS::any_modes_set());
        return f();
    } catch (...) {
        if (PyErr_Occurred()) PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// attention(Q, K, V, scale, n_global or None, global_first, grid, group, kv_count, kv_index, out, stream)
PyObject* attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return ordinary(n, 12, [&]() -> PyObject* {
        const at::Tensor &q = tensor_of(a[0]), &k = tensor_of(a[1]), &v = tensor_of(a[2]);
        need(q.dim() == 4 && q.is_cuda() && q.stride(3) == 1);
        check_like(q, k);
        check_like(q, v);
        const grat_dtype dt = dtype_of(q);
        const float scale = scale_of(a[3]);
        const bool joint = a[4] != Py_None;
        const int64_t n_global = joint ? int_of(a[4]) : 0;
        const int32_t first = joint ? bool_of(a[5]) : 1;
        const Extents grid(a[6]), group(a[7]);
        const Lists lists(a[8], a[9], grid, group, q);
        check_sequence(q.size(2), grid, n_global);
        need(q.size(0) <= INT32_MAX && q.size(1) <= INT32_MAX && q.size(3) <= INT32_MAX);
        const hipStream_t stream = stream_of(a[11]);
        const at::Tensor o = a[10] == Py_None ? at::empty_like(q) : tensor_of(a[10]);
        check_like(q, o);
        void *qp = q.data_ptr(), *kp = k.data_ptr(), *vp = v.data_ptr(), *op = o.data_ptr();
        const int32_t *cp = lists.c(), *ip = lists.i();
        const int32_t B = (int32_t)q.size(0), H = (int32_t)q.size(1), d = (int32_t)q.size(3);
        const int64_t sb = q.stride(0), sh = q.stride(1), sn = q.stride(2);
        return result(without_gil([&] {
            return joint ? g_lib.attention_global(qp, kp, vp, op, dt, B, H, d, sb, sh, sn, scale, (int32_t)n_global, first, grid.n, grid.v,
                                                  group.v, cp, ip, lists.max_kv(), stream)
                         : g_lib.attention(qp, kp, vp, op, dt, B, H, d, sb, sh, sn, scale, grid.n, grid.v, group.v, cp, ip,
                                           lists.max_kv(), stream);
        }), a[10], o);
    });
}

// packed(QKV, scale, n_global, global_first, grid, group, kv_count, kv_index, out, stream)
PyObject* packed(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return ordinary(n, 10, [&]() -> PyObject* {
        const at::Tensor& x = tensor_of(a[0]);
        need(x.dim() == 5 && x.size(2) == 3 && x.is_contiguous() && x.is_cuda());
        const grat_dtype dt = dtype_of(x);
        const float scale = scale_of(a[1]);
        const int64_t n_global = int_of(a[2]);
        const int32_t first = bool_of(a[3]);
        const Extents grid(a[4]), group(a[5]);
        const Lists lists(a[6], a[7], grid, group, x);
        check_sequence(x.size(1), grid, n_global);
        need(x.size(0) <= INT32_MAX && x.size(3) <= INT32_MAX && x.size(4) <= INT32_MAX);
        const hipStream_t stream = stream_of(a[9]);
        const std::array<int64_t, 4> shape = {x.size(0), x.size(1), x.size(3), x.size(4)};
        const at::Tensor o = a[8] == Py_None ? at::empty(shape, x.options()) : tensor_of(a[8]);
        need(o.sizes() == at::IntArrayRef(shape) && o.scalar_type() == x.scalar_type() && o.is_contiguous() && o.device() == x.device());
        void *xp = x.data_ptr(), *op = o.data_ptr();
        const int32_t *cp = lists.c(), *ip = lists.i();
        return result(without_gil([&] {
            return g_lib.attention_packed(xp, op, dt, (int32_t)shape[0], (int32_t)shape[2], (int32_t)shape[3], scale, (int32_t)n_global,
                                          first, grid.n, grid.v, group.v, cp, ip, lists.max_kv(), stream);
        }), a[8], o);
    });
}

// dense(Q, K, V, scale, out, stream)
PyObject* dense(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return ordinary(n, 6, [&]() -> PyObject* {
        const at::Tensor &q = tensor_of(a[0]), &k = tensor_of(a[1]), &v = tensor_of(a[2]);
        need(q.dim() == 4 && q.is_cuda() && q.stride(3) == 1);
        check_like(q, k);
        check_like(q, v);
        const grat_dtype dt = dtype_of(q);
        const float scale = scale_of(a[3]);
        need(q.size(0) <= INT32_MAX && q.size(1) <= INT32_MAX && q.size(3) <= INT32_MAX);
        const hipStream_t stream = stream_of(a[5]);
        const at::Tensor o = a[4] == Py_None ? at::empty_like(q) : tensor_of(a[4]);
        check_like(q, o);
        void *qp = q.data_ptr(), *kp = k.data_ptr(), *vp = v.data_ptr(), *op = o.data_ptr();
        return result(without_gil([&] {
            return g_lib.dense(qp, kp, vp, op, dt, (int32_t)q.size(0), (int32_t)q.size(1), q.size(2), (int32_t)q.size(3), q.stride(0),
                               q.stride(1), q.stride(2), scale, stream);
        }), a[4], o);
    });
}

// block_lists(grid, group, pattern id, radius or None, stream): (kv_count, kv_index) on the current device
PyObject* block_lists(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return ordinary(n, 5, [&]() -> PyObject* {
        const Extents grid(a[0]), group(a[1]);
        need(grid.n == group.n);
        const int64_t id = int_of(a[2]);
        need(id >= GRAT_BLOCK && id <= GRAT_DENSE);
        const grat_pattern pattern = (grat_pattern)id;
        int32_t radius[3];
        const bool has_radius = a[3] != Py_None;
        if (has_radius) {
            const Extents r(a[3]);
            need(r.n == grid.n);
            for (int k = 0; k < r.n; ++k) radius[k] = r.v[k];
        }
        const int32_t* rp = has_radius ? radius : nullptr;
        int32_t groups = 0, max_kv = 0;
        need(g_lib.list_shape(grid.n, grid.v, group.v, pattern, rp, &groups, &max_kv) == GRAT_OK && max_kv >= 1);
        const hipStream_t stream = stream_of(a[4]);
        const at::TensorOptions opt = at::TensorOptions().dtype(at::kInt).device(at::kCUDA);
        const at::Tensor count = at::empty({groups}, opt), index = at::empty({groups, max_kv}, opt);
        int32_t *cp = (int32_t*)count.data_ptr(), *ip = (int32_t*)index.data_ptr();
        const grat_status st = without_gil([&] { return g_lib.build_lists(grid.n, grid.v, group.v, pattern, rp, cp, ip, max_kv, stream); });
        if (st != GRAT_OK) return PyLong_FromLong((long)st);
        PyObject *c = THPVariable_Wrap(count), *i = THPVariable_Wrap(index);
        PyObject* pair = c && i ? PyTuple_Pack(2, c, i) : nullptr;
        Py_XDECREF(c);
        Py_XDECREF(i);
        return pair;
    });
}

PyMethodDef kMethods[] = {
    {"set_library", set_library, METH_VARARGS, nullptr},
    {"attention", (PyCFunction)(void (*)())attention, METH_FASTCALL, nullptr},
    {"packed", (PyCFunction)(void (*)())packed, METH_FASTCALL, nullptr},
    {"dense", (PyCFunction)(void (*)())dense, METH_FASTCALL, nullptr},
    {"block_lists", (PyCFunction)(void (*)())block_lists, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&kModule); }
