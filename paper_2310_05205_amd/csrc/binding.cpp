// Python entry of the calls that a program makes every step: selection,
// collection, priority update and their sharded forms.
//
// A step's kernels take 2 to 20 us on the small workloads, and allocating its
// outputs and marshalling its arguments in Python took longer than that.  Each
// function here allocates the outputs as torch tensors, passes their addresses
// to the C ABI and wraps them, with the interpreter lock released around the
// library call.  The library is reached through the addresses that the Python
// binding hands to bind(), so both use the one it loaded.
//
// Every call returns its results, or the library's negative status as an int.
#include <Python.h>

#include <ATen/Functions.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <exception>
#include <vector>

#include "gear.h"

namespace {

decltype(&gear_select) f_select = nullptr;
decltype(&gear_collect) f_collect = nullptr;
decltype(&gear_select_collect) f_select_collect = nullptr;
decltype(&gear_update_priorities) f_update = nullptr;
decltype(&gear_select_shard) f_select_shard = nullptr;
decltype(&gear_is_weights) f_is_weights = nullptr;
decltype(&gear_topk_merge) f_topk_merge = nullptr;

// One column of a table as its batches are handed out.
struct Column {
    at::ScalarType dtype;
    std::vector<int64_t> shape;  // per step
    int64_t elem_bytes;
};
const char* const kPlanName = "gear column plan";

// A Python error that is already set.
struct PythonError {};

int64_t as_int(PyObject* o) {
    PyObject* i = PyNumber_Index(o);
    if (i == nullptr) throw PythonError();
    const long long v = PyLong_AsLongLong(i);
    Py_DECREF(i);
    if (v == -1 && PyErr_Occurred()) throw PythonError();
    return v;
}

int32_t as_int32(PyObject* o) {
    const int64_t v = as_int(o);
    if (v != (int32_t)v) {
        PyErr_SetString(PyExc_OverflowError, "argument out of the 32-bit range");
        throw PythonError();
    }
    return (int32_t)v;
}

uint64_t as_u64(PyObject* o) {
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
    if (v == (unsigned long long)-1 && PyErr_Occurred()) throw PythonError();
    return v;
}

float as_float(PyObject* o) {
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw PythonError();
    return (float)v;
}

bool as_bool(PyObject* o) {
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw PythonError();
    return v != 0;
}

void* as_ptr(PyObject* o) {
    if (o == Py_None) return nullptr;
    void* p = PyLong_AsVoidPtr(o);
    if (p == nullptr && PyErr_Occurred()) throw PythonError();
    return p;
}

// Device address of a tensor, or of anything else with a data_ptr() method.
void* address_of(PyObject* o) {
    if (THPVariable_Check(o)) return THPVariable_Unpack(o).data_ptr();
    PyObject* v = PyObject_CallMethod(o, "data_ptr", nullptr);
    if (v == nullptr) throw PythonError();
    void* p = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    if (p == nullptr && PyErr_Occurred()) throw PythonError();
    return p;
}

// shape[0], which the library takes as a 32-bit batch size.
int32_t batch_of(PyObject* o) {
    int64_t n;
    if (THPVariable_Check(o)) {
        n = THPVariable_Unpack(o).size(0);
    } else {
        PyObject* shape = PyObject_GetAttrString(o, "shape");
        if (shape == nullptr) throw PythonError();
        PyObject* v = PySequence_GetItem(shape, 0);
        Py_DECREF(shape);
        if (v == nullptr) throw PythonError();
        n = PyLong_AsLongLong(v);
        Py_DECREF(v);
        if (n == -1 && PyErr_Occurred()) throw PythonError();
    }
    if (n != (int32_t)n) {
        PyErr_SetString(PyExc_OverflowError, "batch out of the 32-bit range");
        throw PythonError();
    }
    return (int32_t)n;
}

at::Tensor empty(at::IntArrayRef sizes, at::ScalarType dtype, int32_t device) {
    return at::empty(sizes, at::TensorOptions().dtype(dtype).device(at::Device(at::kCUDA, (at::DeviceIndex)device)));
}

PyObject* wrap(at::Tensor t) {
    PyObject* o = THPVariable_Wrap(std::move(t));
    if (o == nullptr) throw PythonError();
    return o;
}

template <typename F>
int without_gil(F call) {
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return rc;
}

// A tuple that owns the items set so far.
struct Tuple {
    PyObject* t;
    explicit Tuple(Py_ssize_t n) : t(PyTuple_New(n)) {
        if (t == nullptr) throw PythonError();
    }
    ~Tuple() { Py_XDECREF(t); }
    void set(Py_ssize_t i, PyObject* o) { PyTuple_SET_ITEM(t, i, o); }
    void none(Py_ssize_t i) {
        Py_INCREF(Py_None);
        PyTuple_SET_ITEM(t, i, Py_None);
    }
    PyObject* release() {
        PyObject* r = t;
        t = nullptr;
        return r;
    }
};

// The batch buffers of a call: `ids` None for every column, else a list.
struct Batch {
    std::vector<int32_t> ids;
    std::vector<at::Tensor> out;
    std::vector<void*> ptr;
    bool all;

    Batch(PyObject* plan, PyObject* id_list, bool typed, int64_t B, int64_t L, int32_t device) {
        const auto* cols = static_cast<const std::vector<Column>*>(PyCapsule_GetPointer(plan, kPlanName));
        if (cols == nullptr) throw PythonError();
        all = id_list == Py_None;
        if (all) {
            for (size_t c = 0; c < cols->size(); c++) ids.push_back((int32_t)c);
        } else {
            const Py_ssize_t n = PyList_Size(id_list);
            if (n < 0) throw PythonError();
            for (Py_ssize_t k = 0; k < n; k++) {
                int64_t c = as_int(PyList_GET_ITEM(id_list, k));
                // Sizes come from Python's indexing (from the end when
                // negative); the library checks the number itself.
                const int64_t have = (int64_t)cols->size();
                if (c < -have || c >= have) {
                    PyErr_SetString(PyExc_IndexError, "list index out of range");
                    throw PythonError();
                }
                ids.push_back((int32_t)c);
            }
        }
        std::vector<int64_t> sizes;
        for (int32_t id : ids) {
            const Column& c = (*cols)[id < 0 ? id + (int32_t)cols->size() : id];
            if (typed) {
                sizes.assign({B, L});
                sizes.insert(sizes.end(), c.shape.begin(), c.shape.end());
                out.push_back(empty(sizes, c.dtype, device));
            } else {
                out.push_back(empty({B, L * c.elem_bytes}, at::kByte, device));
            }
            ptr.push_back(out.back().data_ptr());
        }
    }
    const int32_t* id_data() const { return all ? nullptr : ids.data(); }
    PyObject* list() {
        PyObject* l = PyList_New((Py_ssize_t)out.size());
        if (l == nullptr) throw PythonError();
        for (size_t k = 0; k < out.size(); k++) {
            PyObject* o = THPVariable_Wrap(out[k]);
            if (o == nullptr) {
                Py_DECREF(l);
                throw PythonError();
            }
            PyList_SET_ITEM(l, (Py_ssize_t)k, o);
        }
        return l;
    }
};

// Every entry: argument count, and C++ exceptions turned into Python ones.
template <typename F>
PyObject* entry(Py_ssize_t have, Py_ssize_t want, F body) {
    if (have != want) {
        PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, have);
        return nullptr;
    }
    HANDLE_TH_ERRORS
    try {
        return body();
    } catch (const PythonError&) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

PyObject* py_bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return entry(n, 7, [&]() -> PyObject* {
        f_select = reinterpret_cast<decltype(f_select)>(as_ptr(a[0]));
        f_collect = reinterpret_cast<decltype(f_collect)>(as_ptr(a[1]));
        f_select_collect = reinterpret_cast<decltype(f_select_collect)>(as_ptr(a[2]));
        f_update = reinterpret_cast<decltype(f_update)>(as_ptr(a[3]));
        f_select_shard = reinterpret_cast<decltype(f_select_shard)>(as_ptr(a[4]));
        f_is_weights = reinterpret_cast<decltype(f_is_weights)>(as_ptr(a[5]));
        f_topk_merge = reinterpret_cast<decltype(f_topk_merge)>(as_ptr(a[6]));
        Py_RETURN_NONE;
    });
}

// plan([(dtype, shape, elem_bytes), ...])
PyObject* py_plan(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return entry(n, 1, [&]() -> PyObject* {
        auto cols = std::make_unique<std::vector<Column>>();
        const Py_ssize_t k = PyList_Size(a[0]);
        if (k < 0) throw PythonError();
        for (Py_ssize_t i = 0; i < k; i++) {
            PyObject *dtype, *shape;
            long long eb;
            if (!PyArg_ParseTuple(PyList_GET_ITEM(a[0], i), "O!O!L", &THPDtypeType, &dtype, &PyTuple_Type, &shape, &eb))
                throw PythonError();
            Column c;
            c.dtype = reinterpret_cast<THPDtype*>(dtype)->scalar_type;
            for (Py_ssize_t d = 0; d < PyTuple_GET_SIZE(shape); d++) c.shape.push_back(as_int(PyTuple_GET_ITEM(shape, d)));
            c.elem_bytes = eb;
            cols->push_back(std::move(c));
        }
        PyObject* cap = PyCapsule_New(cols.get(), kPlanName, [](PyObject* o) {
            delete static_cast<std::vector<Column>*>(PyCapsule_GetPointer(o, kPlanName));
        });
        if (cap == nullptr) throw PythonError();
        cols.release();
        return cap;
    });
}

// select(handle, strategy, B, L, seed, beta, weights, device, stream)
PyObject* py_select(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return entry(n, 9, [&]() -> PyObject* {
        gear_table* t = static_cast<gear_table*>(as_ptr(a[0]));
        const int32_t strategy = as_int32(a[1]), B = as_int32(a[2]), L = as_int32(a[3]), dev = as_int32(a[7]);
        const uint64_t seed = as_u64(a[4]);
        const float beta = as_float(a[5]);
        const bool weights = as_bool(a[6]);
        void* s = as_ptr(a[8]);
        at::Tensor idx = empty({B}, at::kLong, dev), start = empty({B}, at::kInt, dev), w;
        if (weights) w = empty({B}, at::kFloat, dev);
        int64_t* pi = static_cast<int64_t*>(idx.data_ptr());
        int32_t* ps = static_cast<int32_t*>(start.data_ptr());
        float* pw = weights ? static_cast<float*>(w.data_ptr()) : nullptr;
        const int rc = without_gil([&] { return f_select(t, strategy, B, L, seed, beta, pi, ps, pw, s); });
        if (rc != GEAR_OK) return PyLong_FromLong(rc);
        Tuple r(3);
        r.set(0, wrap(std::move(idx)));
        r.set(1, wrap(std::move(start)));
        if (weights) r.set(2, wrap(std::move(w)));
        else r.none(2);
        return r.release();
    });
}

// collect(handle, plan, idx, start, L, ids, typed, device, stream): list of batches
PyObject* py_collect(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return entry(n, 9, [&]() -> PyObject* {
        gear_table* t = static_cast<gear_table*>(as_ptr(a[0]));
        const int32_t B = batch_of(a[2]), L = as_int32(a[4]), dev = as_int32(a[7]);
        void* s = as_ptr(a[8]);
        Batch batch(a[1], a[5], as_bool(a[6]), B, L, dev);
        const int64_t* pi = static_cast<const int64_t*>(address_of(a[2]));
        const int32_t* ps = static_cast<const int32_t*>(address_of(a[3]));
        const int rc = without_gil([&] {
            return f_collect(t, pi, ps, B, L, batch.id_data(), (int32_t)batch.ptr.size(), batch.ptr.data(), s);
        });
        if (rc != GEAR_OK) return PyLong_FromLong(rc);
        return batch.list();
    });
}

// select_collect(handle, plan, strategy, B, L, seed, weights, ids, typed, device, stream)
PyObject* py_select_collect(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return entry(n, 11, [&]() -> PyObject* {
        gear_table* t = static_cast<gear_table*>(as_ptr(a[0]));
        const int32_t strategy = as_int32(a[2]), B = as_int32(a[3]), L = as_int32(a[4]), dev = as_int32(a[9]);
        const uint64_t seed = as_u64(a[5]);
        const bool weights = as_bool(a[6]);
        void* s = as_ptr(a[10]);
        at::Tensor idx = empty({B}, at::kLong, dev), start = empty({B}, at::kInt, dev), w;
        if (weights) w = empty({B}, at::kFloat, dev);
        Batch batch(a[1], a[7], as_bool(a[8]), B, L, dev);
        int64_t* pi = static_cast<int64_t*>(idx.data_ptr());
        int32_t* ps = static_cast<int32_t*>(start.data_ptr());
        float* pw = weights ? static_cast<float*>(w.data_ptr()) : nullptr;
        const int rc = without_gil([&] {
            return f_select_collect(t, strategy, B, L, seed, pi, ps, pw, batch.id_data(), (int32_t)batch.ptr.size(),
                                    batch.ptr.data(), s);
        });
        if (rc != GEAR_OK) return PyLong_FromLong(rc);
        Tuple r(4);
        r.set(0, wrap(std::move(idx)));
        r.set(1, wrap(std::move(start)));
        if (weights) r.set(2, wrap(std::move(w)));
        else r.none(2);
        r.set(3, batch.list());
        return r.release();
    });
}

// update(handle, idx, new, stream)
PyObject* py_update(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return entry(n, 4, [&]() -> PyObject* {
        gear_table* t = static_cast<gear_table*>(as_ptr(a[0]));
        void* s = as_ptr(a[3]);
        const int32_t B = batch_of(a[1]);
        const int64_t* pi = static_cast<const int64_t*>(address_of(a[1]));
        const uint32_t* pp = static_cast<const uint32_t*>(address_of(a[2]));
        return PyLong_FromLong(without_gil([&] { return f_update(t, pi, pp, B, s); }));
    });
}

// select_shard(handle, G, g, totals, base, B, L, seed, device, stream)
PyObject* py_select_shard(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return entry(n, 10, [&]() -> PyObject* {
        gear_table* t = static_cast<gear_table*>(as_ptr(a[0]));
        const int32_t G = as_int32(a[1]), g = as_int32(a[2]), B = as_int32(a[5]), L = as_int32(a[6]);
        const int64_t base = as_int(a[4]);
        const uint64_t seed = as_u64(a[7]);
        const int32_t dev = as_int32(a[8]);
        void* s = as_ptr(a[9]);
        const uint64_t* totals = static_cast<const uint64_t*>(address_of(a[3]));
        at::Tensor idx = empty({B}, at::kLong, dev), start = empty({B}, at::kInt, dev), p = empty({B}, at::kInt, dev);
        int64_t* pi = static_cast<int64_t*>(idx.data_ptr());
        int32_t* ps = static_cast<int32_t*>(start.data_ptr());
        uint32_t* pp = static_cast<uint32_t*>(p.data_ptr());
        const int rc = without_gil([&] { return f_select_shard(t, G, g, totals, base, B, L, seed, pi, ps, pp, s); });
        if (rc != GEAR_OK) return PyLong_FromLong(rc);
        Tuple r(3);
        r.set(0, wrap(std::move(idx)));
        r.set(1, wrap(std::move(start)));
        r.set(2, wrap(std::move(p)));
        return r.release();
    });
}

// is_weights(handle, sel_prio, beta, device, stream)
PyObject* py_is_weights(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return entry(n, 5, [&]() -> PyObject* {
        gear_table* t = static_cast<gear_table*>(as_ptr(a[0]));
        const float beta = as_float(a[2]);
        const int32_t B = batch_of(a[1]), dev = as_int32(a[3]);
        void* s = as_ptr(a[4]);
        at::Tensor w = empty({B}, at::kFloat, dev);
        const uint32_t* pp = static_cast<const uint32_t*>(address_of(a[1]));
        float* pw = static_cast<float*>(w.data_ptr());
        const int rc = without_gil([&] { return f_is_weights(t, pp, B, beta, pw, s); });
        if (rc != GEAR_OK) return PyLong_FromLong(rc);
        return wrap(std::move(w));
    });
}

// topk_merge(prio, gidx, G, K, T, L, seed, device, stream)
PyObject* py_topk_merge(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return entry(n, 9, [&]() -> PyObject* {
        const uint32_t* p = static_cast<const uint32_t*>(address_of(a[0]));
        const int64_t* gi = static_cast<const int64_t*>(address_of(a[1]));
        const int32_t G = as_int32(a[2]), K = as_int32(a[3]), T = as_int32(a[4]), L = as_int32(a[5]);
        const uint64_t seed = as_u64(a[6]);
        const int32_t dev = as_int32(a[7]);
        void* s = as_ptr(a[8]);
        at::Tensor idx = empty({K}, at::kLong, dev), start = empty({K}, at::kInt, dev);
        at::Tensor w = empty({K}, at::kFloat, dev), q = empty({K}, at::kInt, dev);
        int64_t* pi = static_cast<int64_t*>(idx.data_ptr());
        int32_t* ps = static_cast<int32_t*>(start.data_ptr());
        float* pw = static_cast<float*>(w.data_ptr());
        uint32_t* pq = static_cast<uint32_t*>(q.data_ptr());
        const int rc = without_gil([&] { return f_topk_merge(p, gi, G, K, T, L, seed, pi, ps, pw, pq, s); });
        if (rc != GEAR_OK) return PyLong_FromLong(rc);
        Tuple r(4);
        r.set(0, wrap(std::move(idx)));
        r.set(1, wrap(std::move(start)));
        r.set(2, wrap(std::move(w)));
        r.set(3, wrap(std::move(q)));
        return r.release();
    });
}

#define GEAR_METHOD(name, doc) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(py_##name)), METH_FASTCALL, doc}
PyMethodDef methods[] = {
    GEAR_METHOD(bind, "addresses of the library's entry points"),
    GEAR_METHOD(plan, "column plan of a table"),
    GEAR_METHOD(select, "gear_select with allocated outputs"),
    GEAR_METHOD(collect, "gear_collect with allocated batches"),
    GEAR_METHOD(select_collect, "gear_select_collect with allocated outputs"),
    GEAR_METHOD(update, "gear_update_priorities"),
    GEAR_METHOD(select_shard, "gear_select_shard with allocated outputs"),
    GEAR_METHOD(is_weights, "gear_is_weights with allocated output"),
    GEAR_METHOD(topk_merge, "gear_topk_merge with allocated outputs"),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", "Per-step calls of the experience-replay library.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&module); }
