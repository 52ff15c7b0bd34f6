// The checks and the marshalling of the data calls of kvc.py, between Python's tensors and the C entry points.  A small data call is
// host time: the launch takes 2.8 us, and the same checks and a call through ctypes took 1.4 us a call (3 of a prefetch's).
// The entry points are those of the library that kvc.py has loaded (init is given their addresses).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>

#include "kvc.h"

namespace {

struct Entries {
    decltype(&kvc_compress_blocks) compress;
    decltype(&kvc_compress_blocks_mixed) compress_mixed;
    decltype(&kvc_decompress_blocks) decompress;
    decltype(&kvc_gather_decompress) gather;
    decltype(&kvc_prefetch_layers) prefetch;
} e;

// a Python error has been set
struct Raised {};

void require(bool c, const char* what = nullptr) {
    if (c) return;
    if (what)
        PyErr_SetString(PyExc_AssertionError, what);
    else
        PyErr_SetNone(PyExc_AssertionError);
    throw Raised();
}

long long integer(PyObject* o) {
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Raised();
    return v;
}

// A reference that is given back.
struct Ref {
    PyObject* o;
    explicit Ref(PyObject* o) : o(o) {
        if (!o) throw Raised();
    }
    ~Ref() { Py_DECREF(o); }
    Ref(const Ref&) = delete;
};

// An integer that goes straight to a C entry point, where ctypes also took its own integers and what an object names in
// _as_parameter_.
long long passed(PyObject* o) {
    if (PyIndex_Check(o)) return integer(o);
    for (const char* what : {"_as_parameter_", "value"})
        if (PyObject_HasAttrString(o, what)) return passed(Ref(PyObject_GetAttrString(o, what)).o);
    return integer(o);
}

// (None: a codec that has been closed; the library refuses it.  A stream may be one of ctypes' pointers, from a program that made it
// with the runtime.)
template <class T>
T address(PyObject* o) {
    if (o == Py_None) return nullptr;
    if (!PyLong_Check(o)) {
        const Ref ctypes(PyImport_ImportModule("ctypes")), type(PyObject_GetAttrString(ctypes.o, "c_void_p"));
        const Ref pointer(PyObject_CallMethod(ctypes.o, "cast", "OO", o, type.o));
        const Ref value(PyObject_GetAttrString(pointer.o, "value"));
        return address<T>(value.o);
    }
    void* p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) throw Raised();
    return reinterpret_cast<T>(p);
}

// An argument that is to be a tensor.  torch's own are looked at directly; a subclass, or any other object with a tensor's attributes (a
// wrapper of one), is asked as Python code would ask it.
class Tensor {
    const at::Tensor* t = nullptr;
    PyObject* o;

    Ref get(const char* what) const { return Ref(PyObject_GetAttrString(o, what)); }
    Ref call(const char* what) const { return Ref(PyObject_CallMethod(o, what, nullptr)); }
    static bool truth(const Ref& r) {
        const int v = PyObject_IsTrue(r.o);
        if (v < 0) throw Raised();
        return v != 0;
    }

public:
    explicit Tensor(PyObject* o) : o(o) {
        if (THPVariable_CheckExact(o)) {
            t = &THPVariable_Unpack(o);
        } else if (!PyObject_HasAttrString(o, "is_cuda")) {
            PyErr_Format(PyExc_TypeError, "a tensor, not %s", Py_TYPE(o)->tp_name);
            throw Raised();
        }
    }
    bool is_cuda() const { return t ? t->is_cuda() : truth(get("is_cuda")); }
    bool is_contiguous() const { return t ? t->is_contiguous() : truth(call("is_contiguous")); }
    bool holds(at::ScalarType type) const {
        if (t) return t->scalar_type() == type;
        const Ref d = get("dtype");
        return THPDtype_Check(d.o) && reinterpret_cast<THPDtype*>(d.o)->scalar_type == type;
    }
    long long numel() const { return t ? t->numel() : integer(call("numel").o); }
    void* data_ptr() const { return t ? t->data_ptr() : address<void*>(call("data_ptr").o); }
    long long dim() const {
        if (t) return t->dim();
        const Py_ssize_t n = PyObject_Length(get("shape").o);
        if (n < 0) throw Raised();
        return n;
    }
    long long size(int i) const { return t ? t->size(i) : integer(Ref(PySequence_GetItem(get("shape").o, i)).o); }
};

const char kIds[] = "block ids: contiguous int32 CUDA tensor";
void check_ids(const Tensor& t) { require(t.is_cuda() && t.holds(at::kInt) && t.is_contiguous(), kIds); }

// address of an id tensor of at least n entries; None: no list
int32_t* ids_at_least(PyObject* o, long long n) {
    if (o == Py_None) return nullptr;
    const Tensor t(o);
    check_ids(t);
    require(t.numel() >= n, "id tensors shorter than n");
    return static_cast<int32_t*>(t.data_ptr());
}
// ... of exactly n
int32_t* ids_of(PyObject* o, long long n) {
    const Tensor t(o);
    check_ids(t);
    require(t.numel() == n);
    return static_cast<int32_t*>(t.data_ptr());
}

// number of whole blocks the tensor's storage covers: blocks `stride` elements apart that span `span`
struct Blocks {
    void* at;
    long long n;
};
Blocks blocks(PyObject* o, PyObject* stride, PyObject* span) {
    const Tensor t(o);
    require(t.is_cuda() && t.is_contiguous() && t.holds(at::kHalf));
    const long long have = t.numel(), need = integer(span);
    return {t.data_ptr(), have < need ? 0 : (have - need) / integer(stride) + 1};
}

// blocks of a call: as asked for, else of its first list, else all there are
long long count(PyObject* n, PyObject* first, PyObject* second, long long all) {
    if (n == Py_None) return first != Py_None ? Tensor(first).numel() : second != Py_None ? Tensor(second).numel() : all;
    return integer(Ref(PyNumber_Long(n)).o);
}

// rows and columns of a table; an object of another shape cannot be unpacked to them
struct Rows {
    long long n, each;
};
Rows rows(const Tensor& t, bool more_allowed, PyObject* error = PyExc_ValueError) {
    const long long dim = t.dim();
    if (dim < 2 || (dim > 2 && !more_allowed)) {
        PyErr_Format(error, "block table and predictions: a row per sequence, not %lld dimensions", dim);
        throw Raised();
    }
    return {t.size(0), t.size(1)};
}

// (products of sizes that a caller may have got wrong: wide enough not to wrap round to the right number)
typedef __int128 wide;

template <class F>
PyObject* guarded(Py_ssize_t given, Py_ssize_t want, F f) {
    if (given != want) {
        PyErr_SetString(PyExc_TypeError, "number of arguments");
        return nullptr;
    }
    try {
        return PyLong_FromLong(f());
    } catch (const Raised&) {
    } catch (const std::exception& x) {
        PyErr_SetString(PyExc_RuntimeError, x.what());
    } catch (...) {
        PyErr_SetString(PyExc_RuntimeError, "unknown error");
    }
    return nullptr;
}

template <class F>
int unlocked(F f) {
    int rc;
    Py_BEGIN_ALLOW_THREADS;
    rc = f();
    Py_END_ALLOW_THREADS;
    return rc;
}

// init(addresses of the entry points, in the order of Entries)
PyObject* py_init(PyObject*, PyObject* const* a, Py_ssize_t given) {
    return guarded(given, 5, [&] {
        e = Entries{address<decltype(e.compress)>(a[0]), address<decltype(e.compress_mixed)>(a[1]), address<decltype(e.decompress)>(a[2]),
                    address<decltype(e.gather)>(a[3]), address<decltype(e.prefetch)>(a[4])};
        return 0;
    });
}

// compress(ctx, cache, stride, span, n, src_ids, pool_ids, block_scheme, stream)
PyObject* py_compress(PyObject*, PyObject* const* a, Py_ssize_t given) {
    return guarded(given, 9, [&] {
        kvc_ctx* ctx = address<kvc_ctx*>(a[0]);
        const Blocks b = blocks(a[1], a[2], a[3]);
        const long long n = count(a[4], a[5], a[6], b.n);
        const int32_t *src = ids_at_least(a[5], n), *pool = ids_at_least(a[6], n);
        void* stream = address<void*>(a[8]);
        if (a[7] == Py_None) return unlocked([&] { return e.compress(ctx, b.at, b.n, src, pool, (int32_t)n, stream); });
        const Tensor modes(a[7]);
        require(modes.is_cuda() && modes.holds(at::kByte) && modes.numel() >= n);
        const uint8_t* m = static_cast<const uint8_t*>(modes.data_ptr());
        return unlocked([&] { return e.compress_mixed(ctx, b.at, b.n, src, pool, m, (int32_t)n, stream); });
    });
}

// decompress(ctx, out, stride, span, n, pool_ids, dst_ids, stream)
PyObject* py_decompress(PyObject*, PyObject* const* a, Py_ssize_t given) {
    return guarded(given, 8, [&] {
        kvc_ctx* ctx = address<kvc_ctx*>(a[0]);
        const Blocks b = blocks(a[1], a[2], a[3]);
        const long long n = count(a[4], a[5], a[6], b.n);
        const int32_t *pool = ids_at_least(a[5], n), *dst = ids_at_least(a[6], n);
        void* stream = address<void*>(a[7]);
        return unlocked([&] { return e.decompress(ctx, b.at, b.n, pool, dst, (int32_t)n, stream); });
    });
}

// gather(ctx, out, stride, span, block_table, pred, n_layers, pool_blocks_per_layer, stream)
PyObject* py_gather(PyObject*, PyObject* const* a, Py_ssize_t given) {
    return guarded(given, 9, [&] {
        kvc_ctx* ctx = address<kvc_ctx*>(a[0]);
        const Tensor table(a[4]), pred(a[5]);
        check_ids(table);
        check_ids(pred);
        const Rows tr = rows(table, false), pr = rows(pred, true, PyExc_IndexError);
        const long long n_seq = tr.n, k = pr.each, layers = integer(a[6]), per_layer = integer(a[7]);
        require(pr.n == n_seq);
        const Blocks b = blocks(a[1], a[2], a[3]);
        require(b.n == (wide)layers * n_seq * k);
        void* stream = address<void*>(a[8]);
        const int32_t *t = static_cast<const int32_t*>(table.data_ptr()), *p = static_cast<const int32_t*>(pred.data_ptr());
        const int32_t max_blocks = (int32_t)tr.each;
        return unlocked([&] { return e.gather(ctx, b.at, t, max_blocks, p, (int32_t)n_seq, (int32_t)k, (int32_t)layers, per_layer, stream); });
    });
}

// prefetch(ctx, l2, stride, span, tags, fetch, loc, block_table, pred, l1_first, n_layers, layer_begin, layer_end, pool_blocks_per_layer,
// fill_half, stream)
PyObject* py_prefetch(PyObject*, PyObject* const* a, Py_ssize_t given) {
    return guarded(given, 16, [&] {
        kvc_ctx* ctx = address<kvc_ctx*>(a[0]);
        const Rows tr = rows(Tensor(a[7]), false), pr = rows(Tensor(a[8]), true);
        const long long n_seq = tr.n, max_blocks = tr.each, k = pr.each, layers = integer(a[10]);
        const Blocks b = blocks(a[1], a[2], a[3]);
        require(b.n == 2 * ((wide)layers * n_seq * k) && pr.n == n_seq);
        const long long n_slots = b.n / 2;
        int32_t *tags = ids_of(a[4], 2 * n_slots), *fetch = ids_of(a[5], n_slots), *loc = ids_of(a[6], n_slots);
        const int32_t *t = ids_at_least(a[7], 0), *p = ids_at_least(a[8], 0), *l1 = a[9] == Py_None ? nullptr : ids_of(a[9], n_seq);
        const long long begin = passed(a[11]), end = a[12] == Py_None ? layers : passed(a[12]), per_layer = integer(a[13]), half = passed(a[14]);
        void* stream = address<void*>(a[15]);
        return unlocked([&] {
            return e.prefetch(ctx, b.at, tags, fetch, loc, t, (int32_t)max_blocks, p, l1, (int32_t)n_seq, (int32_t)k, (int32_t)layers, (int32_t)begin, (int32_t)end,
                              per_layer, (int32_t)half, stream);
        });
    });
}

#define KVC_METHOD(name, f) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {KVC_METHOD("init", py_init), KVC_METHOD("compress", py_compress), KVC_METHOD("decompress", py_decompress), KVC_METHOD("gather", py_gather),
                         KVC_METHOD("prefetch", py_prefetch), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_kvc_py", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__kvc_py() { return PyModule_Create(&module); }
