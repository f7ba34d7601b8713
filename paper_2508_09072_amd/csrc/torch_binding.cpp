// The Python side of the C ABI as a CPython extension module: takes torch tensors and numpy arrays apart and
// calls the entry points of include/reader.h.  Argument marshalling only; nothing is computed here.
//
// Why native: a verification step of one short prompt takes the GPU about as long as Python needs to take nineteen
// arguments apart (device, layout and type of every tensor, a ctypes object for every pointer: 15 us of host time
// per reader_verify_step and 13 per reader_tree_attn on the machine with the GPU, against 13 to 20 us of kernels);
// here the same checks cost about a tenth of a microsecond per tensor.
//
// The entry points are looked up in the library the ctypes side has loaded (init(handle, dims_type)), so that both see
// the same copy of it; the ctypes type of the dimensions comes with it.  The interpreter lock is released around
// every call, as ctypes does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#define NPY_NO_DEPRECATED_API NPY_1_7_API_VERSION
#include <numpy/arrayobject.h>

#include <c10/hip/HIPStream.h>
#include <dlfcn.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <memory>
#include <new>

#include "reader.h"

namespace {

// ------------------------------------------------------------------ the library's functions
struct Api {
#define READER_FN(name) decltype(&::name) name = nullptr;
#define READER_FNS(X)                                                                                               \
    X(reader_tree_attn) X(reader_tree_attn_noalloc) X(reader_accept_path) X(reader_kv_compact) X(reader_verify_step) \
    X(reader_kv_rearrange) X(reader_target_argmax) X(reader_target_sample) X(reader_kv_compact_layers)               \
    X(reader_trie_insert) X(reader_trie_search_path) X(reader_trie_extract_tree) X(reader_tree_attach_path)
    READER_FNS(READER_FN)
#undef READER_FN
} api;
PyTypeObject *dims_type = nullptr;      // binding.ReaderDims

PyObject *py_init(PyObject *, PyObject *args) {
    PyObject *arg;
    PyTypeObject *type;
    if (!PyArg_ParseTuple(args, "OO!", &arg, &PyType_Type, &type)) return nullptr;
    void *handle = PyLong_AsVoidPtr(arg);
    if (!handle) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null library handle");
        return nullptr;
    }
#define READER_LOOKUP(name)                                                                     \
    api.name = reinterpret_cast<decltype(&::name)>(dlsym(handle, #name));                        \
    if (!api.name) { PyErr_SetString(PyExc_RuntimeError, "library lacks " #name); return nullptr; }
    READER_FNS(READER_LOOKUP)
#undef READER_LOOKUP
    Py_INCREF(type);
    Py_XDECREF(dims_type);
    dims_type = type;
    Py_RETURN_NONE;
}

// ------------------------------------------------------------------ arguments
constexpr at::ScalarType kBf16 = at::kBFloat16, kI32 = at::kInt, kF32 = at::kFloat, kU8 = at::kByte, kAny = at::ScalarType::Undefined;

// The arguments of one call, taken in order; after the first one that does not fit (Python error set) the rest is
// skipped and ok() says so.
class Args {
public:
    Args(PyObject *const *args, Py_ssize_t n, Py_ssize_t want) : a_(args) {
        if (n != want) {
            PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
            ok_ = false;
        }
    }
    bool ok() const { return ok_; }
    PyObject *raw() { return a_[i_++]; }

    // plain data of a ctypes structure
    const reader_dims *dims() {
        if (!ok_) return nullptr;
        PyObject *o = raw();
        // (the type itself is asked for: any other object with bytes enough would be read as dimensions)
        if (!PyObject_TypeCheck(o, dims_type)) {
            PyErr_Format(PyExc_TypeError, "dims must be a ReaderDims, got %.100s", Py_TYPE(o)->tp_name);
            return fail();
        }
        Py_buffer view;
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) return fail();
        if (view.len < (Py_ssize_t)sizeof dims_) {
            PyBuffer_Release(&view);
            PyErr_SetString(PyExc_TypeError, "dims must be a ReaderDims");
            return fail();
        }
        memcpy(&dims_, view.buf, sizeof dims_);
        PyBuffer_Release(&view);
        return &dims_;
    }
    // the tensor itself (for entry points that read its shape), or null with an error set
    const at::Tensor *tensor(at::ScalarType type, bool optional = false) {
        if (!ok_) return nullptr;
        PyObject *o = raw();
        if (o == Py_None) {
            if (!optional) { PyErr_SetString(PyExc_ValueError, "required tensor is None"); ok_ = false; }
            return nullptr;
        }
        if (!THPVariable_Check(o)) {
            PyErr_Format(PyExc_TypeError, "expected a torch tensor, got %.100s", Py_TYPE(o)->tp_name);
            ok_ = false;
            return nullptr;
        }
        const at::Tensor &t = THPVariable_Unpack(o);
        const char *why = !t.is_cuda() ? "tensor must live on the GPU" : !t.is_contiguous() ? "tensor must be contiguous" : nullptr;
        if (why) {
            PyErr_SetString(PyExc_ValueError, why);
            ok_ = false;
            return nullptr;
        }
        if (type != kAny && t.scalar_type() != type) {
            PyErr_Format(PyExc_ValueError, "expected %s, got %s", c10::toString(type), c10::toString(t.scalar_type()));
            ok_ = false;
            return nullptr;
        }
        return &t;
    }
    void *ptr(at::ScalarType type, bool optional = false) {
        const at::Tensor *t = tensor(type, optional);
        return t ? t->data_ptr() : nullptr;
    }
    const int32_t *i32(bool optional = false) { return static_cast<const int32_t *>(ptr(kI32, optional)); }
    int32_t *i32_out(bool optional = false) { return static_cast<int32_t *>(ptr(kI32, optional)); }
    float *f32(bool optional = false) { return static_cast<float *>(ptr(kF32, optional)); }
    // anything Python's int() takes
    int32_t integer() {
        if (!ok_) return 0;
        PyObject *o = raw();
        PyObject *as_long = PyLong_Check(o) ? Py_NewRef_(o) : PyNumber_Long(o);
        if (!as_long) { ok_ = false; return 0; }
        const long long v = PyLong_AsLongLong(as_long);
        Py_DECREF(as_long);
        if (v == -1 && PyErr_Occurred()) ok_ = false;
        return (int32_t)v;
    }
    // anything Python's float() takes
    double number() {
        if (!ok_) return 0.0;
        PyObject *as_float = PyNumber_Float(raw());
        if (!as_float) { ok_ = false; return 0.0; }
        const double v = PyFloat_AS_DOUBLE(as_float);
        Py_DECREF(as_float);
        return v;
    }
    void want_dims(const at::Tensor *t, int64_t n, const char *what) {
        if (!ok_ || t->dim() == n) return;
        PyErr_Format(PyExc_ValueError, "%s needs %lld dimensions, got %lld", what, (long long)n, (long long)t->dim());
        ok_ = false;
    }
    void reject(PyObject *type, const char *why) {
        if (!ok_) return;
        PyErr_SetString(type, why);
        ok_ = false;
    }

private:
    static PyObject *Py_NewRef_(PyObject *o) { Py_INCREF(o); return o; }
    const reader_dims *fail() { ok_ = false; return nullptr; }
    PyObject *const *a_;
    Py_ssize_t i_ = 0;
    bool ok_ = true;
    reader_dims dims_;
};

void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

template <class F>
PyObject *unlocked(F &&call) {
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// No C++ exception may cross into Python (a tensor without storage throws when it is asked for its pointer).
template <PyObject *(*F)(PyObject *const *, Py_ssize_t)>
PyObject *guarded(PyObject *, PyObject *const *args, Py_ssize_t n) {
    try {
        return F(args, n);
    } catch (const std::bad_alloc &) {
        return PyErr_NoMemory();
    } catch (const std::exception &e) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// ------------------------------------------------------------------ the GPU entry points
PyObject *py_tree_attn(PyObject *const *args, Py_ssize_t n) {
    Args a(args, n, 14);
    const reader_dims *d = a.dims();
    const void *q = a.ptr(kBf16), *kt = a.ptr(kBf16, true), *vt = a.ptr(kBf16, true), *kc = a.ptr(kBf16), *vc = a.ptr(kBf16);
    const int32_t *table = a.i32(), *lens = a.i32(), *parents = a.i32();
    void *out = a.ptr(kBf16);
    float *lse = a.f32(true);
    const int32_t max_len = a.integer();
    const at::Tensor *ws = a.tensor(kAny, true);
    int32_t *status = a.i32_out(true);
    if (!a.ok()) return nullptr;
    void *wsp = ws ? ws->data_ptr() : nullptr, *st = stream();
    const size_t ws_bytes = ws ? ws->nbytes() : 0;
    return unlocked([&] { return api.reader_tree_attn(d, q, kt, vt, kc, vc, table, lens, parents, out, lse, max_len, wsp, ws_bytes, status, st); });
}

PyObject *py_tree_attn_noalloc(PyObject *const *args, Py_ssize_t n) {
    Args a(args, n, 13);
    const reader_dims *d = a.dims();
    const bool none = d && d->B == 0;      // the set-up call needs no tensors
    const void *q = a.ptr(kBf16, none), *kt = a.ptr(kBf16, true), *vt = a.ptr(kBf16, true), *kc = a.ptr(kBf16, none), *vc = a.ptr(kBf16, none);
    const int32_t *table = a.i32(none), *lens = a.i32(none), *parents = a.i32(none);
    void *out = a.ptr(kBf16, none);
    float *lse = a.f32(true);
    const int32_t max_len = a.integer();
    int32_t *status = a.i32_out(true);
    if (!a.ok()) return nullptr;
    void *st = stream();
    return unlocked([&] { return api.reader_tree_attn_noalloc(d, q, kt, vt, kc, vc, table, lens, parents, out, lse, max_len, status, st); });
}

PyObject *py_accept_path(PyObject *const *args, Py_ssize_t n) {
    Args a(args, n, 8);
    const reader_dims *d = a.dims();
    const int32_t *draft = a.i32(), *target = a.i32(), *parents = a.i32();
    int32_t *len = a.i32_out(), *path = a.i32_out(), *bonus = a.i32_out(), *status = a.i32_out(true);
    if (!a.ok()) return nullptr;
    void *st = stream();
    return unlocked([&] { return api.reader_accept_path(d, draft, target, parents, len, path, bonus, status, st); });
}

PyObject *py_kv_compact(PyObject *const *args, Py_ssize_t n) {
    Args a(args, n, 10);
    const reader_dims *d = a.dims();
    const void *kt = a.ptr(kBf16), *vt = a.ptr(kBf16);
    const int32_t *path = a.i32(), *len = a.i32();
    void *kc = a.ptr(kBf16), *vc = a.ptr(kBf16);
    const int32_t *table = a.i32();
    int32_t *lens = a.i32_out(), *status = a.i32_out(true);
    if (!a.ok()) return nullptr;
    void *st = stream();
    return unlocked([&] { return api.reader_kv_compact(d, kt, vt, path, len, kc, vc, table, lens, status, st); });
}

PyObject *py_verify_step(PyObject *const *args, Py_ssize_t n) {
    Args a(args, n, 19);
    const reader_dims *d = a.dims();
    const void *q = a.ptr(kBf16), *kt = a.ptr(kBf16, true), *vt = a.ptr(kBf16, true);
    void *kc = a.ptr(kBf16), *vc = a.ptr(kBf16);
    const int32_t *table = a.i32();
    int32_t *lens = a.i32_out();
    const int32_t *parents = a.i32(), *draft = a.i32(), *target = a.i32();
    void *out = a.ptr(kBf16);
    float *lse = a.f32(true);
    int32_t *len = a.i32_out(), *path = a.i32_out(), *bonus = a.i32_out();
    const int32_t max_len = a.integer();
    const at::Tensor *ws = a.tensor(kAny, true);
    int32_t *status = a.i32_out(true);
    if (!a.ok()) return nullptr;
    void *wsp = ws ? ws->data_ptr() : nullptr, *st = stream();
    const size_t ws_bytes = ws ? ws->nbytes() : 0;
    return unlocked([&] {
        return api.reader_verify_step(d, q, kt, vt, kc, vc, table, lens, parents, draft, target, out, lse, len, path, bonus,
                                      max_len, wsp, ws_bytes, status, st);
    });
}

PyObject *py_kv_rearrange(PyObject *const *args, Py_ssize_t n) {
    Args a(args, n, 5);
    const at::Tensor *k = a.tensor(kBf16), *v = a.tensor(kBf16), *valid = a.tensor(kU8), *len = a.tensor(kI32), *scratch = a.tensor(kAny);
    a.want_dims(k, 5, "k_pad");
    if (!a.ok()) return nullptr;
    if (v->sizes() != k->sizes() || valid->dim() != 2 || valid->size(0) != k->size(1) ||
        valid->size(1) != k->size(2) || len->dim() != 1 || len->size(0) != k->size(1)) {
        a.reject(PyExc_AssertionError, "k_pad, v_pad [NL, B, S, Hkv, D], valid [B, S] and new_len [B] do not fit each other");
        return nullptr;
    }
    void *kp = k->data_ptr(), *vp = v->data_ptr(), *vl = valid->data_ptr(), *nl = len->data_ptr(), *sp = scratch->data_ptr(), *st = stream();
    const size_t bytes = scratch->nbytes();
    const int32_t s[5] = {(int32_t)k->size(0), (int32_t)k->size(1), (int32_t)k->size(2), (int32_t)k->size(3), (int32_t)k->size(4)};
    return unlocked([&] {
        return api.reader_kv_rearrange(s[0], s[1], s[2], s[3], s[4], kp, vp, (uint8_t *)vl, (int32_t *)nl, sp, bytes, st);
    });
}

PyObject *py_target_argmax(PyObject *const *args, Py_ssize_t n) {
    Args a(args, n, 2);
    const at::Tensor *logits = a.tensor(kBf16), *out = a.tensor(kI32);
    if (!a.ok()) return nullptr;
    const int64_t V = logits->dim() > 0 ? logits->size(-1) : 0;
    if (V < 1) { a.reject(PyExc_ValueError, "logits need a last dimension"); return nullptr; }
    const int64_t rows = logits->numel() / V;
    if (out->numel() != rows) { a.reject(PyExc_AssertionError, "target_tokens needs one entry per row of logits"); return nullptr; }
    void *lp = logits->data_ptr(), *op = out->data_ptr(), *st = stream();
    return unlocked([&] { return api.reader_target_argmax((int32_t)rows, (int32_t)V, lp, (int32_t *)op, st); });
}

PyObject *py_target_sample(PyObject *const *args, Py_ssize_t n) {
    Args a(args, n, 5);
    const at::Tensor *logits = a.tensor(kBf16), *parents = a.tensor(kI32), *uniforms = a.tensor(kF32);
    const double temperature = a.number();
    const at::Tensor *out = a.tensor(kI32);
    a.want_dims(logits, 3, "logits");
    if (!a.ok()) return nullptr;
    if (parents->sizes() != logits->sizes().slice(0, 2) || uniforms->sizes() != parents->sizes() ||
        out->sizes() != parents->sizes()) {
        a.reject(PyExc_AssertionError, "logits [B, T, V], parents, uniforms and target_tokens [B, T] do not fit each other");
        return nullptr;
    }
    const int32_t B = (int32_t)logits->size(0), T = (int32_t)logits->size(1), V = (int32_t)logits->size(2);
    void *lp = logits->data_ptr(), *pp = parents->data_ptr(), *up = uniforms->data_ptr(), *op = out->data_ptr(), *st = stream();
    return unlocked([&] {
        return api.reader_target_sample(B, T, V, lp, (int32_t *)pp, (float *)up, (float)temperature, (int32_t *)op, st);
    });
}

PyObject *py_kv_compact_layers(PyObject *const *args, Py_ssize_t n) {
    Args a(args, n, 8);
    const reader_dims *d = a.dims();
    const int32_t *path = a.i32(), *len = a.i32();
    const at::Tensor *k = a.tensor(kBf16), *v = a.tensor(kBf16);
    const int32_t *table = a.i32();
    int32_t *lens = a.i32_out(), *status = a.i32_out(true);
    if (!a.ok()) return nullptr;
    if (k->dim() != 5 || v->sizes() != k->sizes()) {
        a.reject(PyExc_AssertionError, "k_cache and v_cache must be [num_layers, num_pages, Hkv, page_size, D]");
        return nullptr;
    }
    void *kp = k->data_ptr(), *vp = v->data_ptr(), *st = stream();
    const int32_t NL = (int32_t)k->size(0);
    return unlocked([&] { return api.reader_kv_compact_layers(d, NL, path, len, kp, vp, table, lens, status, st); });
}

// ------------------------------------------------------------------ the host-side drafter (numpy arrays)

// Whole numbers as a C-contiguous int32 array: the object itself if it is one, else a converted copy.
struct Ints {
    PyArrayObject *arr;
    explicit Ints(PyObject *o) {
        arr = reinterpret_cast<PyArrayObject *>(
            PyArray_FROMANY(o, NPY_INT32, 0, 0, NPY_ARRAY_CARRAY_RO | NPY_ARRAY_FORCECAST));
    }
    ~Ints() { Py_XDECREF(arr); }
    Ints(const Ints &) = delete;
    Ints &operator=(const Ints &) = delete;
    const int32_t *data() const { return static_cast<const int32_t *>(PyArray_DATA(arr)); }
    Py_ssize_t size() const { return PyArray_SIZE(arr); }
};

PyObject *int_array(const int32_t *from, npy_intp n) {
    PyObject *o = PyArray_SimpleNew(1, &n, NPY_INT32);
    if (o && n > 0) memcpy(PyArray_DATA(reinterpret_cast<PyArrayObject *>(o)), from, (size_t)n * sizeof(int32_t));
    return o;
}

bool whole_number(PyObject *o, long long *v) {
    PyObject *as_long = PyNumber_Long(o);
    if (!as_long) return false;
    *v = PyLong_AsLongLong(as_long);
    Py_DECREF(as_long);
    return !(*v == -1 && PyErr_Occurred());
}

// Room for as many tokens as a caller allows (a depth or budget without an end is an ordinary one): left as it comes, so
// that only what is written is paid for (filled with zeros, a limit of 2^20 tokens cost 2 ms a call).
std::unique_ptr<int32_t[]> room(long long n) { return std::unique_ptr<int32_t[]>(new int32_t[(size_t)std::max(n, 1LL)]); }

bool enough(Py_ssize_t n, Py_ssize_t want) {
    if (n == want) return true;
    PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
    return false;
}

PyObject *py_trie_insert(PyObject *const *args, Py_ssize_t n) {      // (trie, tokens)
    if (!enough(n, 2)) return nullptr;
    reader_trie *t = static_cast<reader_trie *>(PyLong_AsVoidPtr(args[0]));
    if (PyErr_Occurred()) return nullptr;
    Ints tokens(args[1]);
    if (!tokens.arr) return nullptr;
    return unlocked([&] { return api.reader_trie_insert(t, tokens.data(), tokens.size()); });
}

PyObject *py_trie_search_path(PyObject *const *args, Py_ssize_t n) {   // (trie, suffix, depth)
    long long depth;
    if (!enough(n, 3) || !whole_number(args[2], &depth)) return nullptr;
    const reader_trie *t = static_cast<const reader_trie *>(PyLong_AsVoidPtr(args[0]));
    if (PyErr_Occurred()) return nullptr;
    Ints suffix(args[1]);
    if (!suffix.arr) return nullptr;
    const auto out = room(depth);
    int32_t k;
    Py_BEGIN_ALLOW_THREADS
    k = api.reader_trie_search_path(t, suffix.data(), (int32_t)suffix.size(), (int32_t)depth, out.get());
    Py_END_ALLOW_THREADS
    if (k < 0) { PyErr_SetString(PyExc_ValueError, "reader_trie_search_path: bad argument"); return nullptr; }
    return int_array(out.get(), k);
}

PyObject *py_trie_extract_tree(PyObject *const *args, Py_ssize_t n) {   // (trie, suffix, max_depth, budget)
    long long depth;
    long long budget;
    if (!enough(n, 4) || !whole_number(args[2], &depth) || !whole_number(args[3], &budget)) return nullptr;
    const reader_trie *t = static_cast<const reader_trie *>(PyLong_AsVoidPtr(args[0]));
    if (PyErr_Occurred()) return nullptr;
    Ints suffix(args[1]);
    if (!suffix.arr) return nullptr;
    const auto tokens = room(budget), parents = room(budget);
    int32_t k;
    Py_BEGIN_ALLOW_THREADS
    k = api.reader_trie_extract_tree(t, suffix.data(), (int32_t)suffix.size(), (int32_t)depth, (int32_t)budget, tokens.get(), parents.get());
    Py_END_ALLOW_THREADS
    if (k < 0) { PyErr_SetString(PyExc_ValueError, "reader_trie_extract_tree: bad argument"); return nullptr; }
    PyObject *x = int_array(tokens.get(), k), *y = int_array(parents.get(), k);
    if (!x || !y) { Py_XDECREF(x); Py_XDECREF(y); return nullptr; }
    return Py_BuildValue("(NN)", x, y);
}

PyObject *py_tree_attach_path(PyObject *const *args, Py_ssize_t n) {   // (tokens, parents, n_nodes, at_node, path)
    long long n_nodes, at_node;
    if (!enough(n, 5) || !whole_number(args[2], &n_nodes) || !whole_number(args[3], &at_node)) return nullptr;
    int32_t *into[2];
    npy_intp sizes[2];
    for (int i = 0; i < 2; ++i) {
        PyArrayObject *arr = reinterpret_cast<PyArrayObject *>(args[i]);
        if (!PyArray_Check(args[i]) || PyArray_TYPE(arr) != NPY_INT32 || !PyArray_IS_C_CONTIGUOUS(arr) || !PyArray_ISWRITEABLE(arr)) {
            PyErr_SetString(PyExc_AssertionError, "tokens and parents must be writable contiguous int32 arrays");
            return nullptr;
        }
        into[i] = static_cast<int32_t *>(PyArray_DATA(arr));
        sizes[i] = PyArray_SIZE(arr);
    }
    if (sizes[0] != sizes[1]) { PyErr_SetString(PyExc_AssertionError, "tokens and parents must have one capacity"); return nullptr; }
    Ints path(args[4]);
    if (!path.arr) return nullptr;
    const int32_t k = api.reader_tree_attach_path(into[0], into[1], (int32_t)n_nodes, (int32_t)sizes[0], (int32_t)at_node, path.data(),
                                                  (int32_t)path.size());
    if (k < 0) { PyErr_SetString(PyExc_ValueError, "reader_tree_attach_path: bad argument"); return nullptr; }
    return PyLong_FromLong(k);
}

#define READER_FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(guarded<py_##name>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"init", py_init, METH_VARARGS, "init(handle, dims_type): look the entry points up in a loaded library"},
    READER_FAST(tree_attn), READER_FAST(tree_attn_noalloc), READER_FAST(accept_path), READER_FAST(kv_compact),
    READER_FAST(verify_step), READER_FAST(kv_rearrange), READER_FAST(target_argmax), READER_FAST(target_sample),
    READER_FAST(kv_compact_layers), READER_FAST(trie_insert), READER_FAST(trie_search_path), READER_FAST(trie_extract_tree),
    READER_FAST(tree_attach_path), {nullptr, nullptr, 0, nullptr}};

PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_reader_torch", "torch and numpy arguments of the reader C ABI", -1, methods,
                          nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__reader_torch(void) {
    import_array();
    return PyModule_Create(&module_def);
}
