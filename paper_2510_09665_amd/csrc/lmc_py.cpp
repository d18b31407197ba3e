// The calls of the store / retrieve path for CPython: what an engine makes for every request or
// layer, with nothing between Python's arguments and include/lmc.h but the reading of addresses.
// Everything else of the C ABI is bound in lmc.py through ctypes, which takes 1 to 3 us a call to
// marshal arguments where these take 0.1 to 0.3 (a layer pointer 0.06): as much as the calls
// themselves for hashing, lookup, clear, acquire and release of a chunk, and a third of a small
// request.  The interpreter lock is released around every call, as ctypes does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <dlfcn.h>

#include <cstdint>
#include <cstring>

#include "../../include/lmc.h"

namespace {

#define LMC_CALLS(X)                                                                                         \
    X(lmc_hash_chunks) X(lmc_lookup) X(lmc_clear) X(lmc_store) X(lmc_retrieve) X(lmc_retrieve_batch)          \
    X(lmc_retrieve_layerwise) X(lmc_store_begin) X(lmc_store_layers) X(lmc_wait_layer) X(lmc_wait) X(lmc_test) \
    X(lmc_chunk_acquire) X(lmc_chunk_release) X(lmc_gather) X(lmc_scatter)

struct Calls {
#define X(name) decltype(&::name) name;
    LMC_CALLS(X)
#undef X
} lib{};

PyObject *failed = nullptr;          // lmc.py's function that raises LMCError
PyObject *ascontiguousarray = nullptr, *empty = nullptr, *frombuffer = nullptr;
PyObject *dt_uint64 = nullptr, *dt_int64 = nullptr, *dt_int32 = nullptr, *dt_uint8 = nullptr;
PyObject *str_data_ptr = nullptr, *str_cuda_stream = nullptr;

PyObject *fail(lmc_ctx_t *c, lmc_status_t rc, const char *what, PyObject *ticket = Py_None) {
    PyObject *r = PyObject_CallFunction(failed, "isOK", int(rc), what, ticket, (unsigned long long)(uintptr_t)c);
    Py_XDECREF(r);
    return nullptr;
}

bool arity(Py_ssize_t got, Py_ssize_t want, const char *what) {
    if (got == want) return true;
    PyErr_Format(PyExc_TypeError, "%s takes %zd arguments, got %zd", what, want, got);
    return false;
}

// A host array of one type, C-contiguous: the caller's own memory where it is that already, else
// a converted copy, as numpy.ascontiguousarray makes it.
class Array {
public:
    Array(PyObject *x, PyObject *dtype, const char *formats, Py_ssize_t item) : item_(item) {
        ok_ = PyObject_GetBuffer(x, &view_, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT) == 0;
        if (ok_ && matches(formats)) return;
        if (ok_) PyBuffer_Release(&view_);
        PyErr_Clear();
        ok_ = false;
        copy_ = PyObject_CallFunctionObjArgs(ascontiguousarray, x, dtype, nullptr);
        if (copy_ == nullptr) return;
        ok_ = PyObject_GetBuffer(copy_, &view_, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT) == 0;
    }
    ~Array() {
        if (ok_) PyBuffer_Release(&view_);
        Py_XDECREF(copy_);
    }
    Array(const Array &) = delete;
    Array &operator=(const Array &) = delete;
    bool ok() const { return ok_; }
    int64_t size() const { return int64_t(view_.len / item_); }
    template <typename T> const T *data() const { return static_cast<const T *>(view_.buf); }

private:
    bool matches(const char *formats) const {
        const char *f = view_.format;
        if (f == nullptr || view_.itemsize != item_) return false;
        if (*f == '@' || *f == '=' || *f == '<') f++;     // this machine is little-endian
        return f[0] != 0 && f[1] == 0 && std::strchr(formats, f[0]) != nullptr;
    }
    Py_buffer view_{};
    PyObject *copy_ = nullptr;
    Py_ssize_t item_;
    bool ok_ = false;
};

struct Ids : Array {
    explicit Ids(PyObject *x) : Array(x, dt_uint64, "LQ", 8) {}
};

bool number(PyObject *x, uint64_t *out) {
    PyObject *i = PyNumber_Index(x);
    if (i == nullptr) return false;
    *out = PyLong_AsUnsignedLongLongMask(i);
    Py_DECREF(i);
    return !(*out == uint64_t(-1) && PyErr_Occurred());
}

// int(x), as for the ids of single chunks
bool as_int(PyObject *x, uint64_t *out) {
    PyObject *i = PyNumber_Long(x);
    if (i == nullptr) return false;
    *out = PyLong_AsUnsignedLongLongMask(i);
    Py_DECREF(i);
    return !(*out == uint64_t(-1) && PyErr_Occurred());
}

// x.data_ptr(), or int(x) for an address; None is a null pointer where it may be one
bool device(PyObject *x, void **out, bool may_be_none = true) {
    *out = nullptr;
    if (x == Py_None && may_be_none) return true;
    uint64_t v = 0;
    if (!PyLong_CheckExact(x)) {
        PyObject *r = PyObject_CallMethodNoArgs(x, str_data_ptr);
        if (r != nullptr) {
            const bool ok = number(r, &v);
            Py_DECREF(r);
            *out = reinterpret_cast<void *>(uintptr_t(v));
            return ok;
        }
        if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return false;
        PyErr_Clear();
        if (PyObject_HasAttr(x, str_data_ptr)) {         // the error came from inside data_ptr()
            r = PyObject_CallMethodNoArgs(x, str_data_ptr);
            Py_XDECREF(r);
            if (r == nullptr) return false;
        }
    }
    if (!as_int(x, &v)) return false;
    *out = reinterpret_cast<void *>(uintptr_t(v));
    return true;
}

bool stream(PyObject *x, void **out) {
    *out = nullptr;
    if (x == Py_None) return true;
    uint64_t v = 0;
    bool ok;
    if (PyLong_CheckExact(x)) {
        ok = number(x, &v);
    } else {
        PyObject *h = PyObject_GetAttr(x, str_cuda_stream);
        if (h == nullptr) {
            if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return false;
            PyErr_Clear();
            ok = number(x, &v);
        } else {
            ok = h == Py_None || number(h, &v);
            Py_DECREF(h);
        }
    }
    *out = reinterpret_cast<void *>(uintptr_t(v));
    return ok;
}

struct Layers {
    void *p[LMC_MAX_LAYERS];
    bool read(PyObject *x, PyObject *num_layers) {
        const Py_ssize_t n = PyObject_Size(x), want = PyLong_AsSsize_t(num_layers);
        if (n < 0 || (want == -1 && PyErr_Occurred())) return false;
        if (n != want || n > LMC_MAX_LAYERS) {
            PyErr_Format(PyExc_ValueError, "expected %zd layer pointers", want);
            return false;
        }
        // a tuple of its own: data_ptr() may run Python code that changes the caller's list meanwhile
        PyObject *seq = PySequence_Tuple(x);
        if (seq == nullptr) return false;
        bool ok = PyTuple_GET_SIZE(seq) == n;
        if (!ok) PyErr_Format(PyExc_ValueError, "expected %zd layer pointers", want);
        for (Py_ssize_t i = 0; ok && i < n; i++) ok = device(PyTuple_GET_ITEM(seq, i), &p[i], false);
        Py_DECREF(seq);
        return ok;
    }
};

bool context(PyObject *x, lmc_ctx_t **out) {
    uint64_t v = 0;
    if (!number(x, &v)) return false;
    *out = reinterpret_cast<lmc_ctx_t *>(uintptr_t(v));
    return true;
}

// the call itself, without the interpreter lock
#define UNLOCKED(rc, expr)          \
    lmc_status_t rc;                \
    Py_BEGIN_ALLOW_THREADS          \
    rc = (expr);                    \
    Py_END_ALLOW_THREADS

PyObject *ticket_or_error(lmc_ctx_t *c, lmc_status_t rc, const char *what, uint64_t ticket) {
    PyObject *t = PyLong_FromUnsignedLongLong(ticket);
    if (t == nullptr || rc == LMC_OK) return t;
    fail(c, rc, what, t);
    Py_DECREF(t);
    return nullptr;
}

PyObject *none_or_error(lmc_ctx_t *c, lmc_status_t rc, const char *what) {
    if (rc != LMC_OK) return fail(c, rc, what);
    Py_RETURN_NONE;
}

// hash_chunks(ctx, tokens, chunk_tokens) -> uint64 array
PyObject *hash_chunks(PyObject *, PyObject *const *a, Py_ssize_t n) {
    lmc_ctx_t *c;
    if (!arity(n, 3, "hash_chunks") || !context(a[0], &c)) return nullptr;
    Array tok(a[1], dt_int32, "il", 4);
    const long ct = PyLong_AsLong(a[2]);
    if (!tok.ok() || (ct == -1 && PyErr_Occurred())) return nullptr;
    PyObject *count = PyLong_FromLongLong(ct > 0 ? tok.size() / ct : 0);
    PyObject *out = count ? PyObject_CallFunctionObjArgs(empty, count, dt_uint64, nullptr) : nullptr;
    Py_XDECREF(count);
    if (out == nullptr) return nullptr;
    Py_buffer w;
    if (PyObject_GetBuffer(out, &w, PyBUF_C_CONTIGUOUS | PyBUF_WRITABLE) != 0) {
        Py_DECREF(out);
        return nullptr;
    }
    int64_t got = 0;
    UNLOCKED(rc, lib.lmc_hash_chunks(c, tok.data<int32_t>(), tok.size(), static_cast<uint64_t *>(w.buf), &got));
    PyBuffer_Release(&w);
    if (rc == LMC_OK) return out;
    Py_DECREF(out);
    return fail(c, rc, "lmc_hash_chunks");
}

// lookup(ctx, ids) -> int
PyObject *lookup(PyObject *, PyObject *const *a, Py_ssize_t n) {
    lmc_ctx_t *c;
    if (!arity(n, 2, "lookup") || !context(a[0], &c)) return nullptr;
    Ids ids(a[1]);
    if (!ids.ok()) return nullptr;
    int64_t hits = 0;
    UNLOCKED(rc, lib.lmc_lookup(c, ids.data<uint64_t>(), ids.size(), &hits));
    return rc == LMC_OK ? PyLong_FromLongLong(hits) : fail(c, rc, "lmc_lookup");
}

// clear(ctx, ids)
PyObject *clear(PyObject *, PyObject *const *a, Py_ssize_t n) {
    lmc_ctx_t *c;
    if (!arity(n, 2, "clear") || !context(a[0], &c)) return nullptr;
    Ids ids(a[1]);
    if (!ids.ok()) return nullptr;
    UNLOCKED(rc, lib.lmc_clear(c, ids.data<uint64_t>(), ids.size()));
    return none_or_error(c, rc, "lmc_clear");
}

// store(ctx, num_layers, kv_layers, slot_mapping, ids, stream) -> ticket
PyObject *store(PyObject *, PyObject *const *a, Py_ssize_t n) {
    lmc_ctx_t *c;
    Layers l;
    void *slots, *st;
    if (!arity(n, 6, "store") || !context(a[0], &c)) return nullptr;
    Ids ids(a[4]);
    if (!ids.ok() || !l.read(a[2], a[1]) || !device(a[3], &slots) || !stream(a[5], &st)) return nullptr;
    uint64_t t = 0;
    UNLOCKED(rc, lib.lmc_store(c, l.p, static_cast<const int64_t *>(slots), ids.data<uint64_t>(), ids.size(), st, &t));
    return ticket_or_error(c, rc, "lmc_store", t);
}

// retrieve(ctx, num_layers, ids, slot_mapping, kv_layers, stream) -> ticket
PyObject *retrieve(PyObject *, PyObject *const *a, Py_ssize_t n) {
    lmc_ctx_t *c;
    Layers l;
    void *slots, *st;
    if (!arity(n, 6, "retrieve") || !context(a[0], &c)) return nullptr;
    Ids ids(a[2]);
    if (!ids.ok() || !device(a[3], &slots) || !l.read(a[4], a[1]) || !stream(a[5], &st)) return nullptr;
    uint64_t t = 0;
    UNLOCKED(rc, lib.lmc_retrieve(c, ids.data<uint64_t>(), ids.size(), static_cast<const int64_t *>(slots), l.p, st, &t));
    return ticket_or_error(c, rc, "lmc_retrieve", t);
}

// retrieve_batch(ctx, num_layers, offsets, ids, slot_mapping, kv_layers, stream) -> ticket
PyObject *retrieve_batch(PyObject *, PyObject *const *a, Py_ssize_t n) {
    lmc_ctx_t *c;
    Layers l;
    void *slots, *st;
    if (!arity(n, 7, "retrieve_batch") || !context(a[0], &c)) return nullptr;
    Array off(a[2], dt_int64, "lq", 8);
    if (!off.ok()) return nullptr;
    Ids ids(a[3]);
    if (!ids.ok() || !device(a[4], &slots) || !l.read(a[5], a[1]) || !stream(a[6], &st)) return nullptr;
    uint64_t t = 0;
    UNLOCKED(rc, lib.lmc_retrieve_batch(c, off.size() - 1, off.data<int64_t>(), ids.data<uint64_t>(),
                                        static_cast<const int64_t *>(slots), l.p, st, &t));
    return ticket_or_error(c, rc, "lmc_retrieve_batch", t);
}

// retrieve_layerwise(ctx, num_layers, ids, slot_mapping, kv_layers, layers_per_step, stream) -> ticket
PyObject *retrieve_layerwise(PyObject *, PyObject *const *a, Py_ssize_t n) {
    lmc_ctx_t *c;
    Layers l;
    void *slots, *st;
    uint64_t step;
    if (!arity(n, 7, "retrieve_layerwise") || !context(a[0], &c)) return nullptr;
    Ids ids(a[2]);
    if (!ids.ok() || !device(a[3], &slots) || !l.read(a[4], a[1]) || !number(a[5], &step) || !stream(a[6], &st)) return nullptr;
    uint64_t t = 0;
    UNLOCKED(rc, lib.lmc_retrieve_layerwise(c, ids.data<uint64_t>(), ids.size(), static_cast<const int64_t *>(slots), l.p,
                                            int32_t(step), st, &t));
    return ticket_or_error(c, rc, "lmc_retrieve_layerwise", t);
}

// store_begin(ctx, slot_mapping, ids, stream) -> ticket
PyObject *store_begin(PyObject *, PyObject *const *a, Py_ssize_t n) {
    lmc_ctx_t *c;
    void *slots, *st;
    if (!arity(n, 4, "store_begin") || !context(a[0], &c)) return nullptr;
    Ids ids(a[2]);
    if (!ids.ok() || !device(a[1], &slots) || !stream(a[3], &st)) return nullptr;
    uint64_t t = 0;
    UNLOCKED(rc, lib.lmc_store_begin(c, static_cast<const int64_t *>(slots), ids.data<uint64_t>(), ids.size(), st, &t));
    return ticket_or_error(c, rc, "lmc_store_begin", t);
}

// store_layers(ctx, num_layers, ticket, first_layer, n_layers, kv_layers, stream)
PyObject *store_layers(PyObject *, PyObject *const *a, Py_ssize_t n) {
    lmc_ctx_t *c;
    Layers l;
    void *st;
    uint64_t t, first, count;
    if (!arity(n, 7, "store_layers") || !context(a[0], &c) || !number(a[2], &t) || !number(a[3], &first) ||
        !number(a[4], &count) || !l.read(a[5], a[1]) || !stream(a[6], &st))
        return nullptr;
    UNLOCKED(rc, lib.lmc_store_layers(c, t, int32_t(first), int32_t(count), l.p, st));
    return none_or_error(c, rc, "lmc_store_layers");
}

// wait_layer(ctx, ticket, layer, stream)
PyObject *wait_layer(PyObject *, PyObject *const *a, Py_ssize_t n) {
    lmc_ctx_t *c;
    void *st;
    uint64_t t, layer;
    if (!arity(n, 4, "wait_layer") || !context(a[0], &c) || !number(a[1], &t) || !number(a[2], &layer) || !stream(a[3], &st))
        return nullptr;
    UNLOCKED(rc, lib.lmc_wait_layer(c, t, int32_t(layer), st));
    return none_or_error(c, rc, "lmc_wait_layer");
}

// wait(ctx, ticket)
PyObject *wait(PyObject *, PyObject *const *a, Py_ssize_t n) {
    lmc_ctx_t *c;
    uint64_t t;
    if (!arity(n, 2, "wait") || !context(a[0], &c) || !number(a[1], &t)) return nullptr;
    UNLOCKED(rc, lib.lmc_wait(c, t));
    return none_or_error(c, rc, "lmc_wait");
}

// test(ctx, ticket) -> bool
PyObject *test(PyObject *, PyObject *const *a, Py_ssize_t n) {
    lmc_ctx_t *c;
    uint64_t t;
    if (!arity(n, 2, "test") || !context(a[0], &c) || !number(a[1], &t)) return nullptr;
    UNLOCKED(rc, lib.lmc_test(c, t));
    if (rc != LMC_OK && rc != LMC_ERR_BUSY) return fail(c, rc, "lmc_test");
    return PyBool_FromLong(rc == LMC_OK);
}

// chunk_acquire(ctx, id, chunk_bytes) -> read-only uint8 array over the chunk in the pool
PyObject *chunk_acquire(PyObject *, PyObject *const *a, Py_ssize_t n) {
    lmc_ctx_t *c;
    uint64_t id;
    if (!arity(n, 3, "chunk_acquire") || !context(a[0], &c) || !as_int(a[1], &id)) return nullptr;
    const Py_ssize_t bytes = PyLong_AsSsize_t(a[2]);
    if (bytes == -1 && PyErr_Occurred()) return nullptr;
    const void *p = nullptr;
    UNLOCKED(rc, lib.lmc_chunk_acquire(c, id, &p));
    if (rc != LMC_OK) return fail(c, rc, "lmc_chunk_acquire");
    PyObject *m = PyMemoryView_FromMemory(static_cast<char *>(const_cast<void *>(p)), bytes, PyBUF_READ);
    PyObject *out = m ? PyObject_CallFunctionObjArgs(frombuffer, m, dt_uint8, nullptr) : nullptr;
    Py_XDECREF(m);
    if (out == nullptr) (void)lib.lmc_chunk_release(c, id);
    return out;
}

// chunk_release(ctx, id)
PyObject *chunk_release(PyObject *, PyObject *const *a, Py_ssize_t n) {
    lmc_ctx_t *c;
    uint64_t id;
    if (!arity(n, 2, "chunk_release") || !context(a[0], &c) || !as_int(a[1], &id)) return nullptr;
    UNLOCKED(rc, lib.lmc_chunk_release(c, id));
    return none_or_error(c, rc, "lmc_chunk_release");
}

// gather(ctx, num_layers, kv_layers, slot_mapping, n_chunks, buffer, stream)
PyObject *gather(PyObject *, PyObject *const *a, Py_ssize_t n) {
    lmc_ctx_t *c;
    Layers l;
    void *slots, *buf, *st;
    uint64_t chunks;
    if (!arity(n, 7, "gather") || !context(a[0], &c) || !l.read(a[2], a[1]) || !device(a[3], &slots) || !number(a[4], &chunks) ||
        !device(a[5], &buf) || !stream(a[6], &st))
        return nullptr;
    UNLOCKED(rc, lib.lmc_gather(c, l.p, static_cast<const int64_t *>(slots), int64_t(chunks), buf, st));
    return none_or_error(c, rc, "lmc_gather");
}

// scatter(ctx, num_layers, buffer, slot_mapping, n_chunks, kv_layers, stream)
PyObject *scatter(PyObject *, PyObject *const *a, Py_ssize_t n) {
    lmc_ctx_t *c;
    Layers l;
    void *slots, *buf, *st;
    uint64_t chunks;
    if (!arity(n, 7, "scatter") || !context(a[0], &c) || !device(a[2], &buf) || !device(a[3], &slots) || !number(a[4], &chunks) ||
        !l.read(a[5], a[1]) || !stream(a[6], &st))
        return nullptr;
    UNLOCKED(rc, lib.lmc_scatter(c, buf, static_cast<const int64_t *>(slots), int64_t(chunks), l.p, st));
    return none_or_error(c, rc, "lmc_scatter");
}

// bind(path of liblmc.so, function that raises LMCError): the library is loaded already
PyObject *bind(PyObject *, PyObject *args) {
    const char *path;
    PyObject *f;
    if (!PyArg_ParseTuple(args, "sO", &path, &f)) return nullptr;
    void *h = dlopen(path, RTLD_NOW | RTLD_LOCAL);
    if (h == nullptr) {
        PyErr_SetString(PyExc_ImportError, dlerror());
        return nullptr;
    }
    Calls found{};
#define X(name)                                                                  \
    found.name = reinterpret_cast<decltype(&::name)>(dlsym(h, #name));           \
    if (found.name == nullptr) {                                                 \
        PyErr_SetString(PyExc_ImportError, "liblmc.so has no " #name);           \
        return nullptr;                                                          \
    }
    LMC_CALLS(X)
#undef X
    PyObject *np = PyImport_ImportModule("numpy");
    if (np == nullptr) return nullptr;
    struct { PyObject **to; const char *name; } attrs[] = {
        {&ascontiguousarray, "ascontiguousarray"}, {&empty, "empty"}, {&frombuffer, "frombuffer"}, {&dt_uint64, "uint64"},
        {&dt_int64, "int64"}, {&dt_int32, "int32"}, {&dt_uint8, "uint8"}};
    bool ok = true;
    for (auto &x : attrs) {
        Py_XDECREF(*x.to);
        *x.to = PyObject_GetAttrString(np, x.name);
        ok = ok && *x.to != nullptr;
    }
    Py_DECREF(np);
    if (!ok) return nullptr;
    Py_INCREF(f);
    Py_XDECREF(failed);
    failed = f;
    lib = found;
    Py_RETURN_NONE;
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    FAST(hash_chunks), FAST(lookup), FAST(clear), FAST(store), FAST(retrieve), FAST(retrieve_batch), FAST(retrieve_layerwise),
    FAST(store_begin), FAST(store_layers), FAST(wait_layer), FAST(wait), FAST(test), FAST(chunk_acquire), FAST(chunk_release),
    FAST(gather), FAST(scatter), {"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_lmc_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__lmc_native(void) {
    str_data_ptr = PyUnicode_InternFromString("data_ptr");
    str_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    return PyModule_Create(&module);
}
