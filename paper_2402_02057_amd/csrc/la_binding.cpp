// Argument marshalling between Python and the C ABI (include/la.h), as a CPython extension module.
//
// What bounds it: nothing but host time.  A decoding step calls an entry point per layer, and a
// short launch takes 5 to 8 us on the GPU; marshalled in Python (a dozen attribute reads per tensor,
// a shape tuple built and compared, ctypes converting every argument, the current stream looked up
// through three Python frames) such a call took 10.0 us of host time, so the host could not keep the
// GPU busy below about that.  Here a tensor is checked in a few loads: 4.4 us per call (the
// step of 121 rows over 1024 keys, 32 heads), most of it the launch itself.
//
// Every function takes its arguments positionally in the order of the Python wrapper in
// binding.py, raises what that wrapper documents (TypeError / ValueError for tensors that do not fit,
// binding.LaError for a code the library returns) and releases the interpreter lock around the call.
#define PY_SSIZE_T_CLEAN
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>

#include <string.h>

#include <initializer_list>
#include <vector>

#include "la.h"

namespace {

struct Raised {};  // a Python exception is set

struct Owned {     // a reference that goes with its scope
    PyObject* const o;
    explicit Owned(PyObject* p) : o(p) {}
    ~Owned() { Py_XDECREF(o); }
    Owned(const Owned&) = delete;
};

struct Unlocked {  // no interpreter lock within its scope
    PyThreadState* const state = PyEval_SaveThread();
    Unlocked() {}
    ~Unlocked() { PyEval_RestoreThread(state); }
    Unlocked(const Unlocked&) = delete;
};

PyObject* g_la_error = nullptr;  // binding.LaError

constexpr at::ScalarType kBF16 = at::kBFloat16, kF32 = at::kFloat, kI32 = at::kInt, kU8 = at::kByte;

const char* dtype_name(at::ScalarType t)
{
    return t == kBF16 ? "torch.bfloat16" : t == kF32 ? "torch.float32" : t == kI32 ? "torch.int32" : "torch.uint8";
}

typedef std::initializer_list<int64_t> Shape;

[[noreturn]] void wrong_shape(const at::Tensor& t, const Shape& shape, const char* name)
{
    PyObject* want = PyTuple_New((Py_ssize_t)shape.size());
    PyObject* got = PyTuple_New(t.dim());
    Py_ssize_t i = 0;
    for (int64_t n : shape) PyTuple_SET_ITEM(want, i++, PyLong_FromLongLong(n));
    for (i = 0; i < t.dim(); ++i) PyTuple_SET_ITEM(got, i, PyLong_FromLongLong(t.size(i)));
    PyErr_Format(PyExc_ValueError, "%s must have shape %R, got %R", name, want, got);
    Py_DECREF(want);
    Py_DECREF(got);
    throw Raised();
}

const at::Tensor& tensor(PyObject* o, const char* name)
{
    if (o == Py_None) {
        PyErr_Format(PyExc_ValueError, "%s is None", name);
        throw Raised();
    }
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s must be a torch.Tensor", name);
        throw Raised();
    }
    return THPVariable_Unpack(o);
}

// Device pointer of a contiguous GPU tensor of the expected type and shape; null if it is empty.
template <class T = void>
T* ptr(PyObject* o, at::ScalarType dtype, const Shape& shape, const char* name, bool or_none = false)
{
    if (or_none && o == Py_None) return nullptr;
    const at::Tensor& t = tensor(o, name);
    if (!t.is_cuda()) {
        PyErr_Format(PyExc_ValueError, "%s must live on the GPU", name);
        throw Raised();
    }
    if (t.scalar_type() != dtype) {
        PyObject* got = PyObject_GetAttrString(o, "dtype");
        PyErr_Format(PyExc_ValueError, "%s must be %s, got %S", name, dtype_name(dtype), got ? got : Py_None);
        Py_XDECREF(got);
        throw Raised();
    }
    const at::IntArrayRef sizes = t.sizes();
    if (sizes.size() != shape.size()) wrong_shape(t, shape, name);
    size_t i = 0;
    for (int64_t n : shape)
        if (sizes[i++] != n) wrong_shape(t, shape, name);
    if (!t.is_contiguous()) {
        PyErr_Format(PyExc_ValueError, "%s must be contiguous", name);
        throw Raised();
    }
    return t.numel() ? static_cast<T*>(t.data_ptr()) : nullptr;
}

int64_t size_of(PyObject* o, int dim, const char* name)
{
    const at::Tensor& t = tensor(o, name);
    if (dim >= t.dim()) {
        PyErr_SetString(PyExc_IndexError, "tuple index out of range");
        throw Raised();
    }
    return t.size(dim);
}

// A size that the C functions take as an int: what does not fit one is refused, before anything is
// compared with the rest of it.
int integer(PyObject* o)
{
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    if (v == -1 && !overflow && PyErr_Occurred()) throw Raised();
    if (overflow || v != (int)v) {
        PyErr_Format(PyExc_ValueError, "%S does not fit 32 bits", o);
        throw Raised();
    }
    return (int)v;
}

int integer(int64_t n, const char* name)
{
    if (n != (int)n) {
        PyErr_Format(PyExc_ValueError, "%s: a size of %lld does not fit 32 bits", name, (long long)n);
        throw Raised();
    }
    return (int)n;
}

// (a descriptor's prefix length may be anything int() takes)
int whole_number(PyObject* o)
{
    if (PyLong_Check(o)) return integer(o);
    const Owned n(PyNumber_Long(o));
    if (!n.o) throw Raised();
    return integer(n.o);
}

int truth(PyObject* o)
{
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw Raised();
    return v;
}

// (anything float() takes)
float real(PyObject* o)
{
    const Owned f(PyNumber_Float(o));
    if (!f.o) throw Raised();
    return (float)PyFloat_AS_DOUBLE(f.o);
}

// None: the current stream of the current device; a torch stream; or a stream handle as a number.
void* stream_of(PyObject* o)
{
    if (o == Py_None) return (void*)c10::hip::getCurrentHIPStream().stream();
    PyObject* handle = PyLong_Check(o) ? (Py_INCREF(o), o) : PyObject_GetAttrString(o, "cuda_stream");
    if (!handle) {
        PyErr_Clear();
        handle = PyNumber_Long(o);
        if (!handle) throw Raised();
    }
    void* const s = PyLong_AsVoidPtr(handle);
    Py_DECREF(handle);
    if (!s && PyErr_Occurred()) throw Raised();
    return s;
}

template <class F>
void call(F&& f)
{
    la_status rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    if (rc == LA_OK) return;
    PyObject* e = PyObject_CallFunction(g_la_error, "is", (int)rc, la_last_error());
    if (e) {
        PyErr_SetObject(g_la_error, e);
        Py_DECREF(e);
    }
    throw Raised();
}

// (W, N, G) and what follows from them
struct Step {
    int W, N, G;
    int64_t T;
    explicit Step(PyObject* const* a) : W(integer(a[0])), N(integer(a[1])), G(integer(a[2])), T(1 + ((int64_t)W + G) * ((int64_t)N - 1)) {}
};

struct Heads {
    int heads, kv, d;
    explicit Heads(PyObject* const* a) : heads(integer(a[0])), kv(integer(a[1])), d(integer(a[2])) {}
};

// ---- values of a descriptor dict

// The key `s` as an interned Python string, made once.
#define KEY(s) ([]() -> PyObject* { static PyObject* const k = PyUnicode_InternFromString(s); return k; }())

// The sequence of descriptors, as a tuple of our own: a list may grow or shrink while a descriptor is
// asked for its values, or, from another thread, while the call runs without the lock.  A value is what x[key] gives, an
// optional one what x.get(key) gives.
class Items {
public:
    explicit Items(PyObject* o) : items(PySequence_Tuple(o))
    {
        if (!items) throw Raised();
    }
    ~Items()
    {
        Py_DECREF(items);
        for (PyObject* v : held) Py_DECREF(v);
    }
    Items(const Items&) = delete;
    int size() const { return (int)PyTuple_GET_SIZE(items); }

    // The value of descriptor i under `k`, valid until this object goes: a dict holds its values, what
    // another mapping hands out may exist nowhere else and is kept here until the call has returned.
    PyObject* at(int i, PyObject* k, bool or_none = false)
    {
        PyObject* const x = PyTuple_GET_ITEM(items, i);
        PyObject* v = nullptr;
        if (PyDict_CheckExact(x)) {
            v = PyDict_GetItemWithError(x, k);
        } else {                               // (a subclass of dict may answer for itself, too)
            PyObject* const get = or_none ? PyObject_GetAttrString(x, "get") : nullptr;
            if (or_none && !get) {
                if (!PyErr_ExceptionMatches(PyExc_AttributeError)) throw Raised();
                PyErr_Clear();
            }
            v = get ? PyObject_CallFunctionObjArgs(get, k, nullptr) : PyObject_GetItem(x, k);
            Py_XDECREF(get);
            if (v) held.push_back(v);
            else if (!or_none || get || !PyErr_ExceptionMatches(PyExc_KeyError)) throw Raised();
            else PyErr_Clear();
        }
        if (!v && !PyErr_Occurred()) {
            if (or_none) v = Py_None;
            else PyErr_SetObject(PyExc_KeyError, k);
        }
        if (!v) throw Raised();
        return v;
    }

private:
    PyObject* items;
    std::vector<PyObject*> held;
};

struct Pages {
    void *k, *v;
    int page_size, n_pages;
};

Pages pages_of(PyObject* k_pages, PyObject* v_pages, int kv_heads, int d)
{
    Pages p;
    p.n_pages = integer(size_of(k_pages, 0, "k_pages"), "k_pages");
    p.page_size = integer(size_of(k_pages, 2, "k_pages"), "k_pages");
    p.k = ptr(k_pages, kBF16, {p.n_pages, kv_heads, p.page_size, d}, "k_pages");
    p.v = ptr(v_pages, kBF16, {p.n_pages, kv_heads, p.page_size, d}, "v_pages");
    return p;
}

const int* table_of(PyObject* table, int64_t rows, int page_size)
{
    const int64_t need = page_size > 0 ? (rows + page_size - 1) / page_size : 0;
    const int64_t n = table == Py_None ? 0 : tensor(table, "block_table").numel();
    if (need > 0 && n < need) {
        PyErr_Format(PyExc_ValueError, "block_table must hold at least %lld entries", (long long)need);
        throw Raised();
    }
    return ptr<int>(table, kI32, {n}, "block_table", true);
}

// ---- entry points (positional arguments as in binding.py; the last one is the stream)

#define LA_ENTRY(name) void name(PyObject* const* a)

template <class F>
void plain_step(F f, PyObject* const* a)
{
    const int P = integer(a[5]);
    const Step s(a + 6);
    const Heads h(a + 9);
    const void* q = ptr(a[0], kBF16, {s.T, h.heads, h.d}, "q");
    const void* kc = ptr(a[1], kBF16, {h.kv, P, h.d}, "k_cache", true);
    const void* vc = ptr(a[2], kBF16, {h.kv, P, h.d}, "v_cache", true);
    const void* sk = ptr(a[3], kBF16, {s.T, h.kv, h.d}, "step_k");
    const void* sv = ptr(a[4], kBF16, {s.T, h.kv, h.d}, "step_v");
    void* out = ptr(a[12], kBF16, {s.T, h.heads, h.d}, "out");
    void* st = stream_of(a[13]);
    call([&] { return f(q, kc, vc, sk, sv, P, s.W, s.N, s.G, h.heads, h.kv, h.d, out, st); });
}

LA_ENTRY(step_attention)
{
    plain_step(la_step_attention, a);
}

LA_ENTRY(step_attention_noalloc)
{
    plain_step(la_step_attention_noalloc, a);
}

LA_ENTRY(step_attention_fp8kv)
{
    const int P = integer(a[7]);
    const Step s(a + 8);
    const Heads h(a + 11);
    const void* q = ptr(a[0], kBF16, {s.T, h.heads, h.d}, "q");
    const void* kc = ptr(a[1], kU8, {h.kv, P, h.d}, "k_cache", true);
    const void* vc = ptr(a[2], kU8, {h.kv, P, h.d}, "v_cache", true);
    const void* sk = ptr(a[3], kU8, {s.T, h.kv, h.d}, "step_k");
    const void* sv = ptr(a[4], kU8, {s.T, h.kv, h.d}, "step_v");
    const float* ks = ptr<float>(a[5], kF32, {h.kv}, "k_scale");
    const float* vs = ptr<float>(a[6], kF32, {h.kv}, "v_scale");
    void* out = ptr(a[14], kBF16, {s.T, h.heads, h.d}, "out");
    void* st = stream_of(a[15]);
    call([&] { return la_step_attention_fp8kv(q, kc, vc, sk, sv, ks, vs, P, s.W, s.N, s.G, h.heads, h.kv, h.d, out, st); });
}

LA_ENTRY(step_attention_cap)
{
    const int P = integer(a[5]);
    const Step s(a + 6);
    const Heads h(a + 9);
    const int64_t cap = size_of(a[1], 1, "k_cache");
    const void* q = ptr(a[0], kBF16, {s.T, h.heads, h.d}, "q");
    const void* kc = ptr(a[1], kBF16, {h.kv, cap, h.d}, "k_cache");
    const void* vc = ptr(a[2], kBF16, {h.kv, cap, h.d}, "v_cache");
    const void* sk = ptr(a[3], kBF16, {s.T, h.kv, h.d}, "step_k");
    const void* sv = ptr(a[4], kBF16, {s.T, h.kv, h.d}, "step_v");
    void* out = ptr(a[12], kBF16, {s.T, h.heads, h.d}, "out");
    void* st = stream_of(a[13]);
    call([&] { return la_step_attention_cap(q, kc, vc, cap, sk, sv, P, s.W, s.N, s.G, h.heads, h.kv, h.d, out, st); });
}

LA_ENTRY(step_rope)
{
    const int P = integer(a[4]);
    const Step s(a + 5);
    const Heads h(a + 8);
    const int n_pos = integer(size_of(a[2], 0, "cos"), "cos");
    void* q = ptr(a[0], kBF16, {s.T, h.heads, h.d}, "q", true);   // None: the keys alone
    void* sk = ptr(a[1], kBF16, {s.T, h.kv, h.d}, "step_k");
    const float* c = ptr<float>(a[2], kF32, {n_pos, h.d / 2}, "cos");
    const float* n = ptr<float>(a[3], kF32, {n_pos, h.d / 2}, "sin");
    const int inter = truth(a[11]);
    void* st = stream_of(a[12]);
    call([&] { return la_step_rope(q, sk, c, n, n_pos, P, s.W, s.N, s.G, h.heads, h.kv, h.d, inter, st); });
}

LA_ENTRY(step_attention_rope)
{
    const int P = integer(a[7]);
    const Step s(a + 8);
    const Heads h(a + 11);
    const int n_pos = integer(size_of(a[5], 0, "cos"), "cos");
    const void* q = ptr(a[0], kBF16, {s.T, h.heads, h.d}, "q");
    const void* kc = ptr(a[1], kBF16, {h.kv, P, h.d}, "k_cache", true);
    const void* vc = ptr(a[2], kBF16, {h.kv, P, h.d}, "v_cache", true);
    const void* sk = ptr(a[3], kBF16, {s.T, h.kv, h.d}, "step_k");
    const void* sv = ptr(a[4], kBF16, {s.T, h.kv, h.d}, "step_v");
    const float* c = ptr<float>(a[5], kF32, {n_pos, h.d / 2}, "cos");
    const float* n = ptr<float>(a[6], kF32, {n_pos, h.d / 2}, "sin");
    void* out = ptr(a[14], kBF16, {s.T, h.heads, h.d}, "out");
    const int inter = truth(a[15]), rotate = truth(a[16]);
    void* st = stream_of(a[17]);
    call([&] {
        return la_step_attention_rope(q, kc, vc, sk, sv, c, n, n_pos, inter, rotate, P, s.W, s.N, s.G, h.heads, h.kv, h.d,
                                      out, st);
    });
}

LA_ENTRY(kv_commit)
{
    const int P = integer(a[4]);
    const Step s(a + 5);
    const int kv = integer(a[8]), d = integer(a[9]);
    const int64_t cap = size_of(a[0], 1, "k_cache");
    void* kc = ptr(a[0], kBF16, {kv, cap, d}, "k_cache");
    void* vc = ptr(a[1], kBF16, {kv, cap, d}, "v_cache");
    const void* sk = ptr(a[2], kBF16, {s.T, kv, d}, "step_k");
    const void* sv = ptr(a[3], kBF16, {s.T, kv, d}, "step_v");
    const int* best = ptr<int>(a[10], kI32, {1}, "best");
    const int* n_out = ptr<int>(a[11], kI32, {1}, "n_out");
    void* st = stream_of(a[12]);
    call([&] { return la_kv_commit(kc, vc, cap, sk, sv, P, s.W, s.N, s.G, kv, d, best, n_out, st); });
}

LA_ENTRY(kv_commit_rope)
{
    const int P = integer(a[6]);
    const Step s(a + 7);
    const int kv = integer(a[10]), d = integer(a[11]);
    const int64_t cap = size_of(a[0], 1, "k_cache");
    const int n_pos = integer(size_of(a[4], 0, "cos"), "cos");
    void* kc = ptr(a[0], kBF16, {kv, cap, d}, "k_cache");
    void* vc = ptr(a[1], kBF16, {kv, cap, d}, "v_cache");
    const void* sk = ptr(a[2], kBF16, {s.T, kv, d}, "step_k");
    const void* sv = ptr(a[3], kBF16, {s.T, kv, d}, "step_v");
    const float* c = ptr<float>(a[4], kF32, {n_pos, d / 2}, "cos");
    const float* n = ptr<float>(a[5], kF32, {n_pos, d / 2}, "sin");
    const int* best = ptr<int>(a[12], kI32, {1}, "best");
    const int* n_out = ptr<int>(a[13], kI32, {1}, "n_out");
    const int inter = truth(a[14]);
    void* st = stream_of(a[15]);
    call([&] {
        return la_kv_commit_rope(kc, vc, cap, sk, sv, c, n, n_pos, inter, P, s.W, s.N, s.G, kv, d, best, n_out, st);
    });
}

LA_ENTRY(step_attention_batch)
{
    Items x(a[0]);
    const Step s(a + 1);
    const Heads h(a + 4);
    std::vector<la_step_desc> d((size_t)x.size());
    for (int i = 0; i < x.size(); ++i) {
        const int P = whole_number(x.at(i, KEY("P")));
        d[i].q = ptr(x.at(i, KEY("q")), kBF16, {s.T, h.heads, h.d}, "q");
        d[i].k_cache = ptr(x.at(i, KEY("k_cache")), kBF16, {h.kv, P, h.d}, "k_cache", true);
        d[i].v_cache = ptr(x.at(i, KEY("v_cache")), kBF16, {h.kv, P, h.d}, "v_cache", true);
        d[i].step_k = ptr(x.at(i, KEY("step_k")), kBF16, {s.T, h.kv, h.d}, "step_k");
        d[i].step_v = ptr(x.at(i, KEY("step_v")), kBF16, {s.T, h.kv, h.d}, "step_v");
        d[i].out = ptr(x.at(i, KEY("out")), kBF16, {s.T, h.heads, h.d}, "out");
        d[i].P = P;
        d[i].reserved = 0;
    }
    void* st = stream_of(a[7]);
    call([&] { return la_step_attention_batch(d.data(), x.size(), s.W, s.N, s.G, h.heads, h.kv, h.d, st); });
}

LA_ENTRY(step_attention_batch_paged)
{
    Items x(a[0]);
    const Step s(a + 3);
    const Heads h(a + 6);
    const Pages pg = pages_of(a[1], a[2], h.kv, h.d);
    std::vector<la_step_desc_paged> d((size_t)x.size());
    for (int i = 0; i < x.size(); ++i) {
        const int P = whole_number(x.at(i, KEY("P")));
        d[i].block_table = table_of(x.at(i, KEY("block_table"), true), P, pg.page_size);
        d[i].q = ptr(x.at(i, KEY("q")), kBF16, {s.T, h.heads, h.d}, "q");
        d[i].step_k = ptr(x.at(i, KEY("step_k")), kBF16, {s.T, h.kv, h.d}, "step_k");
        d[i].step_v = ptr(x.at(i, KEY("step_v")), kBF16, {s.T, h.kv, h.d}, "step_v");
        d[i].out = ptr(x.at(i, KEY("out")), kBF16, {s.T, h.heads, h.d}, "out");
        d[i].P = P;
        d[i].reserved = 0;
    }
    void* st = stream_of(a[9]);
    call([&] {
        return la_step_attention_batch_paged(d.data(), x.size(), pg.k, pg.v, pg.page_size, pg.n_pages, s.W, s.N, s.G, h.heads,
                                             h.kv, h.d, st);
    });
}

LA_ENTRY(step_attention_rows)
{
    const int P = integer(a[6]);
    const Step s(a + 7);
    const Heads h(a + 10);
    const int n = integer(tensor(a[5], "row_ids").numel(), "row_ids");
    const void* q = ptr(a[0], kBF16, {n, h.heads, h.d}, "q");
    const void* kc = ptr(a[1], kBF16, {h.kv, P, h.d}, "k_cache", true);
    const void* vc = ptr(a[2], kBF16, {h.kv, P, h.d}, "v_cache", true);
    const void* sk = ptr(a[3], kBF16, {n, h.kv, h.d}, "step_k");
    const void* sv = ptr(a[4], kBF16, {n, h.kv, h.d}, "step_v");
    const int* ids = ptr<int>(a[5], kI32, {n}, "row_ids");
    void* out = ptr(a[13], kBF16, {n, h.heads, h.d}, "out");
    void* st = stream_of(a[14]);
    call([&] {
        return la_step_attention_rows(q, kc, vc, sk, sv, ids, n, P, s.W, s.N, s.G, h.heads, h.kv, h.d, out, st);
    });
}

LA_ENTRY(step_attention_paged)
{
    const int P = integer(a[6]);
    const Step s(a + 7);
    const Heads h(a + 10);
    const int* table = table_of(a[3], P, integer(size_of(a[1], 2, "k_pages"), "k_pages"));
    const Pages pg = pages_of(a[1], a[2], h.kv, h.d);
    const void* q = ptr(a[0], kBF16, {s.T, h.heads, h.d}, "q");
    const void* sk = ptr(a[4], kBF16, {s.T, h.kv, h.d}, "step_k");
    const void* sv = ptr(a[5], kBF16, {s.T, h.kv, h.d}, "step_v");
    void* out = ptr(a[13], kBF16, {s.T, h.heads, h.d}, "out");
    void* st = stream_of(a[14]);
    call([&] {
        return la_step_attention_paged(q, pg.k, pg.v, table, pg.page_size, pg.n_pages, sk, sv, P, s.W, s.N, s.G, h.heads, h.kv,
                                       h.d, out, st);
    });
}

LA_ENTRY(kv_commit_paged)
{
    const int P = integer(a[5]);
    const Step s(a + 6);
    const int kv = integer(a[9]), d = integer(a[10]);
    const int* table = table_of(a[2], (int64_t)P + s.N, integer(size_of(a[0], 2, "k_pages"), "k_pages"));
    const Pages pg = pages_of(a[0], a[1], kv, d);
    const void* sk = ptr(a[3], kBF16, {s.T, kv, d}, "step_k");
    const void* sv = ptr(a[4], kBF16, {s.T, kv, d}, "step_v");
    const int* best = ptr<int>(a[11], kI32, {1}, "best");
    const int* n_out = ptr<int>(a[12], kI32, {1}, "n_out");
    void* st = stream_of(a[13]);
    call([&] {
        return la_kv_commit_paged(pg.k, pg.v, table, pg.page_size, pg.n_pages, sk, sv, P, s.W, s.N, s.G, kv, d, best, n_out, st);
    });
}

LA_ENTRY(kv_commit_batch)
{
    Items x(a[0]);
    const Step s(a + 1);
    const int kv = integer(a[4]), d = integer(a[5]);
    std::vector<la_commit_desc> c((size_t)x.size());
    int page_size = 0, n_pages = 0;
    for (int i = 0; i < x.size(); ++i) {
        const int P = whole_number(x.at(i, KEY("P")));
        PyObject* const table = x.at(i, KEY("block_table"), true);
        PyObject *const kc = x.at(i, KEY("k_cache")), *const vc = x.at(i, KEY("v_cache"));
        if (table != Py_None) {
            c[i].block_table = table_of(table, (int64_t)P + s.N, integer(size_of(kc, 2, "k_pages"), "k_pages"));
            const Pages pg = pages_of(kc, vc, kv, d);
            if (page_size && (pg.page_size != page_size || pg.n_pages != n_pages)) {
                PyErr_SetString(PyExc_ValueError, "all page pools of a launch must have the same geometry");
                throw Raised();
            }
            page_size = pg.page_size;
            n_pages = pg.n_pages;
            c[i].k_cache = pg.k;
            c[i].v_cache = pg.v;
            c[i].capacity = 0;
        } else {
            const int64_t cap = size_of(kc, 1, "k_cache");
            c[i].k_cache = ptr(kc, kBF16, {kv, cap, d}, "k_cache");
            c[i].v_cache = ptr(vc, kBF16, {kv, cap, d}, "v_cache");
            c[i].block_table = nullptr;
            c[i].capacity = cap;
        }
        c[i].step_k = ptr(x.at(i, KEY("step_k")), kBF16, {s.T, kv, d}, "step_k");
        c[i].step_v = ptr(x.at(i, KEY("step_v")), kBF16, {s.T, kv, d}, "step_v");
        c[i].best = ptr<int>(x.at(i, KEY("best")), kI32, {1}, "best");
        c[i].n_out = ptr<int>(x.at(i, KEY("n_out")), kI32, {1}, "n_out");
        c[i].P = P;
        c[i].reserved = 0;
    }
    void* st = stream_of(a[6]);
    call([&] { return la_kv_commit_batch(c.data(), x.size(), page_size, n_pages, s.W, s.N, s.G, kv, d, st); });
}

LA_ENTRY(verify)
{
    const int G = integer(a[2]), N = integer(a[3]), V = integer(a[4]);
    const float* logits = ptr<float>(a[0], kF32, {G, N - 1, V}, "logits");
    const int* cand = ptr<int>(a[1], kI32, {G, N - 1}, "cand_tokens");
    int* len = ptr<int>(a[5], kI32, {G}, "accept_len");
    int* acc = ptr<int>(a[6], kI32, {G, N - 1}, "accepted");
    void* st = stream_of(a[7]);
    call([&] { return la_verify(logits, cand, G, N, V, len, acc, st); });
}

void fill(la_verify_desc& d, PyObject* cur, PyObject* look, PyObject* cand, PyObject* toks, PyObject* out, PyObject* n_out,
          PyObject* best, PyObject* window, PyObject* len, const Step& s, int V)
{
    d.logits_cur = ptr<float>(cur, kF32, {V}, "logits_cur");
    d.logits_look = ptr<float>(look, kF32, {s.W, V}, "logits_look", true);
    d.logits_cand = ptr<float>(cand, kF32, {s.G, s.N - 1, V}, "logits_cand", true);
    d.cand_tokens = ptr<int>(toks, kI32, {s.G, s.N - 1}, "cand_tokens", true);
    d.out_tokens = ptr<int>(out, kI32, {s.N}, "out_tokens");
    d.n_out = ptr<int>(n_out, kI32, {1}, "n_out");
    d.best = ptr<int>(best, kI32, {1}, "best");
    d.new_window = ptr<int>(window, kI32, {s.W}, "new_window", true);
    d.accept_len = ptr<int>(len, kI32, {s.G}, "accept_len", true);
}

LA_ENTRY(verify_step)
{
    const Step s(a + 4);
    const int V = integer(a[7]);
    la_verify_desc d;
    fill(d, a[0], a[1], a[2], a[3], a[8], a[9], a[10], a[11], a[12], s, V);
    void* st = stream_of(a[13]);
    call([&] {
        return la_verify_step(d.logits_cur, d.logits_look, d.logits_cand, d.cand_tokens, s.W, s.N, s.G, V, d.out_tokens, d.n_out,
                              d.best, d.new_window, d.accept_len, st);
    });
}

LA_ENTRY(verify_step_batch)
{
    Items x(a[0]);
    const Step s(a + 1);
    const int V = integer(a[4]);
    std::vector<la_verify_desc> d((size_t)x.size());
    for (int i = 0; i < x.size(); ++i)
        fill(d[i], x.at(i, KEY("logits_cur")), x.at(i, KEY("logits_look"), true), x.at(i, KEY("logits_cand"), true),
             x.at(i, KEY("cand_tokens"), true), x.at(i, KEY("out_tokens")), x.at(i, KEY("n_out")), x.at(i, KEY("best")),
             x.at(i, KEY("new_window"), true), x.at(i, KEY("accept_len"), true), s, V);
    void* st = stream_of(a[5]);
    call([&] { return la_verify_step_batch(d.data(), x.size(), s.W, s.N, s.G, V, st); });
}

void fill(la_sample_desc& d, PyObject* cur, PyObject* cand, PyObject* toks, PyObject* u_test, PyObject* u_final,
          PyObject* temperature, PyObject* out, PyObject* n_out, int N, int G, int V)
{
    d.logits_cur = ptr<float>(cur, kF32, {V}, "logits_cur");
    d.logits_cand = ptr<float>(cand, kF32, {G, N - 1, V}, "logits_cand", true);
    d.cand_tokens = ptr<int>(toks, kI32, {G, N - 1}, "cand_tokens", true);
    d.u_test = ptr<float>(u_test, kF32, {N - 1, G}, "u_test", true);
    d.u_final = ptr<float>(u_final, kF32, {1}, "u_final");
    d.out_tokens = ptr<int>(out, kI32, {N}, "out_tokens");
    d.n_out = ptr<int>(n_out, kI32, {1}, "n_out");
    d.temperature = real(temperature);
    d.reserved = 0;
}

LA_ENTRY(verify_sample)
{
    const int N = integer(a[6]), G = integer(a[7]), V = integer(a[8]);
    la_sample_desc d;
    fill(d, a[0], a[1], a[2], a[3], a[4], a[5], a[9], a[10], N, G, V);
    void* st = stream_of(a[11]);
    call([&] {
        return la_verify_sample(d.logits_cur, d.logits_cand, d.cand_tokens, d.u_test, d.u_final, d.temperature, N, G, V,
                                d.out_tokens, d.n_out, st);
    });
}

LA_ENTRY(verify_sample_batch)
{
    Items x(a[0]);
    const int N = integer(a[1]), G = integer(a[2]), V = integer(a[3]);
    std::vector<la_sample_desc> d((size_t)x.size());
    for (int i = 0; i < x.size(); ++i)
        fill(d[i], x.at(i, KEY("logits_cur")), x.at(i, KEY("logits_cand"), true), x.at(i, KEY("cand_tokens"), true),
             x.at(i, KEY("u_test"), true), x.at(i, KEY("u_final")), x.at(i, KEY("temperature")), x.at(i, KEY("out_tokens")),
             x.at(i, KEY("n_out")), N, G, V);
    void* st = stream_of(a[4]);
    call([&] { return la_verify_sample_batch(d.data(), x.size(), N, G, V, st); });
}

// ---- the decoding loop's host work (lookahead.py)

// Numbers as a new tensor of the current GPU.  The copy is queued on the current stream and not waited for: it leaves
// from pinned memory that torch's allocator holds back until the copy has run.  (torch.tensor(list, device="cuda") copies
// from pageable memory and waits: 19 us for 121 tokens, here 7.)
PyObject* sent(const std::vector<uint32_t>& words, at::ScalarType type)
{
    at::Tensor on_gpu;
    {
        const Unlocked unlocked;   // (the first pinned block is an allocation of milliseconds)
        const at::Tensor host = at::empty({(int64_t)words.size()}, at::TensorOptions().dtype(type).pinned_memory(true));
        if (!words.empty()) memcpy(host.data_ptr(), words.data(), words.size() * 4);
        on_gpu = host.to(at::TensorOptions().device(at::kCUDA), /*non_blocking=*/true);
    }
    return THPVariable_Wrap(on_gpu);
}

// upload(lists, floats): the numbers of the lists one after the other, in int32 (or fp32)
PyObject* upload(PyObject*, PyObject* const* args, Py_ssize_t n_args)
{
    if (n_args != 2 || !PyList_Check(args[0])) {
        PyErr_SetString(PyExc_TypeError, "a list of lists and a truth value are expected");
        return nullptr;
    }
    try {
        const bool floats = truth(args[1]);
        // Converting an item may run code that changes any of the lists: their sizes are read anew each time, and what is
        // in use is held.
        std::vector<uint32_t> words;
        for (Py_ssize_t i = 0; i < PyList_GET_SIZE(args[0]); ++i) {
            const Owned l(PyList_GET_ITEM(args[0], i));
            Py_INCREF(l.o);
            if (!PyList_Check(l.o)) {
                PyErr_SetString(PyExc_TypeError, "a list of lists is expected");
                return nullptr;
            }
            words.reserve(words.size() + (size_t)PyList_GET_SIZE(l.o));
            for (Py_ssize_t j = 0; j < PyList_GET_SIZE(l.o); ++j) {
                const Owned item(PyList_GET_ITEM(l.o, j));
                Py_INCREF(item.o);
                uint32_t w;
                if (floats) {
                    const double v = PyFloat_AsDouble(item.o);
                    if (v == -1.0 && PyErr_Occurred()) return nullptr;
                    const float f = (float)v;
                    memcpy(&w, &f, 4);
                } else {
                    w = (uint32_t)integer(item.o);
                }
                words.push_back(w);
            }
        }
        return sent(words, floats ? kF32 : kI32);
    } catch (const Raised&) {
        return nullptr;
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// upload_in_range(lists, limit): the same in int32, or None unless this is a list of lists of ints (no subclass of either)
// of 0 .. limit-1
PyObject* upload_in_range(PyObject*, PyObject* const* args, Py_ssize_t n_args)
{
    if (n_args != 2) {
        PyErr_SetString(PyExc_TypeError, "two arguments are expected");
        return nullptr;
    }
    const long long most = PyLong_AsLongLong(args[1]);
    if (most == -1 && PyErr_Occurred()) return nullptr;
    const long long limit = most < (1ll << 31) ? most : 1ll << 31;
    if (!PyList_CheckExact(args[0])) Py_RETURN_NONE;
    try {
        std::vector<uint32_t> words;
        for (Py_ssize_t i = 0; i < PyList_GET_SIZE(args[0]); ++i) {       // (none of this runs code that could change a list)
            PyObject* const l = PyList_GET_ITEM(args[0], i);
            if (!PyList_CheckExact(l)) Py_RETURN_NONE;
            const Py_ssize_t n = PyList_GET_SIZE(l);
            words.reserve(words.size() + (size_t)n);
            for (Py_ssize_t j = 0; j < n; ++j) {
                PyObject* const item = PyList_GET_ITEM(l, j);
                if (!PyLong_CheckExact(item)) Py_RETURN_NONE;
                int overflow = 0;
                const long long v = PyLong_AsLongLongAndOverflow(item, &overflow);
                if (overflow || v < 0 || v >= limit) Py_RETURN_NONE;
                words.push_back((uint32_t)v);
            }
        }
        return sent(words, kI32);
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// Three arguments taken modulo 2^64, as the generators below are defined, and a count.
bool words(PyObject* const* args, Py_ssize_t n_args, Py_ssize_t want, uint64_t* w, Py_ssize_t* count)
{
    if (n_args != want) {
        PyErr_Format(PyExc_TypeError, "%zd arguments are expected, got %zd", want, n_args);
        return false;
    }
    for (Py_ssize_t i = 0; i < want - 1; ++i) {
        w[i] = PyLong_AsUnsignedLongLongMask(args[i]);
        if (w[i] == (uint64_t)-1 && PyErr_Occurred()) return false;
    }
    *count = PyLong_AsSsize_t(args[want - 1]);
    return !(*count == -1 && PyErr_Occurred());
}

// window_random_tokens(seed, step, vocab, count): workloads.window_random_token of columns 0 .. count-1
PyObject* window_random_tokens(PyObject*, PyObject* const* args, Py_ssize_t n_args)
{
    uint64_t w[3];
    Py_ssize_t count;
    if (!words(args, n_args, 4, w, &count)) return nullptr;
    int overflow = 0;
    const long long vocab = PyLong_AsLongLongAndOverflow(args[2], &overflow);
    if (vocab == -1 && !overflow && PyErr_Occurred()) return nullptr;
    if (overflow || vocab < 2) {                    // (tokens of 1 .. vocab-1)
        PyErr_Format(PyExc_ValueError, "no random token of a vocabulary of %S", args[2]);
        return nullptr;
    }
    PyObject* const list = PyList_New(count > 0 ? count : 0);
    for (Py_ssize_t j = 0; list && j < count; ++j) {
        uint64_t h = w[0] * 0x9E3779B97F4A7C15ull + w[1] * 0xBF58476D1CE4E5B9ull + (uint64_t)j * 0x94D049BB133111EBull;
        h ^= h >> 31;
        h *= 0xD6E8FEB86659FD93ull;
        h ^= h >> 29;
        PyObject* const v = PyLong_FromUnsignedLongLong(1 + h % ((uint64_t)vocab - 1));
        if (!v) {
            Py_DECREF(list);
            return nullptr;
        }
        PyList_SET_ITEM(list, j, v);
    }
    return list;
}

// uniform_draws(seed, step, first, count): workloads.uniform_draw of indices first .. first+count-1
PyObject* uniform_draws(PyObject*, PyObject* const* args, Py_ssize_t n_args)
{
    uint64_t w[3];
    Py_ssize_t count;
    if (!words(args, n_args, 4, w, &count)) return nullptr;
    PyObject* const list = PyList_New(count > 0 ? count : 0);
    for (Py_ssize_t j = 0; list && j < count; ++j) {
        uint64_t h = w[0] * 0xD1342543DE82EF95ull + w[1] * 0x9E3779B97F4A7C15ull +
                     (w[2] + (uint64_t)j) * 0xC2B2AE3D27D4EB4Full + 0x165667B19E3779F9ull;
        h ^= h >> 32;
        h *= 0xD6E8FEB86659FD93ull;
        h ^= h >> 32;
        h *= 0xD6E8FEB86659FD93ull;
        h ^= h >> 32;
        PyObject* const v = PyFloat_FromDouble((double)(h >> 40) / (double)(1 << 24));   // (24 bits: a float32)
        if (!v) {
            Py_DECREF(list);
            return nullptr;
        }
        PyList_SET_ITEM(list, j, v);
    }
    return list;
}

// ---- module

template <void (*F)(PyObject* const*), int N_ARGS>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (n != N_ARGS) {
        PyErr_Format(PyExc_TypeError, "%d arguments are expected, got %zd", N_ARGS, n);
        return nullptr;
    }
    try {
        F(args);
    } catch (const Raised&) {
        return nullptr;
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
    Py_RETURN_NONE;
}

PyObject* set_error_class(PyObject*, PyObject* cls)
{
    Py_INCREF(cls);
    Py_XSETREF(g_la_error, cls);
    Py_RETURN_NONE;
}

#define LA_METHOD(name, n_args) {#name, (PyCFunction)(void (*)(void))(entry<name, n_args>), METH_FASTCALL, nullptr}

PyMethodDef methods[] = {
    LA_METHOD(step_attention, 14),
    LA_METHOD(step_attention_noalloc, 14),
    LA_METHOD(step_attention_fp8kv, 16),
    LA_METHOD(step_attention_cap, 14),
    LA_METHOD(step_rope, 13),
    LA_METHOD(step_attention_rope, 18),
    LA_METHOD(kv_commit, 13),
    LA_METHOD(kv_commit_rope, 16),
    LA_METHOD(step_attention_batch, 8),
    LA_METHOD(step_attention_batch_paged, 10),
    LA_METHOD(step_attention_rows, 15),
    LA_METHOD(step_attention_paged, 15),
    LA_METHOD(kv_commit_paged, 14),
    LA_METHOD(kv_commit_batch, 7),
    LA_METHOD(verify, 8),
    LA_METHOD(verify_step, 14),
    LA_METHOD(verify_step_batch, 6),
    LA_METHOD(verify_sample, 12),
    LA_METHOD(verify_sample_batch, 5),
    {"upload", (PyCFunction)(void (*)(void))upload, METH_FASTCALL, nullptr},
    {"upload_in_range", (PyCFunction)(void (*)(void))upload_in_range, METH_FASTCALL, nullptr},
    {"window_random_tokens", (PyCFunction)(void (*)(void))window_random_tokens, METH_FASTCALL, nullptr},
    {"uniform_draws", (PyCFunction)(void (*)(void))uniform_draws, METH_FASTCALL, nullptr},
    {"set_error_class", set_error_class, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_la_native", "Argument marshalling of the C ABI, and the decoding loop's host work.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__la_native() { return PyModule_Create(&module); }
