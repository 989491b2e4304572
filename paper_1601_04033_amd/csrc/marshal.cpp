// Native argument marshalling of the binding's calls (module _marshal): plain
// arguments (contiguous device tensors of the right type and length, integers,
// floats, sequences of them) become the C ABI's arguments without a Python
// bytecode per tensor.  An argument that is not plain in this sense (another
// tensor type or subclass, a wrong length, a number that Python converts by
// its own rules) makes a call return None with nothing done; the binding then
// takes its general way in Python, which converts or rejects it.  The two ways
// make the same library call with the same arguments.
//
// Host time per call, back to back, with the library call in it (3.5 us with
// one kernel launch): a pass of K = 1 / 16 / 32 gradients 8.4 / 20.5 / 33.2 us
// marshalled in Python, 3.7 / 4.0 / 4.2 us here; a selection (two launches)
// 12.3 and 6.3 us, a sparse apply 8.0 and 4.0 us.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <stdint.h>
#include <string.h>

#include "../../include/fasgd.h"

namespace {

// the library's entry points, by the order of kNames
constexpr const char* kNames[] = {
    "fasgd_apply_updates", "sasgd_apply_updates", "bfasgd_select_compact", "bfasgd_select_compact_batch",
    "bfasgd_apply_sparse", "fasgd_apply_with_push", "fasgd_apply_with_push_and_select", "fasgd_apply_pushes",
    "bfasgd_apply_cached", "bfasgd_apply_fetch", "bfasgd_decide_segments", "bfasgd_apply_segments"};
constexpr int kCount = sizeof kNames / sizeof kNames[0];
struct Entry {
    decltype(&::fasgd_apply_updates) fasgd_apply_updates;
    decltype(&::sasgd_apply_updates) sasgd_apply_updates;
    decltype(&::bfasgd_select_compact) bfasgd_select_compact;
    decltype(&::bfasgd_select_compact_batch) bfasgd_select_compact_batch;
    decltype(&::bfasgd_apply_sparse) bfasgd_apply_sparse;
    decltype(&::fasgd_apply_with_push) fasgd_apply_with_push;
    decltype(&::fasgd_apply_with_push_and_select) fasgd_apply_with_push_and_select;
    decltype(&::fasgd_apply_pushes) fasgd_apply_pushes;
    decltype(&::bfasgd_apply_cached) bfasgd_apply_cached;
    decltype(&::bfasgd_apply_fetch) bfasgd_apply_fetch;
    decltype(&::bfasgd_decide_segments) bfasgd_decide_segments;
    decltype(&::bfasgd_apply_segments) bfasgd_apply_segments;
};
static_assert(sizeof(Entry) == kCount * sizeof(void*), "one pointer per name");
Entry g_lib;                          // set by bind(), once, before any other call
PyObject* g_current_stream = nullptr; // callable: the current stream's handle as an int

// One call's arguments.  Every getter returns a usable value while `plain`
// holds; afterwards nothing that they return is used.
struct Args {
    PyObject* const* v;
    bool plain = true;
    Py_buffer state_view{};
    Py_buffer seg_view{};
    PyObject* held[3] = {nullptr, nullptr, nullptr};   // fast sequences of this call
    int n_held = 0;

    explicit Args(PyObject* const* args) : v(args) {}
    ~Args()
    {
        if (state_view.obj) PyBuffer_Release(&state_view);
        if (seg_view.obj) PyBuffer_Release(&seg_view);
        for (int i = 0; i < n_held; ++i) Py_DECREF(held[i]);
    }
    Args(const Args&) = delete;
    Args& operator=(const Args&) = delete;

    // The argument is not plain.  Of the exceptions that its conversion may
    // have raised, those that say so are dropped, as the general way raises
    // them again; any other (an interrupt, a signal handler's, no memory)
    // stays set, and finish() lets it out.
    bool refuse()
    {
        if (PyErr_Occurred() &&
            (PyErr_ExceptionMatches(PyExc_TypeError) || PyErr_ExceptionMatches(PyExc_ValueError) ||
             PyErr_ExceptionMatches(PyExc_OverflowError) || PyErr_ExceptionMatches(PyExc_AttributeError) ||
             PyErr_ExceptionMatches(PyExc_BufferError)))
            PyErr_Clear();
        plain = false;
        return false;
    }

    // the fasgd_state struct (a ctypes Structure, by its buffer)
    fasgd_state* state(int i)
    {
        if (!plain) return nullptr;
        if (PyObject_GetBuffer(v[i], &state_view, PyBUF_WRITABLE) != 0 ||
            state_view.len != static_cast<Py_ssize_t>(sizeof(fasgd_state))) {
            refuse();
            return nullptr;
        }
        return static_cast<fasgd_state*>(state_view.buf);
    }

    // a contiguous device tensor of `type` with at least `least` elements and,
    // when `exactly` >= 0, that many; the element count goes to *n
    void* tensor_of(PyObject* o, c10::ScalarType type, int64_t exactly, int64_t least = 0, int64_t* n = nullptr)
    {
        if (!plain) return nullptr;
        if (!THPVariable_CheckExact(o)) {
            refuse();
            return nullptr;
        }
        try {
            const at::Tensor& t = THPVariable_Unpack(o);
            const int64_t count = t.numel();
            if (!t.is_cuda() || t.scalar_type() != type || !t.is_contiguous() || (exactly >= 0 && count != exactly) ||
                count < least) {
                refuse();
                return nullptr;
            }
            if (n) *n = count;
            return t.data_ptr();
        } catch (...) {   // a tensor without storage: the general way says so
            refuse();
            return nullptr;
        }
    }
    void* tensor(int i, c10::ScalarType type, int64_t exactly, int64_t least = 0, int64_t* n = nullptr)
    {
        return tensor_of(v[i], type, exactly, least, n);
    }
    float* floats(int i, int64_t exactly, int64_t* n = nullptr)
    {
        return static_cast<float*>(tensor(i, c10::ScalarType::Float, exactly, 0, n));
    }
    int32_t* ints(int i, int64_t exactly, int64_t* n = nullptr)
    {
        return static_cast<int32_t*>(tensor(i, c10::ScalarType::Int, exactly, 0, n));
    }
    int64_t* counts(int i, int64_t exactly)
    {
        return static_cast<int64_t*>(tensor(i, c10::ScalarType::Long, exactly));
    }
    // a [B, columns] tensor's columns
    int64_t columns(int i, int64_t B)
    {
        if (!plain) return 0;
        try {
            if (THPVariable_CheckExact(v[i])) {
                const at::Tensor& t = THPVariable_Unpack(v[i]);
                if (t.dim() == 2 && t.size(0) == B) return t.size(1);
            }
        } catch (...) {
        }
        refuse();
        return 0;
    }
    // the list index (None where it may be absent)
    uint32_t* seg_start(int i, int64_t length, bool required, bool whole = false)
    {
        if (!plain || (v[i] == Py_None && !required)) return nullptr;
        return static_cast<uint32_t*>(tensor(i, c10::ScalarType::Int, whole ? length : -1, length));
    }

    int64_t integer_of(PyObject* o)
    {
        if (!plain) return 0;
        PyObject* x = PyNumber_Index(o);   // an int, or what says it is one (numpy's)
        if (!x) {
            refuse();
            return 0;
        }
        int over = 0;
        const long long r = PyLong_AsLongLongAndOverflow(x, &over);
        Py_DECREF(x);
        if (over || (r == -1 && PyErr_Occurred())) {
            refuse();
            return 0;
        }
        return r;
    }
    int64_t int64(int i) { return integer_of(v[i]); }
    int32_t narrow(int64_t r)
    {
        if (r < INT32_MIN || r > INT32_MAX) refuse();
        return static_cast<int32_t>(r);
    }
    int32_t int32(int i) { return narrow(integer_of(v[i])); }
    // any integer, by its low 64 bits
    uint64_t seed(int i)
    {
        if (!plain) return 0;
        PyObject* x = PyNumber_Index(v[i]);
        if (!x) {
            refuse();
            return 0;
        }
        const uint64_t r = PyLong_AsUnsignedLongLongMask(x);
        Py_DECREF(x);
        if (PyErr_Occurred()) refuse();
        return r;
    }
    // what ctypes takes for a float: any number (numpy's too)
    float real(int i)
    {
        if (!plain) return 0.0f;
        const double d = PyFloat_AsDouble(v[i]);
        if (d == -1.0 && PyErr_Occurred()) refuse();
        return static_cast<float>(d);
    }

    // a sequence of n (n < 0: any number, 1 .. most); lists and tuples are taken as they are, so a list's items are
    // read through integer_at() wherever Python code may have run since
    PyObject* sequence(int i, int64_t n, int64_t most, int64_t* count)
    {
        if (!plain) return nullptr;
        if (!PyList_CheckExact(v[i]) && !PyTuple_CheckExact(v[i]) && !PySequence_Check(v[i])) {
            refuse();
            return nullptr;
        }
        PyObject* f = PySequence_Fast(v[i], "");
        if (!f) {
            refuse();
            return nullptr;
        }
        held[n_held++] = f;
        const int64_t k = PySequence_Fast_GET_SIZE(f);
        if ((n >= 0 && k != n) || k < 1 || k > most) {
            refuse();
            return nullptr;
        }
        if (count) *count = k;
        return f;
    }
    // the integer at place k of a sequence: its conversion may run Python code, which may change the sequence
    int64_t integer_at(PyObject* f, int64_t k)
    {
        if (!plain) return 0;
        if (k >= PySequence_Fast_GET_SIZE(f)) {
            refuse();
            return 0;
        }
        PyObject* o = PySequence_Fast_GET_ITEM(f, k);
        Py_INCREF(o);
        const int64_t r = integer_of(o);
        Py_DECREF(o);
        return r;
    }
    int64_t gradients(int i, int64_t P, const float** out, int64_t most)
    {
        int64_t K = 0;
        PyObject* f = sequence(i, -1, most, &K);
        for (int64_t k = 0; plain && k < K; ++k)   // no Python code runs in between
            out[k] = static_cast<const float*>(tensor_of(PySequence_Fast_GET_ITEM(f, k), c10::ScalarType::Float, P));
        return K;
    }
    void clients(int i, int64_t K, int32_t* out)
    {
        PyObject* f = sequence(i, K, K, nullptr);
        for (int64_t k = 0; plain && k < K; ++k) out[k] = narrow(integer_at(f, k));
    }
    void timestamps(int i, int64_t K, int64_t* out)
    {
        PyObject* f = sequence(i, K, K, nullptr);
        for (int64_t k = 0; plain && k < K; ++k) out[k] = integer_at(f, k);
    }
    // host offsets of S + 1 segments: a C-contiguous one-dimensional int64 array
    const int64_t* segments(int i, int32_t* S)
    {
        if (!plain) return nullptr;
        if (PyObject_GetBuffer(v[i], &seg_view, PyBUF_FORMAT | PyBUF_C_CONTIGUOUS) != 0) {
            seg_view.obj = nullptr;
            refuse();
            return nullptr;
        }
        const char* f = seg_view.format;
        if (seg_view.ndim != 1 || seg_view.itemsize != 8 || !f || (f[0] != 'l' && f[0] != 'q') || f[1] ||
            seg_view.len / 8 - 1 < 0 || seg_view.len / 8 - 1 > INT32_MAX) {
            refuse();
            return nullptr;
        }
        *S = static_cast<int32_t>(seg_view.len / 8 - 1);
        return static_cast<const int64_t*>(seg_view.buf);
    }
    // the stream's handle, or it itself; None: the current stream (looked up last, after every tensor was found to be a device one)
    hipStream_t stream(int i)
    {
        if (!plain) return nullptr;
        PyObject* h;
        if (v[i] == Py_None) {
            h = PyObject_CallNoArgs(g_current_stream);
            if (!h) {   // whatever it raises is the call's
                plain = false;
                return nullptr;
            }
        } else if (PyLong_CheckExact(v[i])) {   // a raw handle
            h = v[i];
            Py_INCREF(h);
        } else {
            h = PyObject_GetAttrString(v[i], "cuda_stream");
        }
        if (!h || !PyLong_Check(h)) {
            Py_XDECREF(h);
            refuse();
            return nullptr;
        }
        void* p = PyLong_AsVoidPtr(h);
        Py_DECREF(h);
        if (PyErr_Occurred()) refuse();
        return static_cast<hipStream_t>(p);
    }
};

int64_t index_length(int64_t P) { return P < 1 ? 0 : (P + 255) / 256 + 1; }

// The library call itself, without the interpreter's lock; None unless the arguments were plain, or the exception
// that a getter left set.
template <typename Call>
PyObject* finish(Args& a, Call call)
{
    if (!a.plain) {
        if (PyErr_Occurred()) return nullptr;
        Py_RETURN_NONE;
    }
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = static_cast<int>(call());
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

bool arity(Py_ssize_t n, Py_ssize_t want)
{
    if (n == want && g_current_stream) return true;
    PyErr_SetString(PyExc_TypeError, "_marshal: wrong number of arguments, or bind() not called");
    return false;
}

// (state, grads, clients, grad_ts, stream)
template <bool FASGD>
PyObject* dense(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (!arity(n, 5)) return nullptr;
    Args a(args);
    fasgd_state* st = a.state(0);
    const float* g[FASGD_MAX_K];
    int32_t cl[FASGD_MAX_K];
    int64_t ts[FASGD_MAX_K];
    const int64_t K = a.gradients(1, st ? st->P : 0, g, FASGD_MAX_K);
    a.clients(2, K, cl);
    a.timestamps(3, K, ts);
    hipStream_t s = a.stream(4);
    return finish(a, [&] {
        return (FASGD ? g_lib.fasgd_apply_updates : g_lib.sasgd_apply_updates)(st, g, cl, ts, static_cast<int32_t>(K), s);
    });
}

// (state, grad, c, eps_c, seed, T, client, out_idx, out_val, d_count, workspace, seg_start, stream)
PyObject* select_compact(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (!arity(n, 13)) return nullptr;
    Args a(args);
    fasgd_state* st = a.state(0);
    const int64_t P = st ? st->P : 0;
    int64_t cap = 0, ws = 0;
    const float* g = a.floats(1, P);
    const float c = a.real(2), eps_c = a.real(3);
    const uint64_t seed = a.seed(4);
    const int64_t T = a.int64(5);
    const int32_t client = a.int32(6);
    int32_t* idx = a.ints(7, -1, &cap);
    float* val = a.floats(8, cap);
    int64_t* cnt = a.counts(9, -1);
    void* w = a.tensor(10, c10::ScalarType::Byte, -1, 0, &ws);
    uint32_t* seg = a.seg_start(11, index_length(P), false);
    hipStream_t s = a.stream(12);
    return finish(a, [&] {
        return g_lib.bfasgd_select_compact(st, g, c, eps_c, seed, T, client, idx, val, cap, cnt, seg, w,
                                           static_cast<size_t>(ws), s);
    });
}

// (state, grads, c, eps_c, seed, T, clients, out_idx, out_val, d_count, workspace, seg_start, stream)
PyObject* select_compact_batch(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (!arity(n, 13)) return nullptr;
    Args a(args);
    fasgd_state* st = a.state(0);
    const int64_t P = st ? st->P : 0;
    const float* g[FASGD_MAX_BATCH];
    int64_t T[FASGD_MAX_BATCH], ws = 0;
    int32_t cl[FASGD_MAX_BATCH];
    const int64_t B = a.gradients(1, P, g, FASGD_MAX_BATCH);
    const float c = a.real(2), eps_c = a.real(3);
    const uint64_t seed = a.seed(4);
    a.timestamps(5, B, T);
    a.clients(6, B, cl);
    const int64_t cap = a.columns(7, B);
    a.columns(8, B);
    int32_t* idx = a.ints(7, B * cap);
    float* val = a.floats(8, B * cap);
    int64_t* cnt = a.counts(9, B);
    void* w = a.tensor(10, c10::ScalarType::Byte, -1, 0, &ws);
    if (a.plain && a.v[11] != Py_None && a.columns(11, B) != index_length(P)) a.refuse();
    uint32_t* seg = a.seg_start(11, B * index_length(P), false, true);
    hipStream_t s = a.stream(12);
    return finish(a, [&] {
        return g_lib.bfasgd_select_compact_batch(st, static_cast<int32_t>(B), g, c, eps_c, seed, T, cl, idx, val, cap, cnt,
                                                 seg, w, static_cast<size_t>(ws), s);
    });
}

// (state, idx, val, d_count, client, grad_ts, stream)
PyObject* apply_sparse(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (!arity(n, 7)) return nullptr;
    Args a(args);
    fasgd_state* st = a.state(0);
    int64_t cap = 0;
    const int32_t* idx = a.ints(1, -1, &cap);
    const float* val = a.floats(2, cap);
    const int64_t* cnt = a.counts(3, -1);
    const int32_t client = a.int32(4);
    const int64_t ts = a.int64(5);
    hipStream_t s = a.stream(6);
    return finish(a, [&] { return g_lib.bfasgd_apply_sparse(st, idx, val, cnt, cap, client, ts, s); });
}

// (state, push_idx, push_val, push_count, push_seg_start, push_client, push_grad_ts, grads, clients, grad_ts, stream)
PyObject* with_push(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (!arity(n, 11)) return nullptr;
    Args a(args);
    fasgd_state* st = a.state(0);
    const int64_t P = st ? st->P : 0;
    int64_t cap = 0;
    const float* g[FASGD_MAX_K];
    int32_t cl[FASGD_MAX_K];
    int64_t ts[FASGD_MAX_K];
    const int32_t* idx = a.ints(1, -1, &cap);
    const float* val = a.floats(2, cap);
    const int64_t* cnt = a.counts(3, -1);
    const uint32_t* seg = a.seg_start(4, index_length(P), true);
    const int32_t client = a.int32(5);
    const int64_t push_ts = a.int64(6);
    const int64_t K = a.gradients(7, P, g, FASGD_MAX_K);
    a.clients(8, K, cl);
    a.timestamps(9, K, ts);
    hipStream_t s = a.stream(10);
    return finish(a, [&] {
        return g_lib.fasgd_apply_with_push(st, idx, val, cnt, seg, cap, client, push_ts, g, cl, ts,
                                           static_cast<int32_t>(K), s);
    });
}

// (state, push_idx, push_val, push_count, push_seg_start, push_client, push_grad_ts, grads, clients, grad_ts,
//  next_grad, next_client, c, eps_c, seed, out_idx, out_val, out_count, out_seg_start, workspace, stream)
PyObject* with_push_and_select(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (!arity(n, 21)) return nullptr;
    Args a(args);
    fasgd_state* st = a.state(0);
    const int64_t P = st ? st->P : 0;
    int64_t cap = 0, out_cap = 0, ws = 0;
    const float* g[FASGD_MAX_K];
    int32_t cl[FASGD_MAX_K];
    int64_t ts[FASGD_MAX_K];
    const int32_t* idx = a.ints(1, -1, &cap);
    const float* val = a.floats(2, cap);
    const int64_t* cnt = a.counts(3, -1);
    const uint32_t* seg = a.seg_start(4, index_length(P), true);
    const int32_t client = a.int32(5);
    const int64_t push_ts = a.int64(6);
    const int64_t K = a.gradients(7, P, g, FASGD_MAX_K);
    a.clients(8, K, cl);
    a.timestamps(9, K, ts);
    const float* next = a.floats(10, P);
    const int32_t next_client = a.int32(11);
    const float c = a.real(12), eps_c = a.real(13);
    const uint64_t seed = a.seed(14);
    int32_t* out_idx = a.ints(15, -1, &out_cap);
    float* out_val = a.floats(16, out_cap);
    int64_t* out_cnt = a.counts(17, -1);
    uint32_t* out_seg = a.seg_start(18, index_length(P), false);
    void* w = a.tensor(19, c10::ScalarType::Byte, -1, 0, &ws);
    hipStream_t s = a.stream(20);
    return finish(a, [&] {
        return g_lib.fasgd_apply_with_push_and_select(st, idx, val, cnt, seg, cap, client, push_ts, g, cl, ts,
                                                      static_cast<int32_t>(K), next, next_client, c, eps_c, seed, out_idx,
                                                      out_val, out_cap, out_cnt, out_seg, w, static_cast<size_t>(ws), s);
    });
}

// (state, idx, val, d_count, seg_start, clients, grad_ts, stream)
PyObject* apply_pushes(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (!arity(n, 8)) return nullptr;
    Args a(args);
    fasgd_state* st = a.state(0);
    const int64_t P = st ? st->P : 0;
    int32_t cl[FASGD_MAX_BATCH];
    int64_t ts[FASGD_MAX_BATCH], B = 0;
    PyObject* f = a.sequence(5, -1, FASGD_MAX_BATCH, &B);
    for (int64_t b = 0; a.plain && b < B; ++b) cl[b] = a.narrow(a.integer_at(f, b));
    a.timestamps(6, B, ts);
    const int64_t cap = a.columns(1, B);
    a.columns(2, B);
    const int32_t* idx = a.ints(1, B * cap);
    const float* val = a.floats(2, B * cap);
    const int64_t* cnt = a.counts(3, B);
    if (a.columns(4, B) != index_length(P)) a.refuse();
    const uint32_t* seg = a.seg_start(4, B * index_length(P), true, true);
    hipStream_t s = a.stream(7);
    return finish(a, [&] {
        return g_lib.fasgd_apply_pushes(st, static_cast<int32_t>(B), idx, val, cnt, seg, cap, cl, ts, s);
    });
}

// (state, idx, val, d_count, cache, client, grad_ts, seg_start, stream)
PyObject* apply_cached(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (!arity(n, 9)) return nullptr;
    Args a(args);
    fasgd_state* st = a.state(0);
    const int64_t P = st ? st->P : 0;
    int64_t cap = 0;
    const int32_t* idx = a.ints(1, -1, &cap);
    const float* val = a.floats(2, cap);
    const int64_t* cnt = a.counts(3, -1);
    float* cache = a.floats(4, P);
    const int32_t client = a.int32(5);
    const int64_t ts = a.int64(6);
    const uint32_t* seg = a.seg_start(7, index_length(P), false);
    hipStream_t s = a.stream(8);
    return finish(a, [&] { return g_lib.bfasgd_apply_cached(st, idx, val, cnt, seg, cap, cache, client, ts, s); });
}

// (theta_client, idx, val, d_count, seg_start, stream)
PyObject* apply_fetch(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (!arity(n, 6)) return nullptr;
    Args a(args);
    int64_t P = 0, cap = 0;
    float* copy = a.floats(0, -1, &P);
    const int32_t* idx = a.ints(1, -1, &cap);
    const float* val = a.floats(2, cap);
    const int64_t* cnt = a.counts(3, -1);
    const uint32_t* seg = a.seg_start(4, index_length(P), false);
    hipStream_t s = a.stream(5);
    return finish(a, [&] { return g_lib.bfasgd_apply_fetch(copy, P, idx, val, cnt, seg, cap, s); });
}

// (state, seg, c, eps_c, seed, T, client, d_transmit, workspace, stream)
PyObject* decide_segments(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (!arity(n, 10)) return nullptr;
    Args a(args);
    fasgd_state* st = a.state(0);
    int32_t S = 0;
    int64_t ws = 0;
    const int64_t* seg = a.segments(1, &S);
    const float c = a.real(2), eps_c = a.real(3);
    const uint64_t seed = a.seed(4);
    const int64_t T = a.int64(5);
    const int32_t client = a.int32(6);
    uint8_t* send = static_cast<uint8_t*>(a.tensor(7, c10::ScalarType::Byte, S));
    void* w = a.tensor(8, c10::ScalarType::Byte, -1, 0, &ws);
    hipStream_t s = a.stream(9);
    return finish(a, [&] {
        return g_lib.bfasgd_decide_segments(st, seg, S, c, eps_c, seed, T, client, send, w, static_cast<size_t>(ws), s);
    });
}

// (state, grad, seg, d_transmit, client, grad_ts, stream)
PyObject* apply_segments(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    if (!arity(n, 7)) return nullptr;
    Args a(args);
    fasgd_state* st = a.state(0);
    int32_t S = 0;
    const float* g = a.floats(1, st ? st->P : 0);
    const int64_t* seg = a.segments(2, &S);
    const uint8_t* send = static_cast<const uint8_t*>(a.tensor(3, c10::ScalarType::Byte, -1, S));   // one byte per segment
    const int32_t client = a.int32(4);
    const int64_t ts = a.int64(5);
    hipStream_t s = a.stream(6);
    return finish(a, [&] { return g_lib.bfasgd_apply_segments(st, g, seg, S, send, client, ts, s); });
}

// bind(addresses of the entry points in kNames' order, current-stream callable)
PyObject* bind(PyObject*, PyObject* args)
{
    PyObject *list, *stream;
    if (!PyArg_ParseTuple(args, "O!O", &PyList_Type, &list, &stream)) return nullptr;
    if (PyList_GET_SIZE(list) != kCount || !PyCallable_Check(stream)) {
        PyErr_SetString(PyExc_ValueError, "_marshal.bind: one address per entry point and a callable");
        return nullptr;
    }
    void* p[kCount];
    for (int i = 0; i < kCount; ++i) {
        p[i] = PyLong_AsVoidPtr(PyList_GET_ITEM(list, i));
        if (PyErr_Occurred()) return nullptr;
        if (!p[i]) {
            PyErr_SetString(PyExc_ValueError, "_marshal.bind: NULL address");
            return nullptr;
        }
    }
    memcpy(&g_lib, p, sizeof g_lib);
    Py_INCREF(stream);
    Py_XSETREF(g_current_stream, stream);
    Py_RETURN_NONE;
}

using FastCall = PyObject* (*)(PyObject*, PyObject* const*, Py_ssize_t);
PyCFunction fast(FastCall f) { return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)); }

PyMethodDef kMethods[] = {{"bind", bind, METH_VARARGS, nullptr},
                          {kNames[0], fast(dense<true>), METH_FASTCALL, nullptr},
                          {kNames[1], fast(dense<false>), METH_FASTCALL, nullptr},
                          {kNames[2], fast(select_compact), METH_FASTCALL, nullptr},
                          {kNames[3], fast(select_compact_batch), METH_FASTCALL, nullptr},
                          {kNames[4], fast(apply_sparse), METH_FASTCALL, nullptr},
                          {kNames[5], fast(with_push), METH_FASTCALL, nullptr},
                          {kNames[6], fast(with_push_and_select), METH_FASTCALL, nullptr},
                          {kNames[7], fast(apply_pushes), METH_FASTCALL, nullptr},
                          {kNames[8], fast(apply_cached), METH_FASTCALL, nullptr},
                          {kNames[9], fast(apply_fetch), METH_FASTCALL, nullptr},
                          {kNames[10], fast(decide_segments), METH_FASTCALL, nullptr},
                          {kNames[11], fast(apply_segments), METH_FASTCALL, nullptr},
                          {nullptr, nullptr, 0, nullptr}};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal()
{
    PyObject* m = PyModule_Create(&kModule);
    if (!m) return nullptr;
    PyObject* names = PyTuple_New(kCount);
    if (!names) return nullptr;
    for (int i = 0; i < kCount; ++i) PyTuple_SET_ITEM(names, i, PyUnicode_FromString(kNames[i]));
    if (PyModule_AddObject(m, "ENTRY_POINTS", names) != 0) return nullptr;
    // at::Tensor's layout is that torch's alone
    if (PyModule_AddStringConstant(m, "TORCH_VERSION", FASGD_TORCH_VERSION) != 0) return nullptr;
    return m;
}
