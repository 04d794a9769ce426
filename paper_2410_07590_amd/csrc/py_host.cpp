// Native half of binding.py: reads the arguments of a call (torch tensors, numpy arrays, the shape and the store handle)
// and passes them to the C ABI.  No arithmetic and no state besides the entry points that bind() was given.
//
// A serving loop makes three or four of these calls per layer, each in front of a few microseconds of GPU work.  Through
// ctypes a call cost 8 .. 10 us of Python besides the launches themselves (current stream 3 us, every host array 1.4 us,
// every scalar object 0.1 us), so short requests waited for the host; reading the same arguments here costs about 1 us.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#define NPY_NO_DEPRECATED_API NPY_1_7_API_VERSION
#include <numpy/arrayobject.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/turborag.h"

#include <string.h>
#include <vector>

namespace {

// ---- what bind() records --------------------------------------------------------------------------------------------
#define TR_CALLS(X)                                                                                                          \
    X(tr_last_error) X(tr_plan) X(tr_kv_assemble) X(tr_kv_assemble_raw) X(tr_kv_assemble_batched) X(tr_kv_append)            \
    X(tr_kv_assemble_append) X(tr_kv_append_batched) X(tr_prefill_attn) X(tr_prefill_attn_static) X(tr_prefill_attn_batched) \
    X(tr_prefill_attn_gather) X(tr_decode_attn) X(tr_chunk_prefill_attn) X(tr_sequence_prefill_attn) X(tr_linear)
struct Api {
#define X(name) decltype(&::name) name;
    TR_CALLS(X)
#undef X
} api;
PyObject* error_class = nullptr;    // TurboRagError(code, message)
PyObject* current_device = nullptr; // torch._C._cuda_getDevice
PyObject* current_stream = nullptr; // torch._C._cuda_getCurrentRawStream
PyObject* str_handle = nullptr;
PyObject* str_cuda_stream = nullptr;

struct Failed {}; // a Python error is set

[[noreturn]] void fail(PyObject* type, const char* msg)
{
    PyErr_SetString(type, msg);
    throw Failed();
}

// ---- readers: each throws Failed with the Python error set -----------------------------------------------------------
const at::Tensor& tensor(PyObject* o)
{
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "a torch tensor is expected");
    return THPVariable_Unpack(o);
}
const at::Tensor& device_tensor(PyObject* o)
{
    const at::Tensor& t = tensor(o);
    if (!t.is_cuda() || !t.is_contiguous()) fail(PyExc_AssertionError, "device tensors must be contiguous");
    return t;
}
template <class T = void> T* dev(PyObject* o) { return o == Py_None ? nullptr : (T*)device_tensor(o).data_ptr(); }

int64_t rows(PyObject* o)
{
    const at::Tensor& t = tensor(o);
    if (t.dim() < 1) fail(PyExc_IndexError, "tensor has no rows");
    return t.size(0);
}

int64_t integer(PyObject* o)
{
    PyObject* i = PyNumber_Index(o);
    if (!i) throw Failed();
    const long long v = PyLong_AsLongLong(i);
    Py_DECREF(i);
    if (v == -1 && PyErr_Occurred()) throw Failed();
    return v;
}
int32_t int32(PyObject* o) { return (int32_t)integer(o); }

// tr_shape and the store handle are ctypes objects, whose memory is read through the buffer protocol
void read_buffer(PyObject* o, void* to, size_t n)
{
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE)) throw Failed();
    const bool ok = (size_t)b.len == n;
    if (ok) memcpy(to, b.buf, n);
    PyBuffer_Release(&b);
    if (!ok) fail(PyExc_TypeError, "unexpected size of a ctypes argument");
}
tr_shape shape(PyObject* o)
{
    tr_shape s;
    read_buffer(o, &s, sizeof s);
    return s;
}
const tr_store* store(PyObject* o)
{
    PyObject* h = PyObject_GetAttr(o, str_handle);
    if (!h) throw Failed();
    void* p = nullptr;
    try {
        read_buffer(h, &p, sizeof p);
    } catch (const Failed&) {
        Py_DECREF(h);
        throw;
    }
    Py_DECREF(h);
    return (const tr_store*)p;
}

// A contiguous host array of int32 or int64, converted (as numpy.ascontiguousarray does) only where it is not one already.
template <class T> class Host {
public:
    explicit Host(PyObject* o)
    {
        const int type = sizeof(T) == 4 ? NPY_INT32 : NPY_INT64;
        a_ = (PyArrayObject*)PyArray_FROMANY(o, type, 0, 0, NPY_ARRAY_C_CONTIGUOUS | NPY_ARRAY_ALIGNED | NPY_ARRAY_FORCECAST);
        if (!a_) throw Failed();
    }
    ~Host() { Py_DECREF(a_); }
    Host(const Host&) = delete;
    Host& operator=(const Host&) = delete;
    T* data() const { return (T*)PyArray_DATA(a_); }
    int32_t size() const { return (int32_t)PyArray_SIZE(a_); }

private:
    PyArrayObject* a_;
};

// None: torch's current stream of the current device
void* stream(PyObject* o)
{
    PyObject* v = nullptr;
    if (o == Py_None) {
        PyObject* d = PyObject_CallNoArgs(current_device);
        if (!d) throw Failed();
        v = PyObject_CallOneArg(current_stream, d);
        Py_DECREF(d);
    } else {
        v = PyObject_GetAttr(o, str_cuda_stream);
        if (!v) {
            PyErr_Clear();
            v = PyNumber_Long(o);
        }
    }
    if (!v) throw Failed();
    void* s = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    if (!s && PyErr_Occurred()) throw Failed();
    return s;
}

struct Work {
    void* p = nullptr;
    size_t bytes = 0;
    explicit Work(PyObject* o)
    {
        if (o == Py_None) return;
        const at::Tensor& t = device_tensor(o);
        p = t.data_ptr();
        bytes = (size_t)t.numel() * t.element_size();
    }
};

// The library call runs without the interpreter lock (a full queue can make a launch wait), then its status is looked at.
// `call` holds nothing but the C call on values read before: whatever it threw would reach entry() without the lock.
template <class F> PyObject* run(F&& call)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    if (rc == TR_OK) Py_RETURN_NONE;
    PyObject* e = PyObject_CallFunction(error_class, "is", rc, api.tr_last_error());
    if (e) {
        PyErr_SetObject(error_class, e);
        Py_DECREF(e);
    }
    return nullptr;
}

typedef PyObject* const* Args;

// METH_FASTCALL entry with a fixed argument count
template <int N, PyObject* (*F)(Args)> PyObject* entry(PyObject*, Args a, Py_ssize_t n)
{
    if (!api.tr_last_error) {
        PyErr_SetString(PyExc_RuntimeError, "bind() has not been called");
        return nullptr;
    }
    if (n != N) return PyErr_Format(PyExc_TypeError, "%d arguments are expected, got %zd", N, n);
    try {
        return F(a);
    } catch (const Failed&) {
        return nullptr;
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// ---- one function per call of the C ABI; the arguments are those of binding.py, in its order --------------------------
PyObject* plan(Args a) // store, chunk_ids, pos_mode, want_pos_ids
{
    const tr_store* st = store(a[0]);
    const Host<int32_t> ids(a[1]);
    const int32_t mode = int32(a[2]);
    npy_intp n = (npy_intp)ids.size() + 1;
    PyObject* off = PyArray_SimpleNew(1, &n, NPY_INT64);
    if (!off) return nullptr;
    int64_t* o = (int64_t*)PyArray_DATA((PyArrayObject*)off);
    PyObject* ok = run([&] { return api.tr_plan(st, ids.data(), ids.size(), mode, o, nullptr, 0); });
    const int want = ok ? PyObject_IsTrue(a[3]) : 0;
    PyObject* pos = nullptr;
    if (ok && want > 0) {
        npy_intp total = (npy_intp)o[n - 1];
        pos = PyArray_SimpleNew(1, &total, NPY_INT32);
        if (pos) {
            int32_t* p = (int32_t*)PyArray_DATA((PyArrayObject*)pos);
            Py_DECREF(ok);
            ok = run([&] { return api.tr_plan(st, ids.data(), ids.size(), mode, o, p, total); });
        }
    }
    if (!ok || want < 0 || (want > 0 && !pos)) {
        Py_XDECREF(ok);
        Py_XDECREF(pos);
        Py_DECREF(off);
        return nullptr;
    }
    Py_DECREF(ok);
    if (!pos) {
        pos = Py_None;
        Py_INCREF(pos);
    }
    return Py_BuildValue("(NN)", off, pos);
}

template <bool RAW> PyObject* assemble(Args a) // store, chunk_ids, offsets, pos_mode, out_k, out_v, stream
{
    const tr_store* st = store(a[0]);
    const Host<int32_t> ids(a[1]);
    const Host<int64_t> off(a[2]);
    const int32_t mode = int32(a[3]);
    void *k = dev(a[4]), *v = dev(a[5]), *s = stream(a[6]);
    const int64_t cap = rows(a[4]);
    return run([&] { return (RAW ? api.tr_kv_assemble_raw : api.tr_kv_assemble)(st, ids.data(), off.data(), ids.size(), mode, k, v, cap, s); });
}

PyObject* assemble_batched(Args a) // store, chunk_ids, cu_chunks, pos_modes, cache_row_start, out_k, out_v, stream
{
    const tr_store* st = store(a[0]);
    const Host<int32_t> ids(a[1]), cu(a[2]), modes(a[3]);
    const Host<int64_t> start(a[4]);
    void *k = dev(a[5]), *v = dev(a[6]), *s = stream(a[7]);
    const int64_t cap = rows(a[5]);
    return run([&] { return api.tr_kv_assemble_batched(st, ids.data(), cu.data(), modes.data(), start.data(), modes.size(), k, v, cap, s); });
}

PyObject* append(Args a) // shape, k_new, v_new, q_pos, cache_k, cache_v, dst_row, stream
{
    const tr_shape sh = shape(a[0]);
    const void *k = dev(a[1]), *v = dev(a[2]);
    const int32_t* pos = dev<int32_t>(a[3]);
    void *ck = dev(a[4]), *cv = dev(a[5]);
    const int32_t n = (int32_t)rows(a[1]);
    const int64_t dst = integer(a[6]), cap = rows(a[4]);
    void* s = stream(a[7]);
    return run([&] { return api.tr_kv_append(&sh, k, v, pos, n, ck, cv, dst, cap, s); });
}

PyObject* assemble_append(Args a) // store, chunk_ids, offsets, pos_mode, k_new, v_new, q_pos, out_k, out_v, stream
{
    const tr_store* st = store(a[0]);
    const Host<int32_t> ids(a[1]);
    const Host<int64_t> off(a[2]);
    const int32_t mode = int32(a[3]);
    const void *k = dev(a[4]), *v = dev(a[5]);
    const int32_t* pos = dev<int32_t>(a[6]);
    void *ok = dev(a[7]), *ov = dev(a[8]), *s = stream(a[9]);
    const int32_t n = (int32_t)rows(a[4]);
    const int64_t cap = rows(a[7]);
    return run([&] { return api.tr_kv_assemble_append(st, ids.data(), off.data(), ids.size(), mode, k, v, pos, n, ok, ov, cap, s); });
}

PyObject* append_batched(Args a) // shape, k_new, v_new, q_pos, cu_q, cache_row_start, cache_k, cache_v, stream
{
    const tr_shape sh = shape(a[0]);
    const void *k = dev(a[1]), *v = dev(a[2]);
    const int32_t* pos = dev<int32_t>(a[3]);
    const Host<int32_t> cu(a[4]);
    const Host<int64_t> start(a[5]);
    void *ck = dev(a[6]), *cv = dev(a[7]), *s = stream(a[8]);
    const int64_t cap = rows(a[6]);
    return run([&] { return api.tr_kv_append_batched(&sh, k, v, pos, cu.data(), start.data(), cu.size() - 1, ck, cv, cap, s); });
}

PyObject* prefill(Args a) // shape, q, k, v, q_pos, kv_len, out, workspace, stream
{
    const tr_shape sh = shape(a[0]);
    const void *q = dev(a[1]), *k = dev(a[2]), *v = dev(a[3]);
    const int32_t* pos = dev<int32_t>(a[4]);
    const int32_t n = (int32_t)rows(a[1]);
    const int64_t kv_len = integer(a[5]);
    void* out = dev(a[6]);
    const Work w(a[7]);
    void* s = stream(a[8]);
    return run([&] { return api.tr_prefill_attn(&sh, q, k, v, pos, n, kv_len, out, w.p, w.bytes, s); });
}

PyObject* prefill_static(Args a) // shape, q, k, v, q_pos, kv_len, out, stream
{
    const tr_shape sh = shape(a[0]);
    const void *q = dev(a[1]), *k = dev(a[2]), *v = dev(a[3]);
    const int32_t* pos = dev<int32_t>(a[4]);
    const int32_t n = (int32_t)rows(a[1]);
    const int64_t kv_len = integer(a[5]);
    void *out = dev(a[6]), *s = stream(a[7]);
    return run([&] { return api.tr_prefill_attn_static(&sh, q, k, v, pos, n, kv_len, out, s); });
}

PyObject* prefill_batched(Args a) // shape, q, k, v, q_pos, cu_q, cache_row_start, out, workspace, stream
{
    const tr_shape sh = shape(a[0]);
    const void *q = dev(a[1]), *k = dev(a[2]), *v = dev(a[3]);
    const int32_t* pos = dev<int32_t>(a[4]);
    const Host<int32_t> cu(a[5]);
    const Host<int64_t> start(a[6]);
    void* out = dev(a[7]);
    const Work w(a[8]);
    void* s = stream(a[9]);
    return run([&] { return api.tr_prefill_attn_batched(&sh, q, k, v, pos, cu.data(), start.data(), cu.size() - 1, out, w.p, w.bytes, s); });
}

PyObject* prefill_gather(Args a) // store, chunk_ids, offsets, pos_mode, q, cache_k, cache_v, q_pos, out, workspace, stream
{
    const tr_store* st = store(a[0]);
    const Host<int32_t> ids(a[1]);
    const Host<int64_t> off(a[2]);
    const int32_t mode = int32(a[3]);
    const void *q = dev(a[4]), *ck = dev(a[5]), *cv = dev(a[6]);
    const int32_t* pos = dev<int32_t>(a[7]);
    const int32_t n = (int32_t)rows(a[4]);
    const int64_t cap = rows(a[5]);
    void* out = dev(a[8]);
    const Work w(a[9]);
    void* s = stream(a[10]);
    return run([&] { return api.tr_prefill_attn_gather(st, ids.data(), off.data(), ids.size(), mode, q, ck, cv, pos, n, cap, out, w.p, w.bytes, s); });
}

PyObject* decode(Args a) // shape, q, k, v, q_pos, cache_row_start, out, workspace, stream
{
    const tr_shape sh = shape(a[0]);
    const void *q = dev(a[1]), *k = dev(a[2]), *v = dev(a[3]);
    const int32_t* pos = dev<int32_t>(a[4]);
    const Host<int64_t> start(a[5]);
    void* out = dev(a[6]);
    const Work w(a[7]);
    void* s = stream(a[8]);
    return run([&] { return api.tr_decode_attn(&sh, q, k, v, pos, start.data(), start.size() - 1, out, w.p, w.bytes, s); });
}

PyObject* chunk_prefill(Args a) // shape, q, k, v, cu_chunk_lens, n_chunks, max_chunk_len, out, k_rot_out, workspace, stream
{
    const tr_shape sh = shape(a[0]);
    const void *q = dev(a[1]), *k = dev(a[2]), *v = dev(a[3]);
    const int32_t* cu = dev<int32_t>(a[4]);
    const int32_t n = int32(a[5]), longest = int32(a[6]);
    const int64_t total = rows(a[1]);
    void *out = dev(a[7]), *rot = dev(a[8]);
    const Work w(a[9]);
    void* s = stream(a[10]);
    return run([&] { return api.tr_chunk_prefill_attn(&sh, q, k, v, cu, n, total, longest, out, rot, w.p, w.bytes, s); });
}

PyObject* sequence_prefill(Args a) // shape, q, k, v, seg_start, pos, out, k_rot_out, seg_start_host, workspace, stream
{
    const tr_shape sh = shape(a[0]);
    const void *q = dev(a[1]), *k = dev(a[2]), *v = dev(a[3]);
    const int32_t *seg = dev<int32_t>(a[4]), *pos = dev<int32_t>(a[5]);
    const int64_t total = rows(a[1]);
    void *out = dev(a[6]), *rot = dev(a[7]);
    const Work w(a[9]);
    void* s = stream(a[10]);
    if (a[8] == Py_None)
        return run([&] { return api.tr_sequence_prefill_attn(&sh, q, k, v, seg, pos, nullptr, total, out, rot, w.p, w.bytes, s); });
    const Host<int32_t> host(a[8]);
    return run([&] { return api.tr_sequence_prefill_attn(&sh, q, k, v, seg, pos, host.data(), total, out, rot, w.p, w.bytes, s); });
}

PyObject* linear(Args a) // x, [w], [y], workspace, stream
{
    const at::Tensor& x = device_tensor(a[0]);
    if (x.dim() != 2) fail(PyExc_ValueError, "x has two dimensions");
    if (!PyList_Check(a[1]) || !PyList_Check(a[2])) fail(PyExc_TypeError, "lists of tensors are expected");
    const int64_t M = x.size(0), K = x.size(1);
    const void* xp = x.data_ptr(); // may throw, as every tensor access may: none of them inside run()
    const Py_ssize_t n = PyList_GET_SIZE(a[1]), ny = PyList_GET_SIZE(a[2]);
    std::vector<const void*> w((size_t)n);
    std::vector<void*> y((size_t)ny);
    std::vector<int32_t> f((size_t)n);
    for (Py_ssize_t j = 0; j < n; ++j) {
        const at::Tensor& t = device_tensor(PyList_GET_ITEM(a[1], j));
        if (t.dim() < 2 || t.size(1) != K) fail(PyExc_AssertionError, "w[j] has K columns");
        w[(size_t)j] = t.data_ptr();
        f[(size_t)j] = (int32_t)t.size(0);
    }
    for (Py_ssize_t j = 0; j < ny; ++j) {
        const at::Tensor& t = device_tensor(PyList_GET_ITEM(a[2], j));
        if (j < n && t.numel() != M * f[(size_t)j]) fail(PyExc_AssertionError, "y[j] holds M x n_features[j] values");
        y[(size_t)j] = t.data_ptr();
    }
    if (ny < n) fail(PyExc_AssertionError, "as many outputs as weights are expected");
    const Work ws(a[3]);
    void* s = stream(a[4]);
    return run([&] { return api.tr_linear(xp, (int32_t)M, (int32_t)K, (int32_t)n, w.data(), y.data(), f.data(), ws.p, ws.bytes, s); });
}

// addresses: dict name -> address of the library's entry point; error: the exception class for a failed call
PyObject* bind(PyObject*, PyObject* args)
{
    PyObject *addresses, *error, *device, *raw_stream;
    if (!PyArg_ParseTuple(args, "O!OOO", &PyDict_Type, &addresses, &error, &device, &raw_stream)) return nullptr;
    Api got;
#define X(name)                                                                                 \
    {                                                                                           \
        PyObject* v = PyDict_GetItemString(addresses, #name);                                   \
        if (!v) return PyErr_Format(PyExc_KeyError, "the library has no %s", #name);            \
        got.name = (decltype(got.name))PyLong_AsVoidPtr(v);                                     \
        if (!got.name) return PyErr_Format(PyExc_ValueError, "bad address of %s", #name);       \
    }
    TR_CALLS(X)
#undef X
    Py_INCREF(error);
    Py_INCREF(device);
    Py_INCREF(raw_stream);
    Py_XSETREF(error_class, error);
    Py_XSETREF(current_device, device);
    Py_XSETREF(current_stream, raw_stream);
    api = got;
    Py_RETURN_NONE;
}

#define ENTRY(name, n, f) {name, (PyCFunction)(void (*)(void))(PyObject * (*)(PyObject*, Args, Py_ssize_t)) entry<n, f>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    ENTRY("plan", 4, plan),
    ENTRY("kv_assemble", 7, assemble<false>),
    ENTRY("kv_assemble_raw", 7, assemble<true>),
    ENTRY("kv_assemble_batched", 8, assemble_batched),
    ENTRY("kv_append", 8, append),
    ENTRY("kv_assemble_append", 10, assemble_append),
    ENTRY("kv_append_batched", 9, append_batched),
    ENTRY("prefill_attn", 9, prefill),
    ENTRY("prefill_attn_static", 8, prefill_static),
    ENTRY("prefill_attn_batched", 10, prefill_batched),
    ENTRY("prefill_attn_gather", 11, prefill_gather),
    ENTRY("decode_attn", 9, decode),
    ENTRY("chunk_prefill_attn", 11, chunk_prefill),
    ENTRY("sequence_prefill_attn", 11, sequence_prefill),
    ENTRY("linear", 5, linear),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tr_host", "argument marshalling for binding.py", -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__tr_host(void)
{
    import_array();
    str_handle = PyUnicode_InternFromString("handle");
    str_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    if (!str_handle || !str_cuda_stream) return nullptr;
    return PyModule_Create(&module);
}
