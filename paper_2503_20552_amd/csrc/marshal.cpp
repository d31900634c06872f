// Argument marshalling of the binding's enqueueing calls, in native code (a CPython module).
//
// A call of the binding through ctypes spends 9 to 12 us in the interpreter taking its tensors apart,
// more than the smallest calls take on the GPU.  Each function here does the same for the plain
// case -- plain tensors of the right types and shapes, plain numbers -- and calls the C entry
// point whose address it is given.  Whatever is not plain, including everything the binding
// refuses, it leaves alone: it returns None, nothing has been enqueued, and the binding goes through
// its own checks, which raise what they raise.  Otherwise it returns the entry point's status.
//
// Nothing is kept between calls but the names of attributes and two functions of torch.
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include "../../include/adr.h"

#include <climits>

namespace {

PyObject *name_k, *name_v, *name_k_scale, *name_v_scale, *name_cuda_stream;
PyObject *get_device, *get_raw_stream;

struct NotPlain {};

void need(bool ok)
{
    if (!ok)
        throw NotPlain();
}

const at::Tensor &tensor(PyObject *o)
{
    need(THPVariable_CheckExact(o));
    const at::Tensor &t = THPVariable_Unpack(o);
    need(t.defined() && t.has_storage() && t.layout() == at::kStrided && !t.is_neg() && !t.is_conj());
    return t;
}

const at::Tensor *optional_tensor(PyObject *o) { return o == Py_None ? nullptr : &tensor(o); }

long whole(PyObject *o, long lo, long hi)
{
    need(PyLong_CheckExact(o));
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    need(!overflow && v >= lo && v <= hi);
    return v;
}

int whole_int(PyObject *o) { return (int)whole(o, INT_MIN, INT_MAX); }

float real(PyObject *o)
{
    need(PyFloat_CheckExact(o));
    return (float)PyFloat_AS_DOUBLE(o);
}

// The raw stream handle of None (torch's current stream), an int, or an object with a `cuda_stream`.
void *stream_handle(PyObject *o, const at::Tensor &on)
{
    PyObject *handle;
    if (o == Py_None) {
        need(on.is_cuda() && get_device && get_raw_stream); // (torch has set the device up, then)
        PyObject *device = PyObject_CallNoArgs(get_device);
        handle = device ? PyObject_CallOneArg(get_raw_stream, device) : nullptr;
        Py_XDECREF(device);
    } else if (PyLong_CheckExact(o)) {
        Py_INCREF(o);
        handle = o;
    } else {
        handle = PyObject_GetAttr(o, name_cuda_stream);
    }
    need(handle != nullptr);
    void *p = PyLong_Check(handle) ? PyLong_AsVoidPtr(handle) : nullptr;
    const bool ok = PyLong_Check(handle) && !PyErr_Occurred();
    Py_DECREF(handle);
    need(ok);
    return p;
}

struct Rows { // [B, heads, d] bf16, heads and d contiguous
    const void *data;
    int64_t stride, B, heads, d;
};

Rows rows_view(PyObject *o)
{
    const at::Tensor &t = tensor(o);
    need(t.scalar_type() == at::kBFloat16 && t.dim() == 3);
    Rows r = {nullptr, t.stride(0), t.size(0), t.size(1), t.size(2)};
    need(t.stride(2) == 1 && t.stride(1) == r.d);
    if (r.B <= 1)
        r.stride = std::max(r.stride, r.heads * r.d);
    need(r.B <= INT_MAX && r.heads <= INT_MAX && r.d <= INT_MAX);
    r.data = t.data_ptr();
    return r;
}

const int32_t *int_vector(const at::Tensor &t)
{
    need(t.scalar_type() == at::kInt && t.is_contiguous());
    return (const int32_t *)t.data_ptr();
}

adr_kv_cache cache_struct(PyObject *cache, PyObject *cache_type)
{
    need((PyObject *)Py_TYPE(cache) == cache_type);
    struct Field {
        PyObject *o;
        Field(PyObject *c, PyObject *name) : o(PyObject_GetAttr(c, name)) { need(o != nullptr); }
        ~Field() { Py_XDECREF(o); }
    } k(cache, name_k), v(cache, name_v), ks(cache, name_k_scale), vs(cache, name_v_scale);
    const at::Tensor &kt = tensor(k.o), &vt = tensor(v.o);
    need(kt.dim() == 4 && vt.sizes() == kt.sizes() && vt.scalar_type() == kt.scalar_type());
    need(kt.scalar_type() == at::kBFloat16 || kt.scalar_type() == at::kByte);
    need(kt.is_contiguous() && vt.is_contiguous());
    for (int i = 0; i < 4; ++i)
        need(kt.size(i) <= INT_MAX);
    adr_kv_cache c;
    c.k = kt.data_ptr();
    c.v = vt.data_ptr();
    c.num_pages = (int)kt.size(0);
    c.page_size = (int)kt.size(1);
    c.Hkv = (int)kt.size(2);
    c.d = (int)kt.size(3);
    c.dtype = kt.scalar_type() == at::kBFloat16 ? ADR_BF16 : ADR_FP8_E4M3;
    auto scale = [&](PyObject *o) -> float * {
        const at::Tensor *t = optional_tensor(o);
        if (!t)
            return nullptr;
        need(t->scalar_type() == at::kFloat && t->is_contiguous() && t->dim() == 2 && t->size(0) == kt.size(0) &&
             t->size(1) == kt.size(2));
        return (float *)t->data_ptr();
    };
    c.k_scale = scale(ks.o);
    c.v_scale = scale(vs.o);
    return c;
}

struct Output {
    void *data;
    adr_dtype dtype;
    float *lse;
};

Output output(const at::Tensor &out, PyObject *lse, int64_t B, int64_t heads, int64_t d)
{
    need(out.scalar_type() == at::kBFloat16 || out.scalar_type() == at::kFloat);
    need(out.dim() == 3 && out.size(0) == B && out.size(1) == heads && out.size(2) == d && out.is_contiguous());
    Output o = {out.data_ptr(), out.scalar_type() == at::kBFloat16 ? ADR_BF16 : ADR_F32, nullptr};
    if (const at::Tensor *t = optional_tensor(lse)) {
        need(t->scalar_type() == at::kFloat && t->dim() == 2 && t->size(0) == B && t->size(1) == heads && t->is_contiguous());
        o.lse = (float *)t->data_ptr();
    }
    return o;
}

struct Table {
    const int32_t *data;
    int width;
};

Table table(PyObject *o, int64_t B)
{
    const at::Tensor &t = tensor(o);
    need(t.dim() == 2 && t.size(0) == B && t.size(1) <= INT_MAX);
    return {int_vector(t), (int)t.size(1)};
}

const int32_t *per_row(PyObject *o, int64_t n)
{
    const at::Tensor &t = tensor(o);
    need(t.dim() == 1 && t.size(0) == n);
    return int_vector(t);
}

struct Space {
    void *data;
    size_t bytes;
};

Space workspace(PyObject *o)
{
    const at::Tensor *t = optional_tensor(o);
    if (!t)
        return {nullptr, 0};
    return {t->data_ptr(), (size_t)t->numel() * t->element_size()};
}

// Runs `body`, which checks and then calls; the interpreter lock is given up around the C call alone.
template <class Body> PyObject *guarded(PyObject *const *args, Py_ssize_t n, Py_ssize_t expected, Body body)
{
    if (n != expected) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    try {
        return PyLong_FromLong(body(args));
    } catch (const NotPlain &) {
    } catch (const std::exception &) {
    }
    PyErr_Clear();
    Py_RETURN_NONE;
}

template <class Fn> Fn *entry(PyObject *address) { return (Fn *)PyLong_AsVoidPtr(address); }

#define ADR_WITHOUT_LOCK(CALL)                                                                     \
    int status;                                                                                   \
    Py_BEGIN_ALLOW_THREADS status = (CALL);                                                       \
    Py_END_ALLOW_THREADS return status

// (address, KVCache, out, q, cache, block_table, seq_lens, scale, max_seq_len, partition_tokens, workspace, lse,
//  flags, stream)
PyObject *decode_attention(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded(args, n, 14, [](PyObject *const *a) -> int {
        const Rows q = rows_view(a[3]);
        const at::Tensor &out = tensor(a[2]);
        const Output o = output(out, a[11], q.B, q.heads, q.d);
        const adr_kv_cache cache = cache_struct(a[4], a[1]);
        const Table t = table(a[5], q.B);
        const int32_t *lens = per_row(a[6], q.B);
        const float scale = real(a[7]);
        const int bound = whole_int(a[8]), part = whole_int(a[9]);
        const Space ws = workspace(a[10]);
        const unsigned flags = (unsigned)whole(a[12], 0, UINT_MAX);
        void *stream = stream_handle(a[13], out);
        auto *fn = entry<decltype(adr_decode_attention)>(a[0]);
        ADR_WITHOUT_LOCK(fn(o.data, o.dtype, o.lse, q.data, q.stride, &cache, t.data, t.width, lens, (int)q.B, (int)q.heads,
                            scale, bound, part, ws.data, ws.bytes, flags, stream));
    });
}

// (address, KVCache, out, q, k_new, v_new, cache, block_table, seq_lens, scale, max_seq_len, partition_tokens,
//  workspace, lse, flags, stream)
PyObject *decode_step(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded(args, n, 16, [](PyObject *const *a) -> int {
        const Rows q = rows_view(a[3]), k = rows_view(a[4]), v = rows_view(a[5]);
        const at::Tensor &out = tensor(a[2]);
        const Output o = output(out, a[13], q.B, q.heads, q.d);
        need(k.stride == v.stride && k.B == q.B && v.B == q.B);
        const adr_kv_cache cache = cache_struct(a[6], a[1]);
        const Table t = table(a[7], q.B);
        const int32_t *lens = per_row(a[8], q.B);
        const float scale = real(a[9]);
        const int bound = whole_int(a[10]), part = whole_int(a[11]);
        const Space ws = workspace(a[12]);
        const unsigned flags = (unsigned)whole(a[14], 0, UINT_MAX);
        void *stream = stream_handle(a[15], out);
        auto *fn = entry<decltype(adr_decode_step)>(a[0]);
        ADR_WITHOUT_LOCK(fn(o.data, o.dtype, o.lse, q.data, q.stride, k.data, v.data, k.stride, &cache, t.data, t.width,
                            lens, (int)q.B, (int)q.heads, scale, bound, part, ws.data, ws.bytes, flags, stream));
    });
}

// (address, KVCache, cache, k_new, v_new, block_table, positions, stream)
PyObject *kv_append(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded(args, n, 8, [](PyObject *const *a) -> int {
        const adr_kv_cache cache = cache_struct(a[2], a[1]);
        const Rows k = rows_view(a[3]), v = rows_view(a[4]);
        need(k.stride == v.stride);
        const Table t = table(a[5], k.B);
        const int32_t *positions = per_row(a[6], k.B);
        void *stream = stream_handle(a[7], tensor(a[3]));
        auto *fn = entry<decltype(adr_kv_append)>(a[0]);
        ADR_WITHOUT_LOCK(fn(&cache, k.data, v.data, k.stride, t.data, t.width, positions, (int)k.B, stream));
    });
}

// (address, out, part_o, part_lse, part_offsets, lse_out, stream)
PyObject *lse_merge(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded(args, n, 7, [](PyObject *const *a) -> int {
        const at::Tensor &out = tensor(a[1]), &part_o = tensor(a[2]), &part_lse = tensor(a[3]);
        need(out.dim() == 3);
        const int64_t B = out.size(0), heads = out.size(1), d = out.size(2);
        need(B < INT_MAX && heads <= INT_MAX && d <= INT_MAX);
        const Output o = output(out, Py_None, B, heads, d);
        float *lse = nullptr;
        if (const at::Tensor *t = optional_tensor(a[5]))
            lse = (float *)t->data_ptr(); // (the binding takes any tensor here)
        need(part_o.scalar_type() == at::kFloat && part_lse.scalar_type() == at::kFloat);
        need(part_o.is_contiguous() && part_lse.is_contiguous() && part_o.dim() == 3 && part_o.size(1) == heads &&
             part_o.size(2) == d && part_lse.dim() == 2 && part_lse.size(0) == part_o.size(0) && part_lse.size(1) == heads);
        const int32_t *offsets = per_row(a[4], B + 1);
        void *stream = stream_handle(a[6], out);
        const float *po = (const float *)part_o.data_ptr(), *pl = (const float *)part_lse.data_ptr();
        auto *fn = entry<decltype(adr_lse_merge)>(a[0]);
        ADR_WITHOUT_LOCK(fn(o.data, o.dtype, lse, po, pl, offsets, (int)B, (int)heads, (int)d, stream));
    });
}

// (address, dst, q, k, v, stream)
PyObject *pack_qkv(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded(args, n, 6, [](PyObject *const *a) -> int {
        const at::Tensor &dst = tensor(a[1]);
        const Rows q = rows_view(a[2]), k = rows_view(a[3]), v = rows_view(a[4]);
        need(dst.scalar_type() == at::kBFloat16 && dst.dim() == 2 && dst.size(0) == q.B && dst.stride(1) == 1);
        need(k.B == q.B && k.d == q.d && v.B == k.B && v.heads == k.heads && v.d == k.d &&
             dst.size(1) >= (q.heads + 2 * k.heads) * q.d);
        void *stream = stream_handle(a[5], dst);
        void *p = dst.data_ptr();
        auto *fn = entry<decltype(adr_pack_qkv)>(a[0]);
        ADR_WITHOUT_LOCK(fn(p, dst.stride(0), q.data, q.stride, k.data, k.stride, v.data, v.stride, (int)q.B, (int)q.heads,
                            (int)k.heads, (int)q.d, stream));
    });
}

// (address, dst, src, row_index, stream)
PyObject *scatter_rows(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    return guarded(args, n, 5, [](PyObject *const *a) -> int {
        const at::Tensor &dst = tensor(a[1]), &src = tensor(a[2]), &index = tensor(a[3]);
        for (const at::Tensor *t : {&dst, &src})
            need(t->scalar_type() == at::kBFloat16 && t->dim() == 2 && t->stride(1) == 1 && t->size(0) <= INT_MAX &&
                 t->size(1) <= INT_MAX);
        need(dst.size(1) == src.size(1) && index.scalar_type() == at::kInt && index.numel() == src.size(0));
        void *stream = stream_handle(a[4], dst);
        void *to = dst.data_ptr();
        const void *from = src.data_ptr();
        const int32_t *rows = (const int32_t *)index.data_ptr();
        auto *fn = entry<decltype(adr_scatter_rows)>(a[0]);
        ADR_WITHOUT_LOCK(fn(to, dst.stride(0), (int)dst.size(0), from, src.stride(0), rows, (int)src.size(0),
                            (int)src.size(1), stream));
    });
}

PyMethodDef methods[] = {
    {"decode_attention", (PyCFunction)(void (*)(void))decode_attention, METH_FASTCALL, nullptr},
    {"decode_step", (PyCFunction)(void (*)(void))decode_step, METH_FASTCALL, nullptr},
    {"kv_append", (PyCFunction)(void (*)(void))kv_append, METH_FASTCALL, nullptr},
    {"lse_merge", (PyCFunction)(void (*)(void))lse_merge, METH_FASTCALL, nullptr},
    {"pack_qkv", (PyCFunction)(void (*)(void))pack_qkv, METH_FASTCALL, nullptr},
    {"scatter_rows", (PyCFunction)(void (*)(void))scatter_rows, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__marshal()
{
    name_k = PyUnicode_InternFromString("k");
    name_v = PyUnicode_InternFromString("v");
    name_k_scale = PyUnicode_InternFromString("k_scale");
    name_v_scale = PyUnicode_InternFromString("v_scale");
    name_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    PyObject *torch_c = PyImport_ImportModule("torch._C");
    if (!torch_c)
        return nullptr;
    get_device = PyObject_GetAttrString(torch_c, "_cuda_getDevice"); // (a torch without them: such calls are left alone)
    get_raw_stream = PyObject_GetAttrString(torch_c, "_cuda_getCurrentRawStream");
    PyErr_Clear();
    Py_DECREF(torch_c);
    PyObject *m = PyModule_Create(&module);
    // What it was built for: the binding leaves it aside under any other Python or torch.
    if (m && PyModule_AddStringConstant(m, "built_for", ADR_BUILT_FOR) != 0)
        Py_CLEAR(m);
    return m;
}
