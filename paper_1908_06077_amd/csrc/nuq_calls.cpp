// The library's launching calls from Python without ctypes: tensors are looked at and their addresses gathered in C++, then
// the C entry point of include/nuq.h is called on the current stream.  A step on some ten thousand coordinates is bound by
// this work: 17 to 25 tensors per call, half a microsecond each in Python.  Step on 4 x 65 537 coordinates 38.7 -> 18.9 us,
// decode of as many 15.8 -> 8.0, encode of 8 x 65 537 28.9 -> 11.5.
//
// Every function returns the entry point's code, or None for anything but the plain case: another type of object, a tensor
// of another type, size or placement, a number out of range.  The caller (binding.py) then goes through its own checks,
// which raise what they always raised or accept what they always accepted.  Nothing is launched before that is decided.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/TensorSubclassLikeUtils.h>
#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include <array>

#include "../../include/nuq.h"

namespace {

constexpr uint64_t kMax = 32;       // workers per call (NUQ_MAX_WORKERS)

PyObject *g_get_device, *g_raw_stream;                              // torch._C._cuda_getDevice, _cuda_getCurrentRawStream
PyObject *g_norms, *g_bit_off, *g_words, *g_sync;                   // attribute names

// libnuq.so's entry points, in the order of `bind`'s argument.
#define NUQ_CALLS(X)                                                                                                  \
    X(nuq_num_buckets) X(nuq_num_sync) X(nuq_huffman_num_sync) X(nuq_fixed_words) X(nuq_quantize_encode_batch)       \
    X(nuq_decode_accumulate) X(nuq_decode_momentum_step) X(nuq_quantize_encode_table_batch)                          \
    X(nuq_decode_accumulate_table) X(nuq_quantize_pack_fixed_batch) X(nuq_unpack_accumulate_fixed)                   \
    X(nuq_quantize_pack_fixed_table_batch) X(nuq_unpack_accumulate_fixed_table)                                      \
    X(nuq_quantize_encode_huffman_batch) X(nuq_decode_accumulate_huffman) X(nuq_moments_accumulate)
#define NUQ_POINTER(name) decltype(&::name) p_##name = nullptr;
NUQ_CALLS(NUQ_POINTER)

struct NotPlain {};       // thrown by what follows; becomes None

void need(bool ok)
{
    if (!ok)
        throw NotPlain{};
}

uint64_t whole(PyObject *o, uint64_t top)
{
    need(PyLong_CheckExact(o));
    const unsigned long long x = PyLong_AsUnsignedLongLong(o);
    need(!PyErr_Occurred() && x <= top);
    return x;
}
uint32_t u32(PyObject *o) { return (uint32_t)whole(o, UINT32_MAX); }

double real(PyObject *o)
{
    need(PyFloat_CheckExact(o) || PyLong_CheckExact(o));
    const double x = PyFloat_AsDouble(o);
    need(!PyErr_Occurred());
    return x;
}

int truth(PyObject *o)
{
    need(PyBool_Check(o));
    return o == Py_True ? 1 : 0;
}

// A list or tuple of at most kMax things (its items are borrowed).
struct Items {
    PyObject *seq;
    uint64_t n;
    explicit Items(PyObject *o, uint64_t least = 1, uint64_t most = kMax) : seq(o)
    {
        need(PyList_CheckExact(o) || PyTuple_CheckExact(o));
        n = (uint64_t)PySequence_Fast_GET_SIZE(o);
        need(n >= least && n <= most);
    }
    PyObject *operator[](uint64_t i) const { return PySequence_Fast_GET_ITEM(seq, (Py_ssize_t)i); }
};

const at::Tensor &device_tensor(PyObject *o)
{
    need(THPVariable_CheckExact(o));
    const at::Tensor &t = THPVariable_Unpack(o);
    need(t.is_cuda() && t.layout() == at::kStrided && t.is_contiguous() && t.has_storage() && !at::isTensorSubclassLike(t));
    return t;
}

template <class T>
T *address(PyObject *o, at::ScalarType type, uint64_t least = 0, uint64_t *numel = nullptr)
{
    const at::Tensor &t = device_tensor(o);
    need(t.scalar_type() == type && (uint64_t)t.numel() >= least);
    if (numel)
        *numel = (uint64_t)t.numel();
    return static_cast<T *>(t.data_ptr());
}
template <class T>
T *exactly(PyObject *o, at::ScalarType type, uint64_t n)
{
    uint64_t have;
    T *p = address<T>(o, type, 0, &have);
    need(have == n);
    return p;
}

struct Bytes {
    void *p;
    uint64_t n;
    explicit Bytes(PyObject *o)
    {
        const at::Tensor &t = device_tensor(o);
        p = t.data_ptr();
        n = (uint64_t)t.numel() * t.element_size();
    }
};

template <class T>
using Array = std::array<T, kMax>;

// K gradients of one length.
struct Gradients {
    Array<const float *> v;
    uint64_t K, d;
    explicit Gradients(PyObject *o)
    {
        const Items items(o);
        K = items.n;
        for (uint64_t k = 0; k < K; ++k) {
            uint64_t n;
            v[k] = address<const float>(items[k], at::kFloat, 0, &n);
            need(k == 0 || n == d);
            d = n;
        }
    }
};

struct Seeds {
    Array<uint64_t> x;
    Seeds(PyObject *o, uint64_t K)
    {
        const Items items(o);
        need(items.n == K);
        for (uint64_t k = 0; k < K; ++k) {
            need(PyLong_CheckExact(items[k]));
            x[k] = PyLong_AsUnsignedLongLongMask(items[k]);       // modulo 2^64
        }
    }
};

template <class T>
struct Tensors {
    Array<T *> p;
    Tensors(PyObject *o, uint64_t K, at::ScalarType type, uint64_t least)
    {
        const Items items(o);
        need(items.n == K);
        for (uint64_t k = 0; k < K; ++k)
            p[k] = address<T>(items[k], type, least);
    }
};

// K messages.  sized: every array is looked at for the size that d, bucket and the stride imply.
struct Messages {
    Array<float *> norms;
    Array<uint64_t *> bit_off;
    Array<uint32_t *> words, sync;
    Array<uint64_t> len;
    uint64_t K;
    Messages(PyObject *o, uint64_t d, uint32_t bucket, uint32_t stride, bool huffman = false, bool sized = true)
    {
        const Items items(o);
        K = items.n;
        need(bucket > 0);
        const uint64_t B = p_nuq_num_buckets(d, bucket);
        const uint64_t nsync = B * (huffman ? p_nuq_huffman_num_sync : p_nuq_num_sync)(bucket, stride);
        for (uint64_t k = 0; k < K; ++k) {
            norms[k] = field<float>(items[k], g_norms, at::kFloat, sized ? B : 0, nullptr);
            bit_off[k] = field<uint64_t>(items[k], g_bit_off, at::kLong, sized ? B + 1 : 0, nullptr);
            words[k] = field<uint32_t>(items[k], g_words, at::kInt, 0, &len[k]);
            sync[k] = field<uint32_t>(items[k], g_sync, at::kInt, sized ? nsync : 0, nullptr);
        }
    }
    template <class T>
    static T *field(PyObject *m, PyObject *name, at::ScalarType type, uint64_t least, uint64_t *numel)
    {
        PyObject *o = PyObject_GetAttr(m, name);
        need(o != nullptr);
        struct Release {
            PyObject *o;
            ~Release() { Py_DECREF(o); }               // (the message holds the tensor)
        } release{o};
        if (o == Py_None && !least && !numel)
            return nullptr;
        return address<T>(o, type, least, numel);
    }
};

struct Levels {
    std::array<float, 16> x;
    uint32_t s;
    explicit Levels(PyObject *o)
    {
        const Items items(o, 3, 16);
        s = (uint32_t)items.n - 2u;
        for (uint64_t j = 0; j < items.n; ++j)
            x[j] = (float)real(items[j]);
    }
};

struct Lengths {
    std::array<uint8_t, 16> x;
    Lengths(PyObject *o, uint32_t s)
    {
        const Items items(o, 3, 16);
        need(items.n == (uint64_t)s + 2u);
        for (uint64_t j = 0; j < items.n; ++j)
            x[j] = (uint8_t)whole(items[j], 255);
    }
};

// The current stream of the current device, as torch.cuda.current_stream().
nuq_stream_t stream()
{
    PyObject *dev = PyObject_CallNoArgs(g_get_device);
    need(dev != nullptr);
    PyObject *raw = PyObject_CallOneArg(g_raw_stream, dev);
    Py_DECREF(dev);
    need(raw != nullptr);
    void *p = PyLong_AsVoidPtr(raw);
    Py_DECREF(raw);
    need(!PyErr_Occurred());
    return p;
}

template <class F, class... A>
PyObject *launch(F f, A... args)
{
    const nuq_stream_t st = stream();
    int code;
    Py_BEGIN_ALLOW_THREADS
    code = f(args..., st);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(code);
}

// A METH_FASTCALL function of n arguments from a body that takes them.
template <Py_ssize_t n, PyObject *(*body)(PyObject *const *)>
PyObject *entry(PyObject *, PyObject *const *a, Py_ssize_t got)
{
    try {
        need(got == n);
        return body(a);
    } catch (...) {                     // NotPlain, or what a tensor's method throws
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

PyObject *quantize_encode_batch(PyObject *const *a)      // vs, bucket, s, seeds, stride, messages, workspace
{
    const Gradients g(a[0]);
    const uint32_t bucket = u32(a[1]), s = u32(a[2]), stride = u32(a[4]);
    const Seeds seeds(a[3], g.K);
    const Messages m(a[5], g.d, bucket, stride);
    need(m.K == g.K);
    const Bytes ws(a[6]);
    return launch(p_nuq_quantize_encode_batch, (uint32_t)g.K, g.v.data(), seeds.x.data(), g.d, bucket, s, stride, m.norms.data(),
                  m.bit_off.data(), m.words.data(), m.len.data(), m.sync.data(), ws.p, ws.n);
}

PyObject *decode_accumulate(PyObject *const *a)          // messages, d, bucket, s, stride, scale, accumulate, out
{
    const uint64_t d = whole(a[1], UINT64_MAX);
    const uint32_t bucket = u32(a[2]), s = u32(a[3]), stride = u32(a[4]);
    const Messages m(a[0], d, bucket, stride);
    float *out = exactly<float>(a[7], at::kFloat, d);
    return launch(p_nuq_decode_accumulate, (uint32_t)m.K, m.norms.data(), m.bit_off.data(), m.words.data(), m.len.data(),
                  m.sync.data(), d, bucket, s, stride, (float)real(a[5]), truth(a[6]), out);
}

PyObject *decode_momentum_step(PyObject *const *a)       // messages, d, bucket, s, stride, scale, alpha, mu, l, w, yl
{
    const uint64_t d = whole(a[1], UINT64_MAX);
    const uint32_t bucket = u32(a[2]), s = u32(a[3]), stride = u32(a[4]);
    const Messages m(a[0], d, bucket, stride);
    float *w = exactly<float>(a[9], at::kFloat, d), *yl = exactly<float>(a[10], at::kFloat, d);
    return launch(p_nuq_decode_momentum_step, (uint32_t)m.K, m.norms.data(), m.bit_off.data(), m.words.data(), m.len.data(),
                  m.sync.data(), d, bucket, s, stride, (float)real(a[5]), (float)real(a[6]), (float)real(a[7]),
                  (float)real(a[8]), w, yl);
}

PyObject *quantize_encode_table_batch(PyObject *const *a)    // vs, bucket, levels, norm_kind, seeds, stride, messages, workspace
{
    const Gradients g(a[0]);
    const uint32_t bucket = u32(a[1]), kind = u32(a[3]), stride = u32(a[5]);
    const Levels lev(a[2]);
    const Seeds seeds(a[4], g.K);
    const Messages m(a[6], g.d, bucket, stride);
    need(m.K == g.K);
    const Bytes ws(a[7]);
    return launch(p_nuq_quantize_encode_table_batch, (uint32_t)g.K, g.v.data(), seeds.x.data(), g.d, bucket, lev.s, lev.x.data(),
                  kind, stride, m.norms.data(), m.bit_off.data(), m.words.data(), m.len.data(), m.sync.data(), ws.p, ws.n);
}

PyObject *decode_accumulate_table(PyObject *const *a)    // messages, d, bucket, levels, stride, scale, accumulate, out
{
    const uint64_t d = whole(a[1], UINT64_MAX);
    const uint32_t bucket = u32(a[2]), stride = u32(a[4]);
    const Levels lev(a[3]);
    const Messages m(a[0], d, bucket, stride);
    float *out = exactly<float>(a[7], at::kFloat, d);
    return launch(p_nuq_decode_accumulate_table, (uint32_t)m.K, m.norms.data(), m.bit_off.data(), m.words.data(), m.len.data(),
                  m.sync.data(), d, bucket, lev.s, stride, lev.x.data(), (float)real(a[5]), truth(a[6]), out);
}

PyObject *quantize_pack_fixed_batch(PyObject *const *a)  // vs, bucket, s, b, seeds, norms, packed
{
    const Gradients g(a[0]);
    const uint32_t bucket = u32(a[1]), s = u32(a[2]), b = u32(a[3]);
    const Seeds seeds(a[4], g.K);
    const Tensors<float> norms(a[5], g.K, at::kFloat, 0);
    const Tensors<uint32_t> packed(a[6], g.K, at::kInt, 0);
    return launch(p_nuq_quantize_pack_fixed_batch, (uint32_t)g.K, g.v.data(), seeds.x.data(), g.d, bucket, s, b, norms.p.data(),
                  packed.p.data());
}

PyObject *unpack_accumulate_fixed(PyObject *const *a)    // norms, packed, d, bucket, s, b, scale, accumulate, out
{
    const uint64_t K = Items(a[0]).n, d = whole(a[2], UINT64_MAX);
    const Tensors<const float> norms(a[0], K, at::kFloat, 0);
    const Tensors<const uint32_t> packed(a[1], K, at::kInt, 0);
    float *out = exactly<float>(a[8], at::kFloat, d);
    return launch(p_nuq_unpack_accumulate_fixed, (uint32_t)K, norms.p.data(), packed.p.data(), d, u32(a[3]), u32(a[4]), u32(a[5]),
                  (float)real(a[6]), truth(a[7]), out);
}

PyObject *quantize_pack_fixed_table_batch(PyObject *const *a)    // vs, bucket, levels, norm_kind, b, seeds, norms, packed
{
    const Gradients g(a[0]);
    const uint32_t bucket = u32(a[1]), kind = u32(a[3]), b = u32(a[4]);
    const Levels lev(a[2]);
    const Seeds seeds(a[5], g.K);
    need(bucket > 0);
    const Tensors<float> norms(a[6], g.K, at::kFloat, p_nuq_num_buckets(g.d, bucket));
    const Tensors<uint32_t> packed(a[7], g.K, at::kInt, p_nuq_fixed_words(g.d, bucket, b));
    return launch(p_nuq_quantize_pack_fixed_table_batch, (uint32_t)g.K, g.v.data(), seeds.x.data(), g.d, bucket, lev.s,
                  lev.x.data(), kind, b, norms.p.data(), packed.p.data());
}

PyObject *unpack_accumulate_fixed_table(PyObject *const *a)      // norms, packed, d, bucket, levels, b, scale, accumulate, out
{
    const uint64_t K = Items(a[0]).n, d = whole(a[2], UINT64_MAX);
    const uint32_t bucket = u32(a[3]), b = u32(a[5]);
    const Levels lev(a[4]);
    need(bucket > 0);
    const Tensors<const float> norms(a[0], K, at::kFloat, p_nuq_num_buckets(d, bucket));
    const Tensors<const uint32_t> packed(a[1], K, at::kInt, p_nuq_fixed_words(d, bucket, b));
    float *out = exactly<float>(a[8], at::kFloat, d);
    return launch(p_nuq_unpack_accumulate_fixed_table, (uint32_t)K, norms.p.data(), packed.p.data(), d, bucket, lev.s,
                  lev.x.data(), b, (float)real(a[6]), truth(a[7]), out);
}

PyObject *quantize_encode_huffman_batch(PyObject *const *a)      // vs, bucket, s, seeds, stride, lengths, messages, workspace
{
    const Gradients g(a[0]);
    const uint32_t bucket = u32(a[1]), s = u32(a[2]), stride = u32(a[4]);
    const Seeds seeds(a[3], g.K);
    const Lengths len(a[5], s);
    const Messages m(a[6], g.d, bucket, stride, true, false);
    need(m.K == g.K);
    const Bytes ws(a[7]);
    return launch(p_nuq_quantize_encode_huffman_batch, (uint32_t)g.K, g.v.data(), seeds.x.data(), g.d, bucket, s, stride,
                  len.x.data(), m.norms.data(), m.bit_off.data(), m.words.data(), m.len.data(), m.sync.data(), ws.p, ws.n);
}

PyObject *decode_accumulate_huffman(PyObject *const *a)  // messages, d, bucket, s, stride, lengths, scale, accumulate, out
{
    const uint64_t d = whole(a[1], UINT64_MAX);
    const uint32_t bucket = u32(a[2]), s = u32(a[3]), stride = u32(a[4]);
    const Lengths len(a[5], s);
    const Messages m(a[0], d, bucket, stride, true);
    float *out = exactly<float>(a[8], at::kFloat, d);
    return launch(p_nuq_decode_accumulate_huffman, (uint32_t)m.K, m.norms.data(), m.bit_off.data(), m.words.data(), m.len.data(),
                  m.sync.data(), d, bucket, s, stride, len.x.data(), (float)real(a[6]), truth(a[7]), out);
}

PyObject *moments_accumulate(PyObject *const *a)         // g, total, total_sq
{
    uint64_t d;
    const float *g = address<const float>(a[0], at::kFloat, 0, &d);
    double *total = exactly<double>(a[1], at::kDouble, d), *total_sq = exactly<double>(a[2], at::kDouble, d);
    return launch(p_nuq_moments_accumulate, g, total, total_sq, d);
}

// bind(addresses of the entry points in NUQ_CALLS' order, torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream)
PyObject *bind(PyObject *, PyObject *args)
{
    PyObject *addresses, *get_device, *raw_stream;
    if (!PyArg_ParseTuple(args, "O!OO", &PyTuple_Type, &addresses, &get_device, &raw_stream))
        return nullptr;
    Py_ssize_t i = 0;
#define NUQ_BIND(name)                                                                                                \
    if (i >= PyTuple_GET_SIZE(addresses)) {                                                                           \
        PyErr_SetString(PyExc_ValueError, "an address per entry point");                                              \
        return nullptr;                                                                                               \
    }                                                                                                                 \
    p_##name = reinterpret_cast<decltype(p_##name)>(PyLong_AsVoidPtr(PyTuple_GET_ITEM(addresses, i++)));              \
    if (PyErr_Occurred())                                                                                             \
        return nullptr;
    NUQ_CALLS(NUQ_BIND)
    Py_INCREF(get_device);
    Py_INCREF(raw_stream);
    g_get_device = get_device;
    g_raw_stream = raw_stream;
    Py_RETURN_NONE;
}

PyObject *names(PyObject *, PyObject *)
{
#define NUQ_NAME(name) "s"
    return Py_BuildValue("(" NUQ_CALLS(NUQ_NAME) ")"
#undef NUQ_NAME
#define NUQ_NAME(name) , #name
                         NUQ_CALLS(NUQ_NAME));
}

#define NUQ_METHOD(name, n) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(&entry<n, name>)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    {"names", names, METH_NOARGS, nullptr},
    NUQ_METHOD(quantize_encode_batch, 7),
    NUQ_METHOD(decode_accumulate, 8),
    NUQ_METHOD(decode_momentum_step, 11),
    NUQ_METHOD(quantize_encode_table_batch, 8),
    NUQ_METHOD(decode_accumulate_table, 8),
    NUQ_METHOD(quantize_pack_fixed_batch, 7),
    NUQ_METHOD(unpack_accumulate_fixed, 9),
    NUQ_METHOD(quantize_pack_fixed_table_batch, 8),
    NUQ_METHOD(unpack_accumulate_fixed_table, 9),
    NUQ_METHOD(quantize_encode_huffman_batch, 8),
    NUQ_METHOD(decode_accumulate_huffman, 9),
    NUQ_METHOD(moments_accumulate, 3),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_nuq_calls", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__nuq_calls()
{
    g_norms = PyUnicode_InternFromString("norms");
    g_bit_off = PyUnicode_InternFromString("bit_off");
    g_words = PyUnicode_InternFromString("words");
    g_sync = PyUnicode_InternFromString("sync");
    if (!g_norms || !g_bit_off || !g_words || !g_sync)
        return nullptr;
    PyObject *m = PyModule_Create(&g_module);
    if (m && (PyModule_AddObject(m, "header_key", PyLong_FromUnsignedLongLong(NUQ_HEADER_KEY)) ||      // see build.py
              PyModule_AddStringConstant(m, "torch_version", NUQ_TORCH_VERSION)))
        Py_CLEAR(m);
    return m;
}
