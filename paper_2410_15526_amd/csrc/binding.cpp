// binding.cpp -- native argument marshalling of the Python binding.
//
// What a small call costs is its way from Python to the launch, several
// times the kernel.  Each function here takes the arguments of the Python
// function of the same name, checks its tensors as that function does (on a
// GPU, contiguous, holding the bytes the call touches), and calls the C
// entry point on torch's current stream.  It returns the status, or None for
// anything out of the ordinary -- an argument of another kind, a failed
// check -- without having called: the Python function then takes its own,
// general path, which handles or reports it.  (us per queued call on 10^4
// elements, Python's path and this: encode 8.9-10.7 and 3.4, dequantize-reduce
// with 8 peers 17.5 and 4.0, of which the HIP launch itself is 2.3.)
#include "sdp4.h"

#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <exception>

namespace {

struct Entry {
    decltype(&sdp4_qwd_encode) qwd_encode;
    decltype(&sdp4_qwd_decode) qwd_decode;
    decltype(&sdp4_qwd_encode_sym) qwd_encode_sym;
    decltype(&sdp4_qwd_decode_sym) qwd_decode_sym;
    decltype(&sdp4_grad_quant) grad_quant;
    decltype(&sdp4_grad_quant_sr) grad_quant_sr;
    decltype(&sdp4_dequant_reduce) dequant_reduce;
    decltype(&sdp4_dequant_reduce_sr) dequant_reduce_sr;
} lib; // set once by bind()

// Arguments of one call; `ok` turns false at the first that is not ordinary.
struct Args {
    bool ok = true;

    // n or a tensor's element count in its place
    int64_t count(PyObject *n, PyObject *of)
    {
        if (n != Py_None)
            return integer(n, 0, SDP4_MAX_ELEMENTS);
        const at::Tensor *t = tensor(of);
        return t ? t->numel() : 0;
    }
    int64_t integer(PyObject *o, int64_t lo, int64_t hi)
    {
        if (!PyLong_CheckExact(o)) {
            ok = false;
            return 0;
        }
        int over = 0;
        const int64_t v = PyLong_AsLongLongAndOverflow(o, &over);
        if (over || v < lo || v > hi)
            ok = false;
        return ok ? v : 0;
    }
    uint64_t bits64(PyObject *o)
    {
        if (!PyLong_CheckExact(o)) {
            ok = false;
            return 0;
        }
        return PyLong_AsUnsignedLongLongMask(o);
    }
    const at::Tensor *tensor(PyObject *o)
    {
        if (!THPVariable_CheckExact(o)) {
            ok = false;
            return nullptr;
        }
        const at::Tensor &t = THPVariable_Unpack(o);
        if (!t.is_cuda() || !t.has_storage() || !t.is_contiguous()) {
            ok = false;
            return nullptr;
        }
        return &t;
    }
    // address of an array of at least `bytes`: a tensor, or an address whose size is the caller's
    void *array(PyObject *o, int64_t bytes)
    {
        if (PyLong_CheckExact(o)) {
            void *p = PyLong_AsVoidPtr(o);
            if (!p && PyErr_Occurred()) {
                PyErr_Clear();
                ok = false;
            }
            return p;
        }
        const at::Tensor *t = tensor(o);
        if (!t)
            return nullptr;
        if ((int64_t)t->nbytes() < bytes) {
            ok = false;
            return nullptr;
        }
        return t->data_ptr();
    }
    void *optional_array(PyObject *o, int64_t bytes) { return o == Py_None ? nullptr : array(o, bytes); }
    // model weights: address and element type
    void *weights(PyObject *o, int64_t n, int &dtype)
    {
        const at::Tensor *t = tensor(o);
        if (!t)
            return nullptr;
        const at::ScalarType s = t->scalar_type();
        if (s == at::kFloat)
            dtype = SDP4_F32;
        else if (s == at::kBFloat16 || s == at::kShort || s == at::kUInt16)
            dtype = SDP4_BF16;
        else
            ok = false;
        return ok ? array(o, (dtype == SDP4_F32 ? 4 : 2) * n) : nullptr;
    }
    // P arrays of a list or tuple; at most SDP4_MAX_PEERS of them here
    template <class T>
    int arrays(PyObject *o, int64_t bytes, T **p)
    {
        const bool list = PyList_CheckExact(o);
        if (!list && !PyTuple_CheckExact(o)) {
            ok = false;
            return 0;
        }
        const Py_ssize_t count = list ? PyList_GET_SIZE(o) : PyTuple_GET_SIZE(o);
        if (count > SDP4_MAX_PEERS) {
            ok = false;
            return 0;
        }
        for (Py_ssize_t i = 0; ok && i < count; ++i)
            p[i] = static_cast<T *>(array(list ? PyList_GET_ITEM(o, i) : PyTuple_GET_ITEM(o, i), bytes));
        return (int)count;
    }
    // None (torch's current stream), a stream's address, or a torch stream
    void *stream(PyObject *o)
    {
        if (!ok)
            return nullptr;
        if (o == Py_None)
            return c10::hip::getCurrentHIPStream().stream();
        if (PyLong_CheckExact(o))
            return array(o, 0);
        PyObject *address = PyObject_GetAttrString(o, "cuda_stream");
        void *p = nullptr;
        if (address && PyLong_CheckExact(address))
            p = array(address, 0);
        else
            ok = false;
        PyErr_Clear();
        Py_XDECREF(address);
        return p;
    }
};

int64_t headers(int64_t n, int64_t group) // bytes of the group headers; 0 for a group the library will reject
{
    return group > 0 && (group & (group - 1)) == 0 ? 4 * (n / group) : 0;
}

// One call: `body(args, a)` reads the arguments and, if they are all ordinary, returns a
// callable that makes the call (without the interpreter lock: a launch may wait for the queue).
template <class F>
PyObject *run(bool bound, Py_ssize_t given, Py_ssize_t wanted, F body)
{
    if (!bound || given != wanted)
        Py_RETURN_NONE;
    int rc = 0;
    try {
        Args a;
        auto call = body(a);
        if (!a.ok)
            Py_RETURN_NONE;
        Py_BEGIN_ALLOW_THREADS
        rc = call();
        Py_END_ALLOW_THREADS
    } catch (const std::exception &) { // a tensor without an address, no device: the general path reports it
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    return PyLong_FromLong(rc);
}

#define SDP4_INT(o) (int)a.integer(o, INT32_MIN, INT32_MAX)

// w_new, w_prev, group, codes, scale, minv, n, stream
PyObject *py_qwd_encode(PyObject *, PyObject *const *v, Py_ssize_t nargs)
{
    return run(lib.qwd_encode, nargs, 8, [&](Args &a) {
        const int64_t n = a.count(v[6], v[0]);
        const int group = SDP4_INT(v[2]);
        int dtype = 0;
        auto w_new = (const float *)a.array(v[0], 4 * n);
        void *w_prev = a.weights(v[1], n, dtype);
        auto codes = (uint8_t *)a.array(v[3], n / 2);
        auto scale = (float *)a.array(v[4], headers(n, group));
        auto minv = (float *)a.array(v[5], headers(n, group));
        void *stream = a.stream(v[7]);
        return [=] { return lib.qwd_encode(w_new, w_prev, dtype, n, group, codes, scale, minv, stream); };
    });
}

// codes, scale, minv, group, w_prev, n, stream
PyObject *py_qwd_decode(PyObject *, PyObject *const *v, Py_ssize_t nargs)
{
    return run(lib.qwd_decode, nargs, 7, [&](Args &a) {
        const int64_t n = a.count(v[5], v[4]);
        const int group = SDP4_INT(v[3]);
        int dtype = 0;
        auto codes = (const uint8_t *)a.array(v[0], n / 2);
        auto scale = (const float *)a.array(v[1], headers(n, group));
        auto minv = (const float *)a.array(v[2], headers(n, group));
        void *w_prev = a.weights(v[4], n, dtype);
        void *stream = a.stream(v[6]);
        return [=] { return lib.qwd_decode(codes, scale, minv, n, group, w_prev, dtype, stream); };
    });
}

// w_new, w_prev, group, codes, scale, n, stream
PyObject *py_qwd_encode_sym(PyObject *, PyObject *const *v, Py_ssize_t nargs)
{
    return run(lib.qwd_encode_sym, nargs, 7, [&](Args &a) {
        const int64_t n = a.count(v[5], v[0]);
        const int group = SDP4_INT(v[2]);
        int dtype = 0;
        auto w_new = (const float *)a.array(v[0], 4 * n);
        void *w_prev = a.weights(v[1], n, dtype);
        auto codes = (uint8_t *)a.array(v[3], n / 2);
        auto scale = (float *)a.array(v[4], headers(n, group));
        void *stream = a.stream(v[6]);
        return [=] { return lib.qwd_encode_sym(w_new, w_prev, dtype, n, group, codes, scale, stream); };
    });
}

// codes, scale, group, w_prev, n, stream
PyObject *py_qwd_decode_sym(PyObject *, PyObject *const *v, Py_ssize_t nargs)
{
    return run(lib.qwd_decode_sym, nargs, 6, [&](Args &a) {
        const int64_t n = a.count(v[4], v[3]);
        const int group = SDP4_INT(v[2]);
        int dtype = 0;
        auto codes = (const uint8_t *)a.array(v[0], n / 2);
        auto scale = (const float *)a.array(v[1], headers(n, group));
        void *w_prev = a.weights(v[3], n, dtype);
        void *stream = a.stream(v[5]);
        return [=] { return lib.qwd_decode_sym(codes, scale, n, group, w_prev, dtype, stream); };
    });
}

// x, bits, hadamard_block, group, codes, scale, n, stream
PyObject *py_grad_quant(PyObject *, PyObject *const *v, Py_ssize_t nargs)
{
    return run(lib.grad_quant, nargs, 8, [&](Args &a) {
        const int64_t n = a.count(v[6], v[0]);
        const int bits = (int)a.integer(v[1], 4, 8), block = SDP4_INT(v[2]), group = SDP4_INT(v[3]);
        auto x = (const float *)a.array(v[0], 4 * n);
        void *codes = a.array(v[4], n * bits / 8);
        auto scale = (float *)a.array(v[5], headers(n, group));
        void *stream = a.stream(v[7]);
        return [=] { return lib.grad_quant(x, n, bits, block, group, codes, scale, stream); };
    });
}

// x, bits, hadamard_block, group, seed, offset, codes, scale, n, stream
PyObject *py_grad_quant_sr(PyObject *, PyObject *const *v, Py_ssize_t nargs)
{
    return run(lib.grad_quant_sr, nargs, 10, [&](Args &a) {
        const int64_t n = a.count(v[8], v[0]);
        const int bits = (int)a.integer(v[1], 4, 8), block = SDP4_INT(v[2]), group = SDP4_INT(v[3]);
        const uint64_t seed = a.bits64(v[4]), offset = a.bits64(v[5]);
        auto x = (const float *)a.array(v[0], 4 * n);
        void *codes = a.array(v[6], n * bits / 8);
        auto scale = (float *)a.array(v[7], headers(n, group));
        void *stream = a.stream(v[9]);
        return [=] { return lib.grad_quant_sr(x, n, bits, block, group, seed, offset, codes, scale, stream); };
    });
}

struct Peers {
    const void *codes[SDP4_MAX_PEERS];
    const float *scales[SDP4_MAX_PEERS];
    int P;
    Peers(Args &a, PyObject *c, PyObject *s, int64_t n, int64_t bits, int64_t group)
    {
        P = a.arrays(c, n * bits / 8, codes);
        if (a.arrays(s, headers(n, group), scales) != P)
            a.ok = false;
    }
};

// codes, scales, n_chunk, bits_in, group, bits_out, hadamard_block, out_scale, out_codes, out_scales, out_f32, stream
PyObject *py_dequant_reduce(PyObject *, PyObject *const *v, Py_ssize_t nargs)
{
    return run(lib.dequant_reduce, nargs, 12, [&](Args &a) {
        const int64_t n = a.integer(v[2], 0, SDP4_MAX_ELEMENTS);
        const int bits_in = (int)a.integer(v[3], 4, 8), group = SDP4_INT(v[4]), bits_out = (int)a.integer(v[5], 0, 8);
        const int block = SDP4_INT(v[6]);
        if (!PyFloat_CheckExact(v[7]))
            a.ok = false;
        const float out_scale = a.ok ? (float)PyFloat_AS_DOUBLE(v[7]) : 0.0f;
        const Peers in(a, v[0], v[1], n, bits_in, group);
        void *out_codes = a.optional_array(v[8], n * bits_out / 8);
        auto out_scales = (float *)a.optional_array(v[9], bits_out ? headers(n, group) : 0);
        auto out_f32 = (float *)a.optional_array(v[10], 4 * n);
        void *stream = a.stream(v[11]);
        return [=] {
            return lib.dequant_reduce(in.P, in.codes, in.scales, n, bits_in, group, bits_out, block, out_scale,
                                      out_codes, out_scales, out_f32, stream);
        };
    });
}

// codes, scales, n_chunk, bits_in, group, bits_out, seed, offset, out_codes, out_scales, out_f32, stream
PyObject *py_dequant_reduce_sr(PyObject *, PyObject *const *v, Py_ssize_t nargs)
{
    return run(lib.dequant_reduce_sr, nargs, 12, [&](Args &a) {
        const int64_t n = a.integer(v[2], 0, SDP4_MAX_ELEMENTS);
        const int bits_in = (int)a.integer(v[3], 4, 8), group = SDP4_INT(v[4]), bits_out = (int)a.integer(v[5], 0, 8);
        const uint64_t seed = a.bits64(v[6]), offset = a.bits64(v[7]);
        const Peers in(a, v[0], v[1], n, bits_in, group);
        void *out_codes = a.optional_array(v[8], n * bits_out / 8);
        auto out_scales = (float *)a.optional_array(v[9], bits_out ? headers(n, group) : 0);
        auto out_f32 = (float *)a.optional_array(v[10], 4 * n);
        void *stream = a.stream(v[11]);
        return [=] {
            return lib.dequant_reduce_sr(in.P, in.codes, in.scales, n, bits_in, group, bits_out, seed, offset,
                                         out_codes, out_scales, out_f32, stream);
        };
    });
}

// codes, scales, count, code_bytes, headers: the addresses of `count` consecutive chunks of a message, as a pair
// of lists, or None unless both tensors hold them all (their elements one code byte and one float header wide).
PyObject *py_chunk_addresses(PyObject *, PyObject *const *v, Py_ssize_t nargs)
{
    if (nargs != 5)
        Py_RETURN_NONE;
    Args a;
    const int64_t count = a.integer(v[2], 1, SDP4_MAX_PEERS), code_bytes = a.integer(v[3], 0, SDP4_MAX_ELEMENTS),
                  headers = a.integer(v[4], 0, SDP4_MAX_ELEMENTS);
    uintptr_t at[2] = {0, 0};
    const int64_t step[2] = {code_bytes, 4 * headers};
    try {
        for (int k = 0; a.ok && k < 2; ++k) {
            const at::Tensor *t = a.tensor(v[k]);
            if (t && t->element_size() == (k ? 4 : 1))
                at[k] = (uintptr_t)a.array(v[k], count * step[k]);
            else
                a.ok = false;
        }
    } catch (const std::exception &) {
        a.ok = false;
    }
    PyErr_Clear();
    if (!a.ok)
        Py_RETURN_NONE;
    PyObject *lists = PyTuple_New(2);
    for (int k = 0; lists && k < 2; ++k) {
        PyObject *l = PyList_New(count);
        for (int64_t i = 0; l && i < count; ++i) {
            PyObject *p = PyLong_FromVoidPtr((void *)(at[k] + i * step[k]));
            if (p)
                PyList_SET_ITEM(l, i, p);
            else
                Py_CLEAR(l);
        }
        if (l)
            PyTuple_SET_ITEM(lists, k, l);
        else
            Py_CLEAR(lists);
    }
    return lists;
}

// Addresses of the C entry points, in the order of Entry.
PyObject *py_bind(PyObject *, PyObject *const *v, Py_ssize_t nargs)
{
    void *p[8];
    if (nargs != 8) {
        PyErr_SetString(PyExc_TypeError, "bind: eight addresses");
        return nullptr;
    }
    for (int i = 0; i < 8; ++i) {
        p[i] = PyLong_AsVoidPtr(v[i]);
        if (!p[i]) {
            if (!PyErr_Occurred())
                PyErr_SetString(PyExc_ValueError, "bind: null address");
            return nullptr;
        }
    }
    lib.qwd_encode = (decltype(lib.qwd_encode))p[0];
    lib.qwd_decode = (decltype(lib.qwd_decode))p[1];
    lib.qwd_encode_sym = (decltype(lib.qwd_encode_sym))p[2];
    lib.qwd_decode_sym = (decltype(lib.qwd_decode_sym))p[3];
    lib.grad_quant = (decltype(lib.grad_quant))p[4];
    lib.grad_quant_sr = (decltype(lib.grad_quant_sr))p[5];
    lib.dequant_reduce = (decltype(lib.dequant_reduce))p[6];
    lib.dequant_reduce_sr = (decltype(lib.dequant_reduce_sr))p[7];
    Py_RETURN_NONE;
}

#define SDP4_METHOD(name) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    SDP4_METHOD(bind),          SDP4_METHOD(qwd_encode),      SDP4_METHOD(qwd_decode),     SDP4_METHOD(qwd_encode_sym),
    SDP4_METHOD(qwd_decode_sym), SDP4_METHOD(grad_quant),     SDP4_METHOD(grad_quant_sr),  SDP4_METHOD(dequant_reduce),
    SDP4_METHOD(dequant_reduce_sr), SDP4_METHOD(chunk_addresses), {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__binding()
{
    PyObject *m = PyModule_Create(&module_def);
    if (m && PyModule_AddStringConstant(m, "torch_version", SDP4_TORCH_VERSION) < 0)
        Py_CLEAR(m);
    return m;
}
