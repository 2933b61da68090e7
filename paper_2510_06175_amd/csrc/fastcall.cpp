// Python module _fastcall: the argument checks of binding.py and the library call, in one native call.
//
// The checks of a step's 11 tensors (device, type, shape, contiguity, each an attribute read by the interpreter) and
// the conversion of 20 arguments by ctypes are host time in front of a launch that may itself take less:
// appends of one token to 32 sequences, called back to back, 7.9 us each by ctypes, 5.8 here (the kernel then bounds them);
// steps of 1000 tokens 10.12 -> 9.99 us, longer ones unchanged.
//
// Every function returns the library's status, or None where an argument is not what it expects: binding.py then
// goes through its own checks, which say what is wrong (or accept what only they can judge, such as subclasses
// of torch.Tensor).  Nothing is kept between calls but the library's functions and the one that finds the stream.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <exception>
#include <initializer_list>

#include "../../include/vecinfer.h"

namespace {

decltype(&vecinfer_encode_keys) encode_keys;
decltype(&vecinfer_encode_values) encode_values;
decltype(&vecinfer_append_kv) append_kv;
decltype(&vecinfer_decode_attention) decode_attention;
decltype(&vecinfer_decode_attention_residual) decode_residual;
decltype(&vecinfer_decode_step) decode_step;
PyObject *find_stream;                   // binding._stream

struct Refused {};                       // an argument that the interpreter's checks have to look at
struct Raised {};                        // Python's error is set

const at::Tensor &tensor(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) throw Refused();
    return THPVariable_Unpack(o);
}

// A contiguous tensor on the GPU of this type and shape.
void *pointer(const at::Tensor &t, at::ScalarType type, std::initializer_list<int64_t> shape)
{
    if (!t.is_cuda() || t.scalar_type() != type || !t.sizes().equals(c10::IntArrayRef(shape)) || !t.is_contiguous()) throw Refused();
    return t.data_ptr();
}

void *pointer(PyObject *o, at::ScalarType type, std::initializer_list<int64_t> shape) { return pointer(tensor(o), type, shape); }

int64_t extent(const at::Tensor &t, int64_t dims, int64_t i)
{
    if (t.dim() != dims) throw Refused();
    return t.size(i);
}

int64_t integer(PyObject *o)
{
    if (!PyLong_CheckExact(o)) throw Refused();
    int overflow = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow) throw Refused();
    return v;
}

int32_t integer32(PyObject *o)
{
    const int64_t v = integer(o);
    if (v != (int32_t)v) throw Refused();
    return (int32_t)v;
}

void *address(PyObject *o)
{
    void *p = PyLong_Check(o) ? PyLong_AsVoidPtr(o) : nullptr;
    if (PyErr_Occurred()) {
        PyErr_Clear();
        throw Refused();
    }
    return p;
}

// The stream's handle, asked for after the checks as the interpreter's path does, and what that raises is raised: it may
// be an interrupt, which a second attempt would not see.
void *stream_of(PyObject *o)
{
    PyObject *const r = PyObject_CallFunctionObjArgs(find_stream, o, nullptr);
    if (!r) throw Raised();
    struct Release {
        PyObject *r;
        ~Release() { Py_DECREF(r); }
    } release{r};
    return address(r);
}

// What a call needs of its configuration.
struct Cfg {
    const vecinfer_cfg *c;
    int64_t D, Hq, Hkv;
    explicit Cfg(PyObject *o) : c(static_cast<const vecinfer_cfg *>(address(o)))
    {
        if (!c) throw Refused();
        D = c->head_dim;
        Hq = c->num_q_heads;
        Hkv = c->num_kv_heads;
        if (c->k_sub_dim < 1 || c->v_sub_dim < 1 || c->k_bits < 1 || c->v_bits < 1 || c->k_bits > 30 || c->v_bits > 30) throw Refused();
    }
    int64_t row(bool keys) const { return D / (keys ? c->k_sub_dim : c->v_sub_dim) * (keys ? c->k_bits : c->v_bits) / 8; }
    void *codebook(PyObject *o, bool keys) const
    {
        const int64_t d = keys ? c->k_sub_dim : c->v_sub_dim, bits = keys ? c->k_bits : c->v_bits;
        return bits == 8 ? pointer(o, at::kHalf, {Hkv, D / d, 256, d}) : pointer(o, at::kHalf, {Hkv, (int64_t)1 << bits, d});
    }
    const float *lambda(PyObject *o) const { return static_cast<const float *>(pointer(o, at::kFloat, {Hkv, D})); }
    uint8_t *codes(PyObject *o, bool keys, int64_t B, int64_t n_cap) const
    {
        return static_cast<uint8_t *>(pointer(o, at::kByte, {B, Hkv, n_cap, row(keys)}));
    }
};

// f: a call of the library, which throws nothing.  (Where the interpreter is shutting down, PyEval_RestoreThread ends
// a daemon thread by unwinding it: no destructor and no catch-all may stand in its way, or the process aborts.)
template <typename F>
int without_gil(F &&f)
{
    PyThreadState *const state = PyEval_SaveThread();
    const int rc = f();
    PyEval_RestoreThread(state);
    return rc;
}

// f() -> status; None for anything that is not as expected (also torch's own exceptions: wrapped tensors
// have no data pointer).
template <typename F>
PyObject *guarded(F &&f)
{
    try {
        return PyLong_FromLong(f());
    } catch (const Raised &) {
        return nullptr;
    } catch (const Refused &) {
    } catch (const std::exception &) {
    }
    Py_RETURN_NONE;
}

// encode(cfg, x, lambda or None (values), codebook, codes, pos0, stream)
PyObject *encode(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&] {
        if (n != 7) throw Refused();
        const Cfg cfg(a[0]);
        const bool keys = a[2] != Py_None;
        const at::Tensor &x = tensor(a[1]);
        const int64_t B = extent(x, 4, 0), T = extent(x, 4, 2), n_cap = extent(tensor(a[4]), 4, 2), pos0 = integer(a[5]);
        const void *const px = pointer(x, at::kHalf, {B, cfg.Hkv, T, cfg.D});
        const float *const lam = keys ? cfg.lambda(a[2]) : nullptr;
        const void *const cb = cfg.codebook(a[3], keys);
        uint8_t *const idx = cfg.codes(a[4], keys, B, n_cap);
        if (B != (int32_t)B) throw Refused();
        void *const stream = stream_of(a[6]);
        return without_gil([&] {
            return keys ? encode_keys(cfg.c, px, lam, cb, idx, (int32_t)B, T, pos0, n_cap, stream)
                        : encode_values(cfg.c, px, cb, idx, (int32_t)B, T, pos0, n_cap, stream);
        });
    });
}

// append(cfg, k, v, lambda, cb_k, cb_v, k_idx, v_idx, pos0, stream)
PyObject *append(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&] {
        if (n != 10) throw Refused();
        const Cfg cfg(a[0]);
        const at::Tensor &k = tensor(a[1]);
        const int64_t B = extent(k, 4, 0), T = extent(k, 4, 2), n_cap = extent(tensor(a[6]), 4, 2), pos0 = integer(a[8]);
        const void *const pk = pointer(k, at::kHalf, {B, cfg.Hkv, T, cfg.D}), *const pv = pointer(a[2], at::kHalf, {B, cfg.Hkv, T, cfg.D});
        const float *const lam = cfg.lambda(a[3]);
        const void *const cb_k = cfg.codebook(a[4], true), *const cb_v = cfg.codebook(a[5], false);
        uint8_t *const k_idx = cfg.codes(a[6], true, B, n_cap), *const v_idx = cfg.codes(a[7], false, B, n_cap);
        if (B != (int32_t)B) throw Refused();
        void *const stream = stream_of(a[9]);
        return without_gil([&] { return append_kv(cfg.c, pk, pv, lam, cb_k, cb_v, k_idx, v_idx, (int32_t)B, T, pos0, n_cap, stream); });
    });
}

// decode(cfg, q, lambda, cb_k, cb_v, k_idx, v_idx, workspace, out, lse or None, seq_lens or None, N or None, num_splits,
//        variant, stream [, k_new, v_new] [, k_res, v_res, res_lens or None, R or None])
PyObject *decode(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded([&] {
        if (n != 15 && n != 17 && n != 19) throw Refused();
        const Cfg cfg(a[0]);
        const at::Tensor &q = tensor(a[1]), &ws = tensor(a[7]);
        const int64_t B = extent(q, 3, 0), n_cap = extent(tensor(a[5]), 4, 2), N = a[11] == Py_None ? n_cap : integer(a[11]);
        const void *const pq = pointer(q, at::kHalf, {B, cfg.Hq, cfg.D});
        const float *const lam = cfg.lambda(a[2]);
        const void *const cb_k = cfg.codebook(a[3], true), *const cb_v = cfg.codebook(a[4], false);
        uint8_t *const k_idx = cfg.codes(a[5], true, B, n_cap), *const v_idx = cfg.codes(a[6], false, B, n_cap);
        void *const out = pointer(a[8], at::kHalf, {B, cfg.Hq, cfg.D});
        float *const lse = a[9] == Py_None ? nullptr : static_cast<float *>(pointer(a[9], at::kFloat, {B, cfg.Hq}));
        const int32_t *const lens = a[10] == Py_None ? nullptr : static_cast<const int32_t *>(pointer(a[10], at::kInt, {B}));
        const int32_t splits = integer32(a[12]), variant = integer32(a[13]);
        void *const wp = ws.data_ptr();
        const size_t wb = (size_t)ws.numel() * ws.element_size();
        if (B != (int32_t)B) throw Refused();
        const int32_t b = (int32_t)B;
        if (n == 15) {
            void *const stream = stream_of(a[14]);
            return without_gil([&] {
                return decode_attention(cfg.c, pq, lam, cb_k, cb_v, k_idx, v_idx, lens, b, N, n_cap, splits, variant, wp, wb, out, lse, stream);
            });
        }
        if (n == 17) {
            const void *const k = pointer(a[15], at::kHalf, {B, cfg.Hkv, 1, cfg.D}), *const v = pointer(a[16], at::kHalf, {B, cfg.Hkv, 1, cfg.D});
            void *const stream = stream_of(a[14]);
            return without_gil([&] {
                return decode_step(cfg.c, pq, k, v, lam, cb_k, cb_v, k_idx, v_idx, lens, b, N, n_cap, splits, variant, wp, wb, out, lse, stream);
            });
        }
        const int64_t r_cap = extent(tensor(a[15]), 4, 2);
        const void *const k = pointer(a[15], at::kHalf, {B, cfg.Hkv, r_cap, cfg.D}), *const v = pointer(a[16], at::kHalf, {B, cfg.Hkv, r_cap, cfg.D});
        const int32_t *const res = a[17] == Py_None ? nullptr : static_cast<const int32_t *>(pointer(a[17], at::kInt, {B}));
        if (a[18] == Py_None && r_cap != (int32_t)r_cap) throw Refused();
        const int32_t R = a[18] == Py_None ? (int32_t)r_cap : integer32(a[18]);
        void *const stream = stream_of(a[14]);
        return without_gil([&] {
            return decode_residual(cfg.c, pq, lam, cb_k, cb_v, k_idx, v_idx, lens, b, N, n_cap, k, v, res, R, r_cap, splits, variant, wp, wb, out,
                                   lse, stream);
        });
    });
}

// bind(addresses of the library's functions, in the order of the variables above, then the function for streams)
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != 7) {
        PyErr_SetString(PyExc_TypeError, "bind: six addresses and a function");
        return nullptr;
    }
    void *p[6];
    for (int i = 0; i < 6; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (PyErr_Occurred()) return nullptr;
    }
    Py_INCREF(a[6]);
    Py_XDECREF(find_stream);
    find_stream = a[6];
    encode_keys = reinterpret_cast<decltype(encode_keys)>(p[0]);
    encode_values = reinterpret_cast<decltype(encode_values)>(p[1]);
    append_kv = reinterpret_cast<decltype(append_kv)>(p[2]);
    decode_attention = reinterpret_cast<decltype(decode_attention)>(p[3]);
    decode_residual = reinterpret_cast<decltype(decode_residual)>(p[4]);
    decode_step = reinterpret_cast<decltype(decode_step)>(p[5]);
    Py_RETURN_NONE;
}

#define VECINFER_METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {VECINFER_METHOD(bind), VECINFER_METHOD(encode), VECINFER_METHOD(append), VECINFER_METHOD(decode),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__fastcall()
{
    PyObject *const m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
