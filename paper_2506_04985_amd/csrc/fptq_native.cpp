// The fast path of the Python binding: argument checks, output allocation and the library call in one native call.
//
// What a Python wrapper with ctypes spends before the launch (about 7 us of 10.5 a call: torch.empty from Python 1.7 us each, the
// current stream's object 2.7, pointer objects and argument conversion the rest) is longer than the kernels of a token step
// run.  Every function here takes exactly the arguments of its wrapper in binding.py, positionally, and returns what the
// wrapper returns -- or None whenever anything is not the plain case (an argument of another type, a tensor that is not
// contiguous or not on the device, a buffer too small, an error of the library): then the wrapper goes on in Python, which
// raises what there is to raise.  A failing library call launches nothing, so it can be repeated.  Nothing is kept between calls.
#include <array>
#include <initializer_list>

#include <torch/extension.h>
#include <torch/csrc/autograd/python_variable.h>

#include "fptq.h"

namespace {

// torch._C functions: the device, the raw handle of its current stream, and whether that stream is being captured
PyObject *g_device = nullptr, *g_stream = nullptr, *g_capturing = nullptr;

struct Slow {};        // thrown where the call is left to the Python wrapper

// Runs f without the interpreter lock.  A launch can wait for room in its queue and an allocation for the device; other threads, and a
// host callback that the stream is waiting for, need the lock meanwhile.  It is taken again before anything thrown is handled.
template <class F>
auto without_gil(F f)
{
    struct Released {
        PyThreadState *state = PyEval_SaveThread();
        ~Released() { PyEval_RestoreThread(state); }
    } released;
    return f();
}

int64_t need(int64_t rows, int64_t K) { return (K + 127) / 128 * rows * 64; }

const at::Tensor &device_tensor(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) throw Slow();
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda()) throw Slow();
    return t;
}

const at::Tensor &input(PyObject *o, at::ScalarType type)
{
    const at::Tensor &t = device_tensor(o);
    if (t.scalar_type() != type || !t.is_contiguous()) throw Slow();
    return t;
}

void *input_or_null(PyObject *o, at::ScalarType type) { return o == Py_None ? nullptr : input(o, type).data_ptr(); }

int64_t integer(PyObject *o)
{
    if (!PyLong_CheckExact(o)) throw Slow();
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Slow();
    return v;
}

float number(PyObject *o)
{
    if (PyFloat_CheckExact(o)) return (float)PyFloat_AS_DOUBLE(o);
    if (PyLong_CheckExact(o)) {
        const double v = PyLong_AsDouble(o);
        if (v == -1.0 && PyErr_Occurred()) throw Slow();
        return (float)v;
    }
    throw Slow();
}

bool truth(PyObject *o)
{
    if (o == Py_True) return true;
    if (o == Py_False) return false;
    throw Slow();
}

// An output: the caller's tensor, or a new one, made by `allocate` without the interpreter lock and wrapped by `take` with it.
struct Output {
    PyObject *given = nullptr;       // the caller's, who holds it
    at::Tensor made;
    std::array<int64_t, 2> shape = {0, 1};
    int dims = 0;
    at::ScalarType type = at::kByte;
    at::Device device = at::kCPU;
    void *ptr = nullptr;
    int64_t numel = 0;
    Output() = default;              // none: ptr is NULL
    Output(PyObject *o, std::initializer_list<int64_t> sizes, at::ScalarType t, const at::Tensor &like)
    {
        if (o != Py_None) {
            const at::Tensor &v = device_tensor(o);
            given = o, ptr = v.data_ptr(), numel = v.numel();
            return;
        }
        for (int64_t n : sizes) shape[dims++] = n;
        type = t, device = like.device();
    }
    void allocate()
    {
        if (dims == 0) return;
        made = at::empty(at::IntArrayRef(shape.data(), dims), at::TensorOptions().dtype(type).device(device));
        ptr = made.data_ptr(), numel = made.numel();
    }
    PyObject *take()                 // a new reference to the tensor, None for no output
    {
        PyObject *o = given ? given : Py_None;
        if (made.defined()) {
            o = THPVariable_Wrap(std::move(made));
            if (!o) throw Slow();
            return o;
        }
        Py_INCREF(o);
        return o;
    }
};

PyObject *tuple(std::initializer_list<Output *> outputs)
{
    PyObject *t = PyTuple_New((Py_ssize_t)outputs.size());
    if (!t) throw Slow();
    Py_ssize_t i = 0;
    try {
        for (Output *o : outputs) {
            PyTuple_SET_ITEM(t, i, o->take());
            ++i;
        }
    } catch (...) {
        Py_DECREF(t);
        throw;
    }
    return t;
}

// where a launch goes: the current device and its current stream
struct Where {
    long device;
    void *stream;
};

Where where()
{
    PyObject *d = PyObject_CallNoArgs(g_device);
    if (!d) throw Slow();
    const long index = PyLong_AsLong(d);
    PyObject *s = PyObject_CallOneArg(g_stream, d);
    Py_DECREF(d);
    if (!s) throw Slow();
    void *p = PyLong_AsVoidPtr(s);
    Py_DECREF(s);
    if (PyErr_Occurred()) throw Slow();
    return {index, p};
}

bool capturing()
{
    PyObject *c = PyObject_CallNoArgs(g_capturing);
    if (!c) throw Slow();
    const int yes = PyObject_IsTrue(c);
    Py_DECREF(c);
    if (yes < 0) throw Slow();
    return yes;
}

// The part of a call that may wait: the new outputs, then the library's call.
template <class F>
void launch(std::initializer_list<Output *> outputs, F f)
{
    const int rc = without_gil([&] {
        for (Output *o : outputs) o->allocate();
        return f();
    });
    if (rc != FPTQ_OK) throw Slow();
}

// runs f(args), leaving the call to Python where it throws
template <class F>
PyObject *guarded(Py_ssize_t got, Py_ssize_t want, F f)
{
    try {
        if (got != want) throw Slow();
        return f();
    } catch (...) {
        PyErr_Clear();
    }
    Py_RETURN_NONE;
}

void matrix(const at::Tensor &x, int64_t &M, int64_t &K)
{
    if (x.dim() != 2) throw Slow();
    M = x.size(0), K = x.size(1);
    if (M < 1 || K < 1) throw Slow();
}

// (w_int, out)
PyObject *pack_weights(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 2, [&]() -> PyObject * {
        const at::Tensor &w = input(a[0], at::kChar);
        int64_t N, K;
        matrix(w, N, K);
        Output out(a[1], {need(N, K)}, at::kByte, w);
        void *const st = where().stream;
        launch({&out}, [&] { return fptq_pack_weights((const int8_t *)w.data_ptr(), N, K, out.ptr, out.numel, st); });
        return out.take();
    });
}

// (w_int)
PyObject *weight_row_sums(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 1, [&]() -> PyObject * {
        const at::Tensor &w = input(a[0], at::kChar);
        int64_t N, K;
        matrix(w, N, K);
        Output out(Py_None, {N}, at::kInt, w);
        void *const st = where().stream;
        launch({&out}, [&] { return fptq_weight_row_sums((const int8_t *)w.data_ptr(), N, K, (int32_t *)out.ptr, st); });
        return out.take();
    });
}

// (x, s_a, scale_mode, eps, row_scale_in, out, row_scale_out, want_row_scale, kind, parameter): kind 0 the plain quantizer, 1 behind the
// Hadamard transform with blocks of `parameter`, 2 on the asymmetric grid with that zero point.  The wrapper says which call it is: no
// value of the caller's may.
PyObject *quantize_act(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 10, [&]() -> PyObject * {
        const at::Tensor &x = input(a[0], at::kBFloat16);
        int64_t M, K;
        matrix(x, M, K);
        const float s_a = number(a[1]), eps = number(a[3]);
        const int mode = (int)integer(a[2]);
        const int64_t kind = integer(a[8]), parameter = kind ? integer(a[9]) : 0;
        const float *r_in = (const float *)input_or_null(a[4], at::kFloat);
        Output out(a[5], {need(M, K)}, at::kByte, x), r;
        if (a[6] != Py_None || truth(a[7])) r = Output(a[6], {M}, at::kFloat, x);
        void *const st = where().stream;
        launch({&out, &r}, [&] {
            float *const r_out = (float *)r.ptr;
            if (kind == 1) return fptq_quantize_act_hadamard(x.data_ptr(), M, K, (int)parameter, mode, eps, r_in, s_a, out.ptr, out.numel, r_out, st);
            if (kind == 2) return fptq_quantize_act_asym(x.data_ptr(), M, K, mode, eps, r_in, s_a, (int)parameter, out.ptr, out.numel, r_out, st);
            return fptq_quantize_act(x.data_ptr(), M, K, mode, eps, r_in, s_a, out.ptr, out.numel, r_out, st);
        });
        return tuple({&out, &r});
    });
}

// (x, out, token_scale_out)
PyObject *quantize_act_dynamic(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 3, [&]() -> PyObject * {
        const at::Tensor &x = input(a[0], at::kBFloat16);
        int64_t M, K;
        matrix(x, M, K);
        Output out(a[1], {need(M, K)}, at::kByte, x), s(a[2], {M}, at::kFloat, x);
        void *const st = where().stream;
        launch({&out, &s}, [&] { return fptq_quantize_act_dynamic(x.data_ptr(), M, K, out.ptr, out.numel, (float *)s.ptr, st); });
        return tuple({&out, &s});
    });
}

// (x_res, y_blk, s_a, s_prev, eps, x_next, s_next, out)
PyObject *residual_norm_quantize(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 8, [&]() -> PyObject * {
        const at::Tensor &x = input(a[0], at::kBFloat16), &y = input(a[1], at::kBFloat16);
        int64_t M, K;
        matrix(x, M, K);
        const float s_a = number(a[2]), eps = number(a[4]);
        const float *s_prev = (const float *)input_or_null(a[3], at::kFloat);
        Output x_next(a[5], {M, K}, at::kBFloat16, x), s_next(a[6], {M}, at::kFloat, x), out(a[7], {need(M, K)}, at::kByte, x);
        void *const st = where().stream;
        launch({&x_next, &s_next, &out}, [&] {
            return fptq_residual_norm_quantize(x.data_ptr(), y.data_ptr(), M, K, s_prev, eps, s_a, x_next.ptr, (float *)s_next.ptr, out.ptr,
                                               out.numel, st);
        });
        return tuple({&x_next, &s_next, &out});
    });
}

// (xq, wq, M, N, K, s_a, s_w, row_out_scale, out, want_acc, acc, zero_point, w_row_sum, workspace, kind): kind 0 the plain linear and 3
// the one with a zero point, both with scratch where it pays; 1 with a workspace; 2 the one that allocates nothing
PyObject *linear(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 15, [&]() -> PyObject * {
        const at::Tensor &xq = input(a[0], at::kByte), &wq = input(a[1], at::kByte), &s_w = input(a[6], at::kFloat);
        const int64_t M = integer(a[2]), N = integer(a[3]), K = integer(a[4]);
        if (M < 1 || N < 1 || K < 1 || M > (1ll << 40) / K || N > (1ll << 40) / K || M > (1ll << 40) / N) throw Slow();
        if (xq.numel() < need(M, K) || wq.numel() < need(N, K) || s_w.numel() < N) throw Slow();
        const float s_a = number(a[5]);
        const float *d = (const float *)input_or_null(a[7], at::kFloat);
        const bool want_acc = truth(a[9]);
        const int64_t kind = integer(a[14]);
        const int zp = kind == 3 ? (int)integer(a[11]) : 0;
        const int32_t *wsum = kind == 3 ? (const int32_t *)input(a[12], at::kInt).data_ptr() : nullptr;
        const at::Tensor *const ws = kind == 1 ? &input(a[13], at::kByte) : nullptr;
        Output y(a[8], {M, N}, at::kBFloat16, xq), acc;
        const bool with_acc = want_acc || a[10] != Py_None;
        if (with_acc) acc = Output(a[10], {M, N}, at::kInt, xq);
        const Where w = where();
        void *const st = w.stream;
        // Scratch is handed back when the call returns and then guarded by stream order alone: it has to come from the stream that the
        // launch goes to, i.e. from the current device.  Operands on another one (peer access) go without.
        const bool may_scratch = (kind == 0 || kind == 3) && M > 64 && xq.device().index() == w.device;
        int64_t scratch_bytes = may_scratch ? without_gil([&] { return fptq_linear_scratch_bytes(M, N, K); }) : 0;
        if (scratch_bytes > 0 && capturing()) scratch_bytes = 0;
        at::Tensor scratch;
        launch({&y, &acc}, [&] {
            const void *px = xq.data_ptr(), *pw = wq.data_ptr();
            const float *ps = (const float *)s_w.data_ptr();
            int32_t *const pa = (int32_t *)acc.ptr;
            if (scratch_bytes > 0) {
                try {
                    scratch = at::empty({scratch_bytes}, at::TensorOptions().dtype(at::kByte).device(xq.device()));
                } catch (const c10::Error &) {       // no memory, or none to be had now: the INT8 kernels need none
                }
            }
            if (scratch.defined())
                return fptq_w4a4_linear_scratch(px, pw, M, N, K, s_a, ps, d, zp, wsum, y.ptr, pa, scratch.data_ptr(), scratch_bytes, st);
            if (kind == 1) return fptq_w4a4_linear_ws(px, pw, M, N, K, s_a, ps, d, y.ptr, pa, ws->data_ptr(), ws->numel(), st);
            if (kind == 2) return fptq_w4a4_linear_noalloc(px, pw, M, N, K, s_a, ps, d, y.ptr, pa, st);
            if (kind == 3) return fptq_w4a4_linear_zp(px, pw, M, N, K, s_a, ps, d, zp, wsum, y.ptr, pa, st);
            return fptq_w4a4_linear(px, pw, M, N, K, s_a, ps, d, y.ptr, pa, st);
        });
        return with_acc ? tuple({&y, &acc}) : y.take();
    });
}

#define FPTQ_FAST(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FPTQ_FAST(pack_weights), FPTQ_FAST(weight_row_sums), FPTQ_FAST(quantize_act), FPTQ_FAST(quantize_act_dynamic),
                         FPTQ_FAST(residual_norm_quantize), FPTQ_FAST(linear), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" PyObject *PyInit__native()
{
    PyObject *c = PyImport_ImportModule("torch._C");
    if (!c) return nullptr;
    g_device = PyObject_GetAttrString(c, "_cuda_getDevice");
    g_stream = PyObject_GetAttrString(c, "_cuda_getCurrentRawStream");
    g_capturing = PyObject_GetAttrString(c, "_cuda_isCurrentStreamCapturing");
    Py_DECREF(c);
    if (!g_device || !g_stream || !g_capturing) return nullptr;
    return PyModule_Create(&module);
}
