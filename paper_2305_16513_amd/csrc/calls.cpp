// The binding's small calls in native code: arguments taken from Python, the output allocated, the library's entry called.
//
// A call that the GPU finishes in 3 - 8 us is bound by the host.  In Python a sliding sum over one series takes 6.6 us of it (3.1 in HIP's
// launch, 1.4 in allocating, the rest in look-ups, checks and ctypes), a pooling call 7.2; here 4.3 and 4.5, and three of them are the launch.
//
// Every function returns None where anything is out of the ordinary (another type of argument, a tensor that is no plain one of
// the current device, a mode that watches calls, lengths that do not fit, no memory): binding.py's Python code then does the same call,
// and says what is wrong with it.  Only what the library itself answers is raised here.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "sws.h"

namespace {

PyObject *g_error = nullptr;                          // binding.SwsError

// One call.  Its functions note what is not for here in `odd`, so that a refusal costs a tenth of a microsecond (a C++ exception: 2.9).
struct Call {
    PyObject *const *a;
    bool odd = false;
    int device = -1;                                  // the current one, asked for when a tensor of any is met
    at::Tensor out;
    int rc = SWS_OK;

    // an int of 31 bits
    int32_t num(int i)
    {
        long long v = -1;
        int over = 0;
        if (PyLong_Check(a[i])) v = PyLong_AsLongLongAndOverflow(a[i], &over);
        odd |= over != 0 || v < 0 || v > 0x7fffffff;
        return (int32_t)v;
    }
    float real(int i)
    {
        if (PyFloat_Check(a[i])) return (float)PyFloat_AS_DOUBLE(a[i]);
        long long v = 0;
        int over = 1;
        if (PyLong_Check(a[i])) v = PyLong_AsLongLongAndOverflow(a[i], &over);
        odd |= over != 0;
        return (float)(double)v;
    }
    // a contiguous tensor with memory of the current device, and nothing that wraps or watches it; not looked at where the call is odd
    const at::Tensor &tensor(int i, bool half = false)
    {
        static const at::Tensor none;
        if (!THPVariable_CheckExact(a[i])) { odd = true; return none; }
        const at::Tensor &t = THPVariable_Unpack(a[i]);
        if (!t.defined() || !t.is_cuda() || t.layout() != c10::kStrided || !t.has_storage() || !t.is_contiguous() ||
            t.key_set().has_any(c10::DispatchKeySet({c10::DispatchKey::Python, c10::DispatchKey::Functionalize})) ||
            (half ? t.scalar_type() != at::kBFloat16 && t.scalar_type() != at::kHalf : t.scalar_type() != at::kFloat)) {
            odd = true;
            return none;
        }
        if (device < 0) device = c10::hip::current_device();
        odd |= t.device().index() != device;
        return t;
    }
    static int dtype(const at::Tensor &t) { return t.scalar_type() == at::kHalf ? SWS_DTYPE_F16 : SWS_DTYPE_BF16; }

    // The output, of x's type, and the library's call on it: f(address, stream).  Others run meanwhile: the allocator may wait for the device.
    template <class F> bool run(at::IntArrayRef sizes, const at::Tensor &x, F f)
    {
        const at::TensorOptions like = x.options();
        const hipStream_t stream = c10::hip::getCurrentHIPStream((c10::DeviceIndex)device).stream();
        struct Unlocked {
            PyThreadState *state = PyEval_SaveThread();
            ~Unlocked() { PyEval_RestoreThread(state); }
        } unlocked;
        out = at::empty(sizes, like);
        rc = f(out.data_ptr(), stream);
        return true;
    }
};

// sws_out_len for numbers of 31 bits; 0: not for here
int64_t out_len(int64_t n, int64_t w, int64_t stride, int64_t pad, int64_t dilation = 1)
{
    if (w < 1 || stride < 1 || dilation < 1) return 0;
    const int64_t left = n + 2 * pad - dilation * (w - 1) - 1;
    return left < 0 ? 0 : left / stride + 1;
}

// f(call): false where the call is not for here
template <class F>
PyObject *call(const char *name, PyObject *const *a, Py_ssize_t want, Py_ssize_t n, F f)
{
    if (n != want || c10::impl::TorchDispatchModeTLS::any_modes_set() || at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
    try {
        Call c{a};
        if (!f(c)) Py_RETURN_NONE;
        if (c.rc == SWS_OK) return THPVariable_Wrap(std::move(c.out));
        PyObject *e = PyObject_CallFunction(g_error, "is", c.rc, name);
        if (e) {
            PyErr_SetObject(g_error, e);
            Py_DECREF(e);
        }
        return nullptr;
    } catch (...) {                                   // (what torch throws, no memory for one: the Python code meets it again)
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

typedef const float *fp;
#define SWS_CALL(NAME, N) PyObject *NAME(PyObject *, PyObject *const *a, Py_ssize_t n) { return call("sws_" #NAME, a, N, n, [](Call &c) -> bool
#define SWS_END ); }

int64_t rows(const at::Tensor &t) { return t.numel() / t.size(-1); }

// the sliding sums: rows of x shortened to lo
template <class F>
bool along_rows(Call &c, const at::Tensor &x, int64_t lo, F f)
{
    if (lo < 1) return false;
    c10::SmallVector<int64_t, 6> shape(x.sizes().begin(), x.sizes().end());
    shape.back() = lo;
    const void *const p = x.data_ptr();
    const int64_t many = rows(x), length = x.size(-1);
    return c.run(shape, x, [&](void *y, hipStream_t s) { return f(p, y, many, length, s); });
}

SWS_CALL(slide1d, 4) {
    const int op = c.num(0), w = c.num(2);
    const float scale = c.real(3);
    const at::Tensor &x = c.tensor(1);
    if (c.odd || x.dim() < 1) return false;
    return along_rows(c, x, out_len(x.size(-1), w, 1, 0), [=](const void *p, void *y, int64_t many, int64_t length, hipStream_t s) {
        return sws_slide1d((sws_op)op, (fp)p, (float *)y, many, length, w, scale, s);
    });
} SWS_END

SWS_CALL(slide1d_16, 4) {
    const int op = c.num(0), w = c.num(2);
    const float scale = c.real(3);
    const at::Tensor &x = c.tensor(1, true);
    if (c.odd || x.dim() < 1) return false;
    const int dt = c.dtype(x);
    return along_rows(c, x, out_len(x.size(-1), w, 1, 0), [=](const void *p, void *y, int64_t many, int64_t length, hipStream_t s) {
        return sws_slide1d_16((sws_op)op, (sws_dtype)dt, p, y, many, length, w, scale, s);
    });
} SWS_END

SWS_CALL(slide1d_padded, 7) {
    const int op = c.num(0), w = c.num(2), left = c.num(3), right = c.num(4), mode = c.num(5);
    const float scale = c.real(6);
    const at::Tensor &x = c.tensor(1);
    if (c.odd || x.dim() < 1 || x.size(-1) < 1) return false;
    return along_rows(c, x, out_len(x.size(-1) + left + right, w, 1, 0), [=](const void *p, void *y, int64_t many, int64_t length, hipStream_t s) {
        return sws_slide1d_padded((sws_op)op, (fp)p, (float *)y, many, length, w, left, right, (sws_pad_mode)mode, scale, s);
    });
} SWS_END

SWS_CALL(pool2d, 9) {
    const int op = c.num(0), kh = c.num(2), kw = c.num(3), sh = c.num(4), sw = c.num(5), ph = c.num(6), pw = c.num(7);
    const float scale = c.real(8);
    const at::Tensor &x = c.tensor(1);
    if (c.odd || x.dim() != 4) return false;
    const int64_t N = x.size(0), C = x.size(1), H = x.size(2), W = x.size(3), ho = out_len(H, kh, sh, ph), wo = out_len(W, kw, sw, pw);
    if (ho < 1 || wo < 1) return false;
    const fp p = (fp)x.data_ptr();
    return c.run({N, C, ho, wo}, x, [=](void *y, hipStream_t s) { return sws_pool2d((sws_op)op, p, (float *)y, N, C, H, W, kh, kw, sh, sw, ph, pw, scale, s); });
} SWS_END

SWS_CALL(pool2d_16, 9) {
    const int op = c.num(0), kh = c.num(2), kw = c.num(3), sh = c.num(4), sw = c.num(5), ph = c.num(6), pw = c.num(7);
    const float scale = c.real(8);
    const at::Tensor &x = c.tensor(1, true);
    if (c.odd || x.dim() != 4) return false;
    const int64_t N = x.size(0), C = x.size(1), H = x.size(2), W = x.size(3), ho = out_len(H, kh, sh, ph), wo = out_len(W, kw, sw, pw);
    if (ho < 1 || wo < 1) return false;
    const int dt = c.dtype(x);
    const void *const p = x.data_ptr();
    return c.run({N, C, ho, wo}, x, [=](void *y, hipStream_t s) { return sws_pool2d_16((sws_op)op, (sws_dtype)dt, p, y, N, C, H, W, kh, kw, sh, sw, ph, pw, scale, s); });
} SWS_END

SWS_CALL(maxpool2d_grad, 8) {
    const int kh = c.num(2), kw = c.num(3), sh = c.num(4), sw = c.num(5), ph = c.num(6), pw = c.num(7);
    const at::Tensor &x = c.tensor(0), &gy = c.tensor(1);
    if (c.odd || x.dim() != 4 || gy.dim() != 4) return false;
    const int64_t N = x.size(0), C = x.size(1), H = x.size(2), W = x.size(3), ho = out_len(H, kh, sh, ph), wo = out_len(W, kw, sw, pw);
    if (ho < 1 || wo < 1 || gy.size(0) != N || gy.size(1) != C || gy.size(2) != ho || gy.size(3) != wo) return false;
    const fp p = (fp)x.data_ptr(), q = (fp)gy.data_ptr();
    return c.run({N, C, H, W}, x, [=](void *gx, hipStream_t s) { return sws_maxpool2d_grad(p, q, (float *)gx, N, C, H, W, kh, kw, sh, sw, ph, pw, s); });
} SWS_END

SWS_CALL(avgpool2d_grad, 11) {
    const int H = c.num(1), W = c.num(2), kh = c.num(3), kw = c.num(4), sh = c.num(5), sw = c.num(6), ph = c.num(7), pw = c.num(8), div = c.num(9);
    const float scale = c.real(10);
    const at::Tensor &gy = c.tensor(0);
    if (c.odd || gy.dim() != 4) return false;
    const int64_t N = gy.size(0), C = gy.size(1), ho = out_len(H, kh, sh, ph), wo = out_len(W, kw, sw, pw);
    if (ho < 1 || wo < 1 || gy.size(2) != ho || gy.size(3) != wo) return false;
    const fp p = (fp)gy.data_ptr();
    return c.run({N, C, H, W}, gy, [=](void *gx, hipStream_t s) {
        return sws_avgpool2d_grad(p, (float *)gx, N, C, H, W, kh, kw, sh, sw, ph, pw, (sws_divisor)div, scale, s);
    });
} SWS_END

// layers of several groups: none of their kernels uses a workspace
SWS_CALL(conv1d, 6) {
    const int stride = c.num(2), pad = c.num(3), dil = c.num(4), groups = c.num(5);
    const at::Tensor &x = c.tensor(0), &w = c.tensor(1);
    if (c.odd || x.dim() != 3 || w.dim() != 3 || groups < 2) return false;
    const int64_t b = x.size(0), cin = x.size(1), len = x.size(2), cout = w.size(0), k = w.size(2), lo = out_len(len, k, stride, pad, dil);
    if (lo < 1 || w.size(1) * groups != cin) return false;
    const fp p = (fp)x.data_ptr(), q = (fp)w.data_ptr();
    return c.run({b, cout, lo}, x, [=](void *y, hipStream_t s) { return sws_conv1d(p, q, (float *)y, b, cin, len, cout, (int32_t)k, stride, pad, dil, groups, s); });
} SWS_END

SWS_CALL(conv1d_16, 6) {
    const int stride = c.num(2), pad = c.num(3), dil = c.num(4), groups = c.num(5);
    const at::Tensor &x = c.tensor(0, true), &w = c.tensor(1);
    if (c.odd || x.dim() != 3 || w.dim() != 3) return false;
    const int64_t b = x.size(0), cin = x.size(1), len = x.size(2), cout = w.size(0), k = w.size(2), lo = out_len(len, k, stride, pad, dil);
    if (lo < 1 || w.size(1) * groups != cin) return false;
    const int dt = c.dtype(x);
    const void *const p = x.data_ptr();
    const fp q = (fp)w.data_ptr();
    return c.run({b, cout, lo}, x, [=](void *y, hipStream_t s) {
        return sws_conv1d_16((sws_dtype)dt, p, q, y, b, cin, len, cout, (int32_t)k, stride, pad, dil, groups, s);
    });
} SWS_END

SWS_CALL(conv1d_grad_input, 7) {
    const int len = c.num(2), stride = c.num(3), pad = c.num(4), dil = c.num(5), groups = c.num(6);
    const at::Tensor &gy = c.tensor(0), &w = c.tensor(1);
    if (c.odd || gy.dim() != 3 || w.dim() != 3 || groups < 2) return false;
    const int64_t b = gy.size(0), cout = gy.size(1), lo = gy.size(2), cin = w.size(1) * groups, k = w.size(2);
    if (lo < 1 || w.size(0) != cout || lo != out_len(len, k, stride, pad, dil)) return false;
    const fp p = (fp)gy.data_ptr(), q = (fp)w.data_ptr();
    return c.run({b, cin, len}, gy, [=](void *gx, hipStream_t s) {
        return sws_conv1d_grad_input(p, q, (float *)gx, b, cin, len, cout, (int32_t)k, stride, pad, dil, groups, s);
    });
} SWS_END

SWS_CALL(conv1d_grad_weight, 7) {
    const int k = c.num(2), stride = c.num(3), pad = c.num(4), dil = c.num(5), groups = c.num(6);
    const at::Tensor &x = c.tensor(0), &gy = c.tensor(1);
    if (c.odd || x.dim() != 3 || gy.dim() != 3 || groups < 2) return false;
    const int64_t b = x.size(0), cin = x.size(1), len = x.size(2), cout = gy.size(1), lo = gy.size(2);
    if (lo < 1 || gy.size(0) != b || cin % groups != 0 || lo != out_len(len, k, stride, pad, dil)) return false;
    const fp p = (fp)x.data_ptr(), q = (fp)gy.data_ptr();
    return c.run({cout, cin / groups, k}, x, [=](void *gw, hipStream_t s) {
        return sws_conv1d_grad_weight(p, q, (float *)gw, b, cin, len, cout, k, stride, pad, dil, groups, s);
    });
} SWS_END

PyObject *set_error(PyObject *, PyObject *cls)
{
    Py_INCREF(cls);
    Py_XSETREF(g_error, cls);
    Py_RETURN_NONE;
}

#define SWS_METHOD(NAME) {#NAME, (PyCFunction)(void (*)(void))NAME, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    SWS_METHOD(slide1d), SWS_METHOD(slide1d_16), SWS_METHOD(slide1d_padded), SWS_METHOD(pool2d), SWS_METHOD(pool2d_16), SWS_METHOD(maxpool2d_grad),
    SWS_METHOD(avgpool2d_grad), SWS_METHOD(conv1d), SWS_METHOD(conv1d_16), SWS_METHOD(conv1d_grad_input), SWS_METHOD(conv1d_grad_weight),
    {"set_error", set_error, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// torch_version: the one whose headers this was built with, for binding.py to compare
PyMODINIT_FUNC PyInit__calls()
{
    PyObject *m = PyModule_Create(&module_def);
    if (m && PyModule_AddStringConstant(m, "torch_version", SWS_TORCH_VERSION) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
