// The binding's small calls in native code: arguments taken from Python, the output allocated, the library's entry called.
//
// A call that the GPU finishes in 3 - 8 us is bound by the host.  In Python a sliding sum over one series takes 6.6 us of it (3.1 in HIP's
// launch, 1.4 in allocating, the rest in look-ups, checks and ctypes), a pooling call 7.2; here 4.3 and 4.5, and three of them are the launch.
//
// Every function returns None where anything is out of the ordinary (another type of argument, a tensor that is no plain one of
// the current device, a mode that watches calls, lengths that do not fit): binding.py's Python code then does the same call,
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

struct Odd {};                                        // not for here

// an exact int of 31 bits
int32_t num(PyObject *o)
{
    if (!PyLong_CheckExact(o)) throw Odd();
    int over = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &over);
    if (over || v < 0 || v > 0x7fffffff) throw Odd();
    return (int32_t)v;
}

float real(PyObject *o)
{
    if (PyFloat_CheckExact(o)) return (float)PyFloat_AS_DOUBLE(o);
    return (float)num(o);
}

// a contiguous tensor with memory of the current device, and nothing that wraps or watches it
const at::Tensor &tensor(PyObject *o, int device)
{
    if (!THPVariable_CheckExact(o)) throw Odd();
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.device().index() != device || t.layout() != c10::kStrided || !t.has_storage() || !t.is_contiguous() ||
        t.key_set().has_any(c10::DispatchKeySet({c10::DispatchKey::Python, c10::DispatchKey::Functionalize})))
        throw Odd();
    return t;
}
const at::Tensor &f32(PyObject *o, int device)
{
    const at::Tensor &t = tensor(o, device);
    if (t.scalar_type() != at::kFloat) throw Odd();
    return t;
}
const at::Tensor &half(PyObject *o, int device, int *dtype)
{
    const at::Tensor &t = tensor(o, device);
    if (t.scalar_type() == at::kBFloat16) *dtype = SWS_DTYPE_BF16;
    else if (t.scalar_type() == at::kHalf) *dtype = SWS_DTYPE_F16;
    else throw Odd();
    return t;
}

// sws_out_len for numbers of 31 bits; nothing below 1 goes on here
int64_t out_len(int64_t n, int64_t w, int64_t stride, int64_t pad, int64_t dilation = 1)
{
    if (w < 1 || stride < 1 || dilation < 1) throw Odd();
    const int64_t left = n + 2 * pad - dilation * (w - 1) - 1;
    if (left < 0) throw Odd();
    return left / stride + 1;
}
void same(bool ok) { if (!ok) throw Odd(); }

// F(device, stream) -> the output; F allocates, then calls the library through `go`
struct Call {
    const char *name;
    int device;
    hipStream_t stream;
    at::Tensor out;
    int rc = SWS_OK;
    template <class... P, class... A> void go_on(sws_status (*entry)(P...), A... a)
    {
        PyThreadState *save = PyEval_SaveThread();
        rc = entry(static_cast<P>(a)...);
        PyEval_RestoreThread(save);
    }
    template <class E, class... A> void go(E entry, A... a) { go_on(entry, a..., stream); }
    template <class S> void *alloc(const S &sizes, const at::Tensor &like)
    {
        out = at::empty(sizes, like.options());
        return out.data_ptr();
    }
};

template <class F>
PyObject *call(const char *name, Py_ssize_t want, Py_ssize_t n, F f)
{
    try {
        if (n != want || c10::impl::TorchDispatchModeTLS::any_modes_set() || at::impl::torch_function_mode_enabled()) throw Odd();
        Call c;
        c.name = name;
        c.device = c10::hip::current_device();
        c.stream = c10::hip::getCurrentHIPStream((c10::DeviceIndex)c.device).stream();
        f(c);
        if (c.rc == SWS_OK) return THPVariable_Wrap(std::move(c.out));
        PyObject *e = PyObject_CallFunction(g_error, "is", c.rc, name);
        if (e) {
            PyErr_SetObject(g_error, e);
            Py_DECREF(e);
        }
        return nullptr;
    } catch (...) {                                   // (what torch throws too: the Python code meets it again)
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

typedef const float *fp;
#define SWS_CALL(NAME, N) PyObject *NAME(PyObject *, PyObject *const *a, Py_ssize_t n) { return call("sws_" #NAME, N, n, [&](Call &c)
#define SWS_END ); }

c10::SmallVector<int64_t, 6> with_last(const at::Tensor &t, int64_t last)
{
    same(t.dim() >= 1);
    c10::SmallVector<int64_t, 6> s(t.sizes().begin(), t.sizes().end());
    s.back() = last;
    return s;
}
int64_t rows(const at::Tensor &t) { return t.numel() / t.size(-1); }

SWS_CALL(slide1d, 4) {
    const int op = num(a[0]), w = num(a[2]);
    const at::Tensor &x = f32(a[1], c.device);
    const auto shape = with_last(x, out_len(x.dim() ? x.size(-1) : 0, w, 1, 0));
    float *y = (float *)c.alloc(shape, x);
    c.go(sws_slide1d, op, (fp)x.data_ptr(), y, rows(x), x.size(-1), w, real(a[3]));
} SWS_END

SWS_CALL(slide1d_16, 4) {
    int dt = 0;
    const int op = num(a[0]), w = num(a[2]);
    const at::Tensor &x = half(a[1], c.device, &dt);
    const auto shape = with_last(x, out_len(x.dim() ? x.size(-1) : 0, w, 1, 0));
    void *y = c.alloc(shape, x);
    c.go(sws_slide1d_16, op, dt, (const void *)x.data_ptr(), y, rows(x), x.size(-1), w, real(a[3]));
} SWS_END

SWS_CALL(slide1d_padded, 7) {
    const int op = num(a[0]), w = num(a[2]), left = num(a[3]), right = num(a[4]), mode = num(a[5]);
    const at::Tensor &x = f32(a[1], c.device);
    same(x.dim() >= 1 && x.size(-1) > 0);
    const auto shape = with_last(x, out_len(x.size(-1) + left + right, w, 1, 0));
    float *y = (float *)c.alloc(shape, x);
    c.go(sws_slide1d_padded, op, (fp)x.data_ptr(), y, rows(x), x.size(-1), w, left, right, mode, real(a[6]));
} SWS_END

SWS_CALL(pool2d, 9) {
    const int op = num(a[0]), kh = num(a[2]), kw = num(a[3]), sh = num(a[4]), sw = num(a[5]), ph = num(a[6]), pw = num(a[7]);
    const at::Tensor &x = f32(a[1], c.device);
    same(x.dim() == 4);
    float *y = (float *)c.alloc(at::IntArrayRef{x.size(0), x.size(1), out_len(x.size(2), kh, sh, ph), out_len(x.size(3), kw, sw, pw)}, x);
    c.go(sws_pool2d, op, (fp)x.data_ptr(), y, x.size(0), x.size(1), x.size(2), x.size(3), kh, kw, sh, sw, ph, pw, real(a[8]));
} SWS_END

SWS_CALL(pool2d_16, 9) {
    int dt = 0;
    const int op = num(a[0]), kh = num(a[2]), kw = num(a[3]), sh = num(a[4]), sw = num(a[5]), ph = num(a[6]), pw = num(a[7]);
    const at::Tensor &x = half(a[1], c.device, &dt);
    same(x.dim() == 4);
    void *y = c.alloc(at::IntArrayRef{x.size(0), x.size(1), out_len(x.size(2), kh, sh, ph), out_len(x.size(3), kw, sw, pw)}, x);
    c.go(sws_pool2d_16, op, dt, (const void *)x.data_ptr(), y, x.size(0), x.size(1), x.size(2), x.size(3), kh, kw, sh, sw, ph, pw, real(a[8]));
} SWS_END

SWS_CALL(maxpool2d_grad, 8) {
    const int kh = num(a[2]), kw = num(a[3]), sh = num(a[4]), sw = num(a[5]), ph = num(a[6]), pw = num(a[7]);
    const at::Tensor &x = f32(a[0], c.device), &gy = f32(a[1], c.device);
    same(x.dim() == 4 && gy.dim() == 4 && gy.size(0) == x.size(0) && gy.size(1) == x.size(1) &&
         gy.size(2) == out_len(x.size(2), kh, sh, ph) && gy.size(3) == out_len(x.size(3), kw, sw, pw));
    float *gx = (float *)c.alloc(x.sizes(), x);
    c.go(sws_maxpool2d_grad, (fp)x.data_ptr(), (fp)gy.data_ptr(), gx, x.size(0), x.size(1), x.size(2), x.size(3), kh, kw, sh, sw, ph, pw);
} SWS_END

SWS_CALL(avgpool2d_grad, 11) {
    const int h = num(a[1]), w = num(a[2]), kh = num(a[3]), kw = num(a[4]), sh = num(a[5]), sw = num(a[6]), ph = num(a[7]), pw = num(a[8]), div = num(a[9]);
    const at::Tensor &gy = f32(a[0], c.device);
    same(gy.dim() == 4 && gy.size(2) == out_len(h, kh, sh, ph) && gy.size(3) == out_len(w, kw, sw, pw));
    float *gx = (float *)c.alloc(at::IntArrayRef{gy.size(0), gy.size(1), h, w}, gy);
    c.go(sws_avgpool2d_grad, (fp)gy.data_ptr(), gx, gy.size(0), gy.size(1), (int64_t)h, (int64_t)w, kh, kw, sh, sw, ph, pw, div, real(a[10]));
} SWS_END

// layers of several groups: none of their kernels uses a workspace
SWS_CALL(conv1d, 6) {
    const int stride = num(a[2]), pad = num(a[3]), dil = num(a[4]), groups = num(a[5]);
    const at::Tensor &x = f32(a[0], c.device), &w = f32(a[1], c.device);
    same(x.dim() == 3 && w.dim() == 3 && groups > 1 && w.size(1) * groups == x.size(1));
    float *y = (float *)c.alloc(at::IntArrayRef{x.size(0), w.size(0), out_len(x.size(2), w.size(2), stride, pad, dil)}, x);
    c.go(sws_conv1d, (fp)x.data_ptr(), (fp)w.data_ptr(), y, x.size(0), x.size(1), x.size(2), w.size(0), (int32_t)w.size(2), stride, pad, dil, groups);
} SWS_END

SWS_CALL(conv1d_16, 6) {
    int dt = 0;
    const int stride = num(a[2]), pad = num(a[3]), dil = num(a[4]), groups = num(a[5]);
    const at::Tensor &x = half(a[0], c.device, &dt), &w = f32(a[1], c.device);
    same(x.dim() == 3 && w.dim() == 3 && w.size(1) * groups == x.size(1));
    void *y = c.alloc(at::IntArrayRef{x.size(0), w.size(0), out_len(x.size(2), w.size(2), stride, pad, dil)}, x);
    c.go(sws_conv1d_16, dt, (const void *)x.data_ptr(), (fp)w.data_ptr(), y, x.size(0), x.size(1), x.size(2), w.size(0), (int32_t)w.size(2), stride, pad, dil,
         groups);
} SWS_END

SWS_CALL(conv1d_grad_input, 7) {
    const int length = num(a[2]), stride = num(a[3]), pad = num(a[4]), dil = num(a[5]), groups = num(a[6]);
    const at::Tensor &gy = f32(a[0], c.device), &w = f32(a[1], c.device);
    same(gy.dim() == 3 && w.dim() == 3 && groups > 1 && w.size(0) == gy.size(1) && gy.size(2) == out_len(length, w.size(2), stride, pad, dil));
    const int64_t cin = w.size(1) * groups;
    float *gx = (float *)c.alloc(at::IntArrayRef{gy.size(0), cin, length}, gy);
    c.go(sws_conv1d_grad_input, (fp)gy.data_ptr(), (fp)w.data_ptr(), gx, gy.size(0), cin, (int64_t)length, gy.size(1), (int32_t)w.size(2), stride, pad, dil,
         groups);
} SWS_END

SWS_CALL(conv1d_grad_weight, 7) {
    const int k = num(a[2]), stride = num(a[3]), pad = num(a[4]), dil = num(a[5]), groups = num(a[6]);
    const at::Tensor &x = f32(a[0], c.device), &gy = f32(a[1], c.device);
    same(x.dim() == 3 && gy.dim() == 3 && groups > 1 && gy.size(0) == x.size(0) && x.size(1) % groups == 0 &&
         gy.size(2) == out_len(x.size(2), k, stride, pad, dil));
    float *gw = (float *)c.alloc(at::IntArrayRef{gy.size(1), x.size(1) / groups, k}, x);
    c.go(sws_conv1d_grad_weight, (fp)x.data_ptr(), (fp)gy.data_ptr(), gw, x.size(0), x.size(1), x.size(2), gy.size(1), k, stride, pad, dil, groups);
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

PyMODINIT_FUNC PyInit__calls() { return PyModule_Create(&module_def); }
