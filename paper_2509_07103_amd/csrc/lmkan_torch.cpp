// The per-call part of binding.py in native code: check the tensors, allocate what the caller did not
// bring, find the current stream, call the library.  With tables and batches small enough for one
// launch per call, marshalling in Python took longer than the GPU did (forward 12.4 us per call, of
// which the library and its launch are 4).
//
// Only the ordinary case is handled here.  Anything else (a tensor of the wrong type, shape or device, a
// status other than LMKAN_OK) makes a function return None without having launched anything that
// counts, and binding.py goes its own way, which raises the error that describes it.
#include <Python.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>

#include "lmkan.h"

namespace {

// addresses of the library that binding.py has loaded
struct Library {
    decltype(&lmkan_workspace_bytes) workspace_bytes;
    decltype(&lmkan_packed_bytes) packed_bytes;
    decltype(&lmkan_forward) forward;
    decltype(&lmkan_backward) backward;
    decltype(&lmkan_conv2d_rows) conv2d_rows;
    decltype(&lmkan_conv2d_forward) conv2d_forward;
    decltype(&lmkan_conv2d_backward) conv2d_backward;
    decltype(&lmkan_pack) pack;
} g_lib;

// attribute names, interned once
enum { kNIn, kNOut, kGrid, kOrder, kDtype, kLayout, kFlags, kDescNames };
enum { kN, kH, kW, kCIn, kKh, kKw, kStride, kConvNames };
PyObject *g_desc_names[kDescNames], *g_conv_names[kConvNames];

template <int N>
bool read_ints(PyObject *obj, PyObject *const (&names)[N], int32_t (&out)[N])
{
    for (int i = 0; i < N; ++i) {
        PyObject *v = PyObject_GetAttr(obj, names[i]);
        const long n = v ? PyLong_AsLong(v) : -1;
        Py_XDECREF(v);
        if ((n == -1 && PyErr_Occurred()) || n < INT32_MIN || n > INT32_MAX) {
            PyErr_Clear();
            return false;
        }
        out[i] = (int32_t)n;
    }
    return true;
}

bool read_desc(PyObject *obj, lmkan_desc &d)
{
    int32_t v[kDescNames];
    if (!read_ints(obj, g_desc_names, v)) return false;
    d = {v[kNIn], v[kNOut], v[kGrid], v[kOrder], v[kDtype], v[kLayout], v[kFlags]};
    return d.n_in >= 2 && d.n_out >= 1 && d.grid >= 3 && d.grid <= LMKAN_MAX_GRID && d.coef_dtype >= 0 && d.coef_dtype <= 2;
}

at::ScalarType coef_type(const lmkan_desc &d)
{
    return d.coef_dtype == LMKAN_F32 ? at::kFloat : d.coef_dtype == LMKAN_F16 ? at::kHalf : at::kBFloat16;
}

// the tensor behind a Python object, or nullptr
const at::Tensor *tensor(PyObject *o) { return THPVariable_Check(o) ? &THPVariable_Unpack(o) : nullptr; }

bool fits(const at::Tensor *t, at::ScalarType type, at::IntArrayRef shape)
{
    return t && t->is_cuda() && t->scalar_type() == type && t->sizes() == shape && t->is_contiguous();
}

std::array<int64_t, 4> coef_shape(const lmkan_desc &d) { return {d.grid + 1, d.grid + 1, d.n_in / 2, d.n_out}; }

bool coef_fits(const lmkan_desc &d, const at::Tensor *t)
{
    if (d.coef_layout == LMKAN_LAYOUT_PACKED)
        return fits(t, coef_type(d), {(int64_t)(g_lib.packed_bytes(&d) / (d.coef_dtype == LMKAN_F32 ? 4 : 2))});
    return fits(t, coef_type(d), coef_shape(d));
}

void *data(const at::Tensor &t) { return t.defined() ? t.data_ptr() : nullptr; }

void *current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// the caller's workspace, or one of the size the library asks for
bool workspace(PyObject *given, const lmkan_desc &d, int64_t rows, int pass, const at::Tensor &like, at::Tensor &ws, size_t &bytes)
{
    if (given != Py_None) {
        const at::Tensor *t = tensor(given);
        if (!t || !t->is_cuda() || !t->is_contiguous()) return false;
        ws = *t;
        bytes = t->nbytes();
        return true;
    }
    bytes = g_lib.workspace_bytes(&d, rows, pass);
    if (bytes > 0) ws = at::empty({(int64_t)bytes}, like.options().dtype(at::kByte));
    return true;
}

// an output the caller brought, or a new one
bool output(PyObject *given, at::IntArrayRef shape, const at::Tensor &like, at::Tensor &out)
{
    if (given == Py_None) {
        out = at::empty(shape, like.options());
        return true;
    }
    const at::Tensor *t = tensor(given);
    if (!fits(t, at::kFloat, shape)) return false;
    out = *t;
    return true;
}

PyObject *wrap(const at::Tensor &t)
{
    if (!t.defined()) Py_RETURN_NONE;
    return THPVariable_Wrap(t);
}

// geometry of a convolution (conv not None): shapes of the image and of the output, rows of the layer
struct Rows {
    lmkan_conv2d conv;
    bool is_conv = false;
    int64_t rows = 0;
    std::vector<int64_t> in, out;
};

bool read_rows(PyObject *conv, const lmkan_desc &d, const at::Tensor *x, Rows &r)
{
    if (!x) return false;
    if (conv == Py_None) {
        if (x->dim() != 2) return false;
        r.rows = x->size(0);
        r.in = {r.rows, d.n_in};
        r.out = {r.rows, d.n_out};
    } else {
        int32_t v[kConvNames], oh = 0, ow = 0;
        if (!read_ints(conv, g_conv_names, v)) return false;
        r.conv = {v[kN], v[kH], v[kW], v[kCIn], v[kKh], v[kKw], v[kStride]};
        r.is_conv = true;
        r.rows = g_lib.conv2d_rows(&r.conv, &oh, &ow);
        r.in = {v[kN], v[kH], v[kW], v[kCIn]};
        r.out = {v[kN], oh, ow, d.n_out};
    }
    return r.rows >= 0 && fits(x, at::kFloat, r.in);
}

// The Python exception of a C++ one, as torch's own functions raise it: running out of memory stays
// torch.OutOfMemoryError, which callers catch to go on with a smaller batch
PyObject *raise_in_python(const std::exception_ptr &e)
{
    torch::translate_exception_to_python(e);
    return nullptr;
}

// every function: arguments by position, None when binding.py has to take over
#define LMKAN_GUARDED_BEGIN try {
#define LMKAN_GUARDED_END                                                  \
    }                                                                      \
    catch (...)                                                            \
    {                                                                      \
        return raise_in_python(std::current_exception());                  \
    }

// forward(desc, conv, x, coef, y, workspace) -> y
PyObject *forward(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 6) Py_RETURN_NONE;
    LMKAN_GUARDED_BEGIN
    lmkan_desc d;
    Rows r;
    const at::Tensor *x = tensor(args[2]), *coef = tensor(args[3]);
    at::Tensor y, ws;
    size_t bytes = 0;
    if (!read_desc(args[0], d) || !read_rows(args[1], d, x, r) || !coef_fits(d, coef) ||
        !output(args[4], r.out, *x, y) || !workspace(args[5], d, r.rows, 0, *x, ws, bytes))
        Py_RETURN_NONE;
    lmkan_status st;
    float *xp = static_cast<float *>(data(*x)), *yp = static_cast<float *>(data(y));
    void *s = current_stream(), *cp = data(*coef), *wp = data(ws);
    Py_BEGIN_ALLOW_THREADS
    st = r.is_conv ? g_lib.conv2d_forward(&d, &r.conv, xp, cp, yp, wp, bytes, s)
                   : g_lib.forward(&d, r.rows, xp, cp, yp, wp, bytes, s);
    Py_END_ALLOW_THREADS
    if (st != LMKAN_OK) Py_RETURN_NONE;
    return wrap(y);
    LMKAN_GUARDED_END
}

// backward(desc, conv, x, coef, grad_y, need_x, need_coef, grad_x, grad_coef, workspace) -> (grad_x, grad_coef)
PyObject *backward(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 10) Py_RETURN_NONE;
    LMKAN_GUARDED_BEGIN
    lmkan_desc d;
    Rows r;
    const at::Tensor *x = tensor(args[2]), *coef = tensor(args[3]), *gy = tensor(args[4]);
    const bool need_x = args[5] == Py_True, need_coef = args[6] == Py_True;
    if ((!need_x && args[5] != Py_False) || (!need_coef && args[6] != Py_False)) Py_RETURN_NONE;
    at::Tensor gx, gp, ws;
    size_t bytes = 0;
    if (!read_desc(args[0], d) || !read_rows(args[1], d, x, r) || !(args[3] == Py_None || coef_fits(d, coef)) ||
        !fits(gy, at::kFloat, r.out))
        Py_RETURN_NONE;
    if (need_coef && args[8] == Py_None && (d.flags & LMKAN_FLAG_ACCUMULATE_GRAD_COEF)) Py_RETURN_NONE;
    if ((need_x && !output(args[7], r.in, *x, gx)) || (need_coef && !output(args[8], coef_shape(d), *x, gp)) ||
        !workspace(args[9], d, r.rows, need_x && need_coef ? 1 : need_x ? 2 : 3, *x, ws, bytes))
        Py_RETURN_NONE;
    lmkan_status st;
    float *xp = static_cast<float *>(data(*x)), *gyp = static_cast<float *>(data(*gy));
    float *gxp = static_cast<float *>(data(gx)), *gpp = static_cast<float *>(data(gp));
    void *s = current_stream(), *cp = coef ? data(*coef) : nullptr, *wp = data(ws);
    Py_BEGIN_ALLOW_THREADS
    st = r.is_conv ? g_lib.conv2d_backward(&d, &r.conv, xp, cp, gyp, gxp, gpp, wp, bytes, s)
                   : g_lib.backward(&d, r.rows, xp, cp, gyp, gxp, gpp, wp, bytes, s);
    Py_END_ALLOW_THREADS
    if (st != LMKAN_OK) Py_RETURN_NONE;
    PyObject *a = wrap(gx), *b = wrap(gp), *pair = a && b ? PyTuple_Pack(2, a, b) : nullptr;
    Py_XDECREF(a);
    Py_XDECREF(b);
    return pair;
    LMKAN_GUARDED_END
}

// pack(desc, coef) -> packed table
PyObject *pack(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 2) Py_RETURN_NONE;
    LMKAN_GUARDED_BEGIN
    lmkan_desc d;
    const at::Tensor *coef = tensor(args[1]);
    if (!read_desc(args[0], d) || !fits(coef, coef_type(d), coef_shape(d))) Py_RETURN_NONE;
    const int64_t elems = (int64_t)(g_lib.packed_bytes(&d) / (d.coef_dtype == LMKAN_F32 ? 4 : 2));
    if (elems == 0) Py_RETURN_NONE;
    const at::Tensor out = at::empty({elems}, coef->options());
    lmkan_status st;
    void *s = current_stream(), *src = data(*coef), *dst = data(out);
    Py_BEGIN_ALLOW_THREADS
    st = g_lib.pack(&d, src, dst, s);
    Py_END_ALLOW_THREADS
    if (st != LMKAN_OK) Py_RETURN_NONE;
    return wrap(out);
    LMKAN_GUARDED_END
}

// init(the addresses, in the order of Library)
PyObject *init(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != (Py_ssize_t)(sizeof(Library) / sizeof(void *))) {
        PyErr_SetString(PyExc_ValueError, "init: one address per library function");
        return nullptr;
    }
    for (Py_ssize_t i = 0; i < n; ++i) {
        void *p = PyLong_AsVoidPtr(args[i]);
        if (!p) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "init: null address");
            return nullptr;
        }
        reinterpret_cast<void **>(&g_lib)[i] = p;
    }
    Py_RETURN_NONE;
}

PyMethodDef g_methods[] = {{"init", (PyCFunction)(void (*)(void))init, METH_FASTCALL, nullptr},
                           {"forward", (PyCFunction)(void (*)(void))forward, METH_FASTCALL, nullptr},
                           {"backward", (PyCFunction)(void (*)(void))backward, METH_FASTCALL, nullptr},
                           {"pack", (PyCFunction)(void (*)(void))pack, METH_FASTCALL, nullptr},
                           {nullptr, nullptr, 0, nullptr}};

PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void)
{
    static const char *desc[] = {"n_in", "n_out", "grid", "spline_order", "coef_dtype", "coef_layout", "flags"};
    static const char *conv[] = {"n", "h", "w", "c_in", "kh", "kw", "stride"};
    for (int i = 0; i < kDescNames; ++i) g_desc_names[i] = PyUnicode_InternFromString(desc[i]);
    for (int i = 0; i < kConvNames; ++i) g_conv_names[i] = PyUnicode_InternFromString(conv[i]);
    return PyModule_Create(&g_module);
}
