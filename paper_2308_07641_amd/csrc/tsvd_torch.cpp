// Argument marshalling of the forward entry points for torch tensors, as a CPython extension: the checks, the
// allocation of an omitted result and the call into libtsvd.so (host code only, no arithmetic).
//
// Why native: a small call is bound by the host.  On MI355X the library's own call (one launch) costs 3.7 us of host
// time; reading a dozen tensor properties, looking up the current stream and converting thirteen arguments for ctypes
// in Python cost another 4.7 us (1.9 us of them the stream lookup), more than the GPU works on a 256 x 256 layer: the
// single-token call took 8.4 us through that path and 5.7 us without it.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>

#include <algorithm>
#include <cstdint>
#include <vector>

#include "../../include/tsvd.h"
#include "../../include/tsvd_conv.h"

namespace {

PyObject* error_class = nullptr;       // TsvdError(status, where)
PyObject* raw_stream = nullptr;        // device index -> hipStream_t of torch's current stream, as an int
PyObject *name_ptr, *name_M, *name_N;

struct failed {};                      // a Python error is set

[[noreturn]] void raise(PyObject* type, const char* text) {
    PyErr_SetString(type, text);
    throw failed();
}

int64_t attr_int(PyObject* o, PyObject* name) {
    PyObject* v = PyObject_GetAttr(o, name);
    if (!v) throw failed();
    const long long r = v == Py_None ? 0 : PyLong_AsLongLong(v);
    Py_DECREF(v);
    if (r == -1 && PyErr_Occurred()) throw failed();
    return r;
}

struct handle_view {
    const tsvd_handle* ptr;            // null after tsvd_free: the library rejects it
    int64_t M, N;
};
handle_view handle_of(PyObject* h) {
    return {reinterpret_cast<const tsvd_handle*>((uintptr_t)attr_int(h, name_ptr)), attr_int(h, name_M), attr_int(h, name_N)};
}

const at::Tensor& tensor_of(PyObject* o, const char* what) {
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s must be a torch tensor, not %.100s", what, Py_TYPE(o)->tp_name);
        throw failed();
    }
    return THPVariable_Unpack(o);
}

tsvd_dtype dtype_code(const at::Tensor& t) {
    if (t.scalar_type() == at::kFloat) return TSVD_F32;
    if (t.scalar_type() == at::kBFloat16) return TSVD_BF16;
    PyErr_Format(PyExc_TypeError, "unsupported activation dtype %s", at::toString(t.scalar_type()));
    throw failed();
}

int64_t integer(PyObject* o) {
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw failed();
    return v;
}

void* stream_of(PyObject* stream, const at::Tensor& x) {
    PyObject* v = nullptr;
    if (stream == Py_None) {
        PyObject* index = PyLong_FromLong(x.device().index());
        v = index ? PyObject_CallOneArg(raw_stream, index) : nullptr;
        Py_XDECREF(index);
        if (!v) throw failed();
    } else {
        v = Py_NewRef(stream);
    }
    void* s = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    if (!s && PyErr_Occurred()) throw failed();
    return s;
}

void check(tsvd_status st, const char* where) {
    if (st == TSVD_OK) return;
    PyObject* e = PyObject_CallFunction(error_class, "is", (int)st, where);
    if (e) {
        PyErr_SetObject(error_class, e);
        Py_DECREF(e);
    }
    throw failed();
}

const float* bias_of(PyObject* bias, int64_t M, const char* text) {
    if (bias == Py_None) return nullptr;
    const at::Tensor& b = tensor_of(bias, "bias");
    if (b.scalar_type() != at::kFloat || b.dim() != 1 || b.size(0) != M || !b.is_cuda() || !b.is_contiguous()) raise(PyExc_ValueError, text);
    return static_cast<const float*>(b.data_ptr());
}

struct workspace_view {
    void* ptr;
    size_t bytes;
};
workspace_view workspace_of(PyObject* ws) {
    if (ws == Py_None) return {nullptr, 0};
    const at::Tensor& w = tensor_of(ws, "workspace");
    return {w.data_ptr(), (size_t)w.numel() * w.element_size()};
}

// Activations and result of a call after the checks; `y` is the caller's tensor or a new one.
struct io {
    const at::Tensor* x;
    PyObject* y;                       // new reference
    const at::Tensor* yt;
    int64_t B, ldx, ldy;
    tsvd_dtype x_dtype, y_dtype;
};

struct y_ref {                         // drops the result when the call fails
    PyObject* p;
    ~y_ref() { Py_XDECREF(p); }
    PyObject* release() { PyObject* r = p; p = nullptr; return r; }
};

// rows: the extent of y's first dimension; must_give: no allocation
PyObject* result_of(PyObject* y, int64_t rows, int64_t cols, at::ScalarType dt, const at::Tensor& x, const char* text) {
    if (y == Py_None) return THPVariable_Wrap(at::empty({rows, cols}, x.options().dtype(dt)));
    const at::Tensor& t = tensor_of(y, "y");
    if (t.scalar_type() != dt || t.dim() != 2 || t.size(0) != rows || t.size(1) != cols || t.stride(1) != 1 || !t.is_cuda())
        raise(PyExc_ValueError, text);
    return Py_NewRef(y);
}

int64_t row_pitch(const at::Tensor& t) { return t.size(0) > 1 ? t.stride(0) : std::max<int64_t>(t.size(1), t.stride(0)); }

void need_args(Py_ssize_t got, Py_ssize_t want, const char* name) {
    if (got != want) {
        PyErr_Format(PyExc_TypeError, "%s takes %zd arguments", name, want);
        throw failed();
    }
}

template <typename F>
PyObject* guarded(F&& body) {
    try {
        return body();
    } catch (const failed&) {
        return nullptr;
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// forward(h, x, y, workspace, stream)
PyObject* py_forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        need_args(n, 5, "forward");
        const handle_view h = handle_of(a[0]);
        const at::Tensor& x = tensor_of(a[1], "x");
        if (!x.is_cuda()) raise(PyExc_ValueError, "x must live on the GPU");
        const int64_t d = x.dim();
        // a vector is one token: [N] reads as [N, 1]
        if ((d != 1 && d != 2) || x.size(0) != h.N || (d == 2 && x.stride(1) != 1))
            raise(PyExc_ValueError, "x must be [N,B] with unit column stride");
        const int64_t B = d == 2 ? x.size(1) : 1;
        const int64_t ldx = x.size(0) > 1 ? x.stride(0) : std::max(B, x.stride(0));
        y_ref y{result_of(a[2], h.M, B, at::kFloat, x, "y must be a float32 GPU tensor [M,B] with unit column stride")};
        if (!y.p) throw failed();
        const at::Tensor& yt = THPVariable_Unpack(y.p);
        const workspace_view ws = workspace_of(a[3]);
        void* stream = stream_of(a[4], x);
        const tsvd_dtype xd = dtype_code(x);
        const void* xp = x.data_ptr();
        void* yp = yt.data_ptr();
        const int64_t ldy = row_pitch(yt);
        tsvd_status st;
        Py_BEGIN_ALLOW_THREADS
        st = tsvd_forward(h.ptr, xp, xd, B, ldx, yp, TSVD_F32, ldy, ws.ptr, ws.bytes, stream);
        Py_END_ALLOW_THREADS
        check(st, "tsvd_forward");
        return y.release();
    });
}

// layer(h, x, x_layout, bias, y, y_dtype, y_layout, workspace, stream, entry): the forward entry points with options;
// entry 0 tsvd_forward_ex, 1 tsvd_forward_io, 2 tsvd_forward_noalloc
PyObject* py_layer(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        need_args(n, 10, "layer");
        static const char* const where[] = {"tsvd_forward_ex", "tsvd_forward_io", "tsvd_forward_noalloc"};
        static const char* const y_text[] = {"y must be a GPU tensor [M,B] of the requested type with unit column stride",
                                             "y must be a GPU tensor of the requested type and layout with unit inner stride",
                                             "y must be a GPU tensor [M,B] of the requested type with unit column stride"};
        const int entry = (int)integer(a[9]);
        const handle_view h = handle_of(a[0]);
        const at::Tensor& x = tensor_of(a[1], "x");
        if (!x.is_cuda() || x.dim() != 2 || x.stride(1) != 1) raise(PyExc_ValueError, "x must be a 2-d GPU tensor with unit inner stride");
        const tsvd_layout xl = (tsvd_layout)integer(a[2]), yl = (tsvd_layout)integer(a[6]);
        const int64_t yd = integer(a[5]);
        const bool xt = xl == TSVD_TOKEN_MAJOR, ytm = yl == TSVD_TOKEN_MAJOR;
        const int64_t B = x.size(xt ? 0 : 1);
        if (x.size(xt ? 1 : 0) != h.N) raise(PyExc_ValueError, "x does not have N features");
        y_ref y{result_of(a[4], ytm ? B : h.M, ytm ? h.M : B, yd == TSVD_BF16 ? at::kBFloat16 : at::kFloat, x, y_text[entry])};
        if (!y.p) throw failed();
        const at::Tensor& yt = THPVariable_Unpack(y.p);
        const float* bias = bias_of(a[3], h.M, "bias must be a contiguous float32 GPU tensor [M]");
        const workspace_view ws = workspace_of(a[7]);
        void* stream = stream_of(a[8], x);
        const tsvd_dtype xd = dtype_code(x);
        const void* xp = x.data_ptr();
        void* yp = yt.data_ptr();
        const int64_t ldx = row_pitch(x), ldy = row_pitch(yt);
        tsvd_status st;
        Py_BEGIN_ALLOW_THREADS
        st = entry == 0   ? tsvd_forward_ex(h.ptr, xp, xd, xl, B, ldx, bias, yp, (tsvd_dtype)yd, ldy, ws.ptr, ws.bytes, stream)
             : entry == 1 ? tsvd_forward_io(h.ptr, xp, xd, xl, B, ldx, bias, yp, (tsvd_dtype)yd, yl, ldy, ws.ptr, ws.bytes, stream)
                          : tsvd_forward_noalloc(h.ptr, xp, xd, xl, B, ldx, bias, yp, (tsvd_dtype)yd, ldy, stream);
        Py_END_ALLOW_THREADS
        check(st, where[entry]);
        return y.release();
    });
}

// conv2d(h, form, c_in, c_out, k1, k2, x, stride, pad, dil, bias, y_dtype, stream, groups)
PyObject* py_conv2d(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        need_args(n, 14, "conv2d");
        const handle_view h = handle_of(a[0]);
        auto pair = [&](PyObject* o, int32_t* first, int32_t* second) {
            PyObject* f = PySequence_Fast(o, "stride, pad and dil must be pairs");
            if (!f) throw failed();
            const bool two = PySequence_Fast_GET_SIZE(f) >= 2;
            const long v0 = two ? PyLong_AsLong(PySequence_Fast_GET_ITEM(f, 0)) : 0, v1 = two ? PyLong_AsLong(PySequence_Fast_GET_ITEM(f, 1)) : 0;
            Py_DECREF(f);
            if (PyErr_Occurred()) throw failed();
            if (!two) raise(PyExc_IndexError, "stride, pad and dil must be pairs");
            *first = (int32_t)v0;
            *second = (int32_t)v1;
        };
        tsvd_conv_geometry g;
        g.form = (int32_t)integer(a[1]); g.c_in = (int32_t)integer(a[2]); g.c_out = (int32_t)integer(a[3]);
        g.k1 = (int32_t)integer(a[4]); g.k2 = (int32_t)integer(a[5]);
        const at::Tensor& x = tensor_of(a[6], "x");
        if (!x.is_cuda() || x.scalar_type() != at::kBFloat16 || x.dim() != 4 || x.size(0) != g.c_in || !x.is_contiguous())
            raise(PyExc_ValueError, "x must be a contiguous bf16 GPU tensor [C_in, images, H, W]");
        pair(a[7], &g.stride1, &g.stride2);
        pair(a[8], &g.pad1, &g.pad2);
        pair(a[9], &g.dil1, &g.dil2);
        const tsvd_dtype yd = (tsvd_dtype)integer(a[11]);
        g.groups = (int32_t)integer(a[13]);
        const int64_t images = x.size(1), H = x.size(2), W = x.size(3);
        const size_t nbytes = tsvd_conv2d_workspace_bytes(h.ptr, &g, images, H, W);
        if (nbytes == 0) raise(PyExc_ValueError, "geometry does not fit the packed matrix (or is invalid)");
        const int64_t Ho = (H + 2 * (int64_t)g.pad1 - (int64_t)g.dil1 * (g.k1 - 1) - 1) / g.stride1 + 1;
        const int64_t Wo = (W + 2 * (int64_t)g.pad2 - (int64_t)g.dil2 * (g.k2 - 1) - 1) / g.stride2 + 1;
        const at::Tensor ws = at::empty({(int64_t)nbytes}, x.options().dtype(at::kByte));
        const at::Tensor y = at::empty({g.c_out, images, Ho, Wo}, x.options().dtype(yd == TSVD_BF16 ? at::kBFloat16 : at::kFloat));
        const float* bias = bias_of(a[10], g.c_out, "bias must be a contiguous GPU tensor torch.float32 [C_out]");
        void* stream = stream_of(a[12], x);
        const void* xp = x.data_ptr();
        void *yp = y.data_ptr(), *wp = ws.data_ptr();
        tsvd_status st;
        Py_BEGIN_ALLOW_THREADS
        st = tsvd_conv2d_forward(h.ptr, &g, xp, images, H, W, bias, yp, yd, wp, nbytes, stream);
        Py_END_ALLOW_THREADS
        check(st, "tsvd_conv2d_forward");
        return THPVariable_Wrap(y);
    });
}

// setup(error class, raw stream lookup)
PyObject* py_setup(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        need_args(n, 2, "setup");
        Py_XDECREF(error_class);
        Py_XDECREF(raw_stream);
        error_class = Py_NewRef(a[0]);
        raw_stream = Py_NewRef(a[1]);
        Py_RETURN_NONE;
    });
}

PyMethodDef methods[] = {
    {"setup", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_setup)), METH_FASTCALL, nullptr},
    {"forward", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_forward)), METH_FASTCALL, nullptr},
    {"layer", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_layer)), METH_FASTCALL, nullptr},
    {"conv2d", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_conv2d)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tsvd_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__tsvd_torch() {
    name_ptr = PyUnicode_InternFromString("ptr");
    name_M = PyUnicode_InternFromString("M");
    name_N = PyUnicode_InternFromString("N");
    return PyModule_Create(&module);
}
