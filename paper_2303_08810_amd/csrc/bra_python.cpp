// CPython extension of the binding: argument checks, output and workspace allocation, and the calls into
// libbra, natively.  A small layer on one image takes 12 us of GPU time; checked and marshalled in Python
// (ctypes), its call took 14 us of host time and set the pace.
//
// Functions here take every argument by position; the Python functions of the package give them their names and
// defaults.  No kernel lives here and nothing is computed.
#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/pybind.h>

#include "../../include/bra.h"

namespace {

PyObject *g_bra_error = nullptr;      // class BraError(code, text), set by init()

struct Raised {};                     // a Python exception is set

[[noreturn]] void value_error(const char *text)
{
    PyErr_SetString(PyExc_ValueError, text);
    throw Raised{};
}

void check(int rc)
{
    if (rc == BRA_OK) return;
    PyObject *e = PyObject_CallFunction(g_bra_error, "is", rc, bra_strerror(rc));
    if (e) {
        PyErr_SetObject(g_bra_error, e);
        Py_DECREF(e);
    }
    throw Raised{};
}

const at::Tensor *tensor(PyObject *o)
{
    if (o == Py_None) return nullptr;
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "expected a torch.Tensor, got %s", Py_TYPE(o)->tp_name);
        throw Raised{};
    }
    return &THPVariable_Unpack(o);
}

const at::Tensor &need(PyObject *o)
{
    const at::Tensor *t = tensor(o);
    if (!t) value_error("a required tensor is None");
    return *t;
}

// ints and what converts to one without loss (numpy integers, anything with __index__); no floats, no strings
int integer(PyObject *o)
{
    PyObject *i = PyNumber_Index(o);
    if (!i) throw Raised{};
    const long v = PyLong_AsLong(i);
    Py_DECREF(i);
    if (v == -1 && PyErr_Occurred()) throw Raised{};
    return (int)v;
}

// what float() takes
double real(PyObject *o)
{
    PyObject *f = PyNumber_Float(o);
    if (!f) throw Raised{};
    const double v = PyFloat_AS_DOUBLE(f);
    Py_DECREF(f);
    return v;
}

float scale_of(PyObject *o) { return o == Py_None ? 0.f : (float)real(o); }

int dtype_of(const at::Tensor &X)
{
    if (X.scalar_type() == at::kFloat) return BRA_F32;
    if (X.scalar_type() == at::kBFloat16) return BRA_BF16;
    PyErr_SetString(PyExc_TypeError, "tensors must be float32 or bfloat16");
    throw Raised{};
}

bool dims_are(const at::Tensor &t, std::initializer_list<int64_t> d) { return t.sizes().equals(at::IntArrayRef(d.begin(), d.size())); }

void same_kind(const at::Tensor &t, const at::Tensor &X)
{
    if (!(t.is_cuda() && t.is_contiguous() && t.scalar_type() == X.scalar_type() && t.device() == X.device()))
        value_error("tensors must be contiguous, on one GPU and of one dtype");
}

// The layer's inputs; fills the shape (scale and path apart).
bra_shape layer_shape(const at::Tensor &X, const at::Tensor &Wqkv, const at::Tensor *Wo, const at::Tensor *Wlce, int S,
                      int k, int heads, PyObject *scale, PyObject *path)
{
    const float scale_value = scale_of(scale);
    if (X.dim() != 4) value_error("X must be [B, H, W, C]");
    const int64_t C = X.size(3);
    same_kind(X, X);
    same_kind(Wqkv, X);
    if (Wo) same_kind(*Wo, X);
    if (Wlce) same_kind(*Wlce, X);
    if (!dims_are(Wqkv, {C, 3 * C})) value_error("Wqkv must be [C, 3C]");
    if (Wo && !dims_are(*Wo, {C, C})) value_error("Wo must be [C, C]");
    if (Wlce && !dims_are(*Wlce, {C, 5, 5})) value_error("Wlce must be [C, 5, 5]");
    for (int d = 0; d < 4; ++d)
        if (X.size(d) > INT32_MAX) value_error("X is too large");
    return bra_shape{(int32_t)X.size(0), (int32_t)X.size(1), (int32_t)X.size(2), (int32_t)C, heads, S, k, dtype_of(X),
                     scale_value, integer(path)};
}

void check_index(const at::Tensor *Ir, const bra_shape &s, const char *text)
{
    if (Ir && !(Ir->is_cuda() && Ir->is_contiguous() && Ir->scalar_type() == at::kInt &&
                dims_are(*Ir, {s.B, (int64_t)s.S * s.S, s.k})))
        value_error(text);
}

void *data(const at::Tensor *t) { return t ? t->data_ptr() : nullptr; }
void *stream_of(const at::Tensor &X) { return (void *)c10::hip::getCurrentHIPStream(X.device().index()).stream(); }

at::Tensor scratch(size_t bytes, const at::Tensor &X)
{
    return at::empty({(int64_t)std::max(bytes, (size_t)256)}, X.options().dtype(at::kByte));
}

at::Tensor new_index(const bra_shape &s, const at::Tensor &X)
{
    return at::empty({s.B, (int64_t)s.S * s.S, s.k}, X.options().dtype(at::kInt));
}

PyObject *wrap(at::Tensor t) { return THPVariable_Wrap(std::move(t)); }

PyObject *tuple(std::initializer_list<PyObject *> items)
{
    PyObject *t = PyTuple_New((Py_ssize_t)items.size());
    Py_ssize_t i = 0;
    for (PyObject *o : items) PyTuple_SET_ITEM(t, i++, o);
    return t;
}

// Runs `call` without the interpreter lock and turns its code into an exception.
template <typename F>
void run(F call)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS;
    rc = call();
    Py_END_ALLOW_THREADS;
    check(rc);
}

template <typename F>
PyObject *guarded(Py_ssize_t n, Py_ssize_t want, F body)
{
    if (n != want) {
        PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
        return nullptr;
    }
    try {
        return body();
    } catch (const Raised &) {
        return nullptr;
    } catch (const c10::OutOfMemoryError &e) {
        PyObject *m = PyImport_ImportModule("torch"), *cls = m ? PyObject_GetAttrString(m, "OutOfMemoryError") : nullptr;
        PyErr_SetString(cls ? cls : PyExc_RuntimeError, e.what_without_backtrace());
        Py_XDECREF(cls);
        Py_XDECREF(m);
        return nullptr;
    } catch (const c10::Error &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
        return nullptr;
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// init(BraError)
PyObject *py_init(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 1, [&]() -> PyObject * {
        Py_INCREF(a[0]);
        Py_XDECREF(g_bra_error);
        g_bra_error = a[0];
        Py_RETURN_NONE;
    });
}

// route(X, Wqkv, S, k, heads, want_Ar, path, ws)
PyObject *py_route(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 8, [&]() -> PyObject * {
        const at::Tensor &X = need(a[0]), &Wqkv = need(a[1]);
        const bra_shape s = layer_shape(X, Wqkv, nullptr, nullptr, integer(a[2]), integer(a[3]), integer(a[4]), Py_None, a[6]);
        at::Tensor own;
        const at::Tensor *ws = tensor(a[7]);
        if (!ws) {
            size_t bytes = 0;
            check(bra_workspace_bytes(&s, &bytes));
            own = scratch(bytes, X);
            ws = &own;
        }
        const bool want_ar = PyObject_IsTrue(a[5]);
        at::Tensor Ir = new_index(s, X), Ar;
        const int64_t R = (int64_t)s.S * s.S;
        if (want_ar) Ar = at::empty({s.B, R, R}, X.options().dtype(at::kFloat));
        void *st = stream_of(X);
        run([&] {
            return bra_route(&s, X.data_ptr(), Wqkv.data_ptr(), (int32_t *)Ir.data_ptr(),
                             want_ar ? (float *)Ar.data_ptr() : nullptr, ws->data_ptr(), (size_t)ws->numel(), st);
        });
        return want_ar ? tuple({wrap(Ir), wrap(Ar)}) : wrap(Ir);
    });
}

// forward(X, Wqkv, Wo, Wlce, S, k, heads, scale, Ir_in, want_Ir, path, ws, out)
PyObject *py_forward(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 13, [&]() -> PyObject * {
        const at::Tensor &X = need(a[0]), &Wqkv = need(a[1]), &Wo = need(a[2]), &Wlce = need(a[3]);
        const bra_shape s = layer_shape(X, Wqkv, &Wo, &Wlce, integer(a[4]), integer(a[5]), integer(a[6]), a[7], a[10]);
        const at::Tensor *Ir_in = tensor(a[8]), *ws = tensor(a[11]), *out = tensor(a[12]);
        at::Tensor own, Y, Ir;
        if (!ws) {
            size_t bytes = 0;
            check(bra_workspace_bytes(&s, &bytes));
            own = scratch(bytes, X);
            ws = &own;
        }
        Y = out ? *out : at::empty_like(X);
        const bool want_ir = PyObject_IsTrue(a[9]);
        if (want_ir) Ir = new_index(s, X);
        check_index(Ir_in, s, "Ir_in must be a contiguous int32 [B, S*S, k] device tensor");
        void *st = stream_of(X);
        run([&] {
            return bra_forward(&s, X.data_ptr(), Wqkv.data_ptr(), Wo.data_ptr(), Wlce.data_ptr(), Y.data_ptr(),
                               want_ir ? (int32_t *)Ir.data_ptr() : nullptr, (const int32_t *)data(Ir_in), ws->data_ptr(),
                               (size_t)ws->numel(), st);
        });
        PyObject *y;
        if (out) Py_INCREF(y = a[12]);
        else y = wrap(Y);
        return want_ir ? tuple({y, wrap(Ir)}) : y;
    });
}

// forward_static(X, Wqkv, Wo, Wlce, S, k, heads, out, Ir_out, Ir_in, scale, path)
PyObject *py_forward_static(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 12, [&]() -> PyObject * {
        const at::Tensor &X = need(a[0]), &Wqkv = need(a[1]), &Wo = need(a[2]), &Wlce = need(a[3]), &out = need(a[7]);
        const bra_shape s = layer_shape(X, Wqkv, &Wo, &Wlce, integer(a[4]), integer(a[5]), integer(a[6]), a[10], a[11]);
        const at::Tensor *Ir_out = tensor(a[8]), *Ir_in = tensor(a[9]);
        if (!(out.is_cuda() && out.is_contiguous() && out.scalar_type() == X.scalar_type() && out.sizes().equals(X.sizes())))
            value_error("out must be a contiguous device tensor of X's shape and dtype");
        check_index(Ir_out, s, "Ir_out must be a contiguous int32 [B, S*S, k] device tensor");
        check_index(Ir_in, s, "Ir_in must be a contiguous int32 [B, S*S, k] device tensor");
        void *st = stream_of(X);
        run([&] {
            return bra_forward_static(&s, X.data_ptr(), Wqkv.data_ptr(), Wo.data_ptr(), Wlce.data_ptr(), out.data_ptr(),
                                      (int32_t *)data(Ir_out), (const int32_t *)data(Ir_in), st);
        });
        Py_INCREF(a[7]);
        return a[7];
    });
}

// forward_padded(X, Wqkv, Wo, Wlce, S, k, heads, scale, Ir_in, want_Ir, path)
PyObject *py_forward_padded(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 11, [&]() -> PyObject * {
        const at::Tensor &X = need(a[0]), &Wqkv = need(a[1]), &Wo = need(a[2]), &Wlce = need(a[3]);
        const bra_shape s = layer_shape(X, Wqkv, &Wo, &Wlce, integer(a[4]), integer(a[5]), integer(a[6]), a[7], a[10]);
        size_t bytes = 0;
        check(bra_padded_workspace_bytes(&s, &bytes));
        at::Tensor ws = scratch(bytes, X), Y = at::empty_like(X), Ir;
        const bool want_ir = PyObject_IsTrue(a[9]);
        if (want_ir) Ir = new_index(s, X);
        const at::Tensor *Ir_in = tensor(a[8]);
        check_index(Ir_in, s, "Ir_in must be a contiguous int32 [B, S*S, k] device tensor");
        void *st = stream_of(X);
        run([&] {
            return bra_forward_padded(&s, X.data_ptr(), Wqkv.data_ptr(), Wo.data_ptr(), Wlce.data_ptr(), Y.data_ptr(),
                                      want_ir ? (int32_t *)Ir.data_ptr() : nullptr, (const int32_t *)data(Ir_in),
                                      ws.data_ptr(), (size_t)ws.numel(), st);
        });
        return want_ir ? tuple({wrap(Y), wrap(Ir)}) : wrap(Y);
    });
}

// backward(X, Wqkv, Wo, Wlce, Ir, dY, S, heads, scale, path, ws)
PyObject *py_backward(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 11, [&]() -> PyObject * {
        const at::Tensor &X = need(a[0]), &Wqkv = need(a[1]), &Wo = need(a[2]), &Wlce = need(a[3]), &Ir = need(a[4]),
                         &dY = need(a[5]);
        if (Ir.dim() < 1) value_error("Ir must be a contiguous int32 [B, S*S, k] device tensor");
        const bra_shape s = layer_shape(X, Wqkv, &Wo, &Wlce, integer(a[6]), (int)Ir.size(-1), integer(a[7]), a[8], a[9]);
        check_index(&Ir, s, "Ir must be a contiguous int32 [B, S*S, k] device tensor");
        if (!(dY.is_cuda() && dY.is_contiguous() && dY.scalar_type() == X.scalar_type() && dY.sizes().equals(X.sizes())))
            value_error("dY must match X");
        at::Tensor own;
        const at::Tensor *ws = tensor(a[10]);
        if (!ws) {
            size_t bytes = 0;
            check(bra_backward_workspace_bytes(&s, &bytes));
            own = scratch(bytes, X);
            ws = &own;
        }
        const auto f32 = X.options().dtype(at::kFloat);
        const int64_t C = s.C;
        at::Tensor dX = at::empty_like(X), dWqkv = at::empty({C, 3 * C}, f32), dWo = at::empty({C, C}, f32),
                   dWlce = at::empty({C, 5, 5}, f32);
        void *st = stream_of(X);
        run([&] {
            return bra_backward(&s, X.data_ptr(), Wqkv.data_ptr(), Wo.data_ptr(), Wlce.data_ptr(),
                                (const int32_t *)Ir.data_ptr(), dY.data_ptr(), dX.data_ptr(), (float *)dWqkv.data_ptr(),
                                (float *)dWo.data_ptr(), (float *)dWlce.data_ptr(), ws->data_ptr(), (size_t)ws->numel(), st);
        });
        return tuple({wrap(dX), wrap(dWqkv), wrap(dWo), wrap(dWlce)});
    });
}

// block_forward(X, parameters in the order of bra_block_params (a tuple of 13), S, k, heads, eps, scale, Ir_in, want_Ir,
//               path, ws, out)
PyObject *py_block_forward(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return guarded(n, 12, [&]() -> PyObject * {
        const at::Tensor &X = need(a[0]);
        if (X.dim() != 4) value_error("X must be [B, H, W, C]");
        if (!(X.is_cuda() && X.is_contiguous())) value_error("X must be a contiguous device tensor");
        if (!PyTuple_Check(a[1]) || PyTuple_GET_SIZE(a[1]) != 13) value_error("expected 13 parameter tensors");
        const at::Tensor *p[13];
        for (int i = 0; i < 13; ++i) p[i] = &need(PyTuple_GET_ITEM(a[1], i));
        const int64_t C = X.size(3), hidden = p[9]->dim() == 2 ? p[9]->size(1) : 0;
        const struct { const char *name; bool matrix; int nd; int64_t dims[3]; } want[13] = {
            {"Wpos", true, 3, {C, 3, 3}}, {"bpos", false, 1, {C}}, {"ln1_g", false, 1, {C}}, {"ln1_b", false, 1, {C}},
            {"Wqkv", true, 2, {C, 3 * C}}, {"Wo", true, 2, {C, C}}, {"Wlce", true, 3, {C, 5, 5}}, {"ln2_g", false, 1, {C}},
            {"ln2_b", false, 1, {C}}, {"W1", true, 2, {C, hidden}}, {"b1", false, 1, {hidden}}, {"W2", true, 2, {hidden, C}},
            {"b2", false, 1, {C}}};
        for (int i = 0; i < 13; ++i) {
            const at::Tensor &t = *p[i];
            if (!(t.is_cuda() && t.is_contiguous() && t.device() == X.device() &&
                  t.scalar_type() == (want[i].matrix ? X.scalar_type() : at::kFloat) &&
                  t.sizes().equals(at::IntArrayRef(want[i].dims, (size_t)want[i].nd)))) {
                PyErr_Format(PyExc_ValueError, "%s must be a contiguous device tensor %s, of the shape that fits X and W1",
                             want[i].name, want[i].matrix ? "of X's dtype" : "of float32");
                throw Raised{};
            }
        }
        for (int d = 0; d < 4; ++d)
            if (X.size(d) > INT32_MAX) value_error("X is too large");
        const bra_shape s = {(int32_t)X.size(0), (int32_t)X.size(1), (int32_t)X.size(2), (int32_t)C, integer(a[4]), integer(a[2]),
                             integer(a[3]), dtype_of(X), scale_of(a[6]), integer(a[9])};
        const double eps = real(a[5]);
        at::Tensor own, Xout, Ir;
        const at::Tensor *Ir_in = tensor(a[7]), *ws = tensor(a[10]), *out = tensor(a[11]);
        if (!ws) {
            size_t bytes = 0;
            check(bra_block_workspace_bytes(&s, (int32_t)hidden, &bytes));
            own = scratch(bytes, X);
            ws = &own;
        }
        Xout = out ? *out : at::empty_like(X);
        const bool want_ir = PyObject_IsTrue(a[8]);
        if (want_ir) Ir = new_index(s, X);
        check_index(Ir_in, s, "Ir_in must be a contiguous int32 [B, S*S, k] device tensor");
        const bra_block_params bp = {p[0]->data_ptr(), (const float *)p[1]->data_ptr(), (const float *)p[2]->data_ptr(),
                                     (const float *)p[3]->data_ptr(), p[4]->data_ptr(), p[5]->data_ptr(), p[6]->data_ptr(),
                                     (const float *)p[7]->data_ptr(), (const float *)p[8]->data_ptr(), p[9]->data_ptr(),
                                     (const float *)p[10]->data_ptr(), p[11]->data_ptr(), (const float *)p[12]->data_ptr()};
        void *st = stream_of(X);
        run([&] {
            return bra_block_forward(&s, (int32_t)hidden, (float)eps, X.data_ptr(), &bp, Xout.data_ptr(),
                                     want_ir ? (int32_t *)Ir.data_ptr() : nullptr, (const int32_t *)data(Ir_in), ws->data_ptr(),
                                     (size_t)ws->numel(), st);
        });
        PyObject *y;
        if (out) Py_INCREF(y = a[11]);
        else y = wrap(Xout);
        return want_ir ? tuple({y, wrap(Ir)}) : y;
    });
}

PyMethodDef methods[] = {
    {"init", (PyCFunction)(void *)py_init, METH_FASTCALL, nullptr},
    {"route", (PyCFunction)(void *)py_route, METH_FASTCALL, nullptr},
    {"forward", (PyCFunction)(void *)py_forward, METH_FASTCALL, nullptr},
    {"forward_static", (PyCFunction)(void *)py_forward_static, METH_FASTCALL, nullptr},
    {"forward_padded", (PyCFunction)(void *)py_forward_padded, METH_FASTCALL, nullptr},
    {"backward", (PyCFunction)(void *)py_backward, METH_FASTCALL, nullptr},
    {"block_forward", (PyCFunction)(void *)py_block_forward, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
