// Argument marshalling of the Python surface in native code: the checks, the
// result tensors and the C-ABI call of fit, fit_qr, residuals, fit_batched,
// fit_qr_batched and fit_backward in one step each.  A small fit is a few microseconds of GPU
// work; on the MI355X machine's host a call with two kernel launches took 18.3 us
// with the same steps through ctypes and Python-level tensor calls and 12.6 us
// with them here (9.5 us where a fit takes one launch); the forward and backward of a
// batch through autograd 132 and 86 us.
//
// Every function takes the calls that need nothing but marshalling (plain
// GPU tensors of the right types and shapes, known option names) and returns
// None for any other, which the Python code then handles, errors included.  A
// C-ABI error comes back as its code (an int).  The library's entry points are the
// loaded liblsefit.so's own, handed over by address (init), so that there is one
// copy of the library in the process whatever its path.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>

#include "lsefit.h"

namespace {

struct Api {
    decltype(&::lsefit_workspace_bytes) workspace_bytes = nullptr;
    decltype(&::fit_single) single = nullptr;
    decltype(&::fit_qr) qr = nullptr;
    decltype(&::fit_residuals) residuals = nullptr;
    decltype(&::fit_batched) batched = nullptr;
    decltype(&::fit_backward) backward = nullptr;
    decltype(&::fit_qr_batched) qr_batched = nullptr;
} api;

PyObject* init(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 7) {
        PyErr_SetString(PyExc_TypeError, "init takes seven addresses");
        return nullptr;
    }
    void* p[7];
    for (int i = 0; i < 7; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
            return nullptr;
        }
    }
    api.workspace_bytes = (decltype(api.workspace_bytes))p[0];
    api.single = (decltype(api.single))p[1];
    api.qr = (decltype(api.qr))p[2];
    api.residuals = (decltype(api.residuals))p[3];
    api.batched = (decltype(api.batched))p[4];
    api.backward = (decltype(api.backward))p[5];
    api.qr_batched = (decltype(api.qr_batched))p[6];
    Py_RETURN_NONE;
}

// ---- reading arguments: false means "not a plain call" ----
bool tensor(PyObject* o, const at::Tensor** t) {
    if (!THPVariable_CheckExact(o)) return false;   // subclasses go the Python way
    *t = &THPVariable_Unpack(o);
    // functorch's wrappers (vmap, grad, jvp) have the exact type too, but no memory of their own
    return (*t)->defined() && (*t)->layout() == at::kStrided && (*t)->has_storage();
}
bool integer(PyObject* o, int64_t* v) {
    if (!PyLong_Check(o)) return false;
    int over = 0;
    *v = PyLong_AsLongLongAndOverflow(o, &over);
    return over == 0 && *v >= INT32_MIN && *v <= INT32_MAX;
}
bool number(PyObject* o, double* v) {
    if (PyFloat_CheckExact(o)) {
        *v = PyFloat_AS_DOUBLE(o);
        return true;
    }
    int64_t i;
    if (!integer(o, &i)) return false;
    *v = (double)i;
    return true;
}
bool choice(PyObject* o, const char* zero, const char* one, int32_t* v) {
    if (!PyUnicode_CheckExact(o)) return false;
    if (PyUnicode_CompareWithASCIIString(o, zero) == 0) *v = 0;
    else if (PyUnicode_CompareWithASCIIString(o, one) == 0) *v = 1;
    else return false;
    return true;
}

bool options(PyObject* degree, PyObject* precision, PyObject* refine, PyObject* center, PyObject* scale,
             PyObject* solver, PyObject* basis, lsefit_options* o) {
    memset(o, 0, sizeof(*o));   // with its padding: a plan compares options as bytes
    int64_t deg = 0, ref = 0;
    if (!integer(degree, &deg) || deg < 1 || deg > LSEFIT_MAX_DEGREE_CHEBYSHEV) return false;
    if (!choice(precision, "f64", "f32c", &o->precision) || !choice(solver, "gepp", "cholesky", &o->solver) ||
        !choice(basis, "monomial", "chebyshev", &o->basis) || !integer(refine, &ref))
        return false;
    o->degree = (int32_t)deg;
    o->refine_steps = o->precision == LSEFIT_PREC_F32C ? (int32_t)ref : 0;
    o->range_mode = center == Py_None && scale == Py_None ? LSEFIT_RANGE_AUTO : LSEFIT_RANGE_GIVEN;
    o->center = 0.0;
    o->scale = 1.0;
    o->output_basis = LSEFIT_OUTPUT_X;
    return (center == Py_None || number(center, &o->center)) && (scale == Py_None || number(scale, &o->scale));
}

struct Points {
    const at::Tensor *x, *y;
    const void *px, *py;
    int64_t n;
    int32_t dt;
    void* stream;
};

bool points(PyObject* ox, PyObject* oy, Points* p) {
    if (!tensor(ox, &p->x) || !tensor(oy, &p->y)) return false;
    const at::Tensor &x = *p->x, &y = *p->y;
    if (!x.is_cuda() || x.device() != y.device() || x.scalar_type() != y.scalar_type()) return false;
    if (x.scalar_type() != at::kFloat && x.scalar_type() != at::kDouble) return false;
    if (x.dim() != 1 || y.dim() != 1 || x.numel() != y.numel() || !x.is_contiguous() || !y.is_contiguous()) return false;
    if (x.is_neg() || y.is_neg()) return false;
    p->px = x.data_ptr();
    p->py = y.data_ptr();
    p->n = x.numel();
    p->dt = x.scalar_type() == at::kFloat ? LSEFIT_F32 : LSEFIT_F64;
    p->stream = (void*)c10::hip::getCurrentHIPStream(x.device().index()).stream();
    return true;
}

bool batch(PyObject* ooff, PyObject* odeg, const Points& p, const at::Tensor** off, const at::Tensor** deg) {
    if (!tensor(ooff, off) || !tensor(odeg, deg)) return false;
    const at::Tensor &f = **off, &g = **deg;
    return f.scalar_type() == at::kLong && g.scalar_type() == at::kInt && f.device() == p.x->device() &&
           g.device() == p.x->device() && f.dim() == 1 && g.dim() == 1 && f.numel() == g.numel() + 1 &&
           f.is_contiguous() && g.is_contiguous();
}

// a workspace of at least `bytes`: the caller's, or a new one
bool workspace(PyObject* ows, size_t bytes, const Points& p, at::Tensor* ws) {
    if (bytes == 0) return false;
    if (ows != Py_None) {
        const at::Tensor* t;
        if (!tensor(ows, &t)) return false;
        if (t->scalar_type() != at::kByte || !t->is_contiguous()) return false;
        if ((size_t)t->numel() >= bytes) {
            *ws = *t;
            return true;
        }
    }
    *ws = at::empty({(int64_t)bytes}, p.x->options().dtype(at::kByte).requires_grad(false));
    return true;
}

at::Tensor doubles(const Points& p, int64_t n) {
    return at::empty({n}, p.x->options().dtype(at::kDouble).requires_grad(false));
}
at::Tensor ints(const Points& p, int64_t n) {
    return at::empty({n}, p.x->options().dtype(at::kInt).requires_grad(false));
}
template <class T>
T* at_ptr(const at::Tensor& t) {
    return (T*)t.data_ptr();
}
// a workspace's memory (none with a plan, which brings its own)
struct Space {
    void* p = nullptr;
    size_t bytes = 0;
    Space() = default;
    explicit Space(const at::Tensor& t) : p(t.data_ptr()), bytes((size_t)t.numel()) {}
};

// The library call, with the interpreter released.  Tensors are asked for their
// memory before it (data_ptr may throw, and may run code that needs the
// interpreter); the lambdas hold plain pointers and sizes only.
struct Released {
    PyThreadState* const state = PyEval_SaveThread();
    ~Released() { PyEval_RestoreThread(state); }
};
template <class F>
int call(F&& f) {
    const Released released;
    return (int)f();
}

PyObject* wrap(std::initializer_list<at::Tensor> ts, const lsefit_options* o = nullptr) {
    PyObject* tup = PyTuple_New((Py_ssize_t)ts.size() + (o ? 1 : 0));
    if (!tup) return nullptr;
    Py_ssize_t i = 0;
    for (const at::Tensor& t : ts) PyTuple_SET_ITEM(tup, i++, THPVariable_Wrap(t));
    if (o) PyTuple_SET_ITEM(tup, i, PyBytes_FromStringAndSize((const char*)o, sizeof(*o)));
    return tup;
}

// fit(x, y, degree, precision, refine, center, scale, ws, solver, basis)
//   -> (coef[:m1], coef[m1:], status, moments, ws, options bytes)
PyObject* fit(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Points p;
    lsefit_options o;
    at::Tensor ws;
    if (n != 10 || !points(a[0], a[1], &p) || !options(a[2], a[3], a[4], a[5], a[6], a[8], a[9], &o) ||
        !workspace(a[7], api.workspace_bytes(1, o.degree, nullptr), p, &ws))
        Py_RETURN_NONE;
    const int64_t m1 = o.degree + 1;
    const at::Tensor coef = doubles(p, 2 * m1), status = ints(p, 1), mom = doubles(p, 3 * m1 + 1);
    const Space sp(ws);
    double *pc = at_ptr<double>(coef), *pm = at_ptr<double>(mom);
    int32_t* ps = at_ptr<int32_t>(status);
    const int code = call([&] { return api.single(p.px, p.py, p.n, p.dt, &o, sp.p, sp.bytes, pc, ps, pm, p.stream); });
    if (code) return PyLong_FromLong(code);
    return wrap({coef.narrow(0, 0, m1), coef.narrow(0, m1, m1), status, mom, ws}, &o);
    END_HANDLE_TH_ERRORS
}

// fit_qr(x, y, degree, center, scale, ws, "f64", 0, "gepp", "monomial")
//   -> (coef[:m1], coef[m1:], status, info, ws, options bytes)
PyObject* fit_qr(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Points p;
    lsefit_options o;
    at::Tensor ws;
    if (n != 10 || !points(a[0], a[1], &p) || !options(a[2], a[6], a[7], a[3], a[4], a[8], a[9], &o) ||
        !workspace(a[5], api.workspace_bytes(1, o.degree, nullptr), p, &ws))
        Py_RETURN_NONE;
    const int64_t m1 = o.degree + 1;
    const at::Tensor coef = doubles(p, 2 * m1), status = ints(p, 1), info = doubles(p, 3);
    const Space sp(ws);
    double *pc = at_ptr<double>(coef), *pi = at_ptr<double>(info);
    int32_t* ps = at_ptr<int32_t>(status);
    const int code = call([&] { return api.qr(p.px, p.py, p.n, p.dt, &o, sp.p, sp.bytes, pc, ps, pi, p.stream); });
    if (code) return PyLong_FromLong(code);
    return wrap({coef.narrow(0, 0, m1), coef.narrow(0, m1, m1), status, info, ws}, &o);
    END_HANDLE_TH_ERRORS
}

// residuals(x, y, options address, ws, store) -> (sse, residuals or None)
PyObject* residuals(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Points p;
    const at::Tensor* ws;
    if (n != 5 || !points(a[0], a[1], &p) || !PyLong_Check(a[2]) || !tensor(a[3], &ws) || !PyBool_Check(a[4]))
        Py_RETURN_NONE;
    if (ws->scalar_type() != at::kByte || !ws->is_contiguous()) Py_RETURN_NONE;
    const lsefit_options* given = (const lsefit_options*)PyLong_AsVoidPtr(a[2]);
    if (!given) Py_RETURN_NONE;
    const lsefit_options o = *given;   // its owner may drop it once the interpreter is released
    const at::Tensor sse = doubles(p, 1);
    const bool store = a[4] == Py_True;
    const at::Tensor res = store ? at::empty_like(p.x->detach()) : at::Tensor();
    const Space sp(*ws);
    double* pe = at_ptr<double>(sse);
    void* pr = store ? res.data_ptr() : nullptr;
    const int code = call([&] {
        return api.residuals(p.px, p.py, nullptr, nullptr, 1, p.n, p.dt, &o, nullptr, sp.p, sp.bytes, pe, pr, p.stream);
    });
    if (code) return PyLong_FromLong(code);
    return wrap({sse, res});   // an undefined tensor is None
    END_HANDLE_TH_ERRORS
}

// fit_batched(x, y, offsets, degrees, max_degree, precision, refine, center, scale, plan address or None,
//             coef_stride or None, ws, out coef, out status, solver, basis, output_basis)
//   -> (coef, status, ws or None)
PyObject* fit_batched(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Points p;
    lsefit_options o;
    const at::Tensor *off, *deg;
    if (n != 17 || !points(a[0], a[1], &p) || !batch(a[2], a[3], p, &off, &deg) ||
        !options(a[4], a[5], a[6], a[7], a[8], a[14], a[15], &o) || !choice(a[16], "x", "x_and_t", &o.output_basis))
        Py_RETURN_NONE;
    const int64_t B = deg->numel();
    const bool t_out = o.output_basis == LSEFIT_OUTPUT_X_AND_T && o.basis == LSEFIT_BASIS_MONOMIAL;
    int64_t stride = 0;
    if (a[10] != Py_None && !integer(a[10], &stride)) Py_RETURN_NONE;
    if (stride == 0) stride = t_out ? 2 * o.degree + 4 : o.degree + 1;
    if (stride < 1) Py_RETURN_NONE;
    lsefit_plan* plan = nullptr;
    if (a[9] != Py_None) {
        if (!PyLong_Check(a[9]) || !(plan = (lsefit_plan*)PyLong_AsVoidPtr(a[9]))) Py_RETURN_NONE;
    }
    at::Tensor ws, coef, status;
    if (!plan && !workspace(a[11], api.workspace_bytes(B > 1 ? B : 1, o.degree, nullptr), p, &ws)) Py_RETURN_NONE;
    if (a[12] != Py_None || a[13] != Py_None) {
        const at::Tensor *c, *s;
        if (!tensor(a[12], &c) || !tensor(a[13], &s)) Py_RETURN_NONE;
        coef = *c;
        status = *s;
    } else {
        coef = at::zeros({B, stride}, p.x->options().dtype(at::kDouble).requires_grad(false));
        status = ints(p, B);
    }
    const Space sp = plan ? Space() : Space(ws);
    const int64_t* po = at_ptr<int64_t>(*off);
    const int32_t* pd = at_ptr<int32_t>(*deg);
    double* pc = at_ptr<double>(coef);
    int32_t* ps = at_ptr<int32_t>(status);
    const int code = call([&] {
        return api.batched(p.px, p.py, po, pd, B, p.dt, &o, plan, sp.p, sp.bytes, pc, (int32_t)stride, ps, p.stream);
    });
    if (code) return PyLong_FromLong(code);
    return wrap({coef, status, ws});
    END_HANDLE_TH_ERRORS
}

// fit_backward(x, y, offsets, degrees, max_degree, grad_coef, ws or None, plan address or None, precision,
//              center, scale, solver, basis) -> (grad_x, grad_y)
PyObject* fit_backward(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Points p;
    lsefit_options o;
    const at::Tensor *off, *deg, *g, *ws = nullptr;
    PyObject* zero = n == 13 ? a[4] : nullptr;   // any integer: refine is not used by the adjoint
    if (n != 13 || !points(a[0], a[1], &p) || !batch(a[2], a[3], p, &off, &deg) || !tensor(a[5], &g) ||
        !options(a[4], a[8], zero, a[9], a[10], a[11], a[12], &o))
        Py_RETURN_NONE;
    o.refine_steps = 0;
    if (g->device() != p.x->device() || g->dim() < 1 || g->is_neg()) Py_RETURN_NONE;
    if (a[6] != Py_None && !tensor(a[6], &ws)) Py_RETURN_NONE;
    lsefit_plan* plan = nullptr;
    if (a[7] != Py_None) {
        if (!PyLong_Check(a[7]) || !(plan = (lsefit_plan*)PyLong_AsVoidPtr(a[7]))) Py_RETURN_NONE;
    }
    if (!plan && (!ws || ws->scalar_type() != at::kByte || !ws->is_contiguous())) Py_RETURN_NONE;
    const at::Tensor gc = g->scalar_type() == at::kDouble && g->is_contiguous() ? *g : g->to(at::kDouble).contiguous();
    const at::Tensor gx = at::empty_like(p.x->detach()), gy = at::empty_like(p.y->detach());
    const Space sp = plan ? Space() : Space(*ws);
    const int64_t* po = at_ptr<int64_t>(*off);
    const int32_t* pd = at_ptr<int32_t>(*deg);
    const int64_t B = deg->numel();
    const double* pg = at_ptr<double>(gc);
    const int32_t stride = (int32_t)gc.size(-1);
    void *px = gx.data_ptr(), *py = gy.data_ptr();
    const int code = call([&] {
        return api.backward(p.px, p.py, po, pd, B, p.dt, &o, plan, sp.p, sp.bytes, pg, stride, px, py, p.stream);
    });
    if (code) return PyLong_FromLong(code);
    return wrap({gx, gy});
    END_HANDLE_TH_ERRORS
}

// fit_qr_batched(x, y, offsets, degrees, max_degree, center, scale, coef_stride, ws, coef, status, sse,
//                precision, refine, solver, basis) -> (coef, status, sse, ws); the last four as the options have them
PyObject* fit_qr_batched(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Points p;
    lsefit_options o;
    const at::Tensor *off, *deg;
    if (n != 16 || !points(a[0], a[1], &p) || !batch(a[2], a[3], p, &off, &deg) ||
        !options(a[4], a[12], a[13], a[5], a[6], a[14], a[15], &o))
        Py_RETURN_NONE;
    const int64_t B = deg->numel();
    int64_t stride = 0;
    if (a[7] != Py_None && !integer(a[7], &stride)) Py_RETURN_NONE;
    if (stride == 0) stride = o.degree + 1;
    if (stride < 1) Py_RETURN_NONE;
    at::Tensor ws, coef, status, sse;
    if (!workspace(a[8], api.workspace_bytes(B > 1 ? B : 1, o.degree, nullptr), p, &ws)) Py_RETURN_NONE;
    if (a[9] != Py_None || a[10] != Py_None || a[11] != Py_None) {
        const at::Tensor *c, *s, *e;
        if (!tensor(a[9], &c) || !tensor(a[10], &s) || !tensor(a[11], &e)) Py_RETURN_NONE;
        coef = *c;
        status = *s;
        sse = *e;
    } else {
        coef = at::zeros({B, stride}, p.x->options().dtype(at::kDouble).requires_grad(false));
        status = ints(p, B);
        sse = doubles(p, B);
    }
    const Space sp(ws);
    const int64_t* po = at_ptr<int64_t>(*off);
    const int32_t* pd = at_ptr<int32_t>(*deg);
    double *pc = at_ptr<double>(coef), *pe = at_ptr<double>(sse);
    int32_t* ps = at_ptr<int32_t>(status);
    const int code = call([&] {
        return api.qr_batched(p.px, p.py, po, pd, B, p.dt, &o, sp.p, sp.bytes, pc, (int32_t)stride, ps, pe, p.stream);
    });
    if (code) return PyLong_FromLong(code);
    return wrap({coef, status, sse, ws});
    END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {{"init", (PyCFunction)(void*)init, METH_FASTCALL, nullptr},
                         {"fit", (PyCFunction)(void*)fit, METH_FASTCALL, nullptr},
                         {"fit_qr", (PyCFunction)(void*)fit_qr, METH_FASTCALL, nullptr},
                         {"residuals", (PyCFunction)(void*)residuals, METH_FASTCALL, nullptr},
                         {"fit_batched", (PyCFunction)(void*)fit_batched, METH_FASTCALL, nullptr},
                         {"fit_qr_batched", (PyCFunction)(void*)fit_qr_batched, METH_FASTCALL, nullptr},
                         {"fit_backward", (PyCFunction)(void*)fit_backward, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_bind", "argument marshalling in native code", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__bind() { return PyModule_Create(&module); }
