// What a call from Python needs before the library can be called: the checks of its tensors and their pointers, strides
// and sizes.  In Python they took 1.2 us of a step's 5.0 at n = 4, D = 1,024 and, for separate rows, half a microsecond per row:
// 18 of 37 us at n = 33.  Nothing is kept from one call for the next.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <vector>

#include "../../include/svgd.h"

namespace {

struct Matrix {
    int64_t n, D, ld;
    bool operator!=(const Matrix &o) const { return n != o.n || D != o.D || ld != o.ld; }
    int rows() const { return n > INT_MAX ? INT_MAX : (int)n; } // (refused by the library)
};

bool type_error(const char *format, const char *name)
{
    PyErr_Format(PyExc_TypeError, format, name);
    return false;
}

// A 2-D float32 CUDA tensor with contiguous rows, on `device` unless that is negative.
bool matrix(PyObject *obj, const char *name, long device, Matrix &m)
{
    if (!THPVariable_Check(obj)) return type_error("%s must be a 2-D float32 CUDA tensor", name);
    const at::Tensor &t = THPVariable_Unpack(obj);
    if (t.scalar_type() != at::kFloat || !t.is_cuda() || t.dim() != 2)
        return type_error("%s must be a 2-D float32 CUDA tensor", name);
    m.n = t.size(0);
    m.D = t.size(1);
    m.ld = t.stride(0);
    if ((m.D != 1 && t.stride(1) != 1) || (m.n != 1 && m.ld < m.D))
        return type_error("%s must have contiguous rows, at least D elements apart", name);
    if (m.n == 1) m.ld = m.D;
    if (device >= 0 && t.get_device() != device) { // (a pointer of another GPU would fault)
        PyErr_Format(PyExc_ValueError, "%s is on cuda:%d, the handle on cuda:%ld", name, (int)t.get_device(), device);
        return false;
    }
    return true;
}

void *data(PyObject *tensor) { return THPVariable_Unpack(tensor).data_ptr(); }

bool same(const Matrix &x, const Matrix &m, const char *name)
{
    if (!(m != x)) return true;
    PyErr_Format(PyExc_ValueError, "%s has (n, D, row stride) = (%lld, %lld, %lld), X has (%lld, %lld, %lld)", name, (long long)m.n,
                 (long long)m.D, (long long)m.ld, (long long)x.n, (long long)x.D, (long long)x.ld);
    return false;
}

bool number(PyObject *obj, double &out) // what float() takes
{
    if (PyFloat_CheckExact(obj)) {
        out = PyFloat_AS_DOUBLE(obj);
        return true;
    }
    PyObject *f = PyNumber_Float(obj);
    if (!f) return false;
    out = PyFloat_AsDouble(f);
    Py_DECREF(f);
    return !(out == -1.0 && PyErr_Occurred());
}

// A handle or a stream, as an integer
bool word(PyObject *obj, void *&out)
{
    out = PyLong_AsVoidPtr(obj);
    return !(out == nullptr && PyErr_Occurred());
}

struct Owned { // a reference, given back at the end
    PyObject *p;
    ~Owned() { Py_XDECREF(p); }
};

// What stream_ptr makes of a stream object or of None.  Asked for behind the checks, like eps: both run code of the
// caller's or need a GPU, and what is no tensor on one is to be named first.
bool stream_of(PyObject *stream_ptr, PyObject *stream, void *&out)
{
    const Owned r{PyObject_CallFunctionObjArgs(stream_ptr, stream, nullptr)};
    return r.p && word(r.p, out);
}

// Errors and warnings of torch as its own Python functions raise them: the error that a tensor subclass raised in Python,
// the type of torch's, a warning through Python's filters.
template <class F>
PyObject *guarded(F f)
{
    HANDLE_TH_ERRORS
    return f();
    END_HANDLE_TH_ERRORS
}

bool arguments(Py_ssize_t got, Py_ssize_t want)
{
    if (got == want) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments, %zd expected", got, want);
    return false;
}

// n of a call that succeeded, or its (negative) status
PyObject *result(int rc, int64_t n) { return PyLong_FromLongLong(rc == SVGD_OK ? n : rc); }

// step(handle, device, X, G, eps, stream, stream_ptr).  Pointers are taken last, behind everything that can run other code.
PyObject *step(PyObject *, PyObject *const *a, Py_ssize_t na)
{
    return guarded([&]() -> PyObject * {
        if (!arguments(na, 7)) return nullptr;
        void *h, *stream;
        const long device = PyLong_AsLong(a[1]);
        Matrix x, g;
        double eps;
        if (!word(a[0], h) || (device == -1 && PyErr_Occurred()) || !matrix(a[2], "X", device, x) || !matrix(a[3], "G", device, g) ||
            !same(x, g, "G") || !number(a[4], eps) || !stream_of(a[6], a[5], stream))
            return nullptr;
        void *const xp = data(a[2]), *const gp = data(a[3]);
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = svgd_step_ld((svgd_handle_t)h, (float *)xp, (const float *)gp, x.rows(), x.D, x.ld, (float)eps, stream);
        Py_END_ALLOW_THREADS
        return result(rc, x.n);
    });
}

// phi(handle, device, X, G, PHI, stream, stream_ptr)
PyObject *phi(PyObject *, PyObject *const *a, Py_ssize_t na)
{
    return guarded([&]() -> PyObject * {
        if (!arguments(na, 7)) return nullptr;
        void *h, *stream;
        const long device = PyLong_AsLong(a[1]);
        Matrix x, g, p;
        if (!word(a[0], h) || (device == -1 && PyErr_Occurred()) || !matrix(a[2], "X", device, x) || !matrix(a[3], "G", device, g) ||
            !same(x, g, "G") || !matrix(a[4], "PHI", device, p) || !same(x, p, "PHI") || !stream_of(a[6], a[5], stream))
            return nullptr;
        void *const xp = data(a[2]), *const gp = data(a[3]), *const pp = data(a[4]);
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = svgd_phi_ld((svgd_handle_t)h, (const float *)xp, (const float *)gp, x.rows(), x.D, x.ld, (float *)pp, stream);
        Py_END_ALLOW_THREADS
        return result(rc, x.n);
    });
}

// step_static(current_device, X, G, eps, stream, stream_ptr): the status, or 1 for an X on another device (nothing done)
PyObject *step_static(PyObject *, PyObject *const *a, Py_ssize_t na)
{
    return guarded([&]() -> PyObject * {
        if (!arguments(na, 6)) return nullptr;
        void *stream;
        Matrix x, g;
        double eps;
        if (!matrix(a[1], "X", -1, x) || !matrix(a[2], "G", -1, g)) return nullptr;
        if (g != x) {
            PyErr_SetString(PyExc_ValueError, "G must have the shape and row stride of X");
            return nullptr;
        }
        const Owned current{PyObject_CallNoArgs(a[0])};
        const long device = current.p ? PyLong_AsLong(current.p) : -1;
        if (device == -1 && PyErr_Occurred()) return nullptr;
        if (THPVariable_Unpack(a[1]).get_device() != device) return PyLong_FromLong(1);
        if (!number(a[3], eps) || !stream_of(a[5], a[4], stream)) return nullptr;
        void *const xp = data(a[1]), *const gp = data(a[2]);
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = svgd_step_static((float *)xp, (const float *)gp, x.rows(), x.D, x.ld, (float)eps, stream);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    });
}

// The rows of a tuple: 1-D float32 CUDA tensors of D contiguous elements on `device`.
bool check_rows(PyObject *rows, const char *name, int64_t D, long device)
{
    const Py_ssize_t n = PyTuple_GET_SIZE(rows);
    for (Py_ssize_t i = 0; i < n; ++i) {
        PyObject *row = PyTuple_GET_ITEM(rows, i);
        if (!THPVariable_Check(row)) return type_error("%s must hold contiguous 1-D float32 CUDA tensors of one length", name);
        const at::Tensor &t = THPVariable_Unpack(row);
        if (t.scalar_type() != at::kFloat || !t.is_cuda() || t.dim() != 1 || t.size(0) != D || (D != 1 && t.stride(0) != 1))
            return type_error("%s must hold contiguous 1-D float32 CUDA tensors of one length", name);
        if (t.get_device() != device) {
            PyErr_Format(PyExc_ValueError, "a row of %s is on cuda:%d, the handle on cuda:%ld", name, (int)t.get_device(), device);
            return false;
        }
    }
    return true;
}

std::vector<void *> row_pointers(PyObject *rows)
{
    std::vector<void *> out((size_t)PyTuple_GET_SIZE(rows));
    for (size_t i = 0; i < out.size(); ++i) out[i] = data(PyTuple_GET_ITEM(rows, (Py_ssize_t)i));
    return out;
}

// seq[0], or null with an error set
PyObject *first_item(PyObject *seq)
{
    const Owned zero{PyLong_FromLong(0)};
    return zero.p ? PyObject_GetItem(seq, zero.p) : nullptr;
}

// step_rows(handle, device, X_rows, G_rows, eps, stream, stream_ptr)
PyObject *step_rows(PyObject *, PyObject *const *a, Py_ssize_t na)
{
    return guarded([&]() -> PyObject * {
        if (!arguments(na, 7)) return nullptr;
        void *h, *stream;
        const long device = PyLong_AsLong(a[1]);
        if (!word(a[0], h) || (device == -1 && PyErr_Occurred())) return nullptr;
        const Py_ssize_t n = PyObject_Size(a[2]), ng = n > 0 ? PyObject_Size(a[3]) : 0;
        if (n < 0 || ng < 0) return nullptr;
        if (n < 1 || ng != n) {
            PyErr_SetString(PyExc_ValueError, "X_rows and G_rows must be non-empty sequences of the same length");
            return nullptr;
        }
        // X_rows[0] says how long all are.  What has no length or no order (a generator, a set) is refused: particles
        // and scores would meet by chance.
        const Owned first{first_item(a[2])};
        if (!first.p) return nullptr;
        if (!THPVariable_Check(first.p)) {
            type_error("%s must hold contiguous 1-D float32 CUDA tensors of one length", "X_rows");
            return nullptr;
        }
        const int64_t D = THPVariable_Unpack(first.p).numel();
        const Owned xs{PySequence_Tuple(a[2])}; // the rows are held until the call is done
        if (!xs.p) return nullptr;
        const Owned gs{PySequence_Tuple(a[3])};
        if (!gs.p) return nullptr;
        if (PyTuple_GET_SIZE(xs.p) != n || PyTuple_GET_SIZE(gs.p) != n) { // (not as many as they say)
            PyErr_SetString(PyExc_ValueError, "X_rows and G_rows must be non-empty sequences of the same length");
            return nullptr;
        }
        double eps;
        if (!check_rows(xs.p, "X_rows", D, device) || !check_rows(gs.p, "G_rows", D, device) || !number(a[4], eps) ||
            !stream_of(a[6], a[5], stream))
            return nullptr;
        const std::vector<void *> x = row_pointers(xs.p), g = row_pointers(gs.p);
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = svgd_step_rows((svgd_handle_t)h, (float *const *)x.data(), (const float *const *)g.data(), n > INT_MAX ? INT_MAX : (int)n, D,
                            (float)eps, stream);
        Py_END_ALLOW_THREADS
        return result(rc, n);
    });
}

#define METHOD(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(step), METHOD(phi), METHOD(step_static), METHOD(step_rows), {nullptr, nullptr, 0, nullptr}};
PyModuleDef definition = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__binding()
{
    PyObject *m = PyModule_Create(&definition);
    if (m && PyModule_AddStringConstant(m, "torch_version", SVGD_TORCH_VERSION) < 0) { // (whose C++ interface this is built against)
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
