// sv_op records from a Python list of gates, in C: the binding's
// ops_from_gates spent 0.7 us per gate on it in list comprehensions and numpy
// conversions (255 us for 360 gates, more than the device needs for a
// 12-qubit circuit of them; here 40).  Only the plain case is handled: a list
// or tuple of gates whose fields are tuples or lists of integers, numbers and
// a known name.  Anything else returns -1, and the caller's general code
// converts or rejects it.  Loaded with ctypes.PyDLL (the GIL is held).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>

#include "../../include/sv.h"

namespace {

struct Ref { // an owned reference
    PyObject *p;
    explicit Ref(PyObject *o) : p(o) {}
    ~Ref() { Py_XDECREF(p); }
    Ref(const Ref &) = delete;
    Ref &operator=(const Ref &) = delete;
};

bool as_int(PyObject *o, long long lo, long long hi, long long *out) {
    int overflow = 0;
    long long v;
    if (PyLong_Check(o)) {
        v = PyLong_AsLongLongAndOverflow(o, &overflow);
    } else if (PyIndex_Check(o)) { // numpy integers
        Ref i(PyNumber_Index(o));
        if (!i.p) return false;
        v = PyLong_AsLongLongAndOverflow(i.p, &overflow);
    } else {
        return false;
    }
    if (overflow || (v == -1 && PyErr_Occurred()) || v < lo || v > hi) return false;
    *out = v;
    return true;
}

bool plain_sequence(PyObject *o) { return o && (PyTuple_CheckExact(o) || PyList_CheckExact(o)); }

bool fill(PyObject *g, PyObject *kinds, PyObject *const *names, sv_op *op, bool *matrix) {
    Ref name(PyObject_GetAttr(g, names[0])), targets(PyObject_GetAttr(g, names[1])),
        controls(PyObject_GetAttr(g, names[2])), theta(PyObject_GetAttr(g, names[3])),
        param(PyObject_GetAttr(g, names[4]));
    if (!name.p || !plain_sequence(targets.p) || !plain_sequence(controls.p) || !theta.p || !param.p) return false;
    long long v;
    PyObject *kind = PyDict_GetItemWithError(kinds, name.p); // borrowed
    if (!kind || !as_int(kind, INT32_MIN, INT32_MAX, &v)) return false;
    op->kind = (int32_t)v;
    *matrix = v == SV_GATE_MATRIX;
    const Py_ssize_t nt = PySequence_Fast_GET_SIZE(targets.p);
    if (nt < 1 || nt > INT32_MAX) return false;
    op->n_targets = (int32_t)nt;
    for (Py_ssize_t i = 0; i < 2 && i < nt; ++i) {
        if (i >= PySequence_Fast_GET_SIZE(targets.p)) return false;
        Ref t((Py_NewRef(PySequence_Fast_GET_ITEM(targets.p, i))));
        if (!as_int(t.p, INT32_MIN, INT32_MAX, &v)) return false;
        op->targets[i] = (int32_t)v;
    }
    uint64_t mask = 0;
    for (Py_ssize_t i = 0; i < PySequence_Fast_GET_SIZE(controls.p); ++i) {
        Ref c((Py_NewRef(PySequence_Fast_GET_ITEM(controls.p, i))));
        if (!as_int(c.p, 0, 63, &v) || __builtin_add_overflow(mask, 1ull << v, &mask)) return false;
    }
    op->ctrl_mask = mask;
    if (!as_int(param.p, INT32_MIN, INT32_MAX, &v)) return false;
    op->param_index = (int32_t)v;
    if (PyFloat_Check(theta.p)) op->theta = PyFloat_AS_DOUBLE(theta.p);
    else if (PyLong_Check(theta.p)) op->theta = PyLong_AsDouble(theta.p);
    else return false;
    return !PyErr_Occurred();
}

} // namespace

// Fills out[0 .. len(gates)) (zeroed by the caller; the matrices stay zero).
// Returns the number of gates that carry a matrix, -1 for the general path.
extern "C" Py_ssize_t sv_py_fill_ops(PyObject *gates, PyObject *kinds, sv_op *out, Py_ssize_t n) {
    static const char *const kFields[] = {"name", "targets", "controls", "theta", "param"};
    if (!plain_sequence(gates) || !PyDict_Check(kinds)) return -1;
    PyObject *names[5];
    for (int i = 0; i < 5; ++i) names[i] = PyUnicode_InternFromString(kFields[i]);
    Py_ssize_t matrices = 0;
    bool ok = names[0] && names[1] && names[2] && names[3] && names[4];
    for (Py_ssize_t i = 0; ok && i < n; ++i) {
        // a field's getter may run any code: the list is looked at afresh
        if (PySequence_Fast_GET_SIZE(gates) != n) {
            ok = false;
            break;
        }
        Ref g((Py_NewRef(PySequence_Fast_GET_ITEM(gates, i))));
        bool matrix = false;
        ok = fill(g.p, kinds, names, &out[i], &matrix);
        matrices += matrix;
    }
    for (int i = 0; i < 5; ++i) Py_XDECREF(names[i]);
    if (ok) return matrices;
    PyErr_Clear();
    return -1;
}
