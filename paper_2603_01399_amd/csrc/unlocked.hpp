// Calls of C entry points out of Python (host code): the interpreter's lock and what becomes of an exception.
#pragma once

#define PY_SSIZE_T_CLEAN
#include <Python.h>

namespace quasar {

// The launch runs without the interpreter's lock, as under ctypes; the lock is taken again however the call ends.
struct Unlocked {
    PyThreadState *state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};
template <typename Entry, typename... Args>
int call(Entry entry, Args... args) {
    Unlocked unlocked;
    return entry(args...);
}

// Calls body(); whatever keeps it from an ordinary call - a tensor without storage among them, for which torch throws - is left
// to binding.py.
template <typename Body>
PyObject *status_of(Py_ssize_t got, Py_ssize_t want, Body body) {
    long status = -1;
    try {
        if (got == want) status = body();
    } catch (...) {
    }
    if (PyErr_Occurred()) PyErr_Clear();
    return PyLong_FromLong(status);
}

}  // namespace quasar
