// A call into the library with the interpreter lock given up, as ctypes does.
#pragma once

#include <Python.h>

#include <exception>
#include <new>

// f's status as a Python int.  Where f throws, the lock is taken back first and the exception raised in the interpreter, the call not repeated: what
// it had launched by then stands.  (No guard object: a thread that asks for the lock while the interpreter shuts down is unwound out of
// PyEval_RestoreThread, which must not happen in a destructor or below a catch-all.)
template <typename F>
PyObject *without_lock(F f)
{
    long status = 0;
    std::exception_ptr thrown;
    PyThreadState *state = PyEval_SaveThread();
    try {
        status = (long)f();
    } catch (...) {
        thrown = std::current_exception();
    }
    PyEval_RestoreThread(state);
    if (!thrown) return PyLong_FromLong(status);
    try {
        std::rethrow_exception(thrown);
    } catch (const std::bad_alloc &) {
        PyErr_NoMemory();
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    } catch (...) {
        PyErr_SetString(PyExc_RuntimeError, "unknown C++ exception");
    }
    return nullptr;
}
