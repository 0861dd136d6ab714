// Where C++ exceptions end in the calls of the Python binding (apmm_call.cpp).
#pragma once

#include <Python.h>

#include <cxxabi.h>

// What body returns, or what failed returns if body throws.  Handlers of every exception stand here only, because one kind has to go on: a
// thread that ends inside the body is unwound by one, and a handler that keeps it ends the whole process with abort().  Python 3.10 ends a daemon
// thread that way when it takes the interpreter's lock again (Py_END_ALLOW_THREADS, any call of a Python function) while the interpreter shuts down.
template <class Body, class Failed>
auto end_exceptions(Body body, Failed failed) -> decltype(body())
{
    try {
        return body();
    } catch (abi::__forced_unwind &) {
        throw;
    } catch (...) {
        return failed();
    }
}

// The call itself, without the interpreter's lock, and what follows from its status: true if it is 0, else check(status) has set an error.  An exception
// of the call has no status and no text in the library, so it is reported here and not through check.
template <class Call>
bool call_and_check(PyObject *check, Call call)
{
    constexpr int kThrown = -1;
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = end_exceptions([&] { return (int)call(); }, [] { return (int)kThrown; });  // nothing may pass here without the lock
    Py_END_ALLOW_THREADS
    if (status == 0) return true;
    if (status == kThrown) {
        PyErr_SetString(PyExc_RuntimeError, "apmm: a C++ exception ended the call");
        return false;
    }
    PyObject *r = PyObject_CallFunction(check, "i", status);
    if (r) {
        Py_DECREF(r);
        PyErr_SetString(PyExc_RuntimeError, "apmm: a call failed");
    }
    return false;
}
