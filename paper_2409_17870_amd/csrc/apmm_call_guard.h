// Where C++ exceptions end in the calls of the Python binding (apmm_call.cpp).
#pragma once

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
