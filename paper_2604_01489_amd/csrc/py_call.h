// The two halves of a native method of the binding that do not depend on its arguments: what its body throws, and the call without the GIL.  No torch in here,
// so that the test of the interpreter's end can compile it alone.
#pragma once
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <cxxabi.h>

namespace ge_py {

struct Decline {};                       // thrown where binding.py's own code has to take the call

// The body of a method: its status as an int, or None where it declines.
template <typename F>
PyObject *guarded(Py_ssize_t given, Py_ssize_t wanted, F body)
{
    if (given != wanted) {
        PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", wanted, given);
        return nullptr;
    }
    try {
        return PyLong_FromLong(body());
    } catch (abi::__forced_unwind &) {   // the thread's end (without_gil)
        throw;
    } catch (...) {                      // Decline, and what torch throws of a tensor without storage
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// Nothing that the entry point could throw is handed to binding.py's own code, which would call it again.  A daemon thread that comes back while the interpreter
// shuts down does not get the GIL again: Python ends it there, by unwinding its stack, so no frame from here up may be one that nothing is thrown through.
template <typename F>
long without_gil(F call)
{
    PyThreadState *state = PyEval_SaveThread();
    const long status = [&]() noexcept { return (long)call(); }();
    PyEval_RestoreThread(state);
    return status;
}

}  // namespace ge_py
