// A native method as those of py_marshal.cpp, whose library call takes as long as the test asks for.
#include "../paper_2604_01489_amd/csrc/py_call.h"

#include <unistd.h>

static PyObject *call(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return ge_py::guarded(n, 1, [&]() -> long {
        const long us = PyLong_AsLong(a[0]);
        if (us < 0) throw ge_py::Decline{};
        return ge_py::without_gil([&] { usleep((useconds_t)us); return 7; });
    });
}

static PyMethodDef methods[] = {{"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL, nullptr}, {nullptr, nullptr, 0, nullptr}};
static PyModuleDef module = {PyModuleDef_HEAD_INIT, "py_call_probe", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};
PyMODINIT_FUNC PyInit_py_call_probe(void) { return PyModule_Create(&module); }
