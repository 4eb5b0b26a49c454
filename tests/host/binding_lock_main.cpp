// A library call that throws, as the binding makes it: whether the interpreter's lock is held when the exception arrives.
#include "../../paper_2410_09687_amd/csrc/binding.cpp"

#include <cstdio>
#include <cstdlib>
#include <new>

namespace {
PyObject *throwing(PyObject *const *)
{
    try {
        call("throwing", []() -> int { throw std::bad_alloc(); });
    } catch (const std::bad_alloc &) {
        if (!PyGILState_Check()) {
            std::puts("the lock is not held");
            std::fflush(stdout);
            std::_Exit(3);
        }
        throw;
    }
    Py_RETURN_NONE;
}
PyMethodDef lock_methods[] = {MOIN_ENTRY(throwing, 0), {nullptr, nullptr, 0, nullptr}};
PyModuleDef lock_module = {PyModuleDef_HEAD_INIT, "binding_lock", nullptr, -1, lock_methods, nullptr, nullptr, nullptr, nullptr};
}  // namespace

PyMODINIT_FUNC PyInit_binding_lock() { return PyModule_Create(&lock_module); }
