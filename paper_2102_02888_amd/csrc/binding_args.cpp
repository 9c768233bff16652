// Argument checks of the Python binding, in native code: the fused step passes
// 13 tensors, and type, device, layout and size checks of one tensor through
// Python attributes cost about as much as a kernel launch's third.  Host code
// only; built against torch's headers, for one torch and Python (build.py's
// args_path).
//
//   pointer(tensor, dtype, cols, rows, cuda) -> int
//
// is the device pointer of `tensor` if it passes every check that the binding
// makes (a tensor of `dtype`, on a GPU when `cuda` is true, at most 2-D, unit
// stride in its last dimension, and with cols >= 0 at least `rows` rows of
// `cols` elements), and -1 if it does not; the binding then repeats the checks
// one by one to name the one that failed.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

PyObject *pointer(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    if (nargs != 5) {
        PyErr_SetString(PyExc_TypeError, "pointer(tensor, dtype, cols, rows, cuda)");
        return nullptr;
    }
    const long long cols = PyLong_AsLongLong(args[2]);
    const long long rows = PyLong_AsLongLong(args[3]);
    const int cuda = PyObject_IsTrue(args[4]);
    if (PyErr_Occurred()) return nullptr;
    if (!THPVariable_CheckExact(args[0]) || !THPDtype_Check(args[1])) return PyLong_FromLong(-1);
    try {
        const at::Tensor &t = THPVariable_Unpack(args[0]);
        if (t.scalar_type() != reinterpret_cast<THPDtype *>(args[1])->scalar_type ||
            (cuda && !t.is_cuda()))
            return PyLong_FromLong(-1);
        const int64_t dim = t.dim();
        if (dim > 2 || (dim >= 1 && t.stride(dim - 1) != 1)) return PyLong_FromLong(-1);
        if (cols >= 0) {
            const int64_t have_rows = dim == 2 ? t.size(0) : 1;
            const int64_t have_cols = dim == 2 ? t.size(1) : t.numel();
            if (have_rows < rows || have_cols < cols) return PyLong_FromLong(-1);
        }
        return PyLong_FromUnsignedLongLong(reinterpret_cast<uintptr_t>(t.data_ptr()));
    } catch (...) {  // a tensor without storage or plain strides: the slow path says so
        return PyLong_FromLong(-1);
    }
}

PyMethodDef methods[] = {
    {"pointer", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(pointer)),
     METH_FASTCALL, "Device pointer of a tensor that passes the binding's checks, or -1."},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "onebit_args", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_onebit_args(void) { return PyModule_Create(&module); }
