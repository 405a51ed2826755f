// Operand checks of the Python binding, in native code: a stack call hands the
// library 40 to 70 tensors, and checking each from Python (0.8 us apiece) took
// longer than the call's kernels at small sizes.
//
//   pointers(tensors, count, shape, dtype, device) -> bytes or None
//
// The device addresses of tensors[0 .. count - 1] as an array of `void*`, if
// every one is a plain tensor of exactly `shape` and `dtype`, contiguous and on
// `device`; None otherwise (the binding then finds out what is wrong, and says
// so).
#include <torch/csrc/Device.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <vector>

namespace {

constexpr int kMaxDims = 8;

PyObject* pointers(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  if (nargs != 5) {
    PyErr_SetString(PyExc_TypeError, "pointers(tensors, count, shape, dtype, device)");
    return nullptr;
  }
  PyObject *seq = args[0], *shape = args[2];
  const Py_ssize_t count = PyLong_AsSsize_t(args[1]);
  if (count == -1 && PyErr_Occurred()) return nullptr;
  if (!(PyList_CheckExact(seq) || PyTuple_CheckExact(seq)) || !PyTuple_Check(shape) ||
      !THPDtype_Check(args[3]) || !THPDevice_Check(args[4]) ||
      PySequence_Fast_GET_SIZE(seq) < count || count < 0 || PyTuple_GET_SIZE(shape) > kMaxDims)
    Py_RETURN_NONE;
  int64_t dims[kMaxDims];
  const Py_ssize_t nd = PyTuple_GET_SIZE(shape);
  for (Py_ssize_t i = 0; i < nd; i++) {
    dims[i] = PyLong_AsLongLong(PyTuple_GET_ITEM(shape, i));
    if (dims[i] == -1 && PyErr_Occurred()) return nullptr;
  }
  const auto dtype = reinterpret_cast<THPDtype*>(args[3])->scalar_type;
  const auto device = reinterpret_cast<THPDevice*>(args[4])->device;
  std::vector<void*> out((size_t)count);
  for (Py_ssize_t i = 0; i < count; i++) {
    PyObject* o = PySequence_Fast_ITEMS(seq)[i];
    if (!THPVariable_CheckExact(o)) Py_RETURN_NONE;
    const at::Tensor& t = THPVariable_Unpack(o);
    // strided storage with an address of its own (no fake, wrapped or meta tensor)
    bool ok = t.layout() == c10::kStrided && t.scalar_type() == dtype && t.device() == device &&
              device.type() == c10::kCUDA && !t.unsafeGetTensorImpl()->is_python_dispatch() &&
              t.has_storage() && !t.is_conj() && !t.is_neg() && t.dim() == nd &&
              t.is_contiguous();
    for (Py_ssize_t k = 0; ok && k < nd; k++) ok = t.size(k) == dims[k];
    if (!ok) Py_RETURN_NONE;
    out[(size_t)i] = t.data_ptr();
  }
  return PyBytes_FromStringAndSize(reinterpret_cast<const char*>(out.data()),
                                   count * (Py_ssize_t)sizeof(void*));
}

PyObject* guarded_pointers(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
  try {
    return pointers(self, args, nargs);
  } catch (...) {   // a tensor that has no such property: the binding's own checks decide
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

PyMethodDef methods[] = {
    {"pointers", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(guarded_pointers)),
     METH_FASTCALL, "addresses of tensors that match, or None"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
