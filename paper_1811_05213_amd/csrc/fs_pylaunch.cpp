// fs_pylaunch.cpp - the launch path of runner.DeviceRun as a CPython extension module.
//
// A launch of a small plan is bound by what the host does for it.  hipModuleLaunchKernel takes 2.65 us of a call for any kernel with
// arguments; around it, reading the tensors' addresses in Python, building two ctypes arrays and a foreign call with six arguments
// took 1.7 us (softmax f32 [256,1024]: 4.3 us a launch, the kernel 2.9).  Here the addresses are read and fs_plan_run is called without
// leaving C.  Nothing is kept from one call for the next.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstddef>

namespace {

typedef int (*run_fn)(void* plan, const void* const* inputs, void* const* outputs, void* workspace, size_t workspace_bytes, void* stream);

PyObject* g_data_ptr = nullptr;  // "data_ptr"

// the addresses of a sequence of tensors; false with a Python error set
bool addresses(PyObject* tensors, void** out, Py_ssize_t n) {
  for (Py_ssize_t k = 0; k < n; ++k) {
    PyObject* p = PyObject_CallMethodNoArgs(PySequence_Fast_GET_ITEM(tensors, k), g_data_ptr);
    if (!p) return false;
    out[k] = PyLong_AsVoidPtr(p);
    Py_DECREF(p);
    if (!out[k] && PyErr_Occurred()) return false;
  }
  return true;
}

// launch(fs_plan_run, plan, inputs, outputs, workspace or None, workspace_bytes, stream) -> status
PyObject* launch(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  if (nargs != 7) {
    PyErr_SetString(PyExc_TypeError, "launch takes 7 arguments");
    return nullptr;
  }
  const run_fn run = reinterpret_cast<run_fn>(PyLong_AsVoidPtr(args[0]));
  void* const plan = PyLong_AsVoidPtr(args[1]);
  const size_t workspace_bytes = PyLong_AsSize_t(args[5]);
  void* const stream = PyLong_AsVoidPtr(args[6]);
  if (PyErr_Occurred()) return nullptr;
  if (!run) {
    PyErr_SetString(PyExc_ValueError, "launch: no fs_plan_run");
    return nullptr;
  }
  PyObject* result = nullptr;
  PyObject* const ins = PySequence_Fast(args[2], "inputs is no sequence");
  PyObject* const outs = ins ? PySequence_Fast(args[3], "outputs is no sequence") : nullptr;
  if (outs) {
    const Py_ssize_t ni = PySequence_Fast_GET_SIZE(ins), no = PySequence_Fast_GET_SIZE(outs);
    void* few[64];
    void** many = nullptr;  // (no exception may leave a C entry: no std::vector)
    void** table = few;
    if (ni + no + 2 > 64) {
      table = many = static_cast<void**>(PyMem_Malloc(sizeof(void*) * (size_t)(ni + no + 2)));
      if (!many) {
        Py_DECREF(outs);
        Py_DECREF(ins);
        return PyErr_NoMemory();
      }
    }
    // (each list ends with NULL, which fs_plan_run refuses where the plan has more tensors than were given)
    void** const out_table = table + ni + 1;
    table[ni] = out_table[no] = nullptr;
    void* workspace = nullptr;
    bool ok = addresses(ins, table, ni) && addresses(outs, out_table, no);
    if (ok && args[4] != Py_None) {
      PyObject* p = PyObject_CallMethodNoArgs(args[4], g_data_ptr);
      workspace = p ? PyLong_AsVoidPtr(p) : nullptr;
      ok = p && !(workspace == nullptr && PyErr_Occurred());
      Py_XDECREF(p);
    }
    if (ok) {
      int status;
      Py_BEGIN_ALLOW_THREADS
      status = run(plan, table, out_table, workspace, workspace_bytes, stream);
      Py_END_ALLOW_THREADS
      result = PyLong_FromLong(status);
    }
    PyMem_Free(many);
  }
  Py_XDECREF(outs);
  Py_XDECREF(ins);
  return result;
}

PyMethodDef methods[] = {{"launch", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(launch)), METH_FASTCALL,
                          "launch(fs_plan_run, plan, inputs, outputs, workspace, workspace_bytes, stream) -> status"},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_launch", "fs_plan_run on the addresses of tensors", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__launch(void) {
  g_data_ptr = PyUnicode_InternFromString("data_ptr");
  return g_data_ptr ? PyModule_Create(&module) : nullptr;
}
