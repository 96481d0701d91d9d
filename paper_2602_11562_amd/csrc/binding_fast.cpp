// The marshalling of laser_forward in native code, for calls of the ordinary form: plain device tensors, contiguous, outputs given.
// Anything else returns None, and the caller (binding.py) goes its own way, with its own checks and errors. A small request is 8 us
// of kernels; attribute by attribute in Python, with ctypes, its host part took 10.5 us a call. Torch's accessors are inlined here, so
// the module names the torch that it was built against (`stamp`), and the caller leaves it alone in any other.
#include <torch/csrc/autograd/python_variable.h>

typedef int (*Forward)(const void*, const void*, const void*, const void*, const void*, const void*, const void*, const int32_t*, int, int,
                       int, int, int, int, float, int, int, void*, int32_t*, float*, void*);

// a tensor's data where it is a plain contiguous device tensor of the type, else null
static void* data_of(PyObject* o, at::ScalarType type) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.scalar_type() != type || t.layout() != at::kStrided || !t.has_storage() || !t.is_contiguous())
    return nullptr;
  return t.data_ptr();
}

// whether the number just read was no address: then nothing may be called with it, and nothing returned beside its error
static bool no_address() {
  const bool bad = PyErr_Occurred() != nullptr;
  if (bad) PyErr_Clear();
  return bad;
}

// forward(address of laser_forward, q, k, v, t0, wq, wk, wv, lens, w, gamma, seg_out, seg_cnt, z_out, stream) -> status, or None:
// not a call of this form, nothing done
static PyObject* forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  try {
    if (n != 15 || !PyLong_CheckExact(a[0]) || !PyLong_CheckExact(a[9]) || !PyFloat_CheckExact(a[10])) Py_RETURN_NONE;
    const auto fn = reinterpret_cast<Forward>(PyLong_AsVoidPtr(a[0]));
    int overflow = 0;
    const long w = PyLong_AsLongAndOverflow(a[9], &overflow);
    if (no_address()) Py_RETURN_NONE;
    if (!fn || overflow || w != (int)w || w == 0 || !THPVariable_CheckExact(a[1])) Py_RETURN_NONE;
    const at::Tensor& q = THPVariable_Unpack(a[1]);
    const at::ScalarType type = q.scalar_type();
    if (type != at::kFloat && type != at::kBFloat16) Py_RETURN_NONE;
    void* p[7];
    for (int i = 0; i < 7; ++i)
      if (!(p[i] = data_of(a[1 + i], type))) Py_RETURN_NONE;
    const at::Tensor &v = THPVariable_Unpack(a[3]), &wq = THPVariable_Unpack(a[5]);
    if (q.dim() != 3 || v.dim() < 3 || wq.dim() < 1) Py_RETURN_NONE;
    void *lens = nullptr, *cnt = nullptr, *stream = nullptr;
    if (a[8] != Py_None && !(lens = data_of(a[8], at::kInt))) Py_RETURN_NONE;
    if (a[12] != Py_None && !(cnt = data_of(a[12], at::kInt))) Py_RETURN_NONE;
    void *seg = data_of(a[11], type), *z = data_of(a[13], at::kFloat);
    if (!seg || !z) Py_RETURN_NONE;
    if (a[14] != Py_None) {
      if (!PyLong_CheckExact(a[14])) Py_RETURN_NONE;
      stream = PyLong_AsVoidPtr(a[14]);
      if (no_address()) Py_RETURN_NONE;
    }
    const int64_t sizes[6] = {q.size(0), q.size(1), v.size(1), q.size(2), v.size(2), wq.size(0)};
    for (const int64_t s : sizes)
      if (s != (int)s) Py_RETURN_NONE;
    const float gamma = (float)PyFloat_AS_DOUBLE(a[10]);
    int code;
    Py_BEGIN_ALLOW_THREADS
    code = fn(p[0], p[1], p[2], p[3], p[4], p[5], p[6], static_cast<int32_t*>(lens), (int)sizes[0], (int)sizes[1], (int)sizes[2],
              (int)sizes[3], (int)sizes[4], (int)w, gamma, (int)sizes[5], type == at::kFloat ? 0 : 1, seg, static_cast<int32_t*>(cnt),
              static_cast<float*>(z), stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(code);
  } catch (...) {   // (a tensor without data of its own: as any other form)
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

static PyMethodDef methods[] = {
    {"forward", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(forward)), METH_FASTCALL, nullptr}, {nullptr, nullptr, 0, nullptr}};
static PyModuleDef module = {PyModuleDef_HEAD_INIT, "laser_fast", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};
PyMODINIT_FUNC PyInit_laser_fast() {
  PyObject* m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "stamp", LASER_TORCH_STAMP) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
