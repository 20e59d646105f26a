// The calls of binding.py that launch kernels, from tensors to the C-ABI without a Python object in between: a call of that layer took
// 3 us of checks and conversions beside the 3 us of the library and the launch.  Each function here makes the checks of the Python
// function it stands for; where one fails, or an argument is anything but a plain tensor, it returns None and has done nothing, and the Python
// function goes on to do the same checks and to raise what they raise.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <cstring>

#include "roast.h"

// (build.py looks for it in the file)
extern "C" __attribute__((used, visibility("default"))) const char roast_call_stamp[] = ROAST_CALL_STAMP;

namespace {

// functions of the library that binding.py has loaded, by address
struct Library {
  decltype(&roast_mm_fwd_ws) mm_fwd_ws;
  decltype(&roast_mm_bwd_dx_ws) mm_bwd_dx_ws;
  decltype(&roast_mm_bwd_dM) mm_bwd_dM;
  decltype(&roast_embed_fwd) embed_fwd;
  decltype(&roast_embed_bwd) embed_bwd;
  decltype(&roast_embed_bag_fwd) embed_bag_fwd;
  decltype(&roast_embed_bag_bwd) embed_bag_bwd;
  decltype(&roast_optim_step) optim_step;
  decltype(&roast_m_shadow_bytes) m_shadow_bytes;
  decltype(&roast_m_planes_bytes) m_planes_bytes;
  decltype(&roast_m_shadow_bf16) m_shadow_bf16;
  decltype(&roast_m_planes_bf16) m_planes_bf16;
};
Library lib{};
PyObject *get_device = nullptr, *get_stream = nullptr;   // torch._C._cuda_getDevice, _cuda_getCurrentRawStream
PyObject* classes[3] = {};                               // the descriptors' ctypes structures, see index_of
constexpr int index_of(const roast_mm_desc*) { return 0; }
constexpr int index_of(const roast_embed_desc*) { return 1; }
constexpr int index_of(const roast_optim_desc*) { return 2; }

constexpr long kNothingDone = -1;

// A device tensor with a storage of its own (no subclass, no wrapper of a transform), or null
const at::Tensor* tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  return t.defined() && t.is_cuda() && t.layout() == at::kStrided && t.has_storage() && !t.unsafeGetTensorImpl()->has_symbolic_sizes_strides() ? &t : nullptr;
}
bool vector(PyObject* o, at::ScalarType type, void** p, int64_t* n) {
  const at::Tensor* t = tensor(o);
  if (!t || t->scalar_type() != type || !t->is_contiguous()) return false;
  *p = t->data_ptr();
  *n = t->numel();
  return true;
}
bool matrix(PyObject* o, const at::Tensor** t, void** p, int64_t* ld) {
  *t = tensor(o);
  if (!*t || (*t)->dim() != 2) return false;
  const int64_t rows = (*t)->size(0), cols = (*t)->size(1);
  if (cols > 1 && (*t)->stride(1) != 1) return false;
  *p = (*t)->data_ptr();
  *ld = rows > 1 ? (*t)->stride(0) : std::max(cols, (*t)->stride(0));
  return true;
}
bool workspace(PyObject* o, void** p, size_t* bytes) {
  *p = nullptr;
  *bytes = 0;
  if (o == Py_None) return true;
  const at::Tensor* t = tensor(o);
  if (!t) return false;
  *p = t->data_ptr();
  *bytes = (size_t)t->numel() * t->element_size();
  return true;
}
bool copy_of_m(PyObject* o, int64_t m, bool f32, void** p) {
  *p = nullptr;
  if (o == Py_None) return true;
  int64_t n;
  return vector(o, at::kBFloat16, p, &n) && n == (int64_t)((f32 ? lib.m_planes_bytes(m) : lib.m_shadow_bytes(m)) / 2);
}
bool code(const at::Tensor& t, roast_dtype* dt) {
  if (t.scalar_type() != at::kFloat && t.scalar_type() != at::kBFloat16) return false;
  *dt = t.scalar_type() == at::kFloat ? ROAST_F32 : ROAST_BF16;
  return true;
}
// A descriptor: binding.py's structure for it, or one derived from that, as ctypes takes it
template <typename D>
bool descriptor(PyObject* o, D* d) {
  Py_buffer b;
  if (!PyObject_TypeCheck(o, reinterpret_cast<PyTypeObject*>(classes[index_of(d)]))) return false;
  if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) {
    PyErr_Clear();
    return false;
  }
  const bool ok = b.len >= (Py_ssize_t)sizeof(D);      // (a derived structure may be longer)
  if (ok) memcpy(d, b.buf, sizeof(D));
  PyBuffer_Release(&b);
  return ok;
}
bool current_stream(void** s) {
  PyObject* device = PyObject_CallNoArgs(get_device);
  PyObject* handle = device ? PyObject_CallOneArg(get_stream, device) : nullptr;
  Py_XDECREF(device);
  if (handle) *s = PyLong_AsVoidPtr(handle);
  Py_XDECREF(handle);
  if (PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return true;
}
bool number(PyObject* o, int* v) {
  if (!PyLong_CheckExact(o)) return false;
  const long x = PyLong_AsLong(o);
  if (x == -1 && PyErr_Occurred()) {     // (beyond a long)
    PyErr_Clear();
    return false;
  }
  if (x != (int)x) return false;
  *v = (int)x;
  return true;
}

// The library's function without the interpreter's lock, as a call through ctypes is
template <typename F, typename... A>
long run(F f, A... a) {
  PyThreadState* state = PyEval_SaveThread();
  const long st = f(a...);
  PyEval_RestoreThread(state);
  return st;
}

// desc, A, M, C, copy of M, workspace
template <bool DX>
long mm(PyObject* const* a) {
  roast_mm_desc d;
  const at::Tensor *A, *C;
  void *ap, *cp, *m, *mb, *ws, *s;
  int64_t lda, ldc, n;
  size_t bytes;
  roast_dtype dt;
  if (!descriptor(a[0], &d) || !matrix(a[1], &A, &ap, &lda) || !matrix(a[3], &C, &cp, &ldc) || !code(*A, &dt) || C->scalar_type() != A->scalar_type() ||
      A->size(1) != (DX ? d.O : d.H) || C->size(0) != A->size(0) || C->size(1) != (DX ? d.H : d.O) || !vector(a[2], at::kFloat, &m, &n) ||
      !copy_of_m(a[4], n, dt == ROAST_F32, &mb) || !workspace(a[5], &ws, &bytes) || !current_stream(&s))
    return kNothingDone;
  return run(DX ? lib.mm_bwd_dx_ws : lib.mm_fwd_ws, &d, dt, A->size(0), ap, lda, (const float*)m, mb, cp, ldc, ws, bytes, s);
}
// desc, X, dY, dM, mode, workspace
long mm_bwd_dM(PyObject* const* a) {
  roast_mm_desc d;
  const at::Tensor *X, *Y;
  void *xp, *yp, *dM, *ws, *s;
  int64_t ldx, ldy, n;
  size_t bytes;
  roast_dtype dt;
  int mode;
  if (!descriptor(a[0], &d) || !matrix(a[1], &X, &xp, &ldx) || !matrix(a[2], &Y, &yp, &ldy) || !code(*X, &dt) || Y->scalar_type() != X->scalar_type() ||
      X->size(1) != d.H || Y->size(0) != X->size(0) || Y->size(1) != d.O || !vector(a[3], at::kFloat, &dM, &n) || n != d.m_size || !number(a[4], &mode) ||
      !workspace(a[5], &ws, &bytes) || !current_stream(&s))
    return kNothingDone;
  return run(lib.mm_bwd_dM, &d, dt, X->size(0), xp, ldx, yp, ldy, (float*)dM, (roast_reduce_mode)mode, ws, bytes, s);
}
bool rows_of(PyObject* o, int64_t rows, int64_t cols, void** p) {
  const at::Tensor* t = tensor(o);
  int64_t n;
  return t && t->dim() == 2 && t->size(0) == rows && t->size(1) == cols && vector(o, at::kFloat, p, &n);
}
// desc, rows, table ids, M, out
long embed_fwd(PyObject* const* a) {
  roast_embed_desc d;
  void *rows, *tables, *m, *out, *s;
  int64_t N, nt, n;
  if (!descriptor(a[0], &d) || !vector(a[1], at::kLong, &rows, &N) || !vector(a[2], at::kInt, &tables, &nt) || !vector(a[3], at::kFloat, &m, &n) ||
      !rows_of(a[4], N, d.D, &out) || !current_stream(&s))
    return kNothingDone;
  return run(lib.embed_fwd, &d, N, (const int64_t*)rows, (const uint32_t*)tables, (const float*)m, (float*)out, s);
}
// desc, rows, table ids, dOut, dM, mode, workspace
long embed_bwd(PyObject* const* a) {
  roast_embed_desc d;
  void *rows, *tables, *g, *dM, *ws, *s;
  int64_t N, nt, n;
  size_t bytes;
  int mode;
  if (!descriptor(a[0], &d) || !vector(a[1], at::kLong, &rows, &N) || !vector(a[2], at::kInt, &tables, &nt) || !rows_of(a[3], N, d.D, &g) ||
      !vector(a[4], at::kFloat, &dM, &n) || n != d.m_size || !number(a[5], &mode) || !workspace(a[6], &ws, &bytes) || !current_stream(&s))
    return kNothingDone;
  return run(lib.embed_bwd, &d, N, (const int64_t*)rows, (const uint32_t*)tables, (const float*)g, (float*)dM, (roast_reduce_mode)mode, ws, bytes, s);
}
// desc, rows, table ids, bag offsets, M, out
long embed_bag_fwd(PyObject* const* a) {
  roast_embed_desc d;
  void *rows, *tables, *off, *m, *out, *s;
  int64_t N, nt, B, n;
  if (!descriptor(a[0], &d) || !vector(a[1], at::kLong, &rows, &N) || !vector(a[2], at::kInt, &tables, &nt) || !vector(a[3], at::kLong, &off, &B) || B < 1 ||
      !vector(a[4], at::kFloat, &m, &n) || !rows_of(a[5], B - 1, d.D, &out) || !current_stream(&s))
    return kNothingDone;
  return run(lib.embed_bag_fwd, &d, N, B - 1, (const int64_t*)rows, (const uint32_t*)tables, (const int64_t*)off, (const float*)m, (float*)out, s);
}
// desc, rows, table ids, bag offsets, dOut, dM, mode, workspace
long embed_bag_bwd(PyObject* const* a) {
  roast_embed_desc d;
  void *rows, *tables, *off, *g, *dM, *ws, *s;
  int64_t N, nt, B, n;
  size_t bytes;
  int mode;
  if (!descriptor(a[0], &d) || !vector(a[1], at::kLong, &rows, &N) || !vector(a[2], at::kInt, &tables, &nt) || !vector(a[3], at::kLong, &off, &B) || B < 1 ||
      !rows_of(a[4], B - 1, d.D, &g) || !vector(a[5], at::kFloat, &dM, &n) || n != d.m_size || !number(a[6], &mode) || !workspace(a[7], &ws, &bytes) ||
      !current_stream(&s))
    return kNothingDone;
  return run(lib.embed_bag_bwd, &d, N, B - 1, (const int64_t*)rows, (const uint32_t*)tables, (const int64_t*)off, (const float*)g, (float*)dM, (roast_reduce_mode)mode,
                           ws, bytes, s);
}
// desc, M, dM, state1, state2, copy of M
long optim_step(PyObject* const* a) {
  roast_optim_desc d;
  void *p[4] = {}, *mb, *s;
  int64_t n, k;
  if (!descriptor(a[0], &d) || !vector(a[1], at::kFloat, &p[0], &n)) return kNothingDone;
  for (int i = 1; i < 4; ++i)
    if ((i == 1 || a[1 + i] != Py_None) && (!vector(a[1 + i], at::kFloat, &p[i], &k) || k != n)) return kNothingDone;
  if (!copy_of_m(a[5], n, false, &mb) || !current_stream(&s)) return kNothingDone;
  return run(lib.optim_step, &d, n, (float*)p[0], (float*)p[1], (float*)p[2], (float*)p[3], mb, s);
}
// M, copy (not None)
template <bool F32>
long m_copy(PyObject* const* a) {
  void *m, *mb, *s;
  int64_t n;
  if (!vector(a[0], at::kFloat, &m, &n) || a[1] == Py_None || !copy_of_m(a[1], n, F32, &mb) || !current_stream(&s)) return kNothingDone;
  return run(F32 ? lib.m_planes_bf16 : lib.m_shadow_bf16, (const float*)m, n, mb, s);
}

// The library's status, or None
template <long (*F)(PyObject* const*), int N>
PyObject* call(PyObject*, PyObject* const* a, Py_ssize_t n) {
  long st = kNothingDone;
  if (n == N && get_stream) {
    try {
      st = F(a);
    } catch (...) {                      // (of a check: the library throws nothing)
      st = kNothingDone;
    }
  }
  if (st == kNothingDone) Py_RETURN_NONE;
  return PyLong_FromLong(st);
}

// torch._C, the descriptors' classes, then the addresses of the library's functions in the order of Library
PyObject* connect(PyObject*, PyObject* const* a, Py_ssize_t n) {
  constexpr Py_ssize_t count = sizeof(Library) / sizeof(void*);
  if (n != 4 + count || !PyType_Check(a[1]) || !PyType_Check(a[2]) || !PyType_Check(a[3])) {
    PyErr_SetString(PyExc_TypeError, "connect: torch._C, the classes of the descriptors and the addresses of the library's functions");
    return nullptr;
  }
  void* f[count];
  for (Py_ssize_t i = 0; i < count; ++i)
    if (f[i] = PyLong_AsVoidPtr(a[4 + i]); PyErr_Occurred()) return nullptr;
  for (int i = 0; i < 3; ++i) {
    Py_INCREF(a[1 + i]);
    Py_XSETREF(classes[i], a[1 + i]);
  }
  Py_XSETREF(get_stream, nullptr);
  Py_XSETREF(get_device, PyObject_GetAttrString(a[0], "_cuda_getDevice"));
  if (!get_device) return nullptr;
  get_stream = PyObject_GetAttrString(a[0], "_cuda_getCurrentRawStream");
  if (!get_stream) return nullptr;
  memcpy(&lib, f, sizeof(lib));
  Py_RETURN_NONE;
}

#define CALL(name, f, n) {name, (PyCFunction)(void (*)(void))&call<f, n>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"connect", (PyCFunction)(void (*)(void))&connect, METH_FASTCALL, nullptr},
                         CALL("mm_fwd", mm<false>, 6),
                         CALL("mm_bwd_dx", mm<true>, 6),
                         CALL("mm_bwd_dM", mm_bwd_dM, 6),
                         CALL("embed_fwd", embed_fwd, 5),
                         CALL("embed_bwd", embed_bwd, 7),
                         CALL("embed_bag_fwd", embed_bag_fwd, 6),
                         CALL("embed_bag_bwd", embed_bag_bwd, 8),
                         CALL("optim_step", optim_step, 6),
                         CALL("m_shadow_bf16", m_copy<false>, 2),
                         CALL("m_planes_bf16", m_copy<true>, 2),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_roast_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__roast_call() { return PyModule_Create(&module); }
