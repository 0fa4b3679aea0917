// The way from Python to the device entry points of the C ABI (include/egt.h), as a CPython
// extension module.  A product of a few megabytes is over in 3 to 6 us; marshalling its
// arguments in Python (a ctypes structure, sizes and types of six tensors, the current
// stream) took 9 us of a call, so that a loop of single products waited for the interpreter
// and not for the GPU.  Here the tensors are looked at in C++ and a call is one C function.
//
//  - sparse_gemv, sparse_gemm_smallm, int4_gemv: one product with plain arguments.  They
//    check what the ctypes path of binding.py checks; where anything is not as it should be
//    (a wrong type, a short buffer, a refused argument) they launch nothing and return False, and
//    binding.py goes through its own checks, which say what is wrong.  An error of the HIP runtime is
//    raised from here: the call is not made a second time.
//  - Call: a prepared call, arguments marshalled once; calling it crosses the C ABI.
//
// The module is not linked against libegt.so: binding.py hands over the addresses of the
// entry points of the library it has loaded (bind), whichever build that is.
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include <cstdint>
#include <exception>
#include <memory>
#include <vector>

#include "egt.h"

namespace {

typedef int (*gemv_fn)(const void *, const void *, void *, void *);
typedef int (*read_fn)(const void *, size_t, void *, void *);
typedef int (*gemm_fn)(const void *, const void *, int64_t, void *, int64_t, int, void *);
typedef int (*gemm_ws_fn)(const void *, const void *, int64_t, void *, int64_t, int, void *, size_t, void *);
typedef int (*int4_fn)(const void *, const void *, int, int, int, const void *, void *, void *);
typedef int (*gemv_batch_fn)(const void *, const void *, const void *, int, void *);
typedef int (*gemm_batch_fn)(const void *, const void *, int64_t, const void *, int64_t, int, int, void *);
typedef int (*int4_batch_fn)(const void *, const void *, int, int, int, const void *, const void *, int, void *);
typedef int (*table_fn)(const void *, const void *, void *);

enum Kind { GEMV, READ, GEMM, GEMM_WS, INT4, GEMV_BATCH, GEMM_BATCH, INT4_BATCH, TABLE, KINDS };
constexpr int N_ARGS[KINDS] = {3, 3, 6, 8, 7, 4, 7, 8, 2};      // without the stream

struct Thunk {
  Kind kind;
  uintptr_t fn;
  int64_t a[8];
  void *p(int k) const { return (void *)(uintptr_t)a[k]; }
  int i(int k) const { return (int)a[k]; }
  int operator()(void *s) const {
    switch (kind) {
      case GEMV: return ((gemv_fn)fn)(p(0), p(1), p(2), s);
      case READ: return ((read_fn)fn)(p(0), (size_t)a[1], p(2), s);
      case GEMM: return ((gemm_fn)fn)(p(0), p(1), a[2], p(3), a[4], i(5), s);
      case GEMM_WS: return ((gemm_ws_fn)fn)(p(0), p(1), a[2], p(3), a[4], i(5), p(6), (size_t)a[7], s);
      case INT4: return ((int4_fn)fn)(p(0), p(1), i(2), i(3), i(4), p(5), p(6), s);
      case GEMV_BATCH: return ((gemv_batch_fn)fn)(p(0), p(1), p(2), i(3), s);
      case GEMM_BATCH: return ((gemm_batch_fn)fn)(p(0), p(1), a[2], p(3), a[4], i(5), i(6), s);
      case INT4_BATCH: return ((int4_batch_fn)fn)(p(0), p(1), i(2), i(3), i(4), p(5), p(6), i(7), s);
      default: return ((table_fn)fn)(p(0), p(1), s);
    }
  }
};

// what bind() was given
struct {
  gemv_fn sparse_gemv = nullptr;
  gemm_fn gemm = nullptr, gemm_static = nullptr;
  gemm_ws_fn gemm_ws = nullptr;
  int4_fn int4 = nullptr;
  PyObject *check = nullptr;                          // binding._check: turns a status into an exception
  PyObject *raw_stream = nullptr, *get_device = nullptr;
} B;
struct {
  PyObject *rows, *cols, *n_keep, *group, *val_kind, *row_ptr, *values, *idx, *qparams, *total_slots, *cuda_stream, *stream_ptr, *value;
} S;

// ---------------------------------------------------------------- prepared calls
struct Call {
  PyObject_HEAD
  vectorcallfunc vectorcall;
  std::vector<Thunk> *thunks;
  void *stream;
  PyObject *keep, *dict, *weak;
};

// What ctypes takes for a pointer: an integer, None, or an object that carries one (c_void_p)
bool pointer_of(PyObject *o, void *&p) {
  p = nullptr;
  if (o == Py_None) return true;
  if (PyLong_Check(o)) {
    // (handles are read as the bits they are: negative ones too)
    p = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(o);
    return p || !PyErr_Occurred();
  }
  PyObject *v = PyObject_GetAttr(o, S.value);
  if (!v || !(v == Py_None || PyLong_Check(v))) {
    Py_XDECREF(v);
    PyErr_SetString(PyExc_TypeError, "stream_ptr: expected an integer, None or a c_void_p");
    return false;
  }
  const bool ok = pointer_of(v, p);
  Py_DECREF(v);
  return ok;
}

PyObject *call_call(PyObject *self, PyObject *const *args, size_t nargsf, PyObject *kwnames) {
  Call *c = (Call *)self;
  const Py_ssize_t n = PyVectorcall_NARGS(nargsf), nk = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
  void *stream = c->stream;
  if (n + nk > 0) {
    if (n + nk > 1 || (nk == 1 && PyUnicode_Compare(PyTuple_GET_ITEM(kwnames, 0), S.stream_ptr) != 0)) {
      PyErr_SetString(PyExc_TypeError, "a prepared call takes one argument, stream_ptr");
      return nullptr;
    }
    if (!pointer_of(args[0], stream)) return nullptr;
  }
  int st = 0;
  // (a launch waits when the queue is full: other threads of the program go on meanwhile)
  Py_BEGIN_ALLOW_THREADS
  for (const Thunk &t : *c->thunks)
    if ((st = t(stream)) != 0) break;
  Py_END_ALLOW_THREADS
  if (st != 0) return PyObject_CallFunction(B.check, "i", st);
  Py_RETURN_NONE;
}

// Call(kind, address, [arguments of each launch, ...], stream, keep)
PyObject *call_new(PyTypeObject *type, PyObject *args, PyObject *) try {
  int kind;
  unsigned long long fn, stream;
  PyObject *launches, *keep;
  if (!PyArg_ParseTuple(args, "iKO!KO", &kind, &fn, &PyList_Type, &launches, &stream, &keep)) return nullptr;
  if (kind < 0 || kind >= KINDS || !fn) {
    PyErr_SetString(PyExc_ValueError, "unknown kind of call");
    return nullptr;
  }
  auto thunks = std::make_unique<std::vector<Thunk>>();
  for (Py_ssize_t k = 0; k < PyList_GET_SIZE(launches); ++k) {
    PyObject *a = PyList_GET_ITEM(launches, k);
    if (!PyTuple_Check(a) || PyTuple_GET_SIZE(a) != N_ARGS[kind]) {
      PyErr_SetString(PyExc_ValueError, "wrong number of arguments");
      return nullptr;
    }
    Thunk t{(Kind)kind, (uintptr_t)fn, {}};
    for (int j = 0; j < N_ARGS[kind]; ++j) {
      // pointers and sizes may use all 64 bits
      t.a[j] = (int64_t)PyLong_AsUnsignedLongLongMask(PyTuple_GET_ITEM(a, j));
      if (t.a[j] == -1 && PyErr_Occurred()) return nullptr;
    }
    thunks->push_back(t);
  }
  Call *c = (Call *)type->tp_alloc(type, 0);
  if (!c) return nullptr;
  c->vectorcall = call_call;
  c->thunks = thunks.release();
  c->stream = (void *)(uintptr_t)stream;
  Py_INCREF(keep);
  c->keep = keep;
  c->dict = c->weak = nullptr;
  return (PyObject *)c;
} catch (const std::exception &) {                     // (no memory)
  return PyErr_NoMemory();
}
int call_traverse(PyObject *self, visitproc visit, void *arg) {
  Py_VISIT(((Call *)self)->keep);
  Py_VISIT(((Call *)self)->dict);
  return 0;
}
int call_clear(PyObject *self) {
  Py_CLEAR(((Call *)self)->keep);
  Py_CLEAR(((Call *)self)->dict);
  return 0;
}
void call_dealloc(PyObject *self) {
  PyObject_GC_UnTrack(self);
  if (((Call *)self)->weak) PyObject_ClearWeakRefs(self);
  call_clear(self);
  delete ((Call *)self)->thunks;
  Py_TYPE(self)->tp_free(self);
}
PyTypeObject CallType = {PyVarObject_HEAD_INIT(nullptr, 0)};

// ---------------------------------------------------------------- plain calls
// All helpers answer "is it as it should be"; an exception on the way is dropped, the slow
// path raises its own.
bool get_int(PyObject *o, PyObject *name, int64_t &v) {
  PyObject *a = PyObject_GetAttr(o, name);
  if (!a) return false;
  const bool ok = PyLong_CheckExact(a);
  if (ok) v = PyLong_AsLongLong(a);
  Py_DECREF(a);
  return ok && !(v == -1 && PyErr_Occurred());
}
// device address of a contiguous tensor of at least `bytes` bytes
bool plain_tensor(PyObject *o, int64_t bytes, bool f16, void *&ptr) {
  if (!THPVariable_Check(o)) return false;
  const at::Tensor &t = THPVariable_Unpack(o);
  if (!t.is_cuda() || !t.is_contiguous() || (f16 && t.scalar_type() != at::kHalf) || (int64_t)t.nbytes() < bytes) return false;
  ptr = t.data_ptr();
  return true;
}
bool get_tensor(PyObject *o, PyObject *name, int64_t bytes, bool may_be_none, void *&ptr) {
  THPObjectPtr a(PyObject_GetAttr(o, name));     // (the packed matrix keeps it)
  if (!a) return false;
  ptr = nullptr;
  return a.get() == Py_None ? may_be_none : plain_tensor(a.get(), bytes, false, ptr);
}
bool get_view(PyObject *p, egt_2bitcsr &w) {
  int64_t rows, cols, n, group, kind, total;
  if (!get_int(p, S.rows, rows) || !get_int(p, S.cols, cols) || !get_int(p, S.n_keep, n) || !get_int(p, S.group, group) ||
      !get_int(p, S.val_kind, kind) || !get_int(p, S.total_slots, total))
    return false;
  if (rows < 1 || rows > INT32_MAX || cols < 0 || cols > INT32_MAX || cols % 32 || n < 0 || n > 4 || total < 0 || total > UINT32_MAX) return false;
  const bool fp16 = kind == EGT_VAL_FP16;
  if (kind < 0 || kind > 2 || (fp16 ? group != 0 : group <= 0 || group > INT32_MAX || cols % group)) return false;
  const int64_t slots = n ? rows * n * (cols / 4) : total;
  void *rp, *v, *ix, *qp;
  if (!get_tensor(p, S.row_ptr, 4 * (rows + 1), false, rp) || !get_tensor(p, S.values, fp16 ? 2 * slots : slots / 2, false, v) ||
      !get_tensor(p, S.idx, slots / 4, false, ix) || !get_tensor(p, S.qparams, fp16 ? 0 : 4 * rows * (cols / group), fp16, qp))
    return false;
  w.rows = (int32_t)rows; w.cols = (int32_t)cols; w.n_keep = (int32_t)n; w.group_size = (int32_t)group; w.val_kind = (int32_t)kind;
  w.row_ptr = (uint32_t *)rp; w.values = v; w.idx = (uint16_t *)ix; w.qparams = (uint16_t *)qp; w.total_slots = (uint32_t)total;
  return true;
}
// the stream object's handle, or that of the current stream
bool get_stream(PyObject *stream, void *&s) {
  PyObject *v;
  if (stream == Py_None) {
    PyObject *dev = PyObject_CallNoArgs(B.get_device);
    if (!dev) return false;
    v = PyObject_CallOneArg(B.raw_stream, dev);
    Py_DECREF(dev);
  } else {
    v = PyObject_GetAttr(stream, S.cuda_stream);
  }
  if (!v) return false;
  s = PyLong_AsVoidPtr(v);
  Py_DECREF(v);
  return s || !PyErr_Occurred();
}
PyObject *answer(bool ok) {
  if (!ok) PyErr_Clear();
  return PyBool_FromLong(ok);
}
// ... of a call that has reached the library
PyObject *outcome(int st) {
  if (st != EGT_ERR_HIP) return answer(st == EGT_OK);
  PyErr_Clear();
  return PyObject_CallFunction(B.check, "i", st);      // (raises)
}
// A tensor without memory of its own (under a transform, a fake mode, of a sparse layout) throws
// where its address or its strides are asked for: no exception may cross into the interpreter.
template <PyObject *(*F)(PyObject *, PyObject *const *, Py_ssize_t)>
PyObject *guarded(PyObject *self, PyObject *const *a, Py_ssize_t n) {
  try {
    return F(self, a, n);
  } catch (const std::exception &) {
    return answer(false);
  }
}

// sparse_gemv(p, x, y, stream)
PyObject *sparse_gemv(PyObject *, PyObject *const *a, Py_ssize_t n) {
  egt_2bitcsr w;
  void *x, *y, *s;
  if (n != 4 || !B.sparse_gemv || !get_view(a[0], w) || !plain_tensor(a[1], 2 * (int64_t)w.cols, true, x) ||
      !plain_tensor(a[2], 2 * (int64_t)w.rows, true, y) || !get_stream(a[3], s))
    return answer(false);
  int st;
  Py_BEGIN_ALLOW_THREADS
  st = B.sparse_gemv(&w, x, y, s);
  Py_END_ALLOW_THREADS
  return outcome(st);
}

// X (M, cols) or Y (M, rows): FP16, rows of contiguous elements
bool token_rows(PyObject *o, int64_t M, int64_t cols, void *&ptr, int64_t &ld) {
  if (!THPVariable_Check(o)) return false;
  const at::Tensor &t = THPVariable_Unpack(o);
  if (!t.is_cuda() || t.scalar_type() != at::kHalf || t.dim() != 2 || t.size(1) != cols || (M >= 0 && t.size(0) != M) ||
      (cols > 1 && t.stride(1) != 1))
    return false;
  ptr = t.data_ptr();
  ld = t.stride(0);
  return true;
}
// sparse_gemm_smallm(form, p, X, Y, workspace, stream); form 0: one launch, 1: workspace, 2: the library's scratch
PyObject *sparse_gemm_smallm(PyObject *, PyObject *const *a, Py_ssize_t n) {
  egt_2bitcsr w;
  void *x, *y, *s, *ws = nullptr;
  int64_t ldx, ldy, wb = 0;
  if (n != 6 || !B.gemm || !get_view(a[1], w) || !token_rows(a[2], -1, w.cols, x, ldx)) return answer(false);
  const long form = PyLong_AsLong(a[0]);
  const int64_t M = THPVariable_Unpack(a[2]).size(0);
  if (M < 1 || M > 64 || !token_rows(a[3], M, w.rows, y, ldy) || !get_stream(a[5], s)) return answer(false);
  if (form == 1 && a[4] != Py_None) {                 // (a workspace that is missing or too short is an error status)
    if (!plain_tensor(a[4], 0, false, ws)) return answer(false);
    wb = (int64_t)THPVariable_Unpack(a[4]).nbytes();
  }
  int st;
  Py_BEGIN_ALLOW_THREADS
  st = form == 0 ? B.gemm(&w, x, ldx, y, ldy, (int)M, s)
     : form == 1 ? B.gemm_ws(&w, x, ldx, y, ldy, (int)M, ws, (size_t)wb, s)
                 : B.gemm_static(&w, x, ldx, y, ldy, (int)M, s);
  Py_END_ALLOW_THREADS
  return outcome(st);
}

// int4_gemv(q, qparams, rows, cols, group, x, y, stream)
PyObject *int4_gemv(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 8 || !B.int4 || !PyLong_CheckExact(a[2]) || !PyLong_CheckExact(a[3]) || !PyLong_CheckExact(a[4])) return answer(false);
  const int64_t rows = PyLong_AsLongLong(a[2]), cols = PyLong_AsLongLong(a[3]), group = PyLong_AsLongLong(a[4]);
  void *q, *qp, *x, *y, *s;
  if (rows < 1 || rows > INT32_MAX || cols < 0 || cols > INT32_MAX || group <= 0 || group > INT32_MAX || cols % group ||
      !plain_tensor(a[0], rows * (cols / 2), false, q) || !plain_tensor(a[1], 4 * rows * (cols / group), false, qp) ||
      !plain_tensor(a[5], 2 * cols, true, x) || !plain_tensor(a[6], 2 * rows, true, y) || !get_stream(a[7], s))
    return answer(false);
  int st;
  Py_BEGIN_ALLOW_THREADS
  st = B.int4(q, qp, (int)rows, (int)cols, (int)group, x, y, s);
  Py_END_ALLOW_THREADS
  return outcome(st);
}

// bind(sparse_gemv, gemm, gemm_ws, gemm_static, int4, check, raw_stream, get_device): addresses of the entry
// points; binding._check; current stream handle of a device; current device
PyObject *bind(PyObject *, PyObject *args) {
  unsigned long long f[5];
  PyObject *check, *raw, *dev;
  if (!PyArg_ParseTuple(args, "KKKKKOOO", f, f + 1, f + 2, f + 3, f + 4, &check, &raw, &dev)) return nullptr;
  B.sparse_gemv = (gemv_fn)f[0];
  B.gemm = (gemm_fn)f[1];
  B.gemm_ws = (gemm_ws_fn)f[2];
  B.gemm_static = (gemm_fn)f[3];
  B.int4 = (int4_fn)f[4];
  Py_INCREF(check); Py_XSETREF(B.check, check);
  Py_INCREF(raw); Py_XSETREF(B.raw_stream, raw);
  Py_INCREF(dev); Py_XSETREF(B.get_device, dev);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    {"sparse_gemv", (PyCFunction)(void (*)(void))guarded<sparse_gemv>, METH_FASTCALL, nullptr},
    {"sparse_gemm_smallm", (PyCFunction)(void (*)(void))guarded<sparse_gemm_smallm>, METH_FASTCALL, nullptr},
    {"int4_gemv", (PyCFunction)(void (*)(void))guarded<int4_gemv>, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "egt_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};
// A copy of a call, shallow or deep, is the call itself, as for a function: its pointers are those of its buffers.
PyObject *call_copy(PyObject *self, PyObject *) {
  Py_INCREF(self);
  return self;
}
PyMethodDef call_methods[] = {{"__copy__", call_copy, METH_NOARGS, nullptr}, {"__deepcopy__", call_copy, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyGetSetDef call_getset[] = {{"__dict__", PyObject_GenericGetDict, PyObject_GenericSetDict, nullptr, nullptr}, {nullptr, nullptr, nullptr, nullptr, nullptr}};

}  // namespace

PyMODINIT_FUNC PyInit_egt_call(void) {
  CallType.tp_name = "egt_call.Call";
  CallType.tp_basicsize = sizeof(Call);
  CallType.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_GC | Py_TPFLAGS_HAVE_VECTORCALL;
  CallType.tp_new = call_new;
  CallType.tp_call = PyVectorcall_Call;
  CallType.tp_vectorcall_offset = offsetof(Call, vectorcall);
  CallType.tp_dictoffset = offsetof(Call, dict);
  CallType.tp_weaklistoffset = offsetof(Call, weak);
  CallType.tp_methods = call_methods;
  CallType.tp_traverse = call_traverse;
  CallType.tp_clear = call_clear;
  CallType.tp_dealloc = call_dealloc;
  CallType.tp_getattro = PyObject_GenericGetAttr;
  CallType.tp_setattro = PyObject_GenericSetAttr;
  CallType.tp_getset = call_getset;
  if (PyType_Ready(&CallType) < 0) return nullptr;
  PyObject *m = PyModule_Create(&module);
  if (!m) return nullptr;
  struct { PyObject **at; const char *name; } const names[] = {
      {&S.rows, "rows"}, {&S.cols, "cols"}, {&S.n_keep, "n_keep"}, {&S.group, "group"}, {&S.val_kind, "val_kind"}, {&S.row_ptr, "row_ptr"},
      {&S.values, "values"}, {&S.idx, "idx"}, {&S.qparams, "qparams"}, {&S.total_slots, "total_slots"}, {&S.cuda_stream, "cuda_stream"},
      {&S.stream_ptr, "stream_ptr"}, {&S.value, "value"}};
  for (const auto &n : names)
    if (!(*n.at = PyUnicode_InternFromString(n.name))) return nullptr;
  const char *kinds[KINDS] = {"GEMV", "READ", "GEMM", "GEMM_WS", "INT4", "GEMV_BATCH", "GEMM_BATCH", "INT4_BATCH", "TABLE"};
  for (int k = 0; k < KINDS; ++k)
    if (PyModule_AddIntConstant(m, kinds[k], k) < 0) return nullptr;
  Py_INCREF(&CallType);
  if (PyModule_AddObject(m, "Call", (PyObject *)&CallType) < 0) return nullptr;
  return m;
}
