// The plain calls of the Python binding without an interpreter between the tensors and the C ABI.
//
// A small call costs what its host path costs: a 256^3 product runs 3 us on the device, reading three tensors through
// their Python attributes and handing fifteen integers to ctypes took 4 to 6 us.  The methods of `Calls` read shapes,
// strides and addresses from the tensors themselves.  They serve the plain form of a call only (exact torch tensors with
// storage, no head-split map, integers where integers are expected) and otherwise return -1, having called nothing: the
// binding then takes its general path, which raises what it always raised.  Any other result is the status of the call.
//
// The C ABI is reached through the addresses that the binding passes, so that there is one copy of the library however it
// was loaded, and the interpreter lock is released during a call, as ctypes does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include "../../include/hidet_mi355x.h"

namespace {

constexpr int kGeneral = -1;

struct Calls {
  PyObject_HEAD
  decltype(&hidet_gemm_cfg) gemm;
  decltype(&hidet_batched_gemm_cfg) batched;
  decltype(&hidet_conv2d_implicit_gemm_cfg) conv;
  decltype(&hidet_conv2d_implicit_gemm_packed) packed;
  decltype(&hidet_softmax_rows) softmax;
  decltype(&hidet_reduce_rows) reduce;
  PyObject *epilogue_type, *in_bad_fork, *get_device, *get_stream;
};

// An exact tensor (or parameter) with storage, of a type the library knows; null otherwise.
struct Arg {
  const at::Tensor* t = nullptr;
  int32_t dtype = -1;
  explicit Arg(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return;
    const at::Tensor& x = THPVariable_Unpack(o);
    if (!x.defined() || x.layout() != at::kStrided || !x.has_storage()) return;
    switch (x.scalar_type()) {
      case at::kFloat: dtype = HIDET_F32; break;
      case at::kHalf: dtype = HIDET_F16; break;
      case at::kBFloat16: dtype = HIDET_BF16; break;
      default: return;
    }
    t = &x;
  }
  explicit operator bool() const { return t != nullptr; }
  int64_t dim() const { return t->dim(); }
  int64_t size(int64_t d) const { return t->sizes()[d < 0 ? d + t->dim() : d]; }
  int64_t stride(int64_t d) const { return t->strides()[d < 0 ? d + t->dim() : d]; }
  void* ptr() const { return t->data_ptr(); }
  // leading dimension of the last two axes; false where the rows are not contiguous
  bool ld(int64_t& out) const {
    if (stride(-1) != 1 && size(-1) > 1) return false;
    out = size(-2) > 1 ? stride(-2) : (size(-1) > 1 ? size(-1) : 1);
    return true;
  }
  // rows, columns and leading dimension with the leading axes collapsed
  bool rows(int64_t& r, int64_t& c, int64_t& l) const {
    if (dim() < 1) return false;
    if (dim() == 1) {
      r = 1;
      c = size(0);
      l = c > 1 ? c : 1;
      return true;
    }
    if (dim() == 2) {
      r = size(0);
      c = size(1);
      return ld(l);
    }
    c = size(-1);
    if (c == 0 || !t->is_contiguous()) return false;
    r = t->numel() / c;
    l = c;
    return true;
  }
};

bool flag(PyObject* o, int32_t& v) {
  v = o == Py_True;
  return o == Py_True || o == Py_False;
}
bool whole(PyObject* o, int64_t& v) {
  if (!PyLong_CheckExact(o)) return false;
  v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return true;
}
bool pair(PyObject* o, int64_t (&v)[2]) {
  return PyTuple_CheckExact(o) && PyTuple_GET_SIZE(o) == 2 && whole(PyTuple_GET_ITEM(o, 0), v[0]) &&
         whole(PyTuple_GET_ITEM(o, 1), v[1]);
}
bool whole32(PyObject* o, int32_t& v) {
  int64_t w;
  if (!whole(o, w) || w < INT32_MIN || w > INT32_MAX) return false;
  v = (int32_t)w;
  return true;
}

// The epilogue descriptor of a call, borrowed from the ctypes structure for as long as this lives.
class Epilogue {
 public:
  Epilogue(const Calls* c, PyObject* o) {
    if (o == Py_None) {
      ok_ = true;
    } else if ((PyObject*)Py_TYPE(o) == c->epilogue_type) {
      if (PyObject_GetBuffer(o, &view_, PyBUF_SIMPLE) != 0) {
        PyErr_Clear();
        return;
      }
      held_ = true;
      ok_ = view_.len == (Py_ssize_t)sizeof(hidet_epilogue_t);
    }
  }
  ~Epilogue() {
    if (held_) PyBuffer_Release(&view_);
  }
  Epilogue(const Epilogue&) = delete;
  Epilogue& operator=(const Epilogue&) = delete;
  const hidet_epilogue_t* get() const { return held_ ? static_cast<const hidet_epilogue_t*>(view_.buf) : nullptr; }
  bool plain() const { return ok_ && (!held_ || get()->out_map == HIDET_MAP_PLAIN); }

 private:
  Py_buffer view_;
  bool held_ = false, ok_ = false;
};

// The stream of a call: the one given, or the current one of the current device.
bool stream_of(const Calls* c, PyObject* o, const Arg& a, void*& out) {
  PyObject* v = nullptr;
  if (o != Py_None) {
    v = PyObject_GetAttrString(o, "cuda_stream");
  } else {
    if (!a.t->is_cuda()) return false;
    PyObject* bad = PyObject_CallNoArgs(c->in_bad_fork);
    const bool fine = bad == Py_False;
    Py_XDECREF(bad);
    if (fine) {
      if (PyObject* device = PyObject_CallNoArgs(c->get_device)) {
        v = PyObject_CallOneArg(c->get_stream, device);
        Py_DECREF(device);
      }
    }
  }
  const bool ok = v != nullptr && PyLong_CheckExact(v);
  if (ok) out = PyLong_AsVoidPtr(v);
  Py_XDECREF(v);
  if (PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return ok;
}

template <class F>
PyObject* guarded(F f) {  // (a tensor without memory throws where its address is asked for)
  int status = kGeneral;
  try {
    status = f();
  } catch (...) {
    status = kGeneral;
  }
  return PyLong_FromLong(status);
}

template <class F>
int without_lock(F f) {
  int status;
  Py_BEGIN_ALLOW_THREADS;
  status = (int)f();
  Py_END_ALLOW_THREADS;
  return status;
}

bool expect(Py_ssize_t n, Py_ssize_t want) {
  if (n != want) PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
  return n == want;
}

// gemm / batched(A, B, C, transA, transB, epilogue, stream, config)
template <int DIM>
PyObject* call_gemm(PyObject* self, PyObject* const* args, Py_ssize_t n) {
  if (!expect(n, 8)) return nullptr;
  const Calls* c = reinterpret_cast<const Calls*>(self);
  return guarded([&]() -> int {
    const Arg a(args[0]), b(args[1]), y(args[2]);
    int32_t ta, tb, config;
    if (!a || !b || !y || a.dim() != DIM || b.dim() != DIM || y.dim() != DIM) return kGeneral;
    if (!flag(args[3], ta) || !flag(args[4], tb) || !whole32(args[7], config)) return kGeneral;
    const int64_t M = a.size(ta ? -1 : -2), K = a.size(ta ? -2 : -1), N = b.size(tb ? -2 : -1);
    int64_t lda, ldb, ldy;
    if (b.size(tb ? -1 : -2) != K || y.size(-2) != M || y.size(-1) != N) return kGeneral;
    if (!a.ld(lda) || !b.ld(ldb) || !y.ld(ldy)) return kGeneral;
    const Epilogue e(c, args[5]);
    void* stream;
    if (!e.plain() || !stream_of(c, args[6], a, stream)) return kGeneral;
    void *pa = a.ptr(), *pb = b.ptr(), *py = y.ptr();
    if constexpr (DIM == 2) {
      return without_lock([&] {
        return c->gemm(config, a.dtype, y.dtype, ta, tb, M, N, K, pa, lda, pb, ldb, py, ldy, e.get(), stream);
      });
    } else {
      const int64_t batch = a.size(0);
      if (b.size(0) != batch || y.size(0) != batch) return kGeneral;
      const int64_t sa = batch > 1 ? a.stride(0) : a.size(-2) * lda, sb = batch > 1 ? b.stride(0) : b.size(-2) * ldb,
                    sy = batch > 1 ? y.stride(0) : y.size(-2) * ldy;
      return without_lock([&] {
        return c->batched(config, a.dtype, y.dtype, ta, tb, batch, M, N, K, pa, lda, sa, pb, ldb, sb, py, ldy, sy, e.get(),
                          stream);
      });
    }
  });
}

// conv(x, w, y, stride, pad, epilogue, stream, config); packed(x, w_packed, y, stride, pad, epilogue, stream, config, k_slices)
template <bool PACKED>
PyObject* call_conv(PyObject* self, PyObject* const* args, Py_ssize_t n) {
  if (!expect(n, PACKED ? 9 : 8)) return nullptr;
  const Calls* c = reinterpret_cast<const Calls*>(self);
  return guarded([&]() -> int {
    const Arg x(args[0]), w(args[1]), y(args[2]);
    if (!x || !w || !y || x.dim() != 4 || w.dim() != 4 || y.dim() != 4) return kGeneral;
    if (!x.t->is_contiguous() || !w.t->is_contiguous() || !y.t->is_contiguous()) return kGeneral;
    int64_t s[2], p[2];
    int32_t config, slices = 0;
    if (!pair(args[3], s) || !pair(args[4], p) || !whole32(args[7], config)) return kGeneral;
    if (PACKED && !whole32(args[PACKED ? 8 : 0], slices)) return kGeneral;
    const int64_t Nb = x.size(0), IC = x.size(1), H = x.size(2), W = x.size(3), OC = w.size(0);
    const int64_t KH = w.size(PACKED ? 1 : 2), KW = w.size(PACKED ? 2 : 3);
    if (w.size(PACKED ? 3 : 1) != IC || s[0] <= 0 || s[1] <= 0) return kGeneral;
    // (sums that would overflow are the general path's)
    constexpr int64_t lim = INT64_C(1) << 60;
    if (p[0] < -lim || p[0] > lim || p[1] < -lim || p[1] > lim) return kGeneral;
    const int64_t oh = H + 2 * p[0] - KH, ow = W + 2 * p[1] - KW;
    if (oh < 0 || ow < 0) return kGeneral;
    if (y.size(0) != Nb || y.size(1) != OC || y.size(2) != oh / s[0] + 1 || y.size(3) != ow / s[1] + 1) return kGeneral;
    const Epilogue e(c, args[5]);
    void* stream;
    if (!e.plain() || !stream_of(c, args[6], x, stream)) return kGeneral;
    void *px = x.ptr(), *pw = w.ptr(), *py = y.ptr();
    if constexpr (PACKED) {
      return without_lock([&] {
        return c->packed(config, slices, x.dtype, y.dtype, Nb, IC, H, W, OC, KH, KW, s[0], s[1], p[0], p[1], px, pw, py, e.get(),
                         nullptr, 0, stream);
      });
    } else {
      return without_lock([&] {
        return c->conv(config, x.dtype, y.dtype, Nb, IC, H, W, OC, KH, KW, s[0], s[1], p[0], p[1], px, pw, py, e.get(), stream);
      });
    }
  });
}

PyObject* call_softmax(PyObject* self, PyObject* const* args, Py_ssize_t n) {  // (x, y, stream)
  if (!expect(n, 3)) return nullptr;
  const Calls* c = reinterpret_cast<const Calls*>(self);
  return guarded([&]() -> int {
    const Arg x(args[0]), y(args[1]);
    if (!x || !y || x.dtype != y.dtype || x.t->sizes() != y.t->sizes()) return kGeneral;
    int64_t rows, cols, ldx, ldy;
    if (!x.rows(rows, cols, ldx) || !y.rows(rows, cols, ldy)) return kGeneral;
    void* stream;
    if (!stream_of(c, args[2], x, stream)) return kGeneral;
    void *px = x.ptr(), *py = y.ptr();
    return without_lock([&] { return c->softmax(x.dtype, rows, cols, px, ldx, py, ldy, stream); });
  });
}

PyObject* call_reduce(PyObject* self, PyObject* const* args, Py_ssize_t n) {  // (x, y, op, stream)
  if (!expect(n, 4)) return nullptr;
  const Calls* c = reinterpret_cast<const Calls*>(self);
  return guarded([&]() -> int {
    const Arg x(args[0]), y(args[1]);
    int32_t op;
    int64_t rows, cols, ldx;
    if (!x || !y || !whole32(args[2], op) || !x.rows(rows, cols, ldx)) return kGeneral;
    if (y.t->numel() != rows || !y.t->is_contiguous()) return kGeneral;
    void* stream;
    if (!stream_of(c, args[3], x, stream)) return kGeneral;
    void *px = x.ptr(), *py = y.ptr();
    return without_lock([&] { return c->reduce(x.dtype, y.dtype, op, rows, cols, px, ldx, py, stream); });
  });
}

// Calls((addresses of the six entry points), epilogue type, in_bad_fork, get_device, get_stream)
PyObject* calls_new(PyTypeObject* type, PyObject* args, PyObject*) {
  unsigned long long at[6];
  PyObject *epilogue_type, *in_bad_fork, *get_device, *get_stream;
  if (!PyArg_ParseTuple(args, "(KKKKKK)OOOO", &at[0], &at[1], &at[2], &at[3], &at[4], &at[5], &epilogue_type, &in_bad_fork,
                        &get_device, &get_stream))
    return nullptr;
  for (unsigned long long a : at) {
    if (a == 0) {
      PyErr_SetString(PyExc_ValueError, "null entry point");
      return nullptr;
    }
  }
  Calls* c = reinterpret_cast<Calls*>(type->tp_alloc(type, 0));
  if (!c) return nullptr;
  c->gemm = reinterpret_cast<decltype(c->gemm)>((uintptr_t)at[0]);
  c->batched = reinterpret_cast<decltype(c->batched)>((uintptr_t)at[1]);
  c->conv = reinterpret_cast<decltype(c->conv)>((uintptr_t)at[2]);
  c->packed = reinterpret_cast<decltype(c->packed)>((uintptr_t)at[3]);
  c->softmax = reinterpret_cast<decltype(c->softmax)>((uintptr_t)at[4]);
  c->reduce = reinterpret_cast<decltype(c->reduce)>((uintptr_t)at[5]);
  c->epilogue_type = Py_NewRef(epilogue_type);
  c->in_bad_fork = Py_NewRef(in_bad_fork);
  c->get_device = Py_NewRef(get_device);
  c->get_stream = Py_NewRef(get_stream);
  return reinterpret_cast<PyObject*>(c);
}
void calls_dealloc(PyObject* self) {
  Calls* c = reinterpret_cast<Calls*>(self);
  Py_XDECREF(c->epilogue_type);
  Py_XDECREF(c->in_bad_fork);
  Py_XDECREF(c->get_device);
  Py_XDECREF(c->get_stream);
  Py_TYPE(self)->tp_free(self);
}

using Fast = PyObject* (*)(PyObject*, PyObject* const*, Py_ssize_t);
PyMethodDef method(const char* name, Fast f) { return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}; }
PyMethodDef g_methods[] = {method("gemm", call_gemm<2>),         method("batched_gemm", call_gemm<3>),
                           method("conv2d", call_conv<false>),   method("conv2d_packed", call_conv<true>),
                           method("softmax_rows", call_softmax), method("reduce_rows", call_reduce),
                           {nullptr, nullptr, 0, nullptr}};
PyTypeObject g_type = {PyVarObject_HEAD_INIT(nullptr, 0)};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_host_calls", nullptr, -1, nullptr, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host_calls() {
  g_type.tp_name = "_host_calls.Calls";
  g_type.tp_basicsize = sizeof(Calls);
  g_type.tp_flags = Py_TPFLAGS_DEFAULT;
  g_type.tp_new = calls_new;
  g_type.tp_dealloc = calls_dealloc;
  g_type.tp_methods = g_methods;
  if (PyType_Ready(&g_type) < 0) return nullptr;
  PyObject* m = PyModule_Create(&g_module);
  if (!m) return nullptr;
  // (what this was compiled for: the binding refuses it under another torch or Python, whose tensors it would misread)
  if (PyModule_AddObjectRef(m, "Calls", reinterpret_cast<PyObject*>(&g_type)) < 0 ||
      PyModule_AddStringConstant(m, "built_for", HIDET_BUILT_FOR) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
