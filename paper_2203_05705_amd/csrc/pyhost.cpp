// CPython extension under binding.py: the calls a training step issues, marshalled in native code.
//
// A layer call of this library is one to three kernels of a few microseconds; issued through ctypes the
// host spent 9 us per call on Python statements around a launch of about 2 us, so a small layer or a
// grouped iteration ran at the speed of its Python (784-2048-2048-10 at batch 1024: 127 us of host time
// for 72 us of kernels).  Here a call parses its arguments once, reads sizes and addresses from the tensors
// directly and enters the C ABI; names, arguments, defaults, checks and results are those of binding.py's
// documentation.  The library itself stays behind its C ABI: it is opened at the first call by the path
// binding.py gives, and a missing library raises there.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <structmember.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/full.h>
#include <dlfcn.h>
#include <torch/csrc/Device.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/DynamicTypes.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <string>
#include <type_traits>

#include "../../include/ard.h"

namespace {

struct PyRaised {};  // a Python exception is set
[[noreturn]] void raise(PyObject* type, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  PyErr_FormatV(type, fmt, ap);
  va_end(ap);
  throw PyRaised{};
}

// ---- the library ------------------------------------------------------------------------------

#define ARD_CALLS(X)                                                                                                  \
  X(ard_kept_count) X(ard_compact_dim) X(ard_gemm_workspace_bytes) X(ard_compact_weight) X(ard_drop_gemm_fwd)         \
  X(ard_drop_gemm_bwd_data) X(ard_drop_gemm_bwd_weight) X(ard_drop_gemm_bwd_weight_static) X(ard_batch_begin)         \
  X(ard_batch_launch) X(ard_batch_abort) X(ard_lstm_workspace_bytes) X(ard_lstm_fwd) X(ard_lstm_bwd)                  \
  X(ard_conv_workspace_bytes) X(ard_conv_out_size) X(ard_fmap_drop_conv) X(ard_conv_fwd_blocks) X(ard_conv_bwd_blocks) \
  X(ard_sens_regions) X(ard_sens_predict) X(ard_sens_row_pattern) X(ard_sens_block_pattern) X(ard_last_error)
#define DECLARE(name) decltype(&::name) name = nullptr;
struct Library {
  bool open = false;
  ARD_CALLS(DECLARE)
};
Library g_lib;
std::string g_lib_path;
PyObject *g_error = nullptr, *g_alloc = nullptr, *g_raw_stream = nullptr;  // ArdError; output allocator (NULL: torch.empty)
PyObject *s_dtype, *s_device, *s_cuda_stream;

const Library& lib() {
  if (!g_lib.open) {
    void* h = dlopen(g_lib_path.c_str(), RTLD_NOW | RTLD_LOCAL);
    if (!h) raise(PyExc_RuntimeError, "%s is missing or does not load (%s): build it with `python -m paper_2203_05705_amd.build` "
                  "(or __graft_entry__.build()); there is no fallback path", g_lib_path.c_str(), dlerror());
#define LOOKUP(name)                                                                                     \
  if (!(g_lib.name = reinterpret_cast<decltype(g_lib.name)>(dlsym(h, #name)))) raise(PyExc_RuntimeError, "%s has no " #name, g_lib_path.c_str());
    ARD_CALLS(LOOKUP)
    g_lib.open = true;
  }
  return g_lib;
}

void check(int32_t code) {
  if (code == 0) return;
  PyObject* e = PyObject_CallFunction(g_error, "is", (int)code, lib().ard_last_error());
  if (e) {
    PyErr_SetObject(g_error, e);
    Py_DECREF(e);
  }
  throw PyRaised{};
}

// An enqueueing call of the C ABI, without the interpreter lock (as ctypes makes it).  Its arguments are values: whatever
// of them can raise (a tensor without storage has no address) has done so before the lock is given up.
struct Unlocked {
  PyThreadState* state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};
template <class... P, class... A> void enqueue(int32_t (*f)(P...), A... args) {
  static_assert((std::is_scalar_v<A> && ...), "numbers and addresses only: nothing left to evaluate without the lock");
  int32_t rc;
  {
    Unlocked unlocked;
    rc = f(args...);
  }
  check(rc);
}

// ---- patterns ---------------------------------------------------------------------------------

struct PatternObject {
  PyObject_HEAD
  int kind, dp, b, tile_r, tile_c, count;
  PyObject *keep, *lists;
};
extern PyTypeObject PatternType;

const at::Tensor& tensor_of(PyObject* o, const char* what) {
  if (!o || !THPVariable_Check(o)) raise(PyExc_TypeError, "%s: a torch tensor is wanted, got %s", what, o ? Py_TYPE(o)->tp_name : "nothing");
  return THPVariable_Unpack(o);
}

int pattern_init(PyObject* self, PyObject* args, PyObject* kw) {
  static const char* names[] = {"kind", "dp", "b", "tile_r", "tile_c", "keep", "count", "lists", nullptr};
  PatternObject* p = reinterpret_cast<PatternObject*>(self);
  p->kind = 0, p->dp = 1, p->b = 1, p->tile_r = 0, p->tile_c = 0;
  PyObject *keep = Py_None, *count = Py_None, *lists = Py_None;
  if (!PyArg_ParseTupleAndKeywords(args, kw, "|iiiiiOOO", const_cast<char**>(names), &p->kind, &p->dp, &p->b, &p->tile_r, &p->tile_c, &keep,
                                   &count, &lists))
    return -1;
  if (count != Py_None) {
    p->count = (int)PyLong_AsLong(count);
    if (PyErr_Occurred()) return -1;
  } else {
    p->count = keep != Py_None && THPVariable_Check(keep) ? (int)THPVariable_Unpack(keep).numel() : 0;
  }
  Py_INCREF(keep), Py_INCREF(lists);
  Py_XSETREF(p->keep, keep);
  Py_XSETREF(p->lists, lists);
  return 0;
}
PyObject* pattern_new(PyTypeObject* type, PyObject*, PyObject*) {
  PyObject* self = type->tp_alloc(type, 0);
  if (!self) return nullptr;
  PatternObject* p = reinterpret_cast<PatternObject*>(self);
  p->dp = p->b = 1;
  Py_INCREF(Py_None), Py_INCREF(Py_None);
  p->keep = p->lists = Py_None;
  return self;
}
int pattern_traverse(PyObject* self, visitproc visit, void* arg) {
  PatternObject* p = reinterpret_cast<PatternObject*>(self);
  Py_VISIT(p->keep);
  Py_VISIT(p->lists);
  return 0;
}
int pattern_clear(PyObject* self) {
  PatternObject* p = reinterpret_cast<PatternObject*>(self);
  Py_CLEAR(p->keep);
  Py_CLEAR(p->lists);
  return 0;
}
void pattern_dealloc(PyObject* self) {
  PyObject_GC_UnTrack(self);
  pattern_clear(self);
  Py_TYPE(self)->tp_free(self);
}
int as_int(PyObject* o) {
  const long v = PyLong_AsLong(o);
  if (v == -1 && PyErr_Occurred()) throw PyRaised{};
  if (v < INT32_MIN || v > INT32_MAX) raise(PyExc_OverflowError, "%ld does not fit 32 bits", v);
  return (int)v;
}
// int(o) and float(o): counts and rates are taken from whatever converts (a whole-valued float, a 0-d tensor, a string)
int to_int(PyObject* o) {
  if (PyLong_CheckExact(o)) return as_int(o);
  PyObject* n = PyNumber_Long(o);
  if (!n) throw PyRaised{};
  int overflow = 0;
  const long v = PyLong_AsLongAndOverflow(n, &overflow);
  Py_DECREF(n);
  if (overflow || v < INT32_MIN || v > INT32_MAX) raise(PyExc_OverflowError, "%R does not fit 32 bits", o);
  return (int)v;
}
double to_float(PyObject* o) {
  if (PyFloat_CheckExact(o)) return PyFloat_AS_DOUBLE(o);
  PyObject* f = PyNumber_Float(o);
  if (!f) throw PyRaised{};
  const double v = PyFloat_AS_DOUBLE(f);
  Py_DECREF(f);
  return v;
}
PyMemberDef pattern_members[] = {{"kind", T_INT, offsetof(PatternObject, kind), 0, nullptr},
                                 {"dp", T_INT, offsetof(PatternObject, dp), 0, nullptr},
                                 {"b", T_INT, offsetof(PatternObject, b), 0, nullptr},
                                 {"tile_r", T_INT, offsetof(PatternObject, tile_r), 0, nullptr},
                                 {"tile_c", T_INT, offsetof(PatternObject, tile_c), 0, nullptr},
                                 {"count", T_INT, offsetof(PatternObject, count), 0, nullptr},
                                 {"keep", T_OBJECT, offsetof(PatternObject, keep), 0, nullptr},
                                 {"lists", T_OBJECT, offsetof(PatternObject, lists), 0, nullptr},
                                 {nullptr, 0, 0, 0, nullptr}};
PyTypeObject PatternType = {PyVarObject_HEAD_INIT(nullptr, 0)};

// an optional pattern argument in the C ABI's form
struct PatRef {
  ard_pattern c{};
  const ard_pattern* p = nullptr;
  explicit PatRef(PyObject* o) {
    if (!o || o == Py_None) return;
    if (!PyObject_TypeCheck(o, &PatternType)) raise(PyExc_TypeError, "a Pattern or None is wanted, got %s", Py_TYPE(o)->tp_name);
    const PatternObject* q = reinterpret_cast<const PatternObject*>(o);
    c.kind = q->kind, c.dp = q->dp, c.b = q->b, c.tile_r = q->tile_r, c.tile_c = q->tile_c, c.count = q->count;
    if (q->kind == ARD_PAT_LIST && q->keep && q->keep != Py_None) c.d_keep = (const int32_t*)tensor_of(q->keep, "keep").data_ptr();
    const int lists = q->kind == ARD_PAT_TILE && q->lists ? PyObject_IsTrue(q->lists) : 0;
    if (lists < 0) throw PyRaised{};
    if (lists) {
      auto get = [&](const char* k) {
        PyObject* v = PyMapping_GetItemString(q->lists, k);
        if (!v) throw PyRaised{};
        const void* ptr = nullptr;
        try {
          ptr = tensor_of(v, k).data_ptr();
        } catch (...) {
          Py_DECREF(v);
          throw;
        }
        Py_DECREF(v);
        return ptr;
      };
      c.d_keep = (const int32_t*)get("keep"), c.d_mask = (const uint8_t*)get("mask"), c.d_rowptr = (const int32_t*)get("rowptr");
      c.d_colptr = (const int32_t*)get("colptr"), c.d_csc_rows = (const int32_t*)get("csc_rows");
    }
    p = &c;
  }
};

// ---- arguments --------------------------------------------------------------------------------

// Parameter names of a function, the first `required` without a default.  Arguments come by the vectorcall
// protocol; keyword names are interned, so identity finds them.
struct Sig {
  static constexpr int MAX = 16;
  const char* fn;
  int n, required;
  const char* names[MAX];
  PyObject* interned[MAX];
};
struct Args {
  PyObject* v[Sig::MAX] = {};
  Args(Sig& s, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
    if (!s.interned[0])
      for (int i = 0; i < s.n; ++i) s.interned[i] = PyUnicode_InternFromString(s.names[i]);
    if (nargs > s.n) raise(PyExc_TypeError, "%s() takes at most %d arguments (%zd given)", s.fn, s.n, nargs);
    for (Py_ssize_t i = 0; i < nargs; ++i) v[i] = args[i];
    const Py_ssize_t nk = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    for (Py_ssize_t k = 0; k < nk; ++k) {
      PyObject* name = PyTuple_GET_ITEM(kwnames, k);
      int at = -1;
      for (int i = 0; i < s.n && at < 0; ++i)
        if (s.interned[i] == name) at = i;
      for (int i = 0; i < s.n && at < 0; ++i)
        if (PyUnicode_Compare(s.interned[i], name) == 0) at = i;
      if (at < 0) raise(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", s.fn, name);
      if (v[at]) raise(PyExc_TypeError, "%s() got multiple values for argument '%s'", s.fn, s.names[at]);
      v[at] = args[nargs + k];
    }
    for (int i = 0; i < s.required; ++i)
      if (!v[i]) raise(PyExc_TypeError, "%s() missing a required argument: '%s'", s.fn, s.names[i]);
  }
  bool given(int i) const { return v[i] && v[i] != Py_None; }
  int integer(int i, int dflt) const { return v[i] ? as_int(v[i]) : dflt; }
  double real(int i, double dflt) const { return v[i] ? to_float(v[i]) : dflt; }
  uint64_t u64(int i) const {
    const uint64_t d = PyLong_AsUnsignedLongLongMask(v[i]);
    if (d == (uint64_t)-1 && PyErr_Occurred()) throw PyRaised{};
    return d;
  }
  bool truth(int i, bool dflt) const {
    if (!v[i]) return dflt;
    const int t = PyObject_IsTrue(v[i]);
    if (t < 0) throw PyRaised{};
    return t != 0;
  }
};

int32_t dtype_code(const at::Tensor& t) {
  if (t.scalar_type() == at::kFloat) return ARD_F32;
  if (t.scalar_type() == at::kBFloat16) return ARD_BF16;
  raise(PyExc_TypeError, "unsupported dtype %s", c10::toString(t.scalar_type()));
}
const at::Tensor& device_tensor(PyObject* o, const char* what) {
  const at::Tensor& t = tensor_of(o, what);
  if (!t.is_cuda() || !t.is_contiguous()) raise(PyExc_AssertionError, "device-resident contiguous tensors only");
  return t;
}
const at::Tensor& ranked(const at::Tensor& t, int64_t rank, const char* what) {
  if (t.dim() != rank) raise(PyExc_ValueError, "%s: %d dimensions are wanted, got %d", what, (int)rank, (int)t.dim());
  return t;
}
int dim(const at::Tensor& t, int i) {  // t.shape[i]
  if (i >= t.dim()) raise(PyExc_IndexError, "tuple index out of range");
  const int64_t n = t.size(i);
  if (n > INT32_MAX) raise(PyExc_OverflowError, "a dimension of %lld elements is too large", (long long)n);
  return (int)n;
}
void* ptr(const at::Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }
void* opt_ptr(const Args& a, int i, const char* what) { return a.given(i) ? tensor_of(a.v[i], what).data_ptr() : nullptr; }

// torch.cuda.current_stream() of the current device, or the Stream object passed in
void* stream_of(PyObject* o) {
  PyObject* r;
  if (o && o != Py_None) {
    r = PyObject_GetAttr(o, s_cuda_stream);
  } else {
    static PyObject* minus_one = PyLong_FromLong(-1);
    r = PyObject_CallOneArg(g_raw_stream, minus_one);
  }
  if (!r) throw PyRaised{};
  void* s = PyLong_AsVoidPtr(r);
  Py_DECREF(r);
  if (PyErr_Occurred()) throw PyRaised{};
  return s;
}

// a new output tensor, from the installed allocator or torch.empty
at::Tensor output(at::IntArrayRef shape, at::ScalarType dtype, c10::Device dev) {
  if (!g_alloc) return at::empty(shape, at::TensorOptions().dtype(dtype).device(dev));
  PyObject* sh = PyTuple_New((Py_ssize_t)shape.size());
  for (size_t i = 0; i < shape.size(); ++i) PyTuple_SET_ITEM(sh, i, PyLong_FromLongLong(shape[i]));
  PyObject* kw = PyDict_New();
  PyObject* d = THPDevice_New(dev);
  PyDict_SetItem(kw, s_dtype, reinterpret_cast<PyObject*>(torch::getTHPDtype(dtype)));
  PyDict_SetItem(kw, s_device, d);
  PyObject* args = PyTuple_Pack(1, sh);
  PyObject* r = PyObject_Call(g_alloc, args, kw);
  Py_DECREF(args), Py_DECREF(d), Py_DECREF(kw), Py_DECREF(sh);
  if (!r) throw PyRaised{};
  at::Tensor t;
  try {
    t = tensor_of(r, "output allocator");
  } catch (...) {
    Py_DECREF(r);
    throw;
  }
  Py_DECREF(r);
  return t;
}
at::Tensor filled(at::IntArrayRef shape, int value, c10::Device dev) {
  return at::full(shape, value, at::TensorOptions().dtype(at::kInt).device(dev));
}

PyObject* wrap(const at::Tensor& t) {
  PyObject* o = THPVariable_Wrap(t);
  if (!o) throw PyRaised{};
  return o;
}
PyObject* give(PyObject* o) {
  Py_INCREF(o);
  return o;
}
// result tensor: the caller's own object where it gave one
PyObject* result(const Args& a, int i, const at::Tensor& t) { return a.given(i) ? give(a.v[i]) : wrap(t); }
struct DictOut {
  PyObject* d = PyDict_New();
  void put(const char* k, const at::Tensor& t) {
    PyObject* o = wrap(t);
    PyDict_SetItemString(d, k, o);
    Py_DECREF(o);
  }
};
// d[k]; with `optional` None gives an undefined tensor, whose address is NULL
at::Tensor dict_tensor(PyObject* d, const char* k, bool optional = false) {
  PyObject* v = PyMapping_GetItemString(d, k);
  if (!v) throw PyRaised{};
  at::Tensor t;
  try {
    if (!optional || v != Py_None) t = tensor_of(v, k);
  } catch (...) {
    Py_DECREF(v);
    throw;
  }
  Py_DECREF(v);
  return t;
}
// a, b = o
void unpack_pair(PyObject* o, int* a, int* b) {
  PyObject* f = PySequence_Fast(o, "a pair of integers is wanted");
  if (!f) throw PyRaised{};
  try {
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(f);
    if (n != 2) raise(PyExc_ValueError, n < 2 ? "not enough values to unpack (expected 2, got %zd)" : "too many values to unpack (expected 2, got %zd)", n);
    *a = as_int(PySequence_Fast_GET_ITEM(f, 0)), *b = as_int(PySequence_Fast_GET_ITEM(f, 1));
  } catch (...) {
    Py_DECREF(f);
    throw;
  }
  Py_DECREF(f);
}
// o[i], through `convert`
int item_of(PyObject* o, int i, int (*convert)(PyObject*)) {
  PyObject* k = PyLong_FromLong(i);
  PyObject* v = PyObject_GetItem(o, k);
  Py_DECREF(k);
  if (!v) throw PyRaised{};
  int n;
  try {
    n = convert(v);
  } catch (...) {
    Py_DECREF(v);
    throw;
  }
  Py_DECREF(v);
  return n;
}

struct Workspace {
  at::Tensor own;
  void* p = nullptr;
  size_t bytes = 0;
  // `need` is asked only when the caller brings no workspace
  template <class F> Workspace(const Args& a, int i, c10::Device dev, F&& need) {
    if (a.given(i)) {
      const at::Tensor& t = tensor_of(a.v[i], "ws");
      p = t.data_ptr(), bytes = (size_t)t.numel();
    } else {
      const size_t n = need();
      own = at::empty({(int64_t)(n ? n : 1)}, at::TensorOptions().dtype(at::kByte).device(dev));
      p = own.data_ptr(), bytes = n ? n : 1;
    }
  }
};

int kept(const PatRef& p, int units) {
  const int n = lib().ard_kept_count(p.p, units);
  if (n < 0) check(n);
  return n;
}
int pad8(int n) { return lib().ard_compact_dim(nullptr, n); }
void check_compact(const at::Tensor& t, int count, const char* what) {
  if (dim(t, 1) == pad8(count) && t.is_contiguous()) return;
  std::string sh = "(";
  for (int64_t i = 0; i < t.dim(); ++i) sh += (i ? ", " : "") + std::to_string(t.size(i));
  raise(PyExc_ValueError, "%s: a compact activation has pad8(kept)=%d contiguous columns, got %s)", what, pad8(count), sh.c_str());
}

template <PyObject* (*F)(const Args&)>
PyObject* guarded(Sig& s, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  try {
    lib();
    return F(Args(s, args, nargs, kwnames));
  } catch (const PyRaised&) {
  } catch (...) {  // (torch's own: IndexError, OutOfMemoryError and the others keep their Python types)
    torch::translate_exception_to_python(std::current_exception());
  }
  return nullptr;
}

// ---- layer calls ------------------------------------------------------------------------------

PyObject* compact_weight(const Args& a) {  // W, pat_out, pat_in, out, stream
  const at::Tensor& W = ranked(device_tensor(a.v[0], "W"), 2, "W");
  const int O = dim(W, 0), I = dim(W, 1);
  PatRef po(a.v[1]), pi(a.v[2]);
  const int Ok = kept(po, O), Ik = kept(pi, I);
  const at::Tensor Wc = a.given(3) ? tensor_of(a.v[3], "out") : output({pad8(Ok), pad8(Ik)}, W.scalar_type(), W.device());
  const int32_t dt = dtype_code(W);
  void* st = stream_of(a.v[4]);
  enqueue(lib().ard_compact_weight, dt, I, O, ptr(W), ptr(Wc), po.p, pi.p, st);
  return result(a, 3, Wc);
}

// I and O of a forward or data-gradient call: the weight's own sizes unless given
void layer_sizes(const Args& a, int iI, int iO, int flags, const at::Tensor& W, int* I, int* O) {
  const bool own = !(flags & ARD_W_COMPACT);
  if ((!own && !(a.given(iI) && a.given(iO)))) raise(PyExc_AssertionError, "pass I and O with ARD_W_COMPACT");
  *I = a.given(iI) ? as_int(a.v[iI]) : dim(W, 1);
  *O = a.given(iO) ? as_int(a.v[iO]) : dim(W, 0);
}

PyObject* drop_gemm_fwd(const Args& a) {  // X, W, pat_out, pat_in, alpha, relu, flags, out, ws, stream, I, O
  const at::Tensor &X = device_tensor(a.v[0], "X"), &W = device_tensor(a.v[1], "W");
  const int flags = a.integer(6, 0), B = dim(X, 0);
  int I, O;
  layer_sizes(a, 10, 11, flags, W, &I, &O);
  const int32_t dt = dtype_code(X);
  PatRef po(a.v[2]), pi(a.v[3]);
  if (flags & ARD_IN_COMPACT) check_compact(X, kept(pi, I), "X");
  const float alpha = (float)a.real(4, 1.0);
  const int relu = a.truth(5, false);
  const at::Tensor Y = a.given(7) ? tensor_of(a.v[7], "out")
                                  : output({B, flags & ARD_OUT_COMPACT ? pad8(kept(po, O)) : O}, X.scalar_type(), X.device());
  Workspace ws(a, 8, X.device(), [&] { return lib().ard_gemm_workspace_bytes(dt, B, I, O, po.p, pi.p); });
  void* st = stream_of(a.v[9]);
  enqueue(lib().ard_drop_gemm_fwd, dt, B, I, O, ptr(X), ptr(W), ptr(Y), po.p, pi.p, alpha, relu, flags, ws.p, ws.bytes, st);
  return result(a, 7, Y);
}

PyObject* drop_gemm_bwd_data(const Args& a) {  // dY, W, pat_out, pat_in, alpha, relu_src, flags, out, ws, stream, I, O
  const at::Tensor &dY = device_tensor(a.v[0], "dY"), &W = device_tensor(a.v[1], "W");
  const int flags = a.integer(6, 0), B = dim(dY, 0);
  int I, O;
  layer_sizes(a, 10, 11, flags, W, &I, &O);
  const int32_t dt = dtype_code(dY);
  PatRef po(a.v[2]), pi(a.v[3]);
  if (flags & ARD_OUT_COMPACT) check_compact(dY, kept(po, O), "dY");
  const float alpha = (float)a.real(4, 1.0);
  const at::Tensor dX = a.given(7) ? tensor_of(a.v[7], "out")
                                   : output({B, flags & ARD_IN_COMPACT ? pad8(kept(pi, I)) : I}, dY.scalar_type(), dY.device());
  const void* src = opt_ptr(a, 5, "relu_src");
  Workspace ws(a, 8, dY.device(), [&] { return lib().ard_gemm_workspace_bytes(dt, B, I, O, po.p, pi.p); });
  void* st = stream_of(a.v[9]);
  enqueue(lib().ard_drop_gemm_bwd_data, dt, B, I, O, ptr(dY), ptr(W), ptr(dX), po.p, pi.p, alpha, src, flags, ws.p, ws.bytes, st);
  return result(a, 7, dX);
}

PyObject* drop_gemm_bwd_weight(const Args& a) {  // dY, X, pat_out, pat_in, alpha, beta, flags, out, ws, stream, I, O
  const at::Tensor &dY = device_tensor(a.v[0], "dY"), &X = device_tensor(a.v[1], "X");
  const int flags = a.integer(6, 0), B = dim(dY, 0);
  const int I = a.given(10) ? as_int(a.v[10]) : dim(X, 1), O = a.given(11) ? as_int(a.v[11]) : dim(dY, 1);
  const int32_t dt = dtype_code(dY);
  PatRef po(a.v[2]), pi(a.v[3]);
  if (flags & ARD_OUT_COMPACT) check_compact(dY, kept(po, O), "dY");
  if (flags & ARD_IN_COMPACT) check_compact(X, kept(pi, I), "X");
  const float alpha = (float)a.real(4, 1.0), beta = (float)a.real(5, 0.0);
  at::Tensor dW;
  if (a.given(7)) dW = tensor_of(a.v[7], "out");
  else if (flags & ARD_DW_COMPACT) dW = output({pad8(kept(po, O)), pad8(kept(pi, I))}, dY.scalar_type(), dY.device());
  else dW = output({O, I}, dY.scalar_type(), dY.device());
  Workspace ws(a, 8, dY.device(), [&] { return lib().ard_gemm_workspace_bytes(dt, B, I, O, po.p, pi.p); });
  void* st = stream_of(a.v[9]);
  enqueue(lib().ard_drop_gemm_bwd_weight, dt, B, I, O, ptr(dY), ptr(X), ptr(dW), po.p, pi.p, alpha, beta, flags, ws.p, ws.bytes, st);
  return result(a, 7, dW);
}

PyObject* drop_gemm_bwd_weight_static(const Args& a) {  // dY, X, pat_out, pat_in, out, alpha, beta, flags, stream, I, O
  const at::Tensor &dY = device_tensor(a.v[0], "dY"), &X = device_tensor(a.v[1], "X");
  const at::Tensor& dW = device_tensor(a.v[4], "out");
  const int I = a.given(9) ? as_int(a.v[9]) : dim(X, 1), O = a.given(10) ? as_int(a.v[10]) : dim(dY, 1), B = dim(dY, 0);
  const int32_t dt = dtype_code(dY);
  PatRef po(a.v[2]), pi(a.v[3]);
  const float alpha = (float)a.real(5, 1.0), beta = (float)a.real(6, 0.0);
  const int flags = a.integer(7, 0);
  void* st = stream_of(a.v[8]);
  enqueue(lib().ard_drop_gemm_bwd_weight_static, dt, B, I, O, ptr(dY), ptr(X), ptr(dW), po.p, pi.p, alpha, beta, flags, st);
  return give(a.v[4]);
}

// ---- LSTM -------------------------------------------------------------------------------------

// a tuple (or list) of n output tensors given by the caller
void outputs_given(PyObject* o, int n, at::Tensor* t) {
  PyObject* f = PySequence_Fast(o, "out: a tuple of tensors is wanted");
  if (!f) throw PyRaised{};
  const bool right = PySequence_Fast_GET_SIZE(f) == n;
  try {
    if (!right) raise(PyExc_ValueError, "out: %d tensors are wanted", n);
    for (int i = 0; i < n; ++i) t[i] = tensor_of(PySequence_Fast_GET_ITEM(f, i), "out");
  } catch (...) {
    Py_DECREF(f);
    throw;
  }
  Py_DECREF(f);
}
template <int N> PyObject* tuple_of(const at::Tensor (&t)[N]) {
  PyObject* r = PyTuple_New(N);
  for (int i = 0; i < N; ++i) PyTuple_SET_ITEM(r, i, wrap(t[i]));
  return r;
}

PyObject* lstm_fwd(const Args& a) {  // x, W, pat, ws, stream, out
  const at::Tensor &x = ranked(device_tensor(a.v[0], "x"), 3, "x"), &W = device_tensor(a.v[1], "W");
  const int T = dim(x, 0), B = dim(x, 1), I = dim(x, 2), H = dim(W, 0) / 4;
  if (W.dim() != 2 || W.size(0) != 4 * (int64_t)H || W.size(1) != (int64_t)I + H) raise(PyExc_AssertionError, "W is [4H x (I+H)]");
  const int32_t dt = dtype_code(x);
  at::Tensor o[3];  // h, c, gates
  if (a.given(5)) {
    outputs_given(a.v[5], 3, o);
  } else {
    o[0] = output({T, B, H}, x.scalar_type(), x.device());
    o[1] = output({T, B, H}, at::kFloat, x.device());
    o[2] = output({T, B, 4 * (int64_t)H}, at::kFloat, x.device());
  }
  PatRef p(a.v[2]);
  Workspace ws(a, 3, x.device(), [&] { return lib().ard_lstm_workspace_bytes(dt, T, B, I, H, p.p); });
  void* st = stream_of(a.v[4]);
  enqueue(lib().ard_lstm_fwd, dt, T, B, I, H, ptr(x), ptr(W), p.p, ptr(o[0]), (float*)ptr(o[1]), (float*)ptr(o[2]), ws.p, ws.bytes, st);
  return tuple_of(o);
}

PyObject* lstm_bwd(const Args& a) {  // x, W, pat, h, c, gates, dh, ws, stream, out
  const at::Tensor &x = ranked(device_tensor(a.v[0], "x"), 3, "x"), &W = device_tensor(a.v[1], "W"), &h = device_tensor(a.v[3], "h"),
                   &c = device_tensor(a.v[4], "c"), &g = device_tensor(a.v[5], "gates"), &dh = device_tensor(a.v[6], "dh");
  const int T = dim(x, 0), B = dim(x, 1), I = dim(x, 2), H = dim(W, 0) / 4;
  const int32_t dt = dtype_code(x);
  at::Tensor o[2];  // dx, dW
  if (a.given(9)) {
    outputs_given(a.v[9], 2, o);
  } else {
    o[0] = output(x.sizes(), x.scalar_type(), x.device());
    o[1] = output(W.sizes(), W.scalar_type(), W.device());
  }
  PatRef p(a.v[2]);
  Workspace ws(a, 7, x.device(), [&] { return lib().ard_lstm_workspace_bytes(dt, T, B, I, H, p.p); });
  void* st = stream_of(a.v[8]);
  enqueue(lib().ard_lstm_bwd, dt, T, B, I, H, ptr(x), ptr(W), p.p, ptr(h), (const float*)ptr(c), (const float*)ptr(g), ptr(dh), ptr(o[0]), ptr(o[1]),
          ws.p, ws.bytes, st);
  return tuple_of(o);
}

// ---- convolution ------------------------------------------------------------------------------

struct ConvShape {
  int N, C, H, W, Co, kh, kw, stride, pad;
  void in(const at::Tensor& A) {
    ranked(A, 4, "A");
    N = dim(A, 0), C = dim(A, 1), H = dim(A, 2), W = dim(A, 3);
  }
  void filter(const at::Tensor& Wt) {
    ranked(Wt, 4, "Wt");
    Co = dim(Wt, 0), kh = dim(Wt, 2), kw = dim(Wt, 3);
  }
  size_t ws_bytes(int32_t dt) const { return lib().ard_conv_workspace_bytes(dt, N, C, H, W, Co, kh, kw, stride, pad); }
  void out_hw(int* ho, int* wo) const {
    *ho = lib().ard_conv_out_size(H, kh, stride, pad), *wo = lib().ard_conv_out_size(W, kw, stride, pad);
    if (*ho < 0 || *wo < 0) check(*ho < *wo ? *ho : *wo);
  }
};
// one pass of ard_fmap_drop_conv
struct ConvPass {
  double rate = 0.0;
  int n_keep = 0;
  const void *A = nullptr, *Wt = nullptr, *dY = nullptr;
  void* out = nullptr;
  uint8_t* mask = nullptr;
  int32_t *keep = nullptr, *count = nullptr;
  int64_t* score = nullptr;
  void run(int mode, int32_t dt, const ConvShape& s, const Workspace& ws, void* st) const {
    enqueue(lib().ard_fmap_drop_conv, mode, dt, s.N, s.C, s.H, s.W, s.Co, s.kh, s.kw, s.stride, s.pad, rate, n_keep, A, Wt, dY, out, mask, keep, count,
            score, ws.p, ws.bytes, st);
  }
};

PyObject* conv_select(const Args& a) {  // A, rate, Cout, ksize, stride, pad, ws, stream, out
  const at::Tensor& A = device_tensor(a.v[0], "A");
  ConvShape s;
  s.in(A);
  s.Co = a.integer(2, 1), s.kh = s.kw = 3, s.stride = a.integer(4, 1), s.pad = a.integer(5, 1);
  if (a.v[3]) unpack_pair(a.v[3], &s.kh, &s.kw);
  const int32_t dt = dtype_code(A);
  at::Tensor mask, keep, count, score;
  if (a.given(8)) {
    mask = dict_tensor(a.v[8], "mask", true), keep = dict_tensor(a.v[8], "keep", true), count = dict_tensor(a.v[8], "count", true);
    score = dict_tensor(a.v[8], "score", true);
  } else {
    mask = output({s.C}, at::kByte, A.device());
    keep = output({s.C}, at::kInt, A.device());
    count = at::empty({1}, keep.options());
    score = output({s.C}, at::kLong, A.device());
  }
  Workspace ws(a, 6, A.device(), [&] { return s.ws_bytes(dt); });
  ConvPass p;
  p.rate = a.real(1, 0.0), p.A = ptr(A), p.mask = (uint8_t*)ptr(mask), p.keep = (int32_t*)ptr(keep), p.count = (int32_t*)ptr(count);
  p.score = (int64_t*)ptr(score);
  // (a list made here has room for every channel: the kernel fills its end)
  p.run(ARD_CONV_SELECT | (a.given(8) ? 0 : ARD_CONV_PAD_KEEP), dt, s, ws, stream_of(a.v[7]));
  if (a.given(8)) return give(a.v[8]);
  DictOut d;
  d.put("mask", mask), d.put("keep", keep), d.put("count", count), d.put("score", score);
  return d.d;
}

PyObject* conv_fwd(const Args& a) {  // A, Wt, keep, n_keep, stride, pad, ws, stream, out, reuse
  const at::Tensor &A = device_tensor(a.v[0], "A"), &Wt = device_tensor(a.v[1], "Wt");
  ConvShape s;
  s.in(A), s.filter(Wt);
  s.stride = a.integer(4, 1), s.pad = a.integer(5, 1);
  int ho, wo;
  s.out_hw(&ho, &wo);
  const int32_t dt = dtype_code(A);
  const at::Tensor Y = a.given(8) ? tensor_of(a.v[8], "out") : output({s.N, s.Co, ho, wo}, A.scalar_type(), A.device());
  Workspace ws(a, 6, A.device(), [&] { return s.ws_bytes(dt); });
  ConvPass p;
  p.n_keep = to_int(a.v[3]), p.A = ptr(A), p.Wt = ptr(Wt), p.out = ptr(Y), p.keep = (int32_t*)opt_ptr(a, 2, "keep");
  p.run(ARD_CONV_FWD | a.integer(9, 0), dt, s, ws, stream_of(a.v[7]));
  return result(a, 8, Y);
}

PyObject* conv_bwd_data(const Args& a) {  // dY, Wt, keep, n_keep, in_hw, stride, pad, ws, stream, out, reuse
  const at::Tensor &dY = device_tensor(a.v[0], "dY"), &Wt = device_tensor(a.v[1], "Wt");
  ConvShape s;
  s.filter(Wt);
  s.N = dim(dY, 0), s.C = dim(Wt, 1), s.stride = a.integer(5, 1), s.pad = a.integer(6, 1);
  if (!a.given(9)) s.H = item_of(a.v[4], 0, to_int), s.W = item_of(a.v[4], 1, to_int);
  const int32_t dt = dtype_code(dY);
  const at::Tensor dA = a.given(9) ? tensor_of(a.v[9], "out") : output({s.N, s.C, s.H, s.W}, dY.scalar_type(), dY.device());
  ConvShape o = s;  // (the call takes the activations' sizes from dA)
  o.in(dA);
  o.Co = s.Co;
  Workspace ws(a, 7, dY.device(), [&] { return o.ws_bytes(dt); });
  ConvPass p;
  p.n_keep = to_int(a.v[3]), p.Wt = ptr(Wt), p.dY = ptr(dY), p.out = ptr(dA), p.keep = (int32_t*)opt_ptr(a, 2, "keep");
  p.run(ARD_CONV_BWD_DATA | a.integer(10, 0), dt, o, ws, stream_of(a.v[8]));
  return result(a, 9, dA);
}

PyObject* conv_bwd_weight(const Args& a) {  // dY, A, keep, n_keep, ksize, stride, pad, ws, stream, out, reuse
  const at::Tensor &dY = device_tensor(a.v[0], "dY"), &A = device_tensor(a.v[1], "A");
  ConvShape s;
  s.in(A);
  s.Co = dim(dY, 1), s.kh = s.kw = 3, s.stride = a.integer(5, 1), s.pad = a.integer(6, 1);
  if (a.v[4]) unpack_pair(a.v[4], &s.kh, &s.kw);
  const int32_t dt = dtype_code(A);
  const at::Tensor dW = a.given(9) ? tensor_of(a.v[9], "out") : output({s.Co, s.C, s.kh, s.kw}, A.scalar_type(), A.device());
  Workspace ws(a, 7, A.device(), [&] { return s.ws_bytes(dt); });
  ConvPass p;
  p.n_keep = to_int(a.v[3]), p.A = ptr(A), p.dY = ptr(dY), p.out = ptr(dW), p.keep = (int32_t*)opt_ptr(a, 2, "keep");
  p.run(ARD_CONV_BWD_WEIGHT | a.integer(10, 0), dt, s, ws, stream_of(a.v[8]));
  return result(a, 9, dW);
}

PyObject* conv_fwd_rows(const Args& a) {  // A, Wt, row_pat, n_keep, stride, pad, ws, stream, out
  const at::Tensor &A = device_tensor(a.v[0], "A"), &Wt = device_tensor(a.v[1], "Wt");
  ConvShape s;
  s.in(A), s.filter(Wt);
  s.stride = a.integer(4, 1), s.pad = a.integer(5, 1);
  int ho, wo;
  s.out_hw(&ho, &wo);
  const int32_t dt = dtype_code(A);
  const at::Tensor Y = a.given(8) ? tensor_of(a.v[8], "out") : output({s.N, s.Co, ho, wo}, A.scalar_type(), A.device());
  const at::Tensor keep = dict_tensor(a.v[2], "keep", true), mask = dict_tensor(a.v[2], "mask", true);
  Workspace ws(a, 6, A.device(), [&] { return s.ws_bytes(dt); });
  ConvPass p;
  p.n_keep = to_int(a.v[3]), p.A = ptr(A), p.Wt = ptr(Wt), p.out = ptr(Y), p.keep = (int32_t*)ptr(keep), p.mask = (uint8_t*)ptr(mask);
  p.run(ARD_CONV_FWD_ROWS, dt, s, ws, stream_of(a.v[7]));
  return result(a, 8, Y);
}

// the pair of gradients (dA, dWt): given by the caller or new
void gradient_pair(const Args& a, int i, const at::Tensor& A, const at::Tensor& Wt, at::Tensor (&o)[2]) {
  if (a.given(i)) {
    outputs_given(a.v[i], 2, o);
  } else {
    o[0] = output(A.sizes(), A.scalar_type(), A.device());
    o[1] = output(Wt.sizes(), Wt.scalar_type(), Wt.device());
  }
}

PyObject* conv_bwd_rows(const Args& a) {  // dY, A, Wt, row_pat, stride, pad, ws, stream, out, reuse
  const at::Tensor &dY = device_tensor(a.v[0], "dY"), &A = device_tensor(a.v[1], "A"), &Wt = device_tensor(a.v[2], "Wt");
  ConvShape s;
  s.in(A), s.filter(Wt);
  s.stride = a.integer(4, 1), s.pad = a.integer(5, 1);
  const int32_t dt = dtype_code(A);
  at::Tensor o[2];
  gradient_pair(a, 8, A, Wt, o);
  const at::Tensor mask = dict_tensor(a.v[3], "mask", true);
  Workspace ws(a, 6, A.device(), [&] { return s.ws_bytes(dt); });
  void* st = stream_of(a.v[7]);
  ConvPass d;
  d.Wt = ptr(Wt), d.dY = ptr(dY), d.out = ptr(o[0]), d.mask = (uint8_t*)ptr(mask);
  d.run(ARD_CONV_BWD_DATA_ROWS, dt, s, ws, st);
  ConvPass w;
  w.A = ptr(A), w.dY = ptr(dY), w.out = ptr(o[1]), w.mask = (uint8_t*)ptr(mask);
  w.run(ARD_CONV_BWD_WEIGHT_ROWS | a.integer(9, 0), dt, s, ws, st);
  return tuple_of(o);
}

PyObject* conv_fwd_blocks(const Args& a) {  // A, Wt, block_keep, x, y, stride, pad, ws, stream, out
  const at::Tensor &A = device_tensor(a.v[0], "A"), &Wt = device_tensor(a.v[1], "Wt"), &keep = device_tensor(a.v[2], "block_keep");
  ConvShape s;
  s.in(A), s.filter(Wt);
  s.stride = a.integer(5, 1), s.pad = a.integer(6, 1);
  int ho, wo;
  s.out_hw(&ho, &wo);
  const int32_t dt = dtype_code(A);
  const at::Tensor Y = a.given(9) ? tensor_of(a.v[9], "out") : output({s.N, s.Co, ho, wo}, A.scalar_type(), A.device());
  Workspace ws(a, 7, A.device(), [&] { return s.ws_bytes(dt); });
  const int x = to_int(a.v[3]), y = to_int(a.v[4]);
  void* st = stream_of(a.v[8]);
  enqueue(lib().ard_conv_fwd_blocks, dt, s.N, s.C, s.H, s.W, s.Co, s.kh, s.kw, s.stride, s.pad, x, y, ptr(A), ptr(Wt), (const uint8_t*)ptr(keep), ptr(Y),
          ws.p, ws.bytes, st);
  return result(a, 9, Y);
}

PyObject* conv_bwd_blocks(const Args& a) {  // dY, A, Wt, block_keep, x, y, stride, pad, ws, stream, out
  const at::Tensor &dY = device_tensor(a.v[0], "dY"), &A = device_tensor(a.v[1], "A"), &Wt = device_tensor(a.v[2], "Wt"),
                   &keep = device_tensor(a.v[3], "block_keep");
  ConvShape s;
  s.in(A), s.filter(Wt);
  s.stride = a.integer(6, 1), s.pad = a.integer(7, 1);
  const int32_t dt = dtype_code(A);
  at::Tensor o[2];
  gradient_pair(a, 10, A, Wt, o);
  Workspace ws(a, 8, A.device(), [&] { return s.ws_bytes(dt); });
  const int x = to_int(a.v[4]), y = to_int(a.v[5]);
  void* st = stream_of(a.v[9]);
  // (the weight gradient takes what the data gradient just left in the workspace, where it left it)
  const int modes[2] = {ARD_CONV_BWD_DATA, ARD_CONV_BWD_WEIGHT | ARD_CONV_REUSE_DY};
  for (int i = 0; i < 2; ++i)
    enqueue(lib().ard_conv_bwd_blocks, modes[i], dt, s.N, s.C, s.H, s.W, s.Co, s.kh, s.kw, s.stride, s.pad, x, y, ptr(A), ptr(Wt), ptr(dY),
            (const uint8_t*)ptr(keep), ptr(o[i]), ws.p, ws.bytes, st);
  return tuple_of(o);
}

// ---- sensitivity ------------------------------------------------------------------------------

PyObject* sens_predict(const Args& a) {  // A, ksize, stride, pad, x, y, k_permille, t_permille, threshold, seed, iteration, stream
  const at::Tensor& A = device_tensor(a.v[0], "A");
  ConvShape s;
  s.in(A);
  s.kh = item_of(a.v[1], 0, as_int), s.kw = item_of(a.v[1], 1, as_int);
  s.stride = as_int(a.v[2]), s.pad = as_int(a.v[3]);
  const int x = as_int(a.v[4]), y = as_int(a.v[5]), k = as_int(a.v[6]), t = as_int(a.v[7]);
  const float thr = (float)a.real(8, 0.0);
  const uint64_t seed = a.u64(9), it = a.u64(10);
  int32_t rows, rb, cb;
  check(lib().ard_sens_regions(s.N, s.C, s.H, s.W, s.kh, s.kw, s.stride, s.pad, x, y, &rows, &rb, &cb));
  const int32_t dt = dtype_code(A);
  const at::Tensor count = output({s.N, rb, cb}, at::kInt, A.device()), samples = output({s.N, rb, cb}, at::kInt, A.device()),
                   sens = output({s.N, rb, cb}, at::kByte, A.device());
  void* st = stream_of(a.v[11]);
  enqueue(lib().ard_sens_predict, dt, s.N, s.C, s.H, s.W, s.kh, s.kw, s.stride, s.pad, x, y, k, t, thr, seed, it, ptr(A), (int32_t*)ptr(count),
          (int32_t*)ptr(samples), (uint8_t*)ptr(sens), st);
  DictOut d;
  d.put("count", count), d.put("samples", samples), d.put("sens", sens);
  return d.d;
}

PyObject* sens_row_pattern(const Args& a) {  // sens, rows, x, m, n, seed, iteration, stream
  const at::Tensor& sens = device_tensor(a.v[0], "sens");
  const int N = dim(sens, 0), rows = as_int(a.v[1]), x = as_int(a.v[2]);
  const double m = a.real(3, 0.0), n = a.real(4, 0.0);
  const uint64_t seed = a.u64(5), it = a.u64(6);
  const int64_t total = (int64_t)N * rows;
  const at::Tensor mask = output({total}, at::kByte, sens.device()), keep = filled({total}, -1, sens.device()), count = at::empty({1}, keep.options());
  void* st = stream_of(a.v[7]);
  enqueue(lib().ard_sens_row_pattern, N, rows, x, (const uint8_t*)ptr(sens), m, n, seed, it, (uint8_t*)ptr(mask), (int32_t*)ptr(keep),
          (int32_t*)ptr(count), st);
  DictOut d;
  d.put("mask", mask), d.put("keep", keep), d.put("count", count);
  return d.d;
}

PyObject* sens_block_pattern(const Args& a) {  // pred, balance, m, n, seed, iteration, stream
  const at::Tensor cnt = dict_tensor(a.v[0], "count"), smp = dict_tensor(a.v[0], "samples"), in = dict_tensor(a.v[0], "sens");
  ranked(in, 3, "sens");
  const int N = dim(in, 0), RB = dim(in, 1), CB = dim(in, 2), balance = a.truth(1, false);
  const double m = a.real(2, 0.0), n = a.real(3, 0.0);
  const uint64_t seed = a.u64(4), it = a.u64(5);
  const at::Tensor sens = output({N, RB, CB}, at::kByte, in.device()), keep = output({N, RB, CB}, at::kByte, in.device());
  void* st = stream_of(a.v[6]);
  enqueue(lib().ard_sens_block_pattern, N, RB, CB, (const int32_t*)ptr(cnt), (const int32_t*)ptr(smp), (const uint8_t*)ptr(in), balance, m, n, seed, it,
          (uint8_t*)ptr(sens), (uint8_t*)ptr(keep), st);
  DictOut d;
  d.put("sens", sens), d.put("keep", keep);
  return d.d;
}

// ---- grouped launches -------------------------------------------------------------------------

struct BatchObject {
  PyObject_HEAD
  PyObject* stream;
};
PyTypeObject BatchType = {PyVarObject_HEAD_INIT(nullptr, 0)};
int batch_init(PyObject* self, PyObject* args, PyObject* kw) {
  static const char* names[] = {"stream", nullptr};
  PyObject* s = Py_None;
  if (!PyArg_ParseTupleAndKeywords(args, kw, "|O", const_cast<char**>(names), &s)) return -1;
  Py_INCREF(s);
  Py_XSETREF(reinterpret_cast<BatchObject*>(self)->stream, s);
  return 0;
}
PyMemberDef batch_members[] = {{"stream", T_OBJECT, offsetof(BatchObject, stream), 0, nullptr}, {nullptr, 0, 0, 0, nullptr}};
PyObject* batch_reduce(PyObject* self, PyObject*) {  // copies and pickles: type(self)(stream)
  PyObject* s = reinterpret_cast<BatchObject*>(self)->stream;
  return Py_BuildValue("O(O)", Py_TYPE(self), s ? s : Py_None);
}
void batch_dealloc(PyObject* self) {
  Py_XDECREF(reinterpret_cast<BatchObject*>(self)->stream);
  Py_TYPE(self)->tp_free(self);
}
template <class F> PyObject* method(F&& f) {
  try {
    return f();
  } catch (const PyRaised&) {
  } catch (...) {  // (torch's own: IndexError, OutOfMemoryError and the others keep their Python types)
    torch::translate_exception_to_python(std::current_exception());
  }
  return nullptr;
}
PyObject* batch_enter(PyObject* self, PyObject*) {
  return method([&] {
    check(lib().ard_batch_begin());
    return give(self);
  });
}
PyObject* batch_exit(PyObject* self, PyObject* const* args, Py_ssize_t nargs) {
  return method([&] {
    if (nargs > 0 && args[0] != Py_None) {
      lib().ard_batch_abort();
    } else {
      void* st = stream_of(reinterpret_cast<BatchObject*>(self)->stream);
      enqueue(lib().ard_batch_launch, st);
    }
    return give(Py_False);
  });
}
PyMethodDef batch_methods[] = {{"__enter__", batch_enter, METH_NOARGS, nullptr},
                               {"__exit__", (PyCFunction)(void (*)(void))batch_exit, METH_FASTCALL, nullptr},
                               {"__reduce__", batch_reduce, METH_NOARGS, nullptr},
                               {nullptr, nullptr, 0, nullptr}};

// Pattern constructors: a binding.Pattern, filled directly, also when called through a class a program derived from it
// (whose own __new__ and __init__ may want other arguments).
PyObject* pattern_of(PyObject* cls, int kind, int dp, int b, int tr, int tc, PyObject* lists) {
  PyTypeObject* t = reinterpret_cast<PyTypeObject*>(cls);
  while (t != &PatternType && t->tp_base != &PatternType) t = t->tp_base;
  PyObject* o = t->tp_new(t, nullptr, nullptr);
  if (!o) throw PyRaised{};
  PatternObject* p = reinterpret_cast<PatternObject*>(o);
  p->kind = kind, p->dp = dp, p->b = b, p->tile_r = tr, p->tile_c = tc;
  if (lists) {
    Py_INCREF(lists);
    Py_XSETREF(p->lists, lists);
  }
  return o;
}
PyObject* pattern_row(PyObject* cls, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  static Sig s = {"row", 2, 2, {"dp", "b"}, {}};
  return method([&] {
    Args a(s, args, nargs, kwnames);
    return pattern_of(cls, ARD_PAT_ROW, as_int(a.v[0]), as_int(a.v[1]), 0, 0, nullptr);
  });
}
PyObject* pattern_tile(PyObject* cls, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  static Sig s = {"tile", 5, 4, {"dp", "b", "tile_r", "tile_c", "lists"}, {}};
  return method([&] {
    Args a(s, args, nargs, kwnames);
    return pattern_of(cls, ARD_PAT_TILE, as_int(a.v[0]), as_int(a.v[1]), as_int(a.v[2]), as_int(a.v[3]), a.v[4]);
  });
}
PyMethodDef pattern_methods[] = {
    {"row", (PyCFunction)(void (*)(void))pattern_row, METH_CLASS | METH_FASTCALL | METH_KEYWORDS,
     "row($type, dp, b)\n--\n\nEvery dp-th unit from the b-th on is kept."},
    {"tile", (PyCFunction)(void (*)(void))pattern_tile, METH_CLASS | METH_FASTCALL | METH_KEYWORDS,
     "tile($type, dp, b, tile_r, tile_c, lists=None)\n--\n\nEvery dp-th tile of the weight from the b-th on is kept."},
    {nullptr, nullptr, 0, nullptr}};

// ---- module -----------------------------------------------------------------------------------

#define CALL(name, nargs_, required_, ...)                                                                \
  Sig sig_##name = {#name, nargs_, required_, {__VA_ARGS__}, {}};                                         \
  PyObject* py_##name(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {            \
    return guarded<name>(sig_##name, args, nargs, kwnames);                                               \
  }
CALL(compact_weight, 5, 1, "W", "pat_out", "pat_in", "out", "stream")
CALL(drop_gemm_fwd, 12, 2, "X", "W", "pat_out", "pat_in", "alpha", "relu", "flags", "out", "ws", "stream", "I", "O")
CALL(drop_gemm_bwd_data, 12, 2, "dY", "W", "pat_out", "pat_in", "alpha", "relu_src", "flags", "out", "ws", "stream", "I", "O")
CALL(drop_gemm_bwd_weight, 12, 2, "dY", "X", "pat_out", "pat_in", "alpha", "beta", "flags", "out", "ws", "stream", "I", "O")
CALL(drop_gemm_bwd_weight_static, 11, 5, "dY", "X", "pat_out", "pat_in", "out", "alpha", "beta", "flags", "stream", "I", "O")
CALL(lstm_fwd, 6, 2, "x", "W", "pat", "ws", "stream", "out")
CALL(lstm_bwd, 10, 7, "x", "W", "pat", "h", "c", "gates", "dh", "ws", "stream", "out")
CALL(conv_select, 9, 2, "A", "rate", "Cout", "ksize", "stride", "pad", "ws", "stream", "out")
CALL(conv_fwd, 10, 4, "A", "Wt", "keep", "n_keep", "stride", "pad", "ws", "stream", "out", "reuse")
CALL(conv_bwd_data, 11, 5, "dY", "Wt", "keep", "n_keep", "in_hw", "stride", "pad", "ws", "stream", "out", "reuse")
CALL(conv_bwd_weight, 11, 4, "dY", "A", "keep", "n_keep", "ksize", "stride", "pad", "ws", "stream", "out", "reuse")
CALL(conv_fwd_rows, 9, 4, "A", "Wt", "row_pat", "n_keep", "stride", "pad", "ws", "stream", "out")
CALL(conv_bwd_rows, 10, 4, "dY", "A", "Wt", "row_pat", "stride", "pad", "ws", "stream", "out", "reuse")
CALL(conv_fwd_blocks, 10, 5, "A", "Wt", "block_keep", "x", "y", "stride", "pad", "ws", "stream", "out")
CALL(conv_bwd_blocks, 11, 6, "dY", "A", "Wt", "block_keep", "x", "y", "stride", "pad", "ws", "stream", "out")
CALL(sens_predict, 12, 11, "A", "ksize", "stride", "pad", "x", "y", "k_permille", "t_permille", "threshold", "seed", "iteration", "stream")
CALL(sens_row_pattern, 8, 7, "sens", "rows", "x", "m", "n", "seed", "iteration", "stream")
CALL(sens_block_pattern, 7, 6, "pred", "balance", "m", "n", "seed", "iteration", "stream")

PyObject* py_configure(PyObject*, PyObject* args) {  // library path, ArdError, torch._C._cuda_getCurrentRawStream
  const char* path;
  PyObject *err, *raw;
  if (!PyArg_ParseTuple(args, "sOO", &path, &err, &raw)) return nullptr;
  g_lib_path = path;
  Py_INCREF(err), Py_INCREF(raw);
  Py_XSETREF(g_error, err);
  Py_XSETREF(g_raw_stream, raw);
  Py_RETURN_NONE;
}
PyObject* py_set_allocator(PyObject*, PyObject* fn) {
  PyObject* old = g_alloc;
  g_alloc = fn == Py_None ? nullptr : give(fn);
  Py_XDECREF(old);
  Py_RETURN_NONE;
}

// (the first line of a documentation, up to --, is what inspect.signature reads)
#define ENTRY(name, doc) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL | METH_KEYWORDS, doc}
PyMethodDef methods[] = {
    ENTRY(compact_weight, "compact_weight($module, W, pat_out=None, pat_in=None, out=None, stream=None)\n--\n\n"
                          "Wc[pad8(O') x pad8(I')]: W[kept o, kept i] in the top-left corner, zeros elsewhere."),
    ENTRY(drop_gemm_fwd, "drop_gemm_fwd($module, X, W, pat_out=None, pat_in=None, alpha=1.0, relu=False, flags=0, out=None, ws=None, stream=None, I=None, O=None)\n--\n\n"
                         "Y = X . W^T under the patterns.  With layout flags pass the full sizes I / O explicitly."),
    ENTRY(drop_gemm_bwd_data, "drop_gemm_bwd_data($module, dY, W, pat_out=None, pat_in=None, alpha=1.0, relu_src=None, flags=0, out=None, ws=None, stream=None, "
                              "I=None, O=None)\n--\n\ndX = dY . W under the patterns."),
    ENTRY(drop_gemm_bwd_weight, "drop_gemm_bwd_weight($module, dY, X, pat_out=None, pat_in=None, alpha=1.0, beta=0.0, flags=0, out=None, ws=None, stream=None, "
                                "I=None, O=None)\n--\n\ndW = dY^T . X under the patterns."),
    ENTRY(drop_gemm_bwd_weight_static, "drop_gemm_bwd_weight_static($module, dY, X, pat_out, pat_in, out, alpha=1.0, beta=0.0, flags=0, stream=None, I=None, O=None)\n--\n\n"
                                       "The weight gradient on the library's own scratch: the caller passes every tensor, output included, and nothing is "
                                       "allocated here or in the library."),
    ENTRY(lstm_fwd, "lstm_fwd($module, x, W, pat=None, ws=None, stream=None, out=None)\n--\n\n"
                    "x[T,B,I], W[4H, I+H] -> (h[T,B,H] dtype, c[T,B,H] fp32, gates[T,B,4H] fp32); out: reuse such a triple."),
    ENTRY(lstm_bwd, "lstm_bwd($module, x, W, pat, h, c, gates, dh, ws=None, stream=None, out=None)\n--\n\n"
                    "Returns (dx[T,B,I], dW[4H, I+H]) in the storage dtype; out: reuse such a pair."),
    ENTRY(conv_select, "conv_select($module, A, rate, Cout=1, ksize=(3, 3), stride=1, pad=1, ws=None, stream=None, out=None)\n--\n\n"
                       "Sensitivity scores and channel selection: dict(mask, keep, count, score) (out: reuse such a dict)."),
    ENTRY(conv_fwd, "conv_fwd($module, A, Wt, keep, n_keep, stride=1, pad=1, ws=None, stream=None, out=None, reuse=0)\n--\n\n"),
    ENTRY(conv_bwd_data, "conv_bwd_data($module, dY, Wt, keep, n_keep, in_hw, stride=1, pad=1, ws=None, stream=None, out=None, reuse=0)\n--\n\n"),
    ENTRY(conv_bwd_weight, "conv_bwd_weight($module, dY, A, keep, n_keep, ksize=(3, 3), stride=1, pad=1, ws=None, stream=None, out=None, reuse=0)\n--\n\n"),
    ENTRY(conv_fwd_rows, "conv_fwd_rows($module, A, Wt, row_pat, n_keep, stride=1, pad=1, ws=None, stream=None, out=None)\n--\n\n"
                         "Forward convolution over the kept output positions of a row pattern (dict from sens_row_pattern)."),
    ENTRY(conv_bwd_rows, "conv_bwd_rows($module, dY, A, Wt, row_pat, stride=1, pad=1, ws=None, stream=None, out=None, reuse=0)\n--\n\n"
                         "Gradients (dA, dWt) of conv_fwd_rows: gradient arriving on dropped output positions counts as zero.\n"
                         "reuse: CONV_REUSE_* flags for the weight gradient (grids that conv_fwd_rows and the data gradient left in ws)."),
    ENTRY(conv_fwd_blocks, "conv_fwd_blocks($module, A, Wt, block_keep, x, y, stride=1, pad=1, ws=None, stream=None, out=None)\n--\n\n"
                           "Forward convolution under a block pattern (block_keep from sens_block_pattern, uint8 [N*RB*CB])."),
    ENTRY(conv_bwd_blocks, "conv_bwd_blocks($module, dY, A, Wt, block_keep, x, y, stride=1, pad=1, ws=None, stream=None, out=None)\n--\n\n"
                           "Gradients (dA, dWt) of conv_fwd_blocks."),
    ENTRY(sens_predict, "sens_predict($module, A, ksize, stride, pad, x, y, k_permille, t_permille, threshold, seed, iteration, stream=None)\n--\n\n"
                        "Region-level sensitivity prediction: dict(count, samples, sens), each [N, RB, CB] on the device."),
    ENTRY(sens_row_pattern, "sens_row_pattern($module, sens, rows, x, m, n, seed, iteration, stream=None)\n--\n\n"
                            "Row-based pattern from the per-band sensitivity sens[N, RB, 1]: dict(mask[N*rows], keep, count)."),
    ENTRY(sens_block_pattern, "sens_block_pattern($module, pred, balance, m, n, seed, iteration, stream=None)\n--\n\n"
                              "Block-based pattern from ard_sens_predict's outputs: dict(sens (balanced), keep), each [N, RB, CB]."),
    {"configure", py_configure, METH_VARARGS, nullptr},
    {"set_allocator", py_set_allocator, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_ardcall", "Calls into libard.so, marshalled in native code.", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__ardcall(void) {
  PatternType.tp_name = "paper_2203_05705_amd._ardcall.PatternBase";
  PatternType.tp_doc = "PatternBase(kind=0, dp=1, b=1, tile_r=0, tile_c=0, keep=None, count=None, lists=None)\n--\n\nThe fields of a Pattern.";
  PatternType.tp_basicsize = sizeof(PatternObject);
  PatternType.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_BASETYPE | Py_TPFLAGS_HAVE_GC;
  PatternType.tp_new = pattern_new;
  PatternType.tp_init = pattern_init;
  PatternType.tp_dealloc = pattern_dealloc;
  PatternType.tp_traverse = pattern_traverse;
  PatternType.tp_clear = pattern_clear;
  PatternType.tp_members = pattern_members;
  PatternType.tp_methods = pattern_methods;
  BatchType.tp_name = "paper_2203_05705_amd._ardcall.batch";
  BatchType.tp_doc = "batch(stream=None)\n--\n\nContext manager: the library calls made inside are recorded and issued as one grouped launch on\n"
                     "leaving it (they must be independent of each other and use separate workspaces).";
  BatchType.tp_basicsize = sizeof(BatchObject);
  BatchType.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_BASETYPE;
  BatchType.tp_new = PyType_GenericNew;
  BatchType.tp_init = batch_init;
  BatchType.tp_dealloc = batch_dealloc;
  BatchType.tp_methods = batch_methods;
  BatchType.tp_members = batch_members;
  if (PyType_Ready(&PatternType) < 0 || PyType_Ready(&BatchType) < 0) return nullptr;
  s_dtype = PyUnicode_InternFromString("dtype"), s_device = PyUnicode_InternFromString("device");
  s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  PyObject* m = PyModule_Create(&module_def);
  if (!m) return nullptr;
  Py_INCREF(&PatternType), Py_INCREF(&BatchType);
  PyModule_AddObject(m, "PatternBase", reinterpret_cast<PyObject*>(&PatternType));
  PyModule_AddObject(m, "batch", reinterpret_cast<PyObject*>(&BatchType));
  return m;
}
