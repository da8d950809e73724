// The common calls of binding.py in one native step: checks, output tensors and the library call.
//
// A call on 64 x 16 scores takes 2.5 us on the GPU and took 7.8 in Python: a dozen attribute reads of tensors, the
// allocation of the outputs and the foreign call, each of which costs more than what it does.  Every function here takes
// the arguments of its namesakes in binding.py and returns their result, or None where anything is not as in the common
// case (another type, layout or device, overlapping arrays, an explicit stream, a workspace to be made, a mode that
// watches tensor calls): the Python code then makes the call itself, with its own checks and errors.  Errors of the library
// are raised from here, by the same function.
//   64 x 16 JVP into given arrays 8.3 -> 4.3 us a call, 16384 x 64 VJP 8.3 -> 6.0 (5.2 on the GPU), compact
//   output 10.3 -> 6.4, the last two within a tenth from run to run.  What is left of 4.3: 2.7 the launch, 0.7 the Python
//   function, the rest the checks and the stream.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/TracerMode.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <initializer_list>

namespace {

// entry points of the library, by the numbers that binding.py passes
using FwdFn = int (*)(const void*, int64_t, int64_t, int64_t, double, double, void*, void*);
using JvpFn = int (*)(const void*, const void*, int64_t, int64_t, int64_t, double, double, void*, void*, void*);
using SparseFn = int (*)(const void*, int64_t, int64_t, int64_t, double, double, int64_t, void*, void*, void*, void*);
using LossFn = JvpFn;

constexpr int kMaxEntries = 16;
void* g_entry[kMaxEntries] = {};
PyObject* g_names[kMaxEntries] = {};
PyObject* g_raw_stream = nullptr;   // torch._C._cuda_getCurrentRawStream
PyObject* g_check = nullptr;        // binding._check
int g_ws_device = -1;               // of the registered workspace, -1: none
constexpr int kErrWorkspace = -4;

// a plain tensor object without anything that watches or replaces tensor calls
bool plain_mode() {
  return !at::impl::torch_function_mode_enabled() && !c10::impl::TorchDispatchModeTLS::any_modes_set() &&
         !at::tracer::impl::is_dispatch_enabled();
}

const at::Tensor* matrix(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || t.scalar_type() != at::kFloat || t.dim() != 2 ||
      !t.unsafeGetTensorImpl()->has_storage() || !t.is_contiguous() || (t.numel() > 0 && t.data_ptr() == nullptr))
    return nullptr;
  return &t;
}
const at::Tensor* like(PyObject* o, const at::Tensor& ref) {
  const at::Tensor* t = matrix(o);
  if (t == nullptr || t->sizes() != ref.sizes() || t->get_device() != ref.get_device()) return nullptr;
  return t;
}
bool overlap(const at::Tensor& a, const at::Tensor& b) {
  const char *pa = static_cast<const char*>(a.data_ptr()), *pb = static_cast<const char*>(b.data_ptr());
  const char *ea = pa + a.nbytes(), *eb = pb + b.nbytes();
  return pa < eb && pb < ea;
}

bool number(PyObject* o, double* v) {
  if (PyFloat_CheckExact(o)) *v = PyFloat_AS_DOUBLE(o);
  else if (PyLong_CheckExact(o)) *v = PyLong_AsDouble(o);
  else return false;
  if (PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return true;
}
bool integer(PyObject* o, int64_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  *v = PyLong_AsLongLong(o);
  if (PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return true;
}

// the raw handle of torch.cuda.current_stream()
bool current_stream(void** st) {
  const c10::impl::VirtualGuardImpl impl(c10::DeviceType::CUDA);
  PyObject* index = PyLong_FromLong(impl.getDevice().index());
  if (index == nullptr) return false;
  PyObject* h = PyObject_CallOneArg(g_raw_stream, index);
  Py_DECREF(index);
  if (h == nullptr) return false;
  *st = PyLong_AsVoidPtr(h);
  Py_DECREF(h);
  return !PyErr_Occurred();
}

// 1: done, 0: the Python code is to make the call, -1: an error is set
int outcome(int rc, int entry) {
  if (rc == 0) return 1;
  if (rc == kErrWorkspace) return 0;
  PyObject* r = PyObject_CallFunction(g_check, "iO", rc, g_names[entry]);
  Py_XDECREF(r);
  return r == nullptr ? -1 : 0;
}

// a tuple of new references (all of them taken over; null where one is)
PyObject* tuple_of(std::initializer_list<PyObject*> items) {
  bool whole = true;
  for (PyObject* o : items) whole = whole && o != nullptr;
  PyObject* r = whole ? PyTuple_New(Py_ssize_t(items.size())) : nullptr;
  Py_ssize_t i = 0;
  for (PyObject* o : items) {
    if (r != nullptr) PyTuple_SET_ITEM(r, i++, o);
    else Py_XDECREF(o);
  }
  return r;
}

struct Common {
  const at::Tensor* x;
  int64_t rows, n, k;
  double p, lam;
  void* stream;
};
// entry, x, .., k, p, lam and a stream that is None; false: not the common case (or an error is set)
bool common(PyObject* entry, PyObject* x, PyObject* k, PyObject* p, PyObject* lam, PyObject* stream, int* e, Common* c) {
  int64_t ev;
  if (stream != Py_None || !integer(entry, &ev) || ev < 0 || ev >= kMaxEntries || g_entry[ev] == nullptr ||
      !plain_mode() || !integer(k, &c->k) || !number(p, &c->p) || !number(lam, &c->lam))
    return false;
  *e = int(ev);
  c->x = matrix(x);
  if (c->x == nullptr || (g_ws_device >= 0 && g_ws_device != c->x->get_device())) return false;
  c->rows = c->x->size(0);
  c->n = c->x->size(1);
  return current_stream(&c->stream);
}

#define TOPK_NONE                       \
  do {                                  \
    if (PyErr_Occurred()) return nullptr; \
    Py_RETURN_NONE;                     \
  } while (0)

// fwd(entry, x, k, p, lam, out, stream) -> out
PyObject* fwd(PyObject*, PyObject* const* a, Py_ssize_t count) {
  HANDLE_TH_ERRORS
  int e;
  Common c;
  if (count != 7 || !common(a[0], a[1], a[2], a[3], a[4], a[6], &e, &c)) TOPK_NONE;
  at::Tensor fresh;
  const at::Tensor* out = &fresh;
  if (a[5] == Py_None) {
    fresh = at::empty_like(*c.x);
  } else {
    out = like(a[5], *c.x);
    if (out == nullptr || overlap(*out, *c.x)) TOPK_NONE;
  }
  const void* x = c.x->data_ptr();
  void* o = out->data_ptr();
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = reinterpret_cast<FwdFn>(g_entry[e])(x, c.rows, c.n, c.k, c.p, c.lam, o, c.stream);
  Py_END_ALLOW_THREADS
  if (outcome(rc, e) != 1) TOPK_NONE;
  if (a[5] == Py_None) return THPVariable_Wrap(fresh);
  Py_INCREF(a[5]);
  return a[5];
  END_HANDLE_TH_ERRORS
}

// jvp(entry, x, tangent, k, p, lam, out, jvp_out, want_out, stream) -> (out or None, jvp_out)
PyObject* jvp(PyObject*, PyObject* const* a, Py_ssize_t count) {
  HANDLE_TH_ERRORS
  int e;
  Common c;
  if (count != 10 || !PyBool_Check(a[8]) || !common(a[0], a[1], a[3], a[4], a[5], a[9], &e, &c)) TOPK_NONE;
  const at::Tensor* t = like(a[2], *c.x);
  if (t == nullptr) TOPK_NONE;
  at::Tensor fresh_out, fresh_jvp;
  const at::Tensor *out = nullptr, *d = &fresh_jvp;
  if (a[6] != Py_None) {
    out = like(a[6], *c.x);
    if (out == nullptr || overlap(*out, *c.x) || overlap(*out, *t)) TOPK_NONE;
  }
  if (a[7] != Py_None) {
    d = like(a[7], *c.x);
    if (d == nullptr || overlap(*d, *c.x) || overlap(*d, *t) || (out != nullptr && overlap(*out, *d))) TOPK_NONE;
  }
  if (out == nullptr && a[8] == Py_True) {
    fresh_out = at::empty_like(*c.x);
    out = &fresh_out;
  }
  if (a[7] == Py_None) fresh_jvp = at::empty_like(*c.x);
  const void *x = c.x->data_ptr(), *tp = t->data_ptr();
  void *o = out != nullptr ? out->data_ptr() : nullptr, *dp = d->data_ptr();
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = reinterpret_cast<JvpFn>(g_entry[e])(x, tp, c.rows, c.n, c.k, c.p, c.lam, o, dp, c.stream);
  Py_END_ALLOW_THREADS
  if (outcome(rc, e) != 1) TOPK_NONE;
  PyObject* ro = a[6];
  PyObject* rd = a[7];
  if (ro == Py_None && out != nullptr) ro = THPVariable_Wrap(fresh_out);
  else Py_INCREF(ro);
  if (rd == Py_None) rd = THPVariable_Wrap(fresh_jvp);
  else Py_INCREF(rd);
  return tuple_of({ro, rd});
  END_HANDLE_TH_ERRORS
}

// sparse(entry, x, k, p, lam, max_nnz, stream) -> (idx, val, nnz), all three allocated here
PyObject* sparse(PyObject*, PyObject* const* a, Py_ssize_t count) {
  HANDLE_TH_ERRORS
  int e;
  Common c;
  int64_t width;
  if (count != 7 || !integer(a[5], &width) || width < 1 || !common(a[0], a[1], a[2], a[3], a[4], a[6], &e, &c) ||
      width > c.n)
    TOPK_NONE;
  const auto words = at::TensorOptions().dtype(at::kInt).device(c.x->device());
  at::Tensor idx = at::empty({c.rows, width}, words), val = at::empty({c.rows, width}, words.dtype(at::kFloat)),
             nnz = at::empty({c.rows}, words);
  const void* x = c.x->data_ptr();
  void *ip = idx.data_ptr(), *vp = val.data_ptr(), *np = nnz.data_ptr();
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = reinterpret_cast<SparseFn>(g_entry[e])(x, c.rows, c.n, c.k, c.p, c.lam, width, ip, vp, np, c.stream);
  Py_END_ALLOW_THREADS
  if (outcome(rc, e) != 1) TOPK_NONE;
  return tuple_of({THPVariable_Wrap(idx), THPVariable_Wrap(val), THPVariable_Wrap(nnz)});
  END_HANDLE_TH_ERRORS
}

// loss(entry, x, target, k, p, lam, stream) -> (loss, grad), both allocated here
PyObject* loss(PyObject*, PyObject* const* a, Py_ssize_t count) {
  HANDLE_TH_ERRORS
  int e;
  Common c;
  if (count != 7 || !common(a[0], a[1], a[3], a[4], a[5], a[6], &e, &c)) TOPK_NONE;
  const at::Tensor* t = like(a[2], *c.x);
  if (t == nullptr) TOPK_NONE;
  at::Tensor l = at::empty({c.rows}, c.x->options().requires_grad(false)), g = at::empty_like(*c.x);
  const void *x = c.x->data_ptr(), *tp = t->data_ptr();
  void *lp = l.data_ptr(), *gp = g.data_ptr();
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = reinterpret_cast<LossFn>(g_entry[e])(x, tp, c.rows, c.n, c.k, c.p, c.lam, lp, gp, c.stream);
  Py_END_ALLOW_THREADS
  if (outcome(rc, e) != 1) TOPK_NONE;
  return tuple_of({THPVariable_Wrap(l), THPVariable_Wrap(g)});
  END_HANDLE_TH_ERRORS
}

// setup(raw_stream, check, ((name, address), ..)): entry i is the i-th pair
PyObject* setup(PyObject*, PyObject* args) {
  PyObject *raw, *check, *entries;
  if (!PyArg_ParseTuple(args, "OOO!", &raw, &check, &PyTuple_Type, &entries)) return nullptr;
  const Py_ssize_t count = PyTuple_GET_SIZE(entries);
  if (count > kMaxEntries) {
    PyErr_SetString(PyExc_ValueError, "too many entry points");
    return nullptr;
  }
  for (Py_ssize_t i = 0; i < count; ++i) {
    PyObject *name, *address;
    if (!PyArg_ParseTuple(PyTuple_GET_ITEM(entries, i), "UO", &name, &address)) return nullptr;
    void* ptr = PyLong_AsVoidPtr(address);
    if (PyErr_Occurred()) return nullptr;
    Py_INCREF(name);
    Py_XSETREF(g_names[i], name);
    g_entry[i] = ptr;
  }
  Py_INCREF(raw);
  Py_XSETREF(g_raw_stream, raw);
  Py_INCREF(check);
  Py_XSETREF(g_check, check);
  Py_RETURN_NONE;
}

// workspace_device(index): device of the registered workspace, -1 for none
PyObject* workspace_device(PyObject*, PyObject* o) {
  const long v = PyLong_AsLong(o);
  if (v == -1 && PyErr_Occurred()) return nullptr;
  g_ws_device = int(v);
  Py_RETURN_NONE;
}

// the torch this was built against
PyObject* torch_version(PyObject*, PyObject*) { return PyUnicode_FromString(TOPK_TORCH_VERSION); }

PyMethodDef methods[] = {
    {"fwd", reinterpret_cast<PyCFunction>(fwd), METH_FASTCALL, nullptr},
    {"jvp", reinterpret_cast<PyCFunction>(jvp), METH_FASTCALL, nullptr},
    {"sparse", reinterpret_cast<PyCFunction>(sparse), METH_FASTCALL, nullptr},
    {"loss", reinterpret_cast<PyCFunction>(loss), METH_FASTCALL, nullptr},
    {"torch_version", torch_version, METH_NOARGS, nullptr},
    {"setup", setup, METH_VARARGS, nullptr},
    {"workspace_device", workspace_device, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call(void) { return PyModule_Create(&module); }
