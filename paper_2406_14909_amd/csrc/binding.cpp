// Native call path of the Python binding.
//
// Each function takes the tensors of one library call, checks what the Python
// binding checks (type, shape, contiguity, device, with the same rules) and
// makes the call on torch's current stream.  It answers None, having done
// nothing, wherever anything is out of the ordinary: a wrong shape, another
// current device, a tensor subclass, an active torch mode.  The binding then goes
// its general way, which accepts or refuses the call with its own messages.  A
// call that the library has seen is never made again: a status other than MOA_OK
// raises the binding's error (after a failed launch part of the work may be
// enqueued).  What it saves is host time: about 13 us of interpreted checks per
// call become about 2.
#include <Python.h>

#include <algorithm>
#include <cstring>
#include <new>

#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <ATen/PythonTorchFunctionTLS.h>

#include "moa.h"

namespace {

// Entry points of the loaded library, in the order of the binding's table.
struct Api {
  decltype(&moa_prefill) prefill;
  decltype(&moa_kv_append) kv_append;
  decltype(&moa_decode) decode;
  decltype(&moa_decode_noalloc) decode_noalloc;
  decltype(&moa_kv_append_ragged) kv_append_ragged;
  decltype(&moa_decode_ragged) decode_ragged;
  decltype(&moa_influence) influence;
  decltype(&moa_rule_loss) rule_loss;
};

// What the checks need of a library and a plan; held by a capsule.
struct Bound {
  Api api;
  const moa_plan_t* plan;       // null: for the calls that take no plan
  int64_t hq, hkv, d, rows;
  at::ScalarType dtype;
  PyObject* check;              // the binding's function that raises for a status
  ~Bound() { Py_XDECREF(check); }
};
constexpr const char* kName = "moa.bound";

Bound* bound_of(PyObject* o) {
  return PyCapsule_IsValid(o, kName) ? static_cast<Bound*>(PyCapsule_GetPointer(o, kName)) : nullptr;
}

// A plain strided GPU tensor that no torch transform wraps.
const at::Tensor* plain(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage()) return nullptr;
  using K = c10::DispatchKey;
  const c10::DispatchKeySet odd({K::Python, K::PythonTLSSnapshot, K::Functionalize, K::FuncTorchBatched,
                                 K::FuncTorchGradWrapper, K::Conjugate, K::Negative, K::ZeroTensor});
  return t.key_set().has_any(odd) ? nullptr : &t;
}

bool modes_active() {
  return c10::impl::TorchDispatchModeTLS::any_modes_set() || at::impl::torch_function_mode_enabled();
}

// The shape, type and device of one call's tensors.
struct Check {
  bool ok = true;
  c10::DeviceIndex device = -1;
  const at::Tensor* any(PyObject* o) {
    const at::Tensor* t = ok ? plain(o) : nullptr;
    if (!t || (device >= 0 && t->device().index() != device) || !t->is_contiguous()) {
      ok = false;
      return nullptr;
    }
    device = t->device().index();
    return t;
  }
  const at::Tensor* operator()(PyObject* o, at::ScalarType type, at::IntArrayRef shape) {
    const at::Tensor* t = any(o);
    if (t && (t->scalar_type() != type || t->sizes() != shape)) ok = false;
    return ok ? t : nullptr;
  }
  // Tensors checked and the call's device current.
  bool done() const { return ok && device >= 0 && c10::hip::current_device() == device; }
  void* stream() const { return c10::hip::getCurrentHIPStream(device).stream(); }
};

// Makes the call while other Python threads run; false with a Python exception
// set where it was not MOA_OK.
template <class F>
bool call(const Bound& b, F&& f) {
  moa_status_t st = MOA_OK;
  bool no_memory = false;
  Py_BEGIN_ALLOW_THREADS
  try {
    st = f();
  } catch (...) {                 // of a message's string: nothing else in the library throws
    no_memory = true;
  }
  Py_END_ALLOW_THREADS
  if (no_memory) return PyErr_NoMemory(), false;
  if (st == MOA_OK) return true;
  PyObject* r = PyObject_CallFunction(b.check, "i", static_cast<int>(st));
  if (r) PyErr_Format(PyExc_RuntimeError, "moa status %d", static_cast<int>(st));
  Py_XDECREF(r);
  return false;
}

bool as_int(PyObject* o, int64_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  int over = 0;
  *v = PyLong_AsLongLongAndOverflow(o, &over);
  return over == 0;
}

PyObject* none() { Py_RETURN_NONE; }
PyObject* same(PyObject* o) {
  Py_INCREF(o);
  return o;
}

// The output: `given`, or a new tensor like q where it is None.
struct Out {
  at::Tensor fresh;
  const at::Tensor* t = nullptr;
  PyObject* given;
  Out(PyObject* o, const at::Tensor* q, Check& c) : given(o) {
    if (!c.ok) return;
    if (o != Py_None) {
      t = c(o, q->scalar_type(), q->sizes());
    } else if (c.done()) {
      fresh = at::empty_like(*q);
      t = &fresh;
    }
  }
  PyObject* answer() { return given != Py_None ? same(given) : THPVariable_Wrap(fresh); }
};

#define MOA_ENTER(n)                                   \
  Bound* b = nargs == (n) ? bound_of(args[0]) : nullptr; \
  if (!b || modes_active()) return none();             \
  try {                                                \
    Check c;
#define MOA_LEAVE            \
  }                          \
  catch (...) {              \
    PyErr_Clear();           \
    return none();           \
  }

// prefill(bound, q, k, v, o)
PyObject* prefill(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  MOA_ENTER(5)
  const at::Tensor* q = c.any(args[1]);
  if (!b->plan || !q || q->dim() != 4) return none();
  const int64_t bsz = q->size(0), n = q->size(1);
  c(args[1], b->dtype, {bsz, n, b->hq, b->d});
  const at::Tensor* k = c(args[2], b->dtype, {bsz, n, b->hkv, b->d});
  const at::Tensor* v = c(args[3], b->dtype, {bsz, n, b->hkv, b->d});
  Out o(args[4], q, c);
  if (!c.done() || !o.t || bsz > INT32_MAX) return none();
  void *pq = q->data_ptr(), *pk = k->data_ptr(), *pv = v->data_ptr(), *po = o.t->data_ptr(), *s = c.stream();
  if (!call(*b, [&] { return b->api.prefill(b->plan, pq, pk, pv, po, static_cast<int32_t>(bsz), n, s); })) return nullptr;
  return o.answer();
  MOA_LEAVE
}

// kv_append(bound, k_cache, v_cache, pos_cache, k_new, v_new, start_pos)
PyObject* kv_append(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  MOA_ENTER(7)
  int64_t start;
  const at::Tensor* kn = c.any(args[4]);
  if (!b->plan || !kn || kn->dim() != 4 || !as_int(args[6], &start)) return none();
  const int64_t bsz = kn->size(0), n = kn->size(1);
  c(args[4], b->dtype, {bsz, n, b->hkv, b->d});
  const at::Tensor* vn = c(args[5], b->dtype, {bsz, n, b->hkv, b->d});
  const at::Tensor* kc = c(args[1], b->dtype, {bsz, b->rows, b->d});
  const at::Tensor* vc = c(args[2], b->dtype, {bsz, b->rows, b->d});
  const at::Tensor* pc = c(args[3], at::kInt, {bsz, b->rows});
  if (!c.done() || bsz > INT32_MAX) return none();
  void *pkc = kc->data_ptr(), *pvc = vc->data_ptr(), *pkn = kn->data_ptr(), *pvn = vn->data_ptr(), *s = c.stream();
  int32_t* pp = static_cast<int32_t*>(pc->data_ptr());
  if (!call(*b, [&] { return b->api.kv_append(b->plan, pkc, pvc, pp, pkn, pvn, static_cast<int32_t>(bsz), start, n, s); }))
    return nullptr;
  Py_RETURN_TRUE;
  MOA_LEAVE
}

// kv_append_ragged(bound, k_cache, v_cache, pos_cache, k_new, v_new, positions)
PyObject* kv_append_ragged(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  MOA_ENTER(7)
  const at::Tensor* kn = c.any(args[4]);
  if (!b->plan || !kn || kn->dim() != 4) return none();
  const int64_t bsz = kn->size(0);
  c(args[4], b->dtype, {bsz, 1, b->hkv, b->d});
  const at::Tensor* vn = c(args[5], b->dtype, {bsz, 1, b->hkv, b->d});
  const at::Tensor* kc = c(args[1], b->dtype, {bsz, b->rows, b->d});
  const at::Tensor* vc = c(args[2], b->dtype, {bsz, b->rows, b->d});
  const at::Tensor* pc = c(args[3], at::kInt, {bsz, b->rows});
  const at::Tensor* ps = c(args[6], at::kInt, {bsz});
  if (!c.done() || bsz > INT32_MAX) return none();
  void *pkc = kc->data_ptr(), *pvc = vc->data_ptr(), *pkn = kn->data_ptr(), *pvn = vn->data_ptr(), *s = c.stream();
  int32_t* pp = static_cast<int32_t*>(pc->data_ptr());
  const int32_t* at_ = static_cast<const int32_t*>(ps->data_ptr());
  if (!call(*b, [&] { return b->api.kv_append_ragged(b->plan, pkc, pvc, pp, pkn, pvn, at_, static_cast<int32_t>(bsz), s); }))
    return nullptr;
  Py_RETURN_TRUE;
  MOA_LEAVE
}

// q, k_cache, v_cache of a decode call
struct DecodeTensors {
  const at::Tensor *q, *kc = nullptr, *vc = nullptr;
  int64_t bsz = 0;
  DecodeTensors(const Bound& b, PyObject* const* args, Check& c) : q(c.any(args[1])) {
    if (!b.plan || !q || q->dim() != 3) {
      c.ok = false;
      return;
    }
    bsz = q->size(0);
    c(args[1], b.dtype, {bsz, b.hq, b.d});
    kc = c(args[2], b.dtype, {bsz, b.rows, b.d});
    vc = c(args[3], b.dtype, {bsz, b.rows, b.d});
    if (bsz > INT32_MAX) c.ok = false;
  }
};

// decode(bound, q, k_cache, v_cache, pos, workspace, o)
PyObject* decode(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  MOA_ENTER(7)
  int64_t pos;
  if (!as_int(args[4], &pos)) return none();
  const DecodeTensors t(*b, args, c);
  const at::Tensor* w = c.any(args[5]);
  Out o(args[6], t.q, c);
  if (!c.done() || !o.t) return none();
  void *pq = t.q->data_ptr(), *pk = t.kc->data_ptr(), *pv = t.vc->data_ptr(), *po = o.t->data_ptr();
  void *pw = w->data_ptr(), *s = c.stream();
  const size_t nw = w->nbytes();
  if (!call(*b, [&] { return b->api.decode(b->plan, pq, pk, pv, po, static_cast<int32_t>(t.bsz), pos, pw, nw, s); }))
    return nullptr;
  return o.answer();
  MOA_LEAVE
}

// decode_noalloc(bound, q, k_cache, v_cache, pos, o)
PyObject* decode_noalloc(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  MOA_ENTER(6)
  int64_t pos;
  if (!as_int(args[4], &pos) || args[5] == Py_None) return none();
  const DecodeTensors t(*b, args, c);
  Out o(args[5], t.q, c);
  if (!c.done() || !o.t) return none();
  void *pq = t.q->data_ptr(), *pk = t.kc->data_ptr(), *pv = t.vc->data_ptr(), *po = o.t->data_ptr(), *s = c.stream();
  if (!call(*b, [&] { return b->api.decode_noalloc(b->plan, pq, pk, pv, po, static_cast<int32_t>(t.bsz), pos, s); }))
    return nullptr;
  return o.answer();
  MOA_LEAVE
}

// decode_ragged(bound, q, k_cache, v_cache, positions, workspace, o)
PyObject* decode_ragged(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  MOA_ENTER(7)
  const DecodeTensors t(*b, args, c);
  const at::Tensor* ps = c(args[4], at::kInt, {t.bsz});
  const at::Tensor* w = c.any(args[5]);
  Out o(args[6], t.q, c);
  if (!c.done() || !o.t) return none();
  void *pq = t.q->data_ptr(), *pk = t.kc->data_ptr(), *pv = t.vc->data_ptr(), *po = o.t->data_ptr();
  void *pw = w->data_ptr(), *s = c.stream();
  const int32_t* at_ = static_cast<const int32_t*>(ps->data_ptr());
  const size_t nw = w->nbytes();
  if (!call(*b, [&] { return b->api.decode_ragged(b->plan, pq, pk, pv, po, at_, static_cast<int32_t>(t.bsz), pw, nw, s); }))
    return nullptr;
  return o.answer();
  MOA_LEAVE
}

// influence(bound, q, k, v, dout, ebar, softmax_scale)
PyObject* influence(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  MOA_ENTER(7)
  const at::Tensor* q = c.any(args[1]);
  const at::Tensor* k = c.any(args[2]);
  if (!q || !k || q->dim() != 4 || k->dim() != 4 || !PyFloat_CheckExact(args[6])) return none();
  const int64_t bsz = q->size(0), n = q->size(1), hq = q->size(2), d = q->size(3), hkv = k->size(2);
  c(args[1], at::kBFloat16, {bsz, n, hq, d});
  c(args[2], at::kBFloat16, {bsz, n, hkv, d});
  const at::Tensor* v = c(args[3], at::kBFloat16, {bsz, n, hkv, d});
  const at::Tensor* g = c(args[4], at::kBFloat16, {bsz, n, hq, d});
  if (!c.done() || std::max({bsz, n, hq, hkv, d}) > INT32_MAX) return none();
  const int64_t nb = (n + 63) / 64;
  at::Tensor fresh;
  const at::Tensor* e = &fresh;
  if (args[5] == Py_None) fresh = at::empty({hq, nb, nb}, q->options().dtype(at::kFloat));
  else e = c(args[5], at::kFloat, {hq, nb, nb});
  if (!c.done()) return none();
  moa_desc_t desc = {};
  desc.num_q_heads = static_cast<int32_t>(hq);
  desc.num_kv_heads = static_cast<int32_t>(hkv);
  desc.head_dim = static_cast<int32_t>(d);
  desc.n = n;
  desc.dtype = MOA_BF16;
  desc.softmax_scale = static_cast<float>(PyFloat_AS_DOUBLE(args[6]));
  void *pq = q->data_ptr(), *pk = k->data_ptr(), *pv = v->data_ptr(), *pg = g->data_ptr(), *s = c.stream();
  float* pe = static_cast<float*>(e->data_ptr());
  if (!call(*b, [&] { return b->api.influence(&desc, pq, pk, pv, pg, pe, static_cast<int32_t>(bsz), n, s); })) return nullptr;
  return args[5] == Py_None ? THPVariable_Wrap(fresh) : same(args[5]);
  MOA_LEAVE
}

// A one-dimensional contiguous float64 buffer.
struct Doubles {
  Py_buffer v;
  bool held = false, ok = false;
  explicit Doubles(PyObject* o) {
    if (!PyObject_CheckBuffer(o)) return;
    held = PyObject_GetBuffer(o, &v, PyBUF_FORMAT | PyBUF_C_CONTIGUOUS) == 0;
    if (!held) PyErr_Clear();
    ok = held && v.ndim == 1 && v.itemsize == 8 && v.format && v.format[0] == 'd' && v.format[1] == 0 && v.len > 0;
  }
  ~Doubles() {
    if (held) PyBuffer_Release(&v);
  }
  Doubles(const Doubles&) = delete;
};

// rule_loss(bound, ebar, n, num_sink, alpha, beta, flags) -> (dl, density)
PyObject* rule_loss(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  MOA_ENTER(7)
  int64_t n, sink, flags;
  const at::Tensor* e = c.any(args[1]);
  if (!e || e->dim() != 3 || !as_int(args[2], &n) || !as_int(args[3], &sink) || !as_int(args[6], &flags)) return none();
  const int64_t h = e->size(0), nb = (n + 63) / 64;
  if (n < 1 || sink < 0 || sink > INT32_MAX || flags < 0 || flags > 3 || h > INT32_MAX) return none();
  c(args[1], at::kFloat, {h, nb, nb});
  const Doubles al(args[4]), be(args[5]);
  if (!al.ok || !be.ok || al.v.len != be.v.len || !c.done()) return none();
  const int64_t r = al.v.len / 8;
  if (r > INT32_MAX) return none();
  at::Tensor dl = at::empty({h, r}, e->options().dtype(at::kDouble));
  at::Tensor dens = at::empty({r}, e->options().dtype(at::kDouble));
  const float* pe = static_cast<const float*>(e->data_ptr());
  double *pd = static_cast<double*>(dl.data_ptr()), *pn = static_cast<double*>(dens.data_ptr());
  void* s = c.stream();
  if (!call(*b, [&] {
        return b->api.rule_loss(pe, static_cast<int32_t>(h), n, static_cast<int32_t>(sink), static_cast<uint32_t>(flags),
                                static_cast<const double*>(al.v.buf), static_cast<const double*>(be.v.buf),
                                static_cast<int32_t>(r), pd, pn, s);
      }))
    return nullptr;
  PyObject* pair = PyTuple_New(2);
  if (!pair) return nullptr;
  PyTuple_SET_ITEM(pair, 0, THPVariable_Wrap(dl));
  PyTuple_SET_ITEM(pair, 1, THPVariable_Wrap(dens));
  return pair;
  MOA_LEAVE
}

// bind(addresses of the entry points, plan address or 0, num_q_heads, num_kv_heads, head_dim, cache rows, is bf16,
//      function that raises for a status)
PyObject* bind(PyObject*, PyObject* args) {
  PyObject *table, *check;
  unsigned long long plan;
  long long hq, hkv, d, rows;
  int bf16;
  if (!PyArg_ParseTuple(args, "O!KLLLLpO", &PyTuple_Type, &table, &plan, &hq, &hkv, &d, &rows, &bf16, &check))
    return nullptr;
  constexpr Py_ssize_t kEntries = sizeof(Api) / sizeof(void*);
  void* at_[kEntries];
  if (PyTuple_GET_SIZE(table) != kEntries) {
    PyErr_SetString(PyExc_ValueError, "entry point table of the wrong length");
    return nullptr;
  }
  for (Py_ssize_t i = 0; i < kEntries; ++i) {
    at_[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(table, i));
    if (!at_[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null entry point");
      return nullptr;
    }
  }
  Bound* b = new (std::nothrow) Bound{};
  if (!b) return PyErr_NoMemory();
  memcpy(&b->api, at_, sizeof(b->api));
  b->plan = reinterpret_cast<const moa_plan_t*>(static_cast<uintptr_t>(plan));
  b->hq = hq;
  b->hkv = hkv;
  b->d = d;
  b->rows = rows;
  b->dtype = bf16 ? at::kBFloat16 : at::kFloat;
  b->check = same(check);
  PyObject* o = PyCapsule_New(b, kName, [](PyObject* x) { delete static_cast<Bound*>(PyCapsule_GetPointer(x, kName)); });
  if (!o) delete b;
  return o;
}

#define MOA_FAST(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {
    MOA_FAST(prefill), MOA_FAST(kv_append), MOA_FAST(kv_append_ragged), MOA_FAST(decode), MOA_FAST(decode_noalloc),
    MOA_FAST(decode_ragged), MOA_FAST(influence), MOA_FAST(rule_loss), {"bind", bind, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&kModule); }
