// Native fast path of the Python binding: argument checks, output allocation
// and the library call of the entry points a program calls in a loop, and
// their autograd nodes, without Python or ctypes in between (a call of the
// pair mass on small columns took 12.9 us of host time through ctypes, its
// forward and backward 186 us, most of it the hand-over of the interpreter
// lock to the engine's thread).
//
// Every function returns None where it does not see its way -- an argument of
// another kind, dtype, layout or device than the plain GPU tensors it knows, a
// transform or mode of torch that looks inside (functorch, forward mode,
// dispatch and function modes, tracing), or a refusal by the library (the
// GLV_EINVAL_* statuses, decided before anything is launched): the Python path
// then runs and does, or refuses, what it always did.  GLV_EHIP raises here: a
// kernel may have run by then, and a second call would add to the caller's
// counters twice.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/LegacyTypeDispatch.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/forward_grad.h>
#include <torch/csrc/autograd/python_variable.h>

#include <array>
#include <optional>
#include <vector>

#include "glv.h"

namespace {

using at::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

struct NoGil {
  PyThreadState* s = PyEval_SaveThread();
  ~NoGil() { PyEval_RestoreThread(s); }
};

// Whether nothing in this thread looks inside tensor operations.
bool plain_context() {
  using c10::DispatchKey;
  const auto tls = c10::impl::tls_local_dispatch_key_set();
  return !(tls.included_.has(DispatchKey::FuncTorchDynamicLayerFrontMode) ||
           tls.included_.has(DispatchKey::FuncTorchDynamicLayerBackMode) ||
           tls.included_.has(DispatchKey::Functionalize) || tls.included_.has(DispatchKey::Tracer) ||
           tls.included_.has(DispatchKey::Python) || tls.included_.has(DispatchKey::PythonTLSSnapshot)) &&
         !c10::impl::TorchDispatchModeTLS::any_modes_set() && !at::impl::torch_function_mode_enabled();
}

// Columns of one call: plain contiguous 1-D GPU tensors of one dtype and device.
struct Kind {
  at::ScalarType dtype = at::kFloat;
  c10::Device device{c10::kCPU};
  int64_t n = -1;
  glv_dtype dt() const { return dtype == at::kDouble ? GLV_F64 : GLV_F32; }
  at::TensorOptions opts() const { return at::TensorOptions().dtype(dtype).device(device); }
};

const Tensor* plain_tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided) return nullptr;
  const auto ks = t.key_set();
  using c10::DispatchKey;
  if (ks.has(DispatchKey::Python) || ks.has(DispatchKey::FuncTorchBatched) ||
      ks.has(DispatchKey::FuncTorchGradWrapper) || ks.has(DispatchKey::Functionalize) ||
      ks.has(DispatchKey::ZeroTensor) || ks.has(DispatchKey::Negative) || ks.has(DispatchKey::Conjugate))
    return nullptr;
  return &t;
}

bool column(const Tensor& t, const Kind& k, int64_t n) {
  return t.scalar_type() == k.dtype && t.device() == k.device && t.dim() == 1 && t.is_contiguous() &&
         (n < 0 || t.numel() == n);
}

using Cols = std::vector<Tensor>;

// `count` columns of n elements each (n < 0: any) from a tuple or list; with
// `first` the first column sets the kind.
bool columns(PyObject* seq, size_t count, Kind* k, bool first, int64_t n, Cols* out) {
  if (!PyTuple_CheckExact(seq) && !PyList_CheckExact(seq)) return false;
  if ((size_t)PySequence_Fast_GET_SIZE(seq) != count) return false;
  PyObject** items = PySequence_Fast_ITEMS(seq);
  out->reserve(out->size() + count);
  for (size_t i = 0; i < count; ++i) {
    const Tensor* t = plain_tensor(items[i]);
    if (!t) return false;
    if (first && i == 0) {
      if (t->scalar_type() != at::kDouble && t->scalar_type() != at::kFloat) return false;
      *k = Kind{t->scalar_type(), t->device(), t->numel()};
    }
    if (!column(*t, *k, n < 0 && first ? k->n : n)) return false;
    out->push_back(*t);
  }
  return true;
}

// A 1-D contiguous int64 tensor on the columns' device (offsets).
const Tensor* offsets_of(PyObject* o, c10::Device d) {
  const Tensor* t = plain_tensor(o);
  return t && t->scalar_type() == at::kLong && t->device() == d && t->dim() == 1 && t->is_contiguous() ? t : nullptr;
}

template <size_t K>
struct Ptrs {
  std::array<void*, K> p;
  template <typename V>
  explicit Ptrs(const V& v, size_t at = 0) {
    for (size_t k = 0; k < K; ++k) p[k] = v[at + k].data_ptr();
  }
  void* const* out() const { return p.data(); }
  const void* const* in() const { return p.data(); }
};

Cols empties(const Kind& k, int64_t n, size_t count) {
  Cols c;
  c.reserve(count);
  for (size_t i = 0; i < count; ++i) c.push_back(at::empty({n}, k.opts()));
  return c;
}

void* stream_of(c10::Device d) {
  return c10::hip::getCurrentHIPStreamMasqueradingAsCUDA(d.index()).stream();
}

// ------------------------------------------------------------- arguments

bool coords_arg(PyObject* o, glv_coords* c) {
  if (!PyUnicode_Check(o)) return false;
  static const std::pair<const char*, glv_coords> names[] = {{"PtEtaPhiM", GLV_PTETAPHIM},
                                                             {"PxPyPzE", GLV_PXPYPZE},
                                                             {"PtEtaPhiE", GLV_PTETAPHIE},
                                                             {"PxPyPzM", GLV_PXPYPZM}};
  for (const auto& n : names)
    if (PyUnicode_CompareWithASCIIString(o, n.first) == 0) {
      *c = n.second;
      return true;
    }
  return false;
}

bool mode_arg(PyObject* o, glv_mode* m) {
  if (!PyUnicode_Check(o)) return false;
  if (PyUnicode_CompareWithASCIIString(o, "plain") == 0) *m = GLV_PLAIN;
  else if (PyUnicode_CompareWithASCIIString(o, "compensated") == 0) *m = GLV_COMPENSATED;
  else return false;
  return true;
}

bool int_arg(PyObject* o, int64_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  *v = PyLong_AsLongLong(o);
  if (*v == -1 && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return true;
}

bool double_arg(PyObject* o, double* v) {
  if (PyFloat_CheckExact(o)) {
    *v = PyFloat_AS_DOUBLE(o);
    return true;
  }
  int64_t i;
  if (!int_arg(o, &i)) return false;
  *v = (double)i;
  return true;
}

// The FP64-redo counter: None or one int64 element on the device.
bool counter_arg(PyObject* o, c10::Device d, std::optional<Tensor>* t) {
  if (o == Py_None) return true;
  const Tensor* c = plain_tensor(o);
  if (!c || c->scalar_type() != at::kLong || c->device() != d || c->numel() != 1) return false;
  *t = *c;
  return true;
}

unsigned long long* counter_ptr(const std::optional<Tensor>& t) {
  return t ? reinterpret_cast<unsigned long long*>(t->data_ptr()) : nullptr;
}

PyObject* wrap(const Tensor& t) { return THPVariable_Wrap(t); }

PyObject* wrap_tuple(const Cols& c, size_t at, size_t count) {
  PyObject* r = PyTuple_New((Py_ssize_t)count);
  for (size_t i = 0; i < count; ++i) PyTuple_SET_ITEM(r, (Py_ssize_t)i, wrap(c[at + i]));
  return r;
}

// Sets the Python error a failed library call has in the Python path.
void set_error(const char* fn, glv_status st) {
  PyObject* const mod = PyImport_ImportModule("paper_2312_02756_amd._lib");
  PyObject* const r = mod ? PyObject_CallMethod(mod, "check", "si", fn, (int)st) : nullptr;  // raises GlvError
  Py_XDECREF(r);
  Py_XDECREF(mod);
}

// Runs f, which returns the status of library call fn, without the interpreter
// lock; whether it is done.  If not, the caller returns not_done(): the error
// of a call that failed on the GPU, or None where the library refused it.
// Errors of torch's (memory, hooks) are the caller's to raise as they are.
template <typename F>
bool unlocked(const char* fn, F f) {
  glv_status st;
  {
    NoGil g;
    st = f();
  }
  if (st == GLV_EHIP) set_error(fn, st);
  return st == GLV_OK;
}

PyObject* not_done() {
  if (PyErr_Occurred()) return nullptr;
  Py_RETURN_NONE;
}

// ------------------------------------------------------------ entry points

// mass(a, b, coords, mode, fallback_count)
PyObject* py_mass(PyObject*, PyObject* const* args, Py_ssize_t na) {
  HANDLE_TH_ERRORS
  Kind k;
  Cols c;
  glv_coords co;
  glv_mode mo;
  std::optional<Tensor> fb;
  if (na != 5 || !plain_context() || !columns(args[0], 4, &k, true, -1, &c) ||
      !columns(args[1], 4, &k, false, k.n, &c) || !coords_arg(args[2], &co) || !mode_arg(args[3], &mo) ||
      !counter_arg(args[4], k.device, &fb))
    Py_RETURN_NONE;
  Tensor m;
  if (!unlocked("glv_invariant_mass", [&] {
        m = at::empty({k.n}, k.opts());
        return glv_invariant_mass(k.dt(), co, mo, k.n, Ptrs<4>(c).in(), Ptrs<4>(c, 4).in(), m.data_ptr(),
                                  counter_ptr(fb), stream_of(k.device));
      }))
    return not_done();
  return wrap(m);
  END_HANDLE_TH_ERRORS
}

// mass_histogram(a, b, lo, hi, n_bins, coords, mode, counts, fallback_count)
PyObject* py_mass_histogram(PyObject*, PyObject* const* args, Py_ssize_t na) {
  HANDLE_TH_ERRORS
  Kind k;
  Cols c;
  glv_coords co;
  glv_mode mo;
  double lo, hi;
  int64_t bins;
  std::optional<Tensor> fb;
  if (na != 9 || !plain_context() || !columns(args[0], 4, &k, true, -1, &c) ||
      !columns(args[1], 4, &k, false, k.n, &c) || !double_arg(args[2], &lo) || !double_arg(args[3], &hi) ||
      !int_arg(args[4], &bins) || bins < 1 || bins > (int64_t)1 << 40 || !coords_arg(args[5], &co) ||
      !mode_arg(args[6], &mo) || !counter_arg(args[8], k.device, &fb))
    Py_RETURN_NONE;
  Tensor counts;
  if (args[7] != Py_None) {
    const Tensor* t = plain_tensor(args[7]);
    if (!t || t->scalar_type() != at::kLong || t->device() != k.device || t->numel() != bins + 2 ||
        !t->is_contiguous())
      Py_RETURN_NONE;
    counts = *t;
  }
  if (!unlocked("glv_invariant_mass_histogram", [&] {
        if (!counts.defined()) counts = at::zeros({bins + 2}, k.opts().dtype(at::kLong));
        return glv_invariant_mass_histogram(k.dt(), co, mo, k.n, Ptrs<4>(c).in(), Ptrs<4>(c, 4).in(), lo, hi, bins,
                                            reinterpret_cast<unsigned long long*>(counts.data_ptr()),
                                            counter_ptr(fb), stream_of(k.device));
      }))
    return not_done();
  return wrap(counts);
  END_HANDLE_TH_ERRORS
}

// boost(x, beta)
PyObject* py_boost(PyObject*, PyObject* const* args, Py_ssize_t na) {
  HANDLE_TH_ERRORS
  Kind k;
  Cols c;
  if (na != 2 || !plain_context() || !columns(args[0], 4, &k, true, -1, &c) ||
      !columns(args[1], 3, &k, false, -1, &c))
    Py_RETURN_NONE;
  const int64_t bs = c[4].numel() == k.n ? 1 : 0;
  for (size_t i = 4; i < 7; ++i)
    if (c[i].numel() != (bs ? k.n : 1)) Py_RETURN_NONE;
  Cols y;
  if (!unlocked("glv_boost", [&] {
        y = empties(k, k.n, 4);
        return glv_boost(k.dt(), k.n, Ptrs<4>(c).in(), Ptrs<3>(c, 4).in(), bs, Ptrs<4>(y).out(),
                         stream_of(k.device));
      }))
    return not_done();
  return wrap_tuple(y, 0, 4);
  END_HANDLE_TH_ERRORS
}

// convert(cols, from_coords, to_coords)
PyObject* py_convert(PyObject*, PyObject* const* args, Py_ssize_t na) {
  HANDLE_TH_ERRORS
  Kind k;
  Cols c;
  glv_coords from, to;
  if (na != 3 || !plain_context() || !columns(args[0], 4, &k, true, -1, &c) || !coords_arg(args[1], &from) ||
      !coords_arg(args[2], &to))
    Py_RETURN_NONE;
  Cols y;
  if (!unlocked("glv_convert", [&] {
        y = empties(k, k.n, 4);
        return glv_convert(k.dt(), from, to, k.n, Ptrs<4>(c).in(), Ptrs<4>(y).out(), stream_of(k.device));
      }))
    return not_done();
  return wrap_tuple(y, 0, 4);
  END_HANDLE_TH_ERRORS
}

// transform(x, parameters): 16 columns a Lorentz matrix, 9 a rotation matrix,
// 4 an axis and an angle
PyObject* py_transform(PyObject*, PyObject* const* args, Py_ssize_t na) {
  HANDLE_TH_ERRORS
  Kind k;
  Cols c, m;
  if (na != 2 || !plain_context() || !columns(args[0], 4, &k, true, -1, &c) ||
      (!PyTuple_CheckExact(args[1]) && !PyList_CheckExact(args[1])))
    Py_RETURN_NONE;
  const size_t np = (size_t)PySequence_Fast_GET_SIZE(args[1]);
  if ((np != 16 && np != 9 && np != 4) || !columns(args[1], np, &k, false, -1, &m)) Py_RETURN_NONE;
  const int64_t stride = m[0].numel() == k.n ? 1 : 0;
  for (const Tensor& t : m)
    if (t.numel() != (stride ? k.n : 1)) Py_RETURN_NONE;
  Cols y;
  if (!unlocked(np == 16 ? "glv_lorentz_transform" : np == 9 ? "glv_rotate" : "glv_rotate_axis_angle", [&] {
        y = empties(k, k.n, 4);
        const Ptrs<4> x(c), o(y);
        void* const s = stream_of(k.device);
        if (np == 16) return glv_lorentz_transform(k.dt(), k.n, x.in(), Ptrs<16>(m).in(), stride, o.out(), s);
        if (np == 9) return glv_rotate(k.dt(), k.n, x.in(), Ptrs<9>(m).in(), stride, o.out(), s);
        return glv_rotate_axis_angle(k.dt(), k.n, x.in(), Ptrs<4>(m).in(), stride, o.out(), s);
      }))
    return not_done();
  return wrap_tuple(y, 0, 4);
  END_HANDLE_TH_ERRORS
}

// The pair offsets of `off`.
glv_status pair_offsets(const Tensor& off, Tensor* po) {
  *po = at::empty({off.numel()}, off.options());
  return glv_pair_offsets(off.numel() - 1, off.data_ptr<int64_t>(), po->data_ptr<int64_t>(),
                          stream_of(off.device()));
}

// pair_offsets(offsets)
PyObject* py_pair_offsets(PyObject*, PyObject* const* args, Py_ssize_t na) {
  HANDLE_TH_ERRORS
  if (na != 1 || !plain_context()) Py_RETURN_NONE;
  const Tensor* t = plain_tensor(args[0]);
  if (!t || t->scalar_type() != at::kLong || t->dim() != 1 || !t->is_contiguous() || t->numel() < 1) Py_RETURN_NONE;
  const Tensor off = *t;
  Tensor po;
  if (!unlocked("glv_pair_offsets", [&] { return pair_offsets(off, &po); })) return not_done();
  return wrap(po);
  END_HANDLE_TH_ERRORS
}

// Particle columns, offsets and pair offsets (computed where they are None
// and asked for).
struct Events {
  Kind k;
  Cols p;
  Tensor off, po;
  int64_t ne() const { return off.numel() - 1; }
  bool parse(PyObject* cols, PyObject* offsets, PyObject* pairs) {
    if (!columns(cols, 4, &k, true, -1, &p)) return false;
    const Tensor* t = offsets_of(offsets, k.device);
    if (!t || t->numel() < 1) return false;
    off = *t;
    if (pairs != Py_None) {
      const Tensor* q = offsets_of(pairs, k.device);
      if (!q || q->numel() != off.numel()) return false;
      po = *q;
    }
    return true;
  }
  glv_status need_pairs() { return po.defined() ? GLV_OK : pair_offsets(off, &po); }
  const int64_t* offs() const { return off.data_ptr<int64_t>(); }
  const int64_t* pos() const { return po.defined() ? po.data_ptr<int64_t>() : nullptr; }
};

// Totals (4), event masses and pair masses, in this order.
glv_status reduce_events(Events& e, glv_coords co, glv_mode mo, bool wt, bool we, bool wp, int64_t n_pairs,
                         unsigned long long* fb, Cols* out) {
  const int64_t ne = e.ne();
  Cols t = empties(e.k, ne, wt ? 4 : 0);
  Tensor em, pm;
  if (we) em = at::empty({ne}, e.k.opts());
  if (wp) {
    if (n_pairs < 0) n_pairs = ne > 0 ? e.po.select(0, ne).item<int64_t>() : 0;
    pm = at::empty({n_pairs}, e.k.opts());
  }
  std::array<void*, 4> tp{};
  for (size_t i = 0; i < t.size(); ++i) tp[i] = t[i].data_ptr();
  const glv_status st = glv_event_reduce(e.k.dt(), co, mo, ne, e.offs(), e.pos(), Ptrs<4>(e.p).in(),
                                         wt ? tp.data() : nullptr, we ? em.data_ptr() : nullptr,
                                         wp ? pm.data_ptr() : nullptr, fb, nullptr, stream_of(e.k.device));
  if (st != GLV_OK) return st;
  *out = std::move(t);
  if (we) out->push_back(em);
  if (wp) out->push_back(pm);
  return GLV_OK;
}

bool flag_arg(PyObject* o, bool* b) {
  *b = o == Py_True;
  return o == Py_True || o == Py_False;
}

// event_reduce(p, offsets, pair_offsets, coords, mode, want_total,
//              want_event_m, want_pair_m, fallback_count, n_pairs)
PyObject* py_event_reduce(PyObject*, PyObject* const* args, Py_ssize_t na) {
  HANDLE_TH_ERRORS
  Events e;
  glv_coords co;
  glv_mode mo;
  bool wt, we, wp;
  int64_t np = -1;
  std::optional<Tensor> fb;
  if (na != 10 || !plain_context() || !e.parse(args[0], args[1], args[2]) || !coords_arg(args[3], &co) ||
      !mode_arg(args[4], &mo) || !flag_arg(args[5], &wt) || !flag_arg(args[6], &we) || !flag_arg(args[7], &wp) ||
      !counter_arg(args[8], e.k.device, &fb) || (args[9] != Py_None && (!int_arg(args[9], &np) || np < 0)))
    Py_RETURN_NONE;
  Cols out;
  if (!unlocked("glv_event_reduce", [&] {
        if (wp || (mo == GLV_COMPENSATED && we)) {
          const glv_status st = e.need_pairs();
          if (st != GLV_OK) return st;
        }
        return reduce_events(e, co, mo, wt, we, wp, np, counter_ptr(fb), &out);
      }))
    return not_done();
  PyObject* r = PyTuple_New(3);
  size_t at = 0;
  auto put = [&](Py_ssize_t i, PyObject* o) { PyTuple_SET_ITEM(r, i, o); };
  auto none = [] {
    Py_INCREF(Py_None);
    return Py_None;
  };
  put(0, wt ? wrap_tuple(out, 0, 4) : none());
  at = wt ? 4 : 0;
  put(1, we ? wrap(out[at++]) : none());
  put(2, wp ? wrap(out[at]) : none());
  return r;
  END_HANDLE_TH_ERRORS
}

// event_reduce_best_pair(p, offsets, target, pair_offsets, coords, mode, fallback_count)
PyObject* py_best_pair(PyObject*, PyObject* const* args, Py_ssize_t na) {
  HANDLE_TH_ERRORS
  Events e;
  glv_coords co;
  glv_mode mo;
  double target;
  std::optional<Tensor> fb;
  if (na != 7 || !plain_context() || !e.parse(args[0], args[1], args[3]) || !double_arg(args[2], &target) ||
      !coords_arg(args[4], &co) || !mode_arg(args[5], &mo) || !counter_arg(args[6], e.k.device, &fb))
    Py_RETURN_NONE;
  Cols out(2);
  if (!unlocked("glv_event_reduce_best_pair", [&] {
        const glv_status st = e.need_pairs();
        if (st != GLV_OK) return st;
        out[0] = at::empty({e.ne()}, e.off.options());
        out[1] = at::empty({e.ne()}, e.k.opts());
        return glv_event_reduce_best_pair(e.k.dt(), co, mo, e.ne(), e.offs(), e.pos(), Ptrs<4>(e.p).in(), target,
                                          out[0].data_ptr<int64_t>(), out[1].data_ptr(), counter_ptr(fb), nullptr,
                                          stream_of(e.k.device));
      }))
    return not_done();
  return wrap_tuple(out, 0, 2);
  END_HANDLE_TH_ERRORS
}

// The tiling of the reverse mode of ne events with n_pairs pair upstreams.
std::optional<glv_tiling> bwd_tiling(glv_dtype dt, glv_coords co, int64_t ne, int64_t n_pairs) {
  glv_tiling t;
  if (glv_call_tiling(dt, co, GLV_PLAIN, 1, ne, n_pairs, &t) != GLV_OK) return std::nullopt;
  return t;
}

// event_reduce_bwd(p, offsets, pair_offsets, grad_total, grad_event_m, grad_pair_m, coords)
PyObject* py_event_reduce_bwd(PyObject*, PyObject* const* args, Py_ssize_t na) {
  HANDLE_TH_ERRORS
  Events e;
  glv_coords co;
  if (na != 7 || !plain_context() || !e.parse(args[0], args[1], args[2]) || !coords_arg(args[6], &co))
    Py_RETURN_NONE;
  Cols gt;
  Tensor gem, gpm;
  if (args[3] != Py_None && !columns(args[3], 4, &e.k, false, e.ne(), &gt)) Py_RETURN_NONE;
  for (int i : {4, 5}) {
    if (args[i] == Py_None) continue;
    const Tensor* t = plain_tensor(args[i]);
    if (!t || !column(*t, e.k, i == 4 ? e.ne() : -1)) Py_RETURN_NONE;
    (i == 4 ? gem : gpm) = *t;
  }
  Cols g;
  if (!unlocked("glv_event_reduce_bwd", [&] {
        if (gpm.defined()) {
          const glv_status st = e.need_pairs();
          if (st != GLV_OK) return st;
        }
        g = empties(e.k, e.k.n, 4);
        std::array<void*, 4> tp{};
        for (size_t i = 0; i < gt.size(); ++i) tp[i] = gt[i].data_ptr();
        const auto t = gpm.defined() ? bwd_tiling(e.k.dt(), co, e.ne(), gpm.numel()) : std::nullopt;
        return glv_event_reduce_bwd(e.k.dt(), co, e.ne(), e.offs(), e.pos(), Ptrs<4>(e.p).in(),
                                    gt.empty() ? nullptr : tp.data(), gem.defined() ? gem.data_ptr() : nullptr,
                                    gpm.defined() ? gpm.data_ptr() : nullptr, Ptrs<4>(g).out(), t ? &*t : nullptr,
                                    stream_of(e.k.device));
      }))
    return not_done();
  return wrap_tuple(g, 0, 4);
  END_HANDLE_TH_ERRORS
}

// --------------------------------------------------------------- autograd

// The status of a library call inside an autograd node, without the
// interpreter lock: a failure raises what it does in the Python path.
void check(const char* fn, glv_status st) {
  if (st == GLV_OK) return;
  python_error e;
  const PyGILState_STATE gil = PyGILState_Ensure();
  set_error(fn, st);
  e.persist();  // the error leaves the thread's state before that may go
  PyGILState_Release(gil);
  throw e;
}

Kind kind_of(const Tensor& t) { return {t.scalar_type(), t.device(), t.numel()}; }

// No tangent on any of them (the nodes have no forward mode).
bool no_tangents(const Cols& c) {
  for (const Tensor& t : c)
    if (t._fw_grad(0).defined()) return false;
  return true;
}

variable_list with_none(size_t none, const Cols& g) {
  variable_list r(none);
  r.insert(r.end(), g.begin(), g.end());
  return r;
}

struct InvariantMass : torch::autograd::Function<InvariantMass> {
  static Tensor forward(AutogradContext* ctx, int64_t co, int64_t mo, at::TensorList c) {
    const Kind k = kind_of(c[0]);
    Tensor m = at::empty({k.n}, k.opts());
    check("glv_invariant_mass",
          glv_invariant_mass(k.dt(), (glv_coords)co, (glv_mode)mo, k.n, Ptrs<4>(c).in(), Ptrs<4>(c, 4).in(),
                             m.data_ptr(), nullptr, stream_of(k.device)));
    ctx->saved_data["coords"] = co;
    ctx->saved_data["mode"] = mo;
    ctx->save_for_backward(c.vec());
    return m;
  }
  static variable_list backward(AutogradContext* ctx, variable_list gy) {
    const variable_list c = ctx->get_saved_variables();
    const Kind k = kind_of(c[0]);
    const Tensor gm = gy[0].contiguous();
    Cols g = empties(k, k.n, 8);
    const Ptrs<4> a(c), b(c, 4), ga(g), gb(g, 4);
    void* const s = stream_of(k.device);
    if (ctx->saved_data["mode"].toInt() == GLV_COMPENSATED)
      check("glv_invariant_mass_comp_bwd", glv_invariant_mass_comp_bwd(k.dt(), k.n, a.in(), b.in(), gm.data_ptr(),
                                                                       ga.out(), gb.out(), s));
    else
      check("glv_invariant_mass_bwd",
            glv_invariant_mass_bwd(k.dt(), (glv_coords)ctx->saved_data["coords"].toInt(), k.n, a.in(), b.in(),
                                   gm.data_ptr(), ga.out(), gb.out(), s));
    return with_none(2, g);
  }
};

struct Boost : torch::autograd::Function<Boost> {
  static variable_list forward(AutogradContext* ctx, at::TensorList c) {
    const Kind k = kind_of(c[0]);
    Cols y = empties(k, k.n, 4);
    check("glv_boost", glv_boost(k.dt(), k.n, Ptrs<4>(c).in(), Ptrs<3>(c, 4).in(), c[4].numel() == k.n,
                                 Ptrs<4>(y).out(), stream_of(k.device)));
    ctx->save_for_backward(c.vec());
    return y;
  }
  static variable_list backward(AutogradContext* ctx, variable_list gy) {
    const variable_list c = ctx->get_saved_variables();
    const Kind k = kind_of(c[0]);
    for (Tensor& t : gy) t = t.contiguous();
    const bool per_item = c[4].numel() == k.n;
    const bool want =
        per_item && (ctx->needs_input_grad(4) || ctx->needs_input_grad(5) || ctx->needs_input_grad(6));
    Cols g = empties(k, k.n, want ? 7 : 4);
    check("glv_boost_bwd",
          glv_boost_bwd(k.dt(), k.n, Ptrs<4>(c).in(), Ptrs<3>(c, 4).in(), per_item, Ptrs<4>(gy).in(),
                        Ptrs<4>(g).out(), want ? Ptrs<3>(g, 4).out() : nullptr, stream_of(k.device)));
    g.resize(7);
    return g;
  }
};

struct EventReduce : torch::autograd::Function<EventReduce> {
  static variable_list forward(AutogradContext* ctx, int64_t co, const Tensor& off, const Tensor& po,
                               at::TensorList p) {
    Events e;
    e.k = kind_of(p[0]);
    e.p = p.vec();
    e.off = off;
    e.po = po;
    Cols out;
    check("glv_event_reduce", reduce_events(e, (glv_coords)co, GLV_PLAIN, true, true, true, -1, nullptr, &out));
    ctx->saved_data["coords"] = co;
    variable_list keep{off, po};
    keep.insert(keep.end(), e.p.begin(), e.p.end());
    ctx->save_for_backward(std::move(keep));
    return out;
  }
  static variable_list backward(AutogradContext* ctx, variable_list gy) {
    const variable_list c = ctx->get_saved_variables();
    const Kind k = kind_of(c[2]);
    for (Tensor& t : gy) t = t.contiguous();
    Cols g = empties(k, k.n, 4);
    const glv_coords co = (glv_coords)ctx->saved_data["coords"].toInt();
    const int64_t ne = c[0].numel() - 1;
    const auto t = bwd_tiling(k.dt(), co, ne, gy[5].numel());
    check("glv_event_reduce_bwd",
          glv_event_reduce_bwd(k.dt(), co, ne, c[0].data_ptr<int64_t>(), c[1].data_ptr<int64_t>(),
                               Ptrs<4>(c, 2).in(), Ptrs<4>(gy).in(), gy[4].data_ptr(), gy[5].data_ptr(),
                               Ptrs<4>(g).out(), t ? &*t : nullptr, stream_of(k.device)));
    return with_none(3, g);
  }
};

// autograd_mass(a, b, coords, mode)
PyObject* py_autograd_mass(PyObject*, PyObject* const* args, Py_ssize_t na) {
  HANDLE_TH_ERRORS
  Kind k;
  Cols c;
  glv_coords co;
  glv_mode mo;
  if (na != 4 || !plain_context() || !columns(args[0], 4, &k, true, -1, &c) ||
      !columns(args[1], 4, &k, false, k.n, &c) || !coords_arg(args[2], &co) || !mode_arg(args[3], &mo) ||
      (mo == GLV_COMPENSATED && co != GLV_PTETAPHIM) || !no_tangents(c))
    Py_RETURN_NONE;
  Tensor m;
  if (!unlocked("glv_invariant_mass", [&] {
        m = InvariantMass::apply((int64_t)co, (int64_t)mo, at::TensorList(c));
        return GLV_OK;
      }))
    return not_done();
  return wrap(m);
  END_HANDLE_TH_ERRORS
}

// autograd_boost(x, beta)
PyObject* py_autograd_boost(PyObject*, PyObject* const* args, Py_ssize_t na) {
  HANDLE_TH_ERRORS
  Kind k;
  Cols c;
  if (na != 2 || !plain_context() || !columns(args[0], 4, &k, true, -1, &c) ||
      !columns(args[1], 3, &k, false, -1, &c) || !no_tangents(c))
    Py_RETURN_NONE;
  const int64_t nb = c[4].numel() == k.n ? k.n : 1;
  for (size_t i = 4; i < 7; ++i)
    if (c[i].numel() != nb) Py_RETURN_NONE;
  Cols y;
  if (!unlocked("glv_boost", [&] {
        y = Boost::apply(at::TensorList(c));
        return GLV_OK;
      }))
    return not_done();
  return wrap_tuple(y, 0, 4);
  END_HANDLE_TH_ERRORS
}

// autograd_event_reduce(p, offsets, pair_offsets, coords): the totals, event masses and pair masses
PyObject* py_autograd_event_reduce(PyObject*, PyObject* const* args, Py_ssize_t na) {
  HANDLE_TH_ERRORS
  Events e;
  glv_coords co;
  if (na != 4 || !plain_context() || !e.parse(args[0], args[1], args[2]) || !coords_arg(args[3], &co) ||
      !no_tangents(e.p))
    Py_RETURN_NONE;
  Cols out;
  if (!unlocked("glv_pair_offsets", [&] {
        const glv_status st = e.need_pairs();
        if (st == GLV_OK) out = EventReduce::apply((int64_t)co, e.off, e.po, at::TensorList(e.p));
        return st;
      }))
    return not_done();
  return wrap_tuple(out, 0, 6);
  END_HANDLE_TH_ERRORS
}

template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyMethodDef method(const char* name) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(F)), METH_FASTCALL, nullptr};
}

}  // namespace

PyMODINIT_FUNC PyInit__native() {
  static PyMethodDef methods[] = {method<py_mass>("mass"),
                                  method<py_mass_histogram>("mass_histogram"),
                                  method<py_boost>("boost"),
                                  method<py_convert>("convert"),
                                  method<py_transform>("transform"),
                                  method<py_pair_offsets>("pair_offsets"),
                                  method<py_event_reduce>("event_reduce"),
                                  method<py_event_reduce_bwd>("event_reduce_bwd"),
                                  method<py_best_pair>("event_reduce_best_pair"),
                                  method<py_autograd_mass>("autograd_mass"),
                                  method<py_autograd_boost>("autograd_boost"),
                                  method<py_autograd_event_reduce>("autograd_event_reduce"),
                                  {nullptr, nullptr, 0, nullptr}};
  static PyModuleDef def = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};
  return PyModule_Create(&def);
}
