// The Python entry points' host side: one native call per entry point.
//
// What a small revisit costs is not its kernel (about 7 us) but the checks and the
// argument blocks: in Python some thirty attribute, shape and pointer look-ups, a ctypes
// structure per descriptor and four output allocations, 28 us per revisit call and 37 us
// per reassign + rebind pair on the host (8 and 12 now).  Here the same checks read the
// tensors' own fields, and the lock that serialises Python is given up once, around the
// allocations and the launch.
//
// A function either does the whole call, and returns its result (a tensor, a tuple, True,
// or the status of a launch that the HIP runtime refused), or has done nothing and returns
// None.  It returns None for whatever is not the plain case: an argument of another type
// than the entry point's own or of a subclass, a value that binding.py's checks refuse, an
// allocation that fails, an active function mode.  binding.py then takes the call itself,
// and refuses it (or not) with its own checks and messages.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <optional>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/StreamGuard.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <torch/csrc/Device.h>
#include <torch/csrc/Stream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "prcr.h"

namespace {

struct Skip {};   // not the plain case: binding.py takes the call

PyObject *g_rope, *g_memory, *g_cache;   // the classes, exactly these
PyObject *g_modes;                       // mode name -> number
PyObject *g_raw_stream;                  // device index -> the current stream's handle

#define PRCR_NAMES(X)                                                                     \
  X(k) X(v) X(coords) X(n_visual) X(v_slot) X(device) X(block_table) X(paged) X(head_dim) \
  X(sections) X(interleaved) X(theta) X(cuda_stream)
#define PRCR_DECLARE(n) PyObject *s_##n;
PRCR_NAMES(PRCR_DECLARE)
#undef PRCR_DECLARE

// An owned reference.
class Ref {
 public:
  explicit Ref(PyObject *o) : o_(o) {
    if (o_ == nullptr) throw Skip();
  }
  Ref(const Ref &) = delete;
  Ref &operator=(const Ref &) = delete;
  ~Ref() { Py_XDECREF(o_); }
  PyObject *get() const { return o_; }
  PyObject *release() {
    PyObject *o = o_;
    o_ = nullptr;
    return o;
  }

 private:
  PyObject *o_;
};

// Gives up the interpreter lock for a scope: an allocation may wait for the GPU or call
// back into Python, and a launch waits while the queue is full.
class Unlocked {
 public:
  Unlocked() : state_(PyEval_SaveThread()) {}
  ~Unlocked() { PyEval_RestoreThread(state_); }

 private:
  PyThreadState *state_;
};

Ref attr(PyObject *o, PyObject *name) { return Ref(PyObject_GetAttr(o, name)); }

// A tensor argument, kept alive by the copy (another thread may drop the caller's).
at::Tensor tensor(PyObject *o) {
  if (!THPVariable_CheckExact(o)) throw Skip();
  return THPVariable_Unpack(o);
}
at::Tensor tensor_or_none(PyObject *o) { return o == Py_None ? at::Tensor() : tensor(o); }
at::Tensor tensor_attr(PyObject *o, PyObject *name) { return tensor(attr(o, name).get()); }
at::Tensor tensor_attr_or_none(PyObject *o, PyObject *name) { return tensor_or_none(attr(o, name).get()); }

int32_t to_int32(int64_t v) {
  if (v < INT32_MIN || v > INT32_MAX) throw Skip();
  return static_cast<int32_t>(v);
}
int32_t int32_of(PyObject *o) {
  if (!PyLong_CheckExact(o)) throw Skip();
  int overflow = 0;
  const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
  if (overflow != 0) throw Skip();
  return to_int32(v);
}
double double_of(PyObject *o) {
  if (!PyFloat_CheckExact(o)) throw Skip();
  return PyFloat_AS_DOUBLE(o);
}
bool bool_of(PyObject *o) {
  if (!PyBool_Check(o)) throw Skip();
  return o == Py_True;
}
int32_t mode_of(PyObject *o) {
  if (!PyUnicode_CheckExact(o)) throw Skip();
  PyObject *v = PyDict_GetItemWithError(g_modes, o);   // borrowed
  if (v == nullptr) throw Skip();
  return int32_of(v);
}
void only(PyObject *o, PyObject *cls) {
  if (reinterpret_cast<PyObject *>(Py_TYPE(o)) != cls) throw Skip();
}

// What binding.py's _need checks.
void need(const at::Tensor &t, at::Device device) {
  if (!t.is_cuda() || t.device() != device || !t.is_contiguous()) throw Skip();
}
void need(const at::Tensor &t, at::ScalarType type, at::Device device, at::IntArrayRef shape) {
  need(t, device);
  if (t.scalar_type() != type || t.sizes() != shape) throw Skip();
}

prcr_dtype dtype_of(const at::Tensor &t) {
  if (t.scalar_type() == at::kFloat) return PRCR_F32;
  if (t.scalar_type() == at::kBFloat16) return PRCR_BF16;
  throw Skip();
}

template <typename T>
T *ptr(const at::Tensor &t) {
  return t.defined() ? static_cast<T *>(t.data_ptr()) : nullptr;
}

void no_overlap(const at::Tensor &a, const at::Tensor &b) {
  if (a.numel() == 0 || b.numel() == 0) return;
  const uintptr_t x = reinterpret_cast<uintptr_t>(a.data_ptr()), y = reinterpret_cast<uintptr_t>(b.data_ptr());
  if (x < y + b.nbytes() && y < x + a.nbytes()) throw Skip();
}

at::Device device_of(PyObject *owner) {
  const Ref d = attr(owner, s_device);
  if (!THPDevice_Check(d.get())) throw Skip();
  return reinterpret_cast<THPDevice *>(d.get())->device;
}

hipStream_t handle_of(PyObject *number) {
  const Ref h(number);
  if (!PyLong_CheckExact(h.get())) throw Skip();
  const unsigned long long v = PyLong_AsUnsignedLongLong(h.get());
  if (v == static_cast<unsigned long long>(-1) && PyErr_Occurred()) throw Skip();
  return reinterpret_cast<hipStream_t>(static_cast<uintptr_t>(v));
}

// The stream of a call, and the memory made for the call.  On another stream than torch's
// current one that memory is the other stream's: one of the current stream's blocks might
// still be read there when the kernels write it, and would be handed out again, once the
// call has dropped it, while they run.  What the caller is given is used on the current
// stream, so it is recorded there and is not handed out again before that use.
class Launch {
 public:
  Launch(PyObject *stream, at::Device device) : device_(device) {
    const Ref index(PyLong_FromLong(device.index()));
    handle_ = handle_of(PyObject_CallOneArg(g_raw_stream, index.get()));
    if (stream == Py_None) return;
    const hipStream_t current = handle_;
    handle_ = handle_of(PyObject_GetAttr(stream, s_cuda_stream));
    other_ = handle_ != current;
    if (other_ && THPStream_Check(stream)) {
      const THPStream *s = reinterpret_cast<const THPStream *>(stream);
      on_ = c10::Stream::unpack3(s->stream_id, static_cast<c10::DeviceIndex>(s->device_index),
                                 static_cast<c10::DeviceType>(s->device_type));
    }
  }
  hipStream_t handle() const { return handle_; }
  at::Tensor fresh(at::IntArrayRef shape, at::ScalarType type, bool given) const {
    const auto options = at::TensorOptions().dtype(type).device(device_);
    if (!other_) return at::empty(shape, options);
    if (!on_ || on_->device() != device_) throw Skip();   // no stream of torch's
    const c10::impl::VirtualGuardImpl streams(device_.type());
    const c10::Stream current = streams.getStream(device_);
    const c10::StreamGuard guard(*on_);
    at::Tensor t = at::empty(shape, options);
    if (given) streams.recordDataPtrOnStream(t.storage().data_ptr(), current);
    return t;
  }

 private:
  at::Device device_;
  hipStream_t handle_;
  bool other_ = false;
  std::optional<c10::Stream> on_;
};

at::Tensor err_of(PyObject *o, at::Device device) {
  at::Tensor t = tensor_or_none(o);
  if (t.defined()) {
    need(t, device);
    if (t.scalar_type() != at::kInt || t.dim() != 1 || t.size(0) < 1) throw Skip();
  }
  return t;
}

prcr_rope rope_of(PyObject *o) {
  only(o, g_rope);
  prcr_rope r{};
  r.head_dim = int32_of(attr(o, s_head_dim).get());
  const Ref sections = attr(o, s_sections);
  if (!PyTuple_CheckExact(sections.get()) || PyTuple_GET_SIZE(sections.get()) != 3) throw Skip();
  for (int i = 0; i < 3; ++i) r.section[i] = int32_of(PyTuple_GET_ITEM(sections.get(), i));
  r.interleaved = bool_of(attr(o, s_interleaved).get()) ? 1 : 0;
  r.theta = double_of(attr(o, s_theta).get());
  return r;
}

// A Memory's tensors, held for the call, and its descriptor.
struct Mem {
  explicit Mem(PyObject *o)
      : owner((only(o, g_memory), o)), device(device_of(o)), k(tensor_attr(o, s_k)), v(tensor_attr_or_none(o, s_v)),
        coords(tensor_attr(o, s_coords)), n_visual(tensor_attr(o, s_n_visual)),
        v_slot(tensor_attr_or_none(o, s_v_slot)) {
    if (k.dim() != 5) throw Skip();
    c.k = ptr<void>(k);
    c.v = ptr<void>(v);
    c.coords = ptr<int32_t>(coords);
    c.n_visual = ptr<int32_t>(n_visual);
    c.batch = to_int32(k.size(0));
    c.max_visual = to_int32(k.size(1));
    c.n_layers = to_int32(k.size(2));
    c.n_kv_heads = to_int32(k.size(3));
    c.head_dim = to_int32(k.size(4));
    c.dtype = dtype_of(k);
    c.v_slot = ptr<int32_t>(v_slot);
  }
  PyObject *owner;
  at::Device device;
  at::Tensor k, v, coords, n_visual, v_slot;
  prcr_mem c{};
};

// A Cache's tensors, held for the call, and its descriptor.
struct Store {
  explicit Store(PyObject *o)
      : owner((only(o, g_cache), o)), device(device_of(o)), k(tensor_attr(o, s_k)), v(tensor_attr(o, s_v)),
        paged(bool_of(attr(o, s_paged).get())) {
    if (k.dim() != 5) throw Skip();
    c.k = ptr<void>(k);
    c.v = ptr<void>(v);
    c.paged = paged ? 1 : 0;
    if (paged) {
      table = tensor_attr(o, s_block_table);
      if (table.dim() != 2) throw Skip();
      c.block_table = ptr<int32_t>(table);
      c.block_size = to_int32(k.size(2));
      c.max_blocks = to_int32(table.size(1));
      c.n_blocks = to_int32(k.size(1));
    } else {
      c.s_max = to_int32(k.size(3));
    }
  }
  int64_t n_layers() const { return k.size(paged ? 0 : 1); }
  int64_t n_kv_heads() const { return k.size(paged ? 3 : 2); }
  int64_t rows() const { return paged ? table.size(0) : k.size(0); }   // sequences
  void check_matches(const Mem &m) const {
    if (k.scalar_type() != m.k.scalar_type() || rows() != m.c.batch || n_layers() != m.c.n_layers ||
        n_kv_heads() != m.c.n_kv_heads || k.size(4) != m.c.head_dim)
      throw Skip();
  }
  PyObject *owner;
  at::Device device;
  at::Tensor k, v, table;
  bool paged;
  prcr_cache c{};
};

// The selection both calls of a revisit take.
struct Selection {
  Selection(const Mem &m, PyObject *o, PyObject *i) : off(tensor(o)), idx(tensor(i)) {
    need(off, at::kInt, m.device, {int64_t{m.c.batch} + 1});
    need(idx, m.device);
    if (idx.scalar_type() != at::kInt || idx.dim() != 1) throw Skip();
    k = to_int32(idx.size(0));
  }
  at::Tensor off, idx;
  int32_t k;
};

// An output: the caller's tensor, checked, or one made here (inside Unlocked).
struct Out {
  Out(PyObject *o, at::ScalarType type_, at::Device device, at::DimVector shape_)
      : t(tensor_or_none(o)), type(type_), shape(std::move(shape_)) {
    if (t.defined()) need(t, type, device, shape);
  }
  void make(const Launch &on) {
    if (!t.defined()) t = on.fresh(shape, type, true);
  }
  at::Tensor t;
  at::ScalarType type;
  at::DimVector shape;
};

// Whether the call was done.  A launch that the runtime refused is not tried again: its
// status is returned.  Every other status comes from the host checks, before any launch,
// and binding.py finds it, or an earlier refusal of its own, again.
bool done(prcr_status st, PyObject **failed) {
  *failed = nullptr;
  if (st == PRCR_OK) return true;
  if (st != PRCR_ERR_HIP) throw Skip();
  *failed = PyLong_FromLong(st);
  return false;
}

// The positional arguments of a call; a wrong number is a mistake of binding.py's.
using Args = PyObject *const *;
template <int kCount, PyObject *(*kBody)(Args)>
PyObject *entry(PyObject *, Args a, Py_ssize_t n) {
  if (n != kCount) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  try {
    if (g_rope != nullptr && g_raw_stream != nullptr && !at::impl::torch_function_mode_enabled()) return kBody(a);
  } catch (...) {
    PyErr_Clear();
  }
  Py_RETURN_NONE;
}

// A call's result.  The launch is behind it, so an error here (memory) is raised and does
// not hand the call to binding.py, which would launch again.
PyObject *wrap(const at::Tensor &t) noexcept {
  try {
    return t.defined() ? THPVariable_Wrap(t) : Py_NewRef(Py_None);
  } catch (...) {
    return PyErr_Occurred() ? nullptr : PyErr_NoMemory();
  }
}
template <typename... T>
PyObject *tuple_of(const T &...t) noexcept {
  PyObject *out = PyTuple_New(sizeof...(T));
  if (out == nullptr) return nullptr;
  Py_ssize_t i = 0;
  bool ok = true;
  auto put = [&](const at::Tensor &x) {
    PyObject *o = ok ? wrap(x) : nullptr;
    ok = ok && o != nullptr;
    PyTuple_SET_ITEM(out, i++, o);
  };
  (put(t), ...);
  if (ok) return out;
  Py_DECREF(out);
  return nullptr;
}

// (mem, layer, raw_k, raw_v, vis_rows, err, stream)
PyObject *store_raw(Args a) {
  const Mem m(a[0]);
  const int32_t layer = int32_of(a[1]);
  const at::Tensor raw_k = tensor(a[2]), raw_v = tensor_or_none(a[3]), rows = tensor(a[4]);
  if (raw_k.dim() != 4) throw Skip();
  const at::DimVector shape{m.c.batch, raw_k.size(1), m.c.n_kv_heads, m.c.head_dim};
  need(raw_k, m.k.scalar_type(), m.device, shape);
  if (m.v.defined() && !raw_v.defined()) throw Skip();
  if (raw_v.defined()) need(raw_v, m.k.scalar_type(), m.device, shape);
  need(rows, at::kInt, m.device, {m.c.batch, m.c.max_visual});
  const at::Tensor err = err_of(a[5], m.device);
  const Launch on(a[6], m.device);
  const int32_t s_src = to_int32(raw_k.size(1));
  prcr_status st;
  {
    Unlocked u;
    st = prcr_store_raw(&m.c, layer, ptr<void>(raw_k), ptr<void>(raw_v), s_src, ptr<int32_t>(rows),
                        ptr<int32_t>(err), on.handle());
  }
  PyObject *failed;
  return done(st, &failed) ? Py_NewRef(Py_True) : failed;
}

// (mem, sel_off, sel_idx, p_txt, mode, l_ext, new_pos, next_pos, err, stream)
PyObject *reassign_coords(Args a) {
  const Mem m(a[0]);
  const Selection sel(m, a[1], a[2]);
  const at::Tensor p_txt = tensor(a[3]);
  need(p_txt, at::kInt, m.device, {m.c.batch});
  const int32_t mode = mode_of(a[4]), l_ext = int32_of(a[5]);
  Out new_pos(a[6], at::kDouble, m.device, {sel.k, 3}), next_pos(a[7], at::kInt, m.device, {m.c.batch});
  const at::Tensor err = err_of(a[8], m.device);
  const Launch on(a[9], m.device);
  prcr_status st;
  {
    Unlocked u;
    new_pos.make(on);
    next_pos.make(on);
    no_overlap(next_pos.t, sel.off);
    no_overlap(next_pos.t, m.n_visual);
    st = prcr_reassign_coords(&m.c, ptr<int32_t>(sel.off), ptr<int32_t>(sel.idx), sel.k, ptr<int32_t>(p_txt),
                              static_cast<prcr_mode>(mode), l_ext, ptr<double>(new_pos.t),
                              ptr<int32_t>(next_pos.t), ptr<int32_t>(err), on.handle());
  }
  PyObject *failed;
  return done(st, &failed) ? tuple_of(new_pos.t, next_pos.t) : failed;
}

// (rope, mem, sel_off, sel_idx, new_pos, cache, cache_len, new_cache_len, slot_mapping, err, stream)
PyObject *rebind_inject(Args a) {
  const prcr_rope rope = rope_of(a[0]);
  const Mem m(a[1]);
  const Selection sel(m, a[2], a[3]);
  const at::Tensor new_pos = tensor(a[4]), cache_len = tensor(a[6]);
  const Store cache(a[5]);
  cache.check_matches(m);
  need(new_pos, at::kDouble, m.device, {sel.k, 3});
  need(cache_len, at::kInt, m.device, {m.c.batch});
  Out new_len(a[7], at::kInt, m.device, {m.c.batch}), slots(a[8], at::kLong, m.device, {sel.k});
  const at::Tensor err = err_of(a[9], m.device);
  const Launch on(a[10], m.device);
  prcr_status st;
  {
    Unlocked u;
    new_len.make(on);
    slots.make(on);
    no_overlap(new_len.t, cache_len);
    no_overlap(new_len.t, sel.off);
    st = prcr_rebind_inject(&rope, &m.c, ptr<int32_t>(sel.off), ptr<int32_t>(sel.idx), sel.k,
                            ptr<double>(new_pos), &cache.c, ptr<int32_t>(cache_len), ptr<int32_t>(new_len.t),
                            ptr<int64_t>(slots.t), ptr<int32_t>(err), on.handle());
  }
  PyObject *failed;
  return done(st, &failed) ? tuple_of(new_len.t, slots.t) : failed;
}

// (rope, mem, sel_off, sel_idx, p_txt, cache, cache_len, mode, l_ext, new_pos, next_pos,
//  new_cache_len, slot_mapping, err, stream, store_positions)
PyObject *revisit(Args a) {
  const prcr_rope rope = rope_of(a[0]);
  const Mem m(a[1]);
  const Selection sel(m, a[2], a[3]);
  const at::Tensor p_txt = tensor(a[4]), cache_len = tensor(a[6]);
  const Store cache(a[5]);
  cache.check_matches(m);
  need(p_txt, at::kInt, m.device, {m.c.batch});
  need(cache_len, at::kInt, m.device, {m.c.batch});
  const int32_t mode = mode_of(a[7]), l_ext = int32_of(a[8]);
  Out new_pos(a[9], at::kDouble, m.device, {sel.k, 3}), next_pos(a[10], at::kInt, m.device, {m.c.batch}),
      new_len(a[11], at::kInt, m.device, {m.c.batch}), slots(a[12], at::kLong, m.device, {sel.k});
  const at::Tensor err = err_of(a[13], m.device);
  const Launch on(a[14], m.device);
  const bool positions = bool_of(a[15]);
  prcr_status st;
  {
    Unlocked u;
    if (positions) new_pos.make(on);
    next_pos.make(on);
    new_len.make(on);
    slots.make(on);
    const at::Tensor *next_apart[] = {&p_txt, &cache_len, &sel.off, &m.n_visual, &new_len.t};
    for (const at::Tensor *t : next_apart) no_overlap(next_pos.t, *t);
    const at::Tensor *len_apart[] = {&cache_len, &sel.off, &p_txt};
    for (const at::Tensor *t : len_apart) no_overlap(new_len.t, *t);
    st = prcr_revisit(&rope, &m.c, ptr<int32_t>(sel.off), ptr<int32_t>(sel.idx), sel.k, ptr<int32_t>(p_txt),
                      static_cast<prcr_mode>(mode), l_ext, &cache.c, ptr<int32_t>(cache_len),
                      ptr<double>(new_pos.t), ptr<int32_t>(next_pos.t), ptr<int32_t>(new_len.t),
                      ptr<int64_t>(slots.t), ptr<int32_t>(err), on.handle());
  }
  PyObject *failed;
  return done(st, &failed) ? tuple_of(new_pos.t, next_pos.t, new_len.t, slots.t) : failed;
}

// (rope, mem, layer, raw_k, raw_v, pos, n_tokens, vis_index, cache, cache_start, write_coords, err, stream)
PyObject *prefill_capture(Args a) {
  const prcr_rope rope = rope_of(a[0]);
  const Mem m(a[1]);
  const int32_t layer = int32_of(a[2]);
  const at::Tensor raw_k = tensor(a[3]), raw_v = tensor(a[4]), pos = tensor(a[5]), n_tokens = tensor(a[6]),
                   vis = tensor(a[7]), start = tensor(a[9]);
  const Store cache(a[8]);
  cache.check_matches(m);
  if (raw_k.dim() != 4) throw Skip();
  const int64_t B = m.c.batch, S = raw_k.size(1);
  const at::DimVector shape{B, S, m.c.n_kv_heads, m.c.head_dim};
  need(raw_k, m.k.scalar_type(), m.device, shape);
  need(raw_v, m.k.scalar_type(), m.device, shape);
  need(pos, at::kInt, m.device, {B, S, 3});
  need(n_tokens, at::kInt, m.device, {B});
  need(vis, at::kInt, m.device, {B, S});
  need(start, at::kInt, m.device, {B});
  const bool write_coords = bool_of(a[10]);
  const at::Tensor err = err_of(a[11], m.device);
  const Launch on(a[12], m.device);
  const int32_t s_src = to_int32(S);
  prcr_status st;
  {
    Unlocked u;
    st = prcr_prefill_capture(&rope, &m.c, layer, ptr<void>(raw_k), ptr<void>(raw_v), s_src, ptr<int32_t>(pos),
                              ptr<int32_t>(n_tokens), ptr<int32_t>(vis), write_coords ? 1 : 0, &cache.c,
                              ptr<int32_t>(start), ptr<int32_t>(err), on.handle());
  }
  PyObject *failed;
  return done(st, &failed) ? Py_NewRef(Py_True) : failed;
}

// Both decode calls: (rope, cache, layer, q, q_pos, cache_len, scale, out, [workspace,] err, stream)
template <bool kStatic>
PyObject *decode(Args a) {
  const prcr_rope rope = rope_of(a[0]);
  const Store cache(a[1]);
  const int32_t layer = int32_of(a[2]);
  const at::Tensor q = tensor(a[3]), q_pos = tensor(a[4]), cache_len = tensor(a[5]);
  if (q.dim() != 3) throw Skip();
  const int64_t B = q.size(0), Hq = q.size(1), D = cache.k.size(4);
  need(q, cache.k.scalar_type(), cache.device, {B, Hq, D});
  if (cache.rows() != B) throw Skip();
  need(q_pos, at::kInt, cache.device, {B});
  need(cache_len, at::kInt, cache.device, {B});
  const double scale = a[6] == Py_None ? std::pow(static_cast<double>(D), -0.5) : double_of(a[6]);
  Out out(a[7], at::kFloat, cache.device, {B, Hq, D});
  at::Tensor ws = kStatic ? at::Tensor() : tensor_or_none(a[8]);
  constexpr int kErr = kStatic ? 8 : 9;
  const at::Tensor err = err_of(a[kErr], cache.device);
  const Launch on(a[kErr + 1], cache.device);
  const prcr_dtype dtype = dtype_of(cache.k);
  const int32_t b = to_int32(B), hq = to_int32(Hq), nl = to_int32(cache.n_layers()),
                h = to_int32(cache.n_kv_heads());
  prcr_status st;
  if constexpr (kStatic) {
    Unlocked u;
    out.make(on);
    st = prcr_decode_attention_static(&rope, &cache.c, dtype, b, nl, h, layer, ptr<void>(q), hq,
                                      ptr<int32_t>(q_pos), ptr<int32_t>(cache_len), static_cast<float>(scale),
                                      ptr<float>(out.t), ptr<int32_t>(err), on.handle());
  } else {
    size_t bytes = 0;
    if (prcr_decode_workspace_size(&cache.c, b, hq, h, to_int32(D), &bytes) != PRCR_OK) throw Skip();
    if (ws.defined()) {
      need(ws, cache.device);
      if (ws.nbytes() < bytes) throw Skip();
    }
    Unlocked u;
    out.make(on);
    if (!ws.defined())
      ws = on.fresh({static_cast<int64_t>((std::max(bytes, size_t{4}) + 3) / 4)}, at::kFloat, false);
    st = prcr_decode_attention(&rope, &cache.c, dtype, b, nl, h, layer, ptr<void>(q), hq, ptr<int32_t>(q_pos),
                               ptr<int32_t>(cache_len), static_cast<float>(scale), ptr<float>(out.t),
                               ptr<void>(ws), ws.nbytes(), ptr<int32_t>(err), on.handle());
  }
  PyObject *failed;
  return done(st, &failed) ? wrap(out.t) : failed;
}

// (Rope, Memory, Cache, MODES), once.
PyObject *setup(PyObject *, Args a, Py_ssize_t n) {
  if (n != 4 || !PyDict_CheckExact(a[3])) {
    PyErr_SetString(PyExc_TypeError, "setup(Rope, Memory, Cache, MODES)");
    return nullptr;
  }
  PyObject **to[] = {&g_rope, &g_memory, &g_cache, &g_modes};
  for (int i = 0; i < 4; ++i) Py_XSETREF(*to[i], Py_NewRef(a[i]));
  Py_RETURN_NONE;
}

#define PRCR_ENTRY(name, count, body) \
  {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<count, body>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"setup", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&setup)), METH_FASTCALL, nullptr},
    PRCR_ENTRY(store_raw, 7, store_raw),
    PRCR_ENTRY(reassign_coords, 10, reassign_coords),
    PRCR_ENTRY(rebind_inject, 11, rebind_inject),
    PRCR_ENTRY(revisit, 16, revisit),
    PRCR_ENTRY(prefill_capture, 13, prefill_capture),
    PRCR_ENTRY(decode_attention, 11, decode<false>),
    PRCR_ENTRY(decode_attention_static, 10, decode<true>),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_prcr_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__prcr_native() {
#define PRCR_INTERN(n) \
  if ((s_##n = PyUnicode_InternFromString(#n)) == nullptr) return nullptr;
  PRCR_NAMES(PRCR_INTERN)
#undef PRCR_INTERN
  // A torch without GPU support has no current stream: every call is binding.py's then.
  PyObject *torch_c = PyImport_ImportModule("torch._C");
  if (torch_c == nullptr) return nullptr;
  g_raw_stream = PyObject_GetAttrString(torch_c, "_cuda_getCurrentRawStream");
  if (g_raw_stream == nullptr) PyErr_Clear();
  Py_DECREF(torch_c);
  PyObject *m = PyModule_Create(&module);
  if (m != nullptr && PyModule_AddStringConstant(m, "built_for", PRCR_BUILT_FOR) != 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
