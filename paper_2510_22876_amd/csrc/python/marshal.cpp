// Native argument marshalling of the Python binding (specdec.py).
//
// Each function here does for one entry point what the wrapper in specdec.py
// does: the same checks on the same torch tensors, then the library call.
// Checking and converting some thirty arguments in Python took longer than
// the kernels of a small step (tiny step 20.7 us a call, of which about 17 in
// the wrapper; 1 us here).  A function returns
// NotImplemented, with nothing called, for any argument that it does not take
// as it stands (a wrong type, shape or device, a tensor subclass, an integer
// beyond 32 bits): the wrapper then goes on in Python and reports it.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include <initializer_list>

#include "specdec.h"

namespace {

// Library functions, by the addresses of the library that specdec.py loaded.
struct Library {
  decltype(&specdec_workspace_bytes) workspace_bytes;
  decltype(&specdec_sample_workspace_bytes) sample_workspace_bytes;
  decltype(&specdec_verify_greedy) verify_greedy;
  decltype(&specdec_verify_sample) verify_sample;
  decltype(&specdec_step) step;
  decltype(&specdec_step_noalloc) step_noalloc;
  decltype(&specdec_step_sample) step_sample;
  decltype(&specdec_gather_batch) gather_batch;
  decltype(&specdec_scatter_accepted) scatter_accepted;
  decltype(&specdec_varlen_rollback) varlen_rollback;
} lib;
PyObject* get_device = nullptr;   // torch's current device, and the current stream of a device as an integer
PyObject* get_stream = nullptr;

// An argument that the Python wrapper has to look at.
struct Leave {};
void need(bool ok) {
  if (!ok) throw Leave{};
}

const at::Tensor& tensor(PyObject* o) {
  need(THPVariable_CheckExact(o));
  return THPVariable_Unpack(o);
}

template <typename P = void>
P* pointer(const at::Tensor& t) {
  return static_cast<P*>(const_cast<void*>(static_cast<const void*>(t.data_ptr())));
}

// A contiguous device tensor of the given type and shape; its address.
template <typename P>
P* dense(PyObject* o, at::ScalarType type, std::initializer_list<int64_t> shape) {
  const at::Tensor& t = tensor(o);
  need(t.is_cuda() && t.scalar_type() == type && t.sizes().equals(at::IntArrayRef(shape)) && t.is_contiguous());
  return pointer<P>(t);
}
template <typename P>
P* dense_or_none(PyObject* o, at::ScalarType type, std::initializer_list<int64_t> shape) {
  return o == Py_None ? nullptr : dense<P>(o, type, shape);
}
int32_t* ints(PyObject* o, std::initializer_list<int64_t> shape) { return dense<int32_t>(o, at::kInt, shape); }
int32_t* ints_or_none(PyObject* o, std::initializer_list<int64_t> shape) {
  return dense_or_none<int32_t>(o, at::kInt, shape);
}
uint32_t* status(PyObject* o) { return dense_or_none<uint32_t>(o, at::kInt, {1}); }

// A 2-dimensional tensor of `rows` rows and any width.
template <typename P>
P* rows(PyObject* o, at::ScalarType type, int64_t n, int64_t* width) {
  const at::Tensor& t = tensor(o);
  need(t.dim() == 2);
  *width = t.size(1);
  return dense<P>(o, type, {n, *width});
}

int32_t integer(PyObject* o) {
  need(PyLong_Check(o));
  int over = 0;
  const long long v = PyLong_AsLongLongAndOverflow(o, &over);
  need(!over && v >= INT32_MIN && v <= INT32_MAX);
  return static_cast<int32_t>(v);
}

struct Logits {
  const void* data;
  int32_t dtype, B, k, V;
  at::ScalarType type;
};
Logits logits_of(PyObject* o) {
  const at::Tensor& t = tensor(o);
  Logits l;
  l.type = t.scalar_type();
  l.dtype = l.type == at::kFloat ? SPECDEC_F32 : l.type == at::kBFloat16 ? SPECDEC_BF16 : SPECDEC_F16;
  need((l.dtype != SPECDEC_F16 || l.type == at::kHalf) && t.dim() == 3 && t.is_cuda() && t.is_contiguous());
  need(t.size(0) <= INT32_MAX && t.size(1) >= 1 && t.size(1) <= INT32_MAX && t.size(2) <= INT32_MAX);
  l.B = static_cast<int32_t>(t.size(0));
  l.k = static_cast<int32_t>(t.size(1)) - 1;
  l.V = static_cast<int32_t>(t.size(2));
  l.data = pointer(t);
  return l;
}

specdec_kv_t cache(PyObject* o) {
  const at::Tensor& t = tensor(o);
  need(t.dim() == 6 && t.size(1) == 2 && t.scalar_type() == at::kBFloat16 && t.is_contiguous() && t.is_cuda());
  for (int d : {0, 2, 3, 5}) need(t.size(d) <= INT32_MAX);
  return {pointer(t), static_cast<int32_t>(t.size(0)), static_cast<int32_t>(t.size(2)), static_cast<int32_t>(t.size(3)),
          static_cast<int32_t>(t.size(5)), t.size(4)};
}

specdec_varlen_t flat_cache(PyObject* o) {
  const at::Tensor& t = tensor(o);
  need(t.dim() == 5 && t.size(1) == 2 && t.scalar_type() == at::kBFloat16 && t.is_contiguous() && t.is_cuda());
  for (int d : {0, 3, 4}) need(t.size(d) <= INT32_MAX);
  return {pointer(t), static_cast<int32_t>(t.size(0)), static_cast<int32_t>(t.size(3)), static_cast<int32_t>(t.size(4)),
          t.size(2)};
}

struct Workspace {
  void* data;
  size_t bytes;
};
Workspace workspace(PyObject* o, size_t least) {
  const at::Tensor& t = tensor(o);
  const size_t bytes = static_cast<size_t>(t.numel()) * t.itemsize();
  need(t.is_cuda() && bytes >= least);
  return {pointer(t), bytes};
}

// The stream given as an integer or None; else torch's current one.
void* stream_of(PyObject* o) {
  if (o != Py_None) {
    need(PyLong_Check(o));
    void* s = PyLong_AsVoidPtr(o);
    if (PyErr_Occurred()) {
      PyErr_Clear();
      throw Leave{};
    }
    return s;
  }
  PyObject* dev = PyObject_CallNoArgs(get_device);
  PyObject* st = dev ? PyObject_CallOneArg(get_stream, dev) : nullptr;
  Py_XDECREF(dev);
  void* s = st ? PyLong_AsVoidPtr(st) : nullptr;
  Py_XDECREF(st);
  if (PyErr_Occurred()) {
    PyErr_Clear();
    throw Leave{};
  }
  return s;
}

// Runs the library call without the interpreter lock, as ctypes does.
template <typename F>
specdec_status_t unlocked(F&& f) {
  specdec_status_t s;
  Py_BEGIN_ALLOW_THREADS
  s = f();
  Py_END_ALLOW_THREADS
  return s;
}

template <typename F>
PyObject* guarded(Py_ssize_t given, Py_ssize_t wanted, F&& f) {
  if (given != wanted) {
    PyErr_Format(PyExc_TypeError, "%zd arguments given, %zd wanted", given, wanted);
    return nullptr;
  }
  try {
    return f();
  } catch (const Leave&) {
  } catch (const std::exception&) {   // torch's: a tensor without storage, for one
  }
  PyErr_Clear();
  Py_RETURN_NOTIMPLEMENTED;
}

// The arguments that the fused steps share, in the order of specdec.py's
// wrappers: ..., W_in, src, dst, tokens, n_acc, bonus, pad_out, w_new, pos, mask.
struct Step {
  int32_t W_in;
  specdec_kv_t src, dst;
  int32_t *tokens, *n_acc, *bonus, *pad_out, *w_new;
  int64_t* pos;
  uint8_t* mask;
  int64_t pm_cap;
  uint32_t* dev_status;
  int32_t *s_in = nullptr, *s_out = nullptr, pad_id;
  int64_t s_in_stride = 0, s_out_stride = 0;
  bool sync;
  int32_t host = -1;
  void* stream;
  Step(const Logits& l, PyObject* const* a, PyObject* dev, PyObject* sync_, PyObject* stream_, PyObject* sin, PyObject* sout,
       PyObject* pad) {
    const int64_t B = l.B;
    W_in = integer(a[0]);
    src = cache(a[1]);
    dst = cache(a[2]);
    need(src.B == l.B);
    tokens = ints(a[3], {B, l.k + 1});
    n_acc = ints(a[4], {B});
    bonus = ints_or_none(a[5], {B});
    pad_out = ints(a[6], {B});
    w_new = ints(a[7], {1});
    pos = rows<int64_t>(a[8], at::kLong, B, &pm_cap);
    mask = dense<uint8_t>(a[9], at::kByte, {B, pm_cap});
    dev_status = status(dev);
    need(PyBool_Check(sync_));
    sync = sync_ == Py_True;
    need((sin == Py_None) == (sout == Py_None));
    if (sin != Py_None) {
      s_in = rows<int32_t>(sin, at::kInt, B, &s_in_stride);
      s_out = rows<int32_t>(sout, at::kInt, B, &s_out_stride);
    }
    pad_id = integer(pad);
    stream = stream_of(stream_);
  }
  PyObject* result(specdec_status_t s) const {
    return sync && s == SPECDEC_OK ? Py_BuildValue("(ii)", static_cast<int>(s), static_cast<int>(host)) : PyLong_FromLong(s);
  }
};

// (logits, draft, pad_in, W_in, src, dst, tokens, n_acc, bonus, pad_out, w_new,
//  pos, mask, workspace or None for the library's scratch, dev_status, sync,
//  stream, s_in, s_out, pad_id)
PyObject* step(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 20, [&] {
    const Logits l = logits_of(a[0]);
    const int32_t* draft = ints(a[1], {l.B, l.k});
    const int32_t* pad_in = ints(a[2], {l.B});
    Step s(l, a + 3, a[14], a[15], a[16], a[17], a[18], a[19]);
    const bool noalloc = a[13] == Py_None;
    const Workspace ws = noalloc ? Workspace{} : workspace(a[13], lib.workspace_bytes(l.B, l.k, l.V));
    int32_t* host = s.sync ? &s.host : nullptr;
    return s.result(unlocked([&] {
      return noalloc ? lib.step_noalloc(l.data, l.dtype, draft, pad_in, l.B, l.k, l.V, s.W_in, &s.src, &s.dst, s.tokens,
                                        s.n_acc, s.bonus, s.pad_out, s.w_new, s.pos, s.mask, s.pm_cap, s.s_in,
                                        s.s_in_stride, s.s_out, s.s_out_stride, s.pad_id, s.dev_status, host, s.stream)
                     : lib.step(l.data, l.dtype, draft, pad_in, l.B, l.k, l.V, s.W_in, &s.src, &s.dst, s.tokens, s.n_acc,
                                s.bonus, s.pad_out, s.w_new, s.pos, s.mask, s.pm_cap, s.s_in, s.s_in_stride, s.s_out,
                                s.s_out_stride, s.pad_id, ws.data, ws.bytes, s.dev_status, host, s.stream);
    }));
  });
}

struct Sampled {
  const void* draft_logits;
  const int32_t *draft, *pad_in;
  const float *u_accept, *u_sample;
  float temperature;
  Sampled(const Logits& l, PyObject* const* a) {
    draft_logits = dense<void>(a[0], l.type, {l.B, l.k, l.V});
    draft = ints(a[1], {l.B, l.k});
    pad_in = ints(a[2], {l.B});
    u_accept = dense<float>(a[3], at::kFloat, {l.B, l.k});
    u_sample = dense<float>(a[4], at::kFloat, {l.B});
    need(PyFloat_CheckExact(a[5]));
    temperature = static_cast<float>(PyFloat_AS_DOUBLE(a[5]));
  }
};

// (logits, draft_logits, draft, pad_in, u_accept, u_sample, temperature, W_in,
//  src, dst, tokens, n_acc, bonus, pad_out, w_new, pos, mask, workspace,
//  dev_status, sync, stream, s_in, s_out, pad_id)
PyObject* step_sample(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 24, [&] {
    const Logits l = logits_of(a[0]);
    const Sampled d(l, a + 1);
    Step s(l, a + 7, a[18], a[19], a[20], a[21], a[22], a[23]);
    const Workspace ws = workspace(a[17], lib.sample_workspace_bytes(l.B, l.k, l.V));
    return s.result(unlocked([&] {
      return lib.step_sample(l.data, d.draft_logits, l.dtype, d.draft, d.pad_in, d.u_accept, d.u_sample, d.temperature, l.B,
                             l.k, l.V, s.W_in, &s.src, &s.dst, s.tokens, s.n_acc, s.bonus, s.pad_out, s.w_new, s.pos,
                             s.mask, s.pm_cap, s.s_in, s.s_in_stride, s.s_out, s.s_out_stride, s.pad_id, ws.data, ws.bytes,
                             s.dev_status, s.sync ? &s.host : nullptr, s.stream);
    }));
  });
}

// (logits, draft, pad_in, W_in, tokens, n_acc, bonus, pad_out, w_new,
//  workspace, dev_status, stream)
PyObject* verify_greedy(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 12, [&] {
    const Logits l = logits_of(a[0]);
    const int64_t B = l.B;
    const int32_t *draft = ints(a[1], {B, l.k}), *pad_in = ints(a[2], {B}), W_in = integer(a[3]);
    int32_t *tokens = ints(a[4], {B, l.k + 1}), *n_acc = ints(a[5], {B}), *bonus = ints_or_none(a[6], {B});
    int32_t *pad_out = ints(a[7], {B}), *w_new = ints(a[8], {1});
    const Workspace ws = workspace(a[9], lib.workspace_bytes(l.B, l.k, l.V));
    uint32_t* dev = status(a[10]);
    void* st = stream_of(a[11]);
    return PyLong_FromLong(unlocked([&] {
      return lib.verify_greedy(l.data, l.dtype, draft, pad_in, l.B, l.k, l.V, W_in, tokens, n_acc, bonus, pad_out, w_new,
                               ws.data, ws.bytes, dev, st);
    }));
  });
}

// (logits, draft_logits, draft, pad_in, u_accept, u_sample, temperature, W_in,
//  tokens, n_acc, bonus, pad_out, w_new, workspace, dev_status, stream)
PyObject* verify_sample(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 16, [&] {
    const Logits l = logits_of(a[0]);
    const int64_t B = l.B;
    const Sampled d(l, a + 1);
    const int32_t W_in = integer(a[7]);
    int32_t *tokens = ints(a[8], {B, l.k + 1}), *n_acc = ints(a[9], {B}), *bonus = ints_or_none(a[10], {B});
    int32_t *pad_out = ints(a[11], {B}), *w_new = ints(a[12], {1});
    const Workspace ws = workspace(a[13], lib.sample_workspace_bytes(l.B, l.k, l.V));
    uint32_t* dev = status(a[14]);
    void* st = stream_of(a[15]);
    return PyLong_FromLong(unlocked([&] {
      return lib.verify_sample(l.data, d.draft_logits, l.dtype, d.draft, d.pad_in, d.u_accept, d.u_sample, d.temperature,
                               l.B, l.k, l.V, W_in, tokens, n_acc, bonus, pad_out, w_new, ws.data, ws.bytes, dev, st);
    }));
  });
}

// (pool, pool_tok, lens, slots, Lb, batch, pads, batch_tok, pos, mask, k,
//  pad_id, dev_status, stream)
PyObject* gather_batch(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 14, [&] {
    const specdec_kv_t pool = cache(a[0]), batch = cache(a[5]);
    const int64_t B = batch.B, N = pool.B;
    const int32_t *lens = ints(a[2], {N}), *slots = ints(a[3], {B}), *pool_tok = nullptr;
    int32_t *pads = ints(a[6], {B}), *batch_tok = nullptr;
    int64_t tok_stride = 0, btok_stride = 0, pm_cap = 0;
    if (a[7] != Py_None) {
      pool_tok = rows<int32_t>(a[1], at::kInt, N, &tok_stride);
      batch_tok = rows<int32_t>(a[7], at::kInt, B, &btok_stride);
    }
    int64_t* pos = nullptr;
    uint8_t* mask = nullptr;
    if (a[8] != Py_None || a[9] != Py_None) {
      pos = rows<int64_t>(a[8], at::kLong, B, &pm_cap);
      mask = dense<uint8_t>(a[9], at::kByte, {B, pm_cap});
    }
    const int32_t Lb = integer(a[4]), k = integer(a[10]), pad_id = integer(a[11]);
    uint32_t* dev = status(a[12]);
    void* st = stream_of(a[13]);
    return PyLong_FromLong(unlocked([&] {
      return lib.gather_batch(&pool, pool_tok, tok_stride, lens, slots, static_cast<int32_t>(B), Lb, k, &batch, batch_tok,
                              btok_stride, pad_id, pads, pos, mask, pm_cap, dev, st);
    }));
  });
}

// (batch, pads, tokens, n_acc, slots, Lb, pool, pool_tok, lens, batch_tok, mode,
//  dev_status, stream)
PyObject* scatter_accepted(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 13, [&] {
    const specdec_kv_t batch = cache(a[0]), pool = cache(a[6]);
    const int64_t B = batch.B;
    int64_t kp1 = 0, tok_stride = 0, btok_stride = 0;
    const int32_t* tokens = rows<int32_t>(a[2], at::kInt, B, &kp1);
    need(kp1 >= 1 && kp1 <= INT32_MAX);
    const int32_t *pads = ints(a[1], {B}), *n_acc = ints(a[3], {B}), *slots = ints(a[4], {B});
    int32_t* lens = ints(a[8], {pool.B});
    int32_t* pool_tok = rows<int32_t>(a[7], at::kInt, pool.B, &tok_stride);
    int32_t* batch_tok = a[9] != Py_None ? rows<int32_t>(a[9], at::kInt, B, &btok_stride) : nullptr;
    const int32_t Lb = integer(a[5]), mode = integer(a[10]);
    uint32_t* dev = status(a[11]);
    void* st = stream_of(a[12]);
    return PyLong_FromLong(unlocked([&] {
      return lib.scatter_accepted(&batch, pads, tokens, n_acc, slots, static_cast<int32_t>(B), static_cast<int32_t>(kp1 - 1),
                                  Lb, &pool, pool_tok, tok_stride, lens, batch_tok, btok_stride, mode, dev, st);
    }));
  });
}

// (src, dst, cu_in, n_acc, k, max_len, cu_out, pos, dev_status, stream)
PyObject* varlen_rollback(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 10, [&] {
    const specdec_varlen_t src = flat_cache(a[0]), dst = flat_cache(a[1]);
    const int64_t B = tensor(a[2]).numel() - 1;
    need(B >= 0 && B <= INT32_MAX);
    const int32_t *cu_in = ints(a[2], {B + 1}), *n_acc = ints(a[3], {B});
    const int32_t k = integer(a[4]), max_len = integer(a[5]);
    int32_t* cu_out = ints(a[6], {B + 1});
    const int64_t pos_cap = a[7] != Py_None ? tensor(a[7]).numel() : 0;
    int64_t* pos = dense_or_none<int64_t>(a[7], at::kLong, {pos_cap});
    uint32_t* dev = status(a[8]);
    void* st = stream_of(a[9]);
    return PyLong_FromLong(unlocked([&] {
      return lib.varlen_rollback(&src, &dst, cu_in, n_acc, static_cast<int32_t>(B), k, max_len, cu_out, pos, pos_cap, dev, st);
    }));
  });
}

// connect(current device, raw stream of a device, {name: address of a library function})
PyObject* connect(PyObject*, PyObject* args) {
  PyObject *dev, *st, *at;
  if (!PyArg_ParseTuple(args, "OOO!", &dev, &st, &PyDict_Type, &at)) return nullptr;
  struct {
    const char* name;
    void** to;
  } const table[] = {
#define SPECDEC_FN(f) {"specdec_" #f, reinterpret_cast<void**>(&lib.f)}
      SPECDEC_FN(workspace_bytes), SPECDEC_FN(sample_workspace_bytes), SPECDEC_FN(verify_greedy), SPECDEC_FN(verify_sample),
      SPECDEC_FN(step), SPECDEC_FN(step_noalloc), SPECDEC_FN(step_sample), SPECDEC_FN(gather_batch),
      SPECDEC_FN(scatter_accepted), SPECDEC_FN(varlen_rollback)
#undef SPECDEC_FN
  };
  for (const auto& f : table) {
    PyObject* v = PyDict_GetItemString(at, f.name);
    void* p = v ? PyLong_AsVoidPtr(v) : nullptr;
    if (PyErr_Occurred()) return nullptr;
    if (!p) {
      PyErr_Format(PyExc_ValueError, "no address of %s", f.name);
      return nullptr;
    }
    *f.to = p;
  }
  Py_INCREF(dev);
  Py_INCREF(st);
  Py_XSETREF(get_device, dev);
  Py_XSETREF(get_stream, st);
  Py_RETURN_NONE;
}

#define FAST(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"connect", connect, METH_VARARGS, nullptr},
                         FAST(step),
                         FAST(step_sample),
                         FAST(verify_greedy),
                         FAST(verify_sample),
                         FAST(gather_batch),
                         FAST(scatter_accepted),
                         FAST(varlen_rollback),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", "Native argument marshalling of specdec.py.", -1, methods};

}  // namespace

// built_for: the torch whose headers were inlined above and the ABI of the
// library's declarations, for specdec.py to compare with what it has loaded.
PyMODINIT_FUNC PyInit__marshal(void) {
  PyObject* m = PyModule_Create(&module);
  PyObject* built_for = m ? Py_BuildValue("(si)", SPECDEC_TORCH_VERSION, SPECDEC_ABI_VERSION) : nullptr;
  if (!built_for || PyModule_AddObject(m, "built_for", built_for) < 0) {
    Py_XDECREF(built_for);
    Py_XDECREF(m);
    return nullptr;
  }
  return m;
}
