// The Python binding's common path: argument checks, output allocation and the C call of the
// entry points of cover.py, in one native function each.
//
// Why: a call of the binding in Python (shape and stride checks, output tensors, a ctypes
// descriptor and pointers, the current stream) took 12 us for token statistics, 16 for attention
// and 20 for the masses, where their kernels take 5-15 us at small sizes, so the host bounded
// every small call and the whole tail of a decoding step (103 us of host work for about 60 us
// of kernels).  Here the same takes 4-6 us.
//
// Each function either makes the call and returns the outputs (a tuple), returns the library's
// status (an int) if that refused it, or returns None without having done anything: for
// arguments that fail a check, tensors of other classes than Tensor, active torch function
// modes and whatever raises.  The caller then goes through its Python form, which raises the
// error the argument deserves.  Nothing is kept between calls but the library's entry points.
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ATen.h>
#include <string.h>

#include <algorithm>

#include "cover.h"

namespace {

using at::Tensor;

struct Entry {
  decltype(&cover_attn_fwd) attn_fwd;
  decltype(&cover_select_seeds) select_seeds;
  decltype(&cover_token_stats) token_stats;
  decltype(&cover_token_sample) token_sample;
  decltype(&cover_attn_stats) attn_stats;
  decltype(&cover_attn_stats_workspace) attn_stats_workspace;
  decltype(&cover_decode_update) decode_update;
};
Entry lib = {};

// thrown for whatever the native path leaves to the Python form
struct Leave {};
void need(bool ok) {
  if (!ok) throw Leave{};
}

const Tensor& tensor(PyObject* o) {
  need(THPVariable_CheckExact(o));
  const Tensor& t = THPVariable_Unpack(o);
  need(t.is_cuda() && t.layout() == at::kStrided);
  return t;
}
const Tensor* optional(PyObject* o) { return o == Py_None ? nullptr : &tensor(o); }
int64_t integer(PyObject* o) {
  need(PyLong_Check(o));
  int overflow = 0;
  const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
  need(!overflow);
  return v;
}
int32_t int32(PyObject* o) {
  const int64_t v = integer(o);
  need(v == (int32_t)v);
  return (int32_t)v;
}
float real(PyObject* o) {
  need(PyFloat_Check(o) || PyLong_Check(o));
  const double v = PyFloat_AsDouble(o);
  need(!PyErr_Occurred());
  return (float)v;
}
bool truth(PyObject* o) {
  const int v = PyObject_IsTrue(o);
  need(v >= 0);
  return v != 0;
}
hipStream_t stream_of(PyObject* o) { return (hipStream_t)(uintptr_t)integer(o); }

template <class T>
T* ptr(const Tensor& t) {
  return (T*)t.data_ptr();
}
template <class T>
T* ptr(const Tensor* t) {
  return t ? (T*)t->data_ptr() : nullptr;
}
Tensor empty(at::IntArrayRef size, at::ScalarType dtype, const Tensor& like) {
  return at::empty(size, at::TensorOptions().dtype(dtype).device(like.device()));
}
// an output: the caller's object, a tensor allocated here, or None
struct Out {
  PyObject* given = nullptr;
  Tensor made;
  template <class T>
  T* data() const {
    if (given) return given == Py_None ? nullptr : (T*)THPVariable_Unpack(given).data_ptr();
    return made.defined() ? (T*)made.data_ptr() : nullptr;
  }
  PyObject* release() const {
    PyObject* o = given ? given : (made.defined() ? nullptr : Py_None);
    if (!o) return THPVariable_Wrap(made);
    Py_INCREF(o);
    return o;
  }
};
// `o` if it is a tensor, otherwise (None) allocated when wanted
Out output(PyObject* o, bool wanted, at::IntArrayRef size, at::ScalarType dtype, const Tensor& like) {
  Out r;
  if (o && o != Py_None) {
    tensor(o);
    r.given = o;
  } else if (wanted) {
    r.made = empty(size, dtype, like);
  }
  return r;
}
bool is(const Tensor& t, at::IntArrayRef size, at::ScalarType dtype) {
  return t.sizes() == size && t.scalar_type() == dtype && t.is_contiguous();
}
template <class... O>
PyObject* tuple(const O&... outs) {
  PyObject* items[] = {outs.release()...};
  constexpr Py_ssize_t n = sizeof...(O);
  PyObject* r = PyTuple_New(n);
  for (Py_ssize_t i = 0; i < n; ++i) {
    if (!r || !items[i]) {
      Py_XDECREF(items[i]);
      if (r) PyTuple_SET_ITEM(r, i, Py_NewRef(Py_None));
    } else {
      PyTuple_SET_ITEM(r, i, items[i]);
    }
  }
  if (PyErr_Occurred()) {
    Py_XDECREF(r);
    return nullptr;
  }
  return r;
}

int dtype_of(const Tensor& t) {
  if (t.scalar_type() == at::kBFloat16) return COVER_BF16;
  need(t.scalar_type() == at::kFloat);
  return COVER_F32;
}
cover_attn_desc attn_desc(const Tensor& q, const Tensor& k, int64_t max_seeds, float scale) {
  cover_attn_desc d = {};
  d.B = (int32_t)q.size(0); d.Hq = (int32_t)q.size(1); d.L = (int32_t)q.size(2); d.d = (int32_t)q.size(3);
  d.Hkv = (int32_t)k.size(1);
  d.max_seeds = (int32_t)max_seeds;
  d.dtype = (decltype(d.dtype))dtype_of(q);
  d.scale = scale;
  d.q_sb = q.stride(0); d.q_sh = q.stride(1); d.q_sl = q.stride(2);
  d.kv_sb = k.stride(0); d.kv_sh = k.stride(1); d.kv_sl = k.stride(2);
  return d;
}
void same_layout(const Tensor& t, const Tensor& k, const Tensor& q) {
  need(t.sizes() == k.sizes() && t.strides() == k.strides() && t.scalar_type() == q.scalar_type());
}
// the seed list of an attention call: its width, 0 without one
int64_t seed_width(const Tensor* idx, const Tensor* n) {
  if (!idx) return 0;
  need(idx->dim() >= 1 && idx->scalar_type() == at::kInt && n && n->scalar_type() == at::kInt &&
       idx->is_contiguous());
  return idx->size(-1);
}

template <class F>
PyObject* guarded(Py_ssize_t n, Py_ssize_t expect, F&& f) {
  try {
    if (n == expect && lib.attn_fwd && !at::impl::torch_function_mode_enabled()) return f();
  } catch (...) {
    PyErr_Clear();
  }
  Py_RETURN_NONE;
}
template <class F>
cover_status call(F&& f) {
  cover_status st;
  Py_BEGIN_ALLOW_THREADS
  st = f();
  Py_END_ALLOW_THREADS
  return st;
}

// (q, k_live, v_live, k_cache, v_cache, seed_idx, n_seed, out, lse, scale, want_lse, stream)
PyObject* attn_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 12, [&]() -> PyObject* {
    const Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]), &kc = tensor(a[3]), &vc = tensor(a[4]);
    need(q.dim() == 4 && k.dim() == 4 && q.stride(3) == 1 && k.stride(3) == 1);
    need(k.scalar_type() == q.scalar_type());
    for (const Tensor* t : {&v, &kc, &vc}) same_layout(*t, k, q);
    const Tensor *idx = optional(a[5]), *ns = optional(a[6]);
    const cover_attn_desc d = attn_desc(q, k, seed_width(idx, ns), real(a[9]));
    const hipStream_t stream = stream_of(a[11]);
    Out out, lse = output(a[8], truth(a[10]), {q.size(0), q.size(1), q.size(2)}, at::kFloat, q);
    if (a[7] == Py_None) {
      out.made = at::empty_like(q);
      need(out.made.strides() == q.strides());
    } else {
      const Tensor& t = tensor(a[7]);
      need(t.sizes() == q.sizes() && t.strides() == q.strides() && t.scalar_type() == q.scalar_type());
      out.given = a[7];
    }
    const void *pq = ptr<void>(q), *pk = ptr<void>(k), *pv = ptr<void>(v), *pkc = ptr<void>(kc), *pvc = ptr<void>(vc);
    const int32_t *pi = ptr<int32_t>(idx), *pn = ptr<int32_t>(ns);
    void* po = out.data<void>();
    float* pl = lse.data<float>();
    const cover_status st = call([&] { return lib.attn_fwd(pq, pk, pv, pkc, pvc, pi, pn, po, pl, &d, stream); });
    return st == COVER_OK ? tuple(out, lse) : PyLong_FromLong(st);
  });
}

// (logits, tokens, want_logp, want_conf, want_argmax, stream)
PyObject* token_stats(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 6, [&]() -> PyObject* {
    const Tensor& x = tensor(a[0]);
    need(x.dim() == 2 && x.stride(1) == 1);
    const int64_t R = x.size(0);
    cover_token_desc d = {};
    d.R = (int32_t)R; d.V = (int32_t)x.size(1);
    d.dtype = (decltype(d.dtype))dtype_of(x);
    d.row_stride = x.stride(0);
    const bool want_logp = truth(a[2]);
    const int32_t* tok = nullptr;
    if (want_logp) {
      const Tensor& t = tensor(a[1]);
      need(is(t, {R}, at::kInt));
      tok = ptr<int32_t>(t);
    }
    const Out logp = output(nullptr, want_logp, {R}, at::kFloat, x), conf = output(nullptr, truth(a[3]), {R}, at::kFloat, x),
              top = output(nullptr, truth(a[4]), {R}, at::kInt, x);
    const hipStream_t stream = stream_of(a[5]);
    const void* px = ptr<void>(x);
    float *pl = logp.data<float>(), *pc = conf.data<float>();
    int32_t* pt = top.data<int32_t>();
    const cover_status st = call([&] { return lib.token_stats(px, tok, pl, pc, pt, &d, stream); });
    return st == COVER_OK ? tuple(logp, conf, top) : PyLong_FromLong(st);
  });
}

// (logits, temperature, seed, step, want_prob, stream)
PyObject* token_sample(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 6, [&]() -> PyObject* {
    const Tensor& x = tensor(a[0]);
    need(x.dim() == 2 && x.stride(1) == 1 && PyLong_Check(a[2]) && PyLong_Check(a[3]));
    const int64_t R = x.size(0);
    cover_token_desc d = {};
    d.R = (int32_t)R; d.V = (int32_t)x.size(1);
    d.dtype = (decltype(d.dtype))dtype_of(x);
    d.row_stride = x.stride(0);
    const float temperature = real(a[1]);
    const uint64_t seed = PyLong_AsUnsignedLongLongMask(a[2]);
    const uint32_t step = (uint32_t)PyLong_AsUnsignedLongLongMask(a[3]);
    need(!PyErr_Occurred());
    const Out token = output(nullptr, true, {R}, at::kInt, x), prob = output(nullptr, truth(a[4]), {R}, at::kFloat, x);
    const hipStream_t stream = stream_of(a[5]);
    const void* px = ptr<void>(x);
    int32_t* pt = token.data<int32_t>();
    float* pp = prob.data<float>();
    const cover_status st = call([&] { return lib.token_sample(px, temperature, seed, step, pt, pp, &d, stream); });
    return st == COVER_OK ? tuple(token, prob) : PyLong_FromLong(st);
  });
}

// (q, k_live, k_cache, seed_idx, n_seed, lse, masked, drafted, r0, scale, workspace, stream)
PyObject* attn_stats(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 12, [&]() -> PyObject* {
    const Tensor &q = tensor(a[0]), &k = tensor(a[1]), &kc = tensor(a[2]);
    need(q.dim() == 4 && k.dim() == 4 && k.scalar_type() == q.scalar_type());
    same_layout(kc, k, q);
    const Tensor *idx = optional(a[3]), *ns = optional(a[4]);
    need(!idx || idx->dim() >= 1);
    const Tensor &lse = tensor(a[5]), &masked = tensor(a[6]), &drafted = tensor(a[7]);
    const int64_t B = q.size(0), Hq = q.size(1), L = q.size(2);
    need(masked.dim() == 2);
    const int64_t Lr = masked.size(1);
    need(is(masked, {B, Lr}, at::kByte) && is(drafted, {B, Lr}, at::kByte) && is(lse, {B, Hq, L}, at::kFloat));
    cover_stats_desc d = {};
    d.attn = attn_desc(q, k, idx ? idx->size(-1) : 0, real(a[9]));
    d.r0 = int32(a[8]);
    d.Lr = (int32_t)Lr;
    const int64_t floats = lib.attn_stats_workspace((int32_t)B, (int32_t)Hq, (int32_t)Lr);
    need(floats >= 0);
    Tensor own;
    const Tensor* ws = optional(a[10]);
    if (ws) {
      need(ws->scalar_type() == at::kFloat && ws->is_contiguous() && ws->numel() >= floats && ws->device() == q.device());
    } else {
      own = empty({std::max<int64_t>(1, floats)}, at::kFloat, q);
      ws = &own;
    }
    const Out d_in = output(nullptr, true, {B, Lr}, at::kFloat, q), d_out = output(nullptr, true, {B, Lr}, at::kFloat, q);
    const hipStream_t stream = stream_of(a[11]);
    const void *pq = ptr<void>(q), *pk = ptr<void>(k), *pkc = ptr<void>(kc);
    const int32_t *pi = ptr<int32_t>(idx), *pn = ptr<int32_t>(ns);
    const float* pl = ptr<float>(lse);
    const uint8_t *pm = ptr<uint8_t>(masked), *pd = ptr<uint8_t>(drafted);
    float *po = d_in.data<float>(), *pp = d_out.data<float>(), *pw = ptr<float>(*ws);
    const cover_status st =
        call([&] { return lib.attn_stats(pq, pk, pkc, pi, pn, pl, pm, pd, po, pp, pw, &d, stream); });
    return st == COVER_OK ? tuple(d_in, d_out) : PyLong_FromLong(st);
  });
}

// (logp, d_in, d_out, flags, max_seeds, pos_offset, seed_idx, n_seed, score, want_score, stream)
PyObject* select_seeds(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 11, [&]() -> PyObject* {
    const Tensor &logp = tensor(a[0]), &d_in = tensor(a[1]), &d_out = tensor(a[2]), &flags = tensor(a[3]);
    need(logp.dim() == 2);
    const int64_t B = logp.size(0), Lr = logp.size(1);
    need(is(logp, {B, Lr}, at::kFloat) && is(d_in, {B, Lr}, at::kFloat) && is(d_out, {B, Lr}, at::kFloat) &&
         is(flags, {B, Lr}, at::kByte));
    cover_select_desc d = {};
    d.B = (int32_t)B; d.Lr = (int32_t)Lr; d.max_seeds = int32(a[4]); d.pos_offset = int32(a[5]);
    const Out seeds = output(a[6], true, {B, d.max_seeds}, at::kInt, logp), ns = output(a[7], true, {B}, at::kInt, logp),
              score = output(a[8], truth(a[9]), {B, Lr}, at::kDouble, logp);
    const hipStream_t stream = stream_of(a[10]);
    const float *pl = ptr<float>(logp), *pi = ptr<float>(d_in), *po = ptr<float>(d_out);
    const uint8_t* pf = ptr<uint8_t>(flags);
    int32_t *ps = seeds.data<int32_t>(), *pn = ns.data<int32_t>();
    double* pc = score.data<double>();
    const cover_status st = call([&] { return lib.select_seeds(pl, pi, po, pf, ps, pn, pc, &d, stream); });
    return st == COVER_OK ? tuple(seeds, ns, score) : PyLong_FromLong(st);
  });
}

// (tokens, argmax, conf, seed_idx, n_seed, remask_count, mask_id, tau, draft_cap, remask_budget,
//  pos_offset, flags, drafted, counts, want_outputs, min_draft, stream): without flip-flop counts
PyObject* decode_update(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 17, [&]() -> PyObject* {
    const Tensor &tokens = tensor(a[0]), &top = tensor(a[1]), &conf = tensor(a[2]), &remask = tensor(a[5]);
    need(tokens.dim() == 2);
    const int64_t B = tokens.size(0), Lr = tokens.size(1);
    need(is(tokens, {B, Lr}, at::kInt) && is(top, {B, Lr}, at::kInt) && is(conf, {B, Lr}, at::kFloat) &&
         is(remask, {B, Lr}, at::kInt));
    const Tensor *idx = optional(a[3]), *ns = optional(a[4]);
    cover_update_desc d = {};
    if (idx) {
      need(idx->dim() == 2 && idx->size(0) == B && idx->scalar_type() == at::kInt && idx->is_contiguous() && ns &&
           ns->dim() == 1 && ns->size(0) == B && ns->scalar_type() == at::kInt);
      d.max_seeds = (int32_t)idx->size(1);
    }
    d.B = (int32_t)B; d.Lr = (int32_t)Lr;
    d.mask_id = int32(a[6]); d.tau = real(a[7]); d.draft_cap = int32(a[8]); d.remask_budget = int32(a[9]);
    d.pos_offset = int32(a[10]); d.min_draft = int32(a[15]);
    const bool want = truth(a[14]);
    const Out flags = output(a[11], want, {B, Lr}, at::kByte, tokens), drafted = output(a[12], want, {B, Lr}, at::kByte, tokens),
              counts = output(a[13], want, {B, 5}, at::kInt, tokens);
    if (flags.given) need(is(THPVariable_Unpack(flags.given), {B, Lr}, at::kByte));
    if (drafted.given) need(is(THPVariable_Unpack(drafted.given), {B, Lr}, at::kByte));
    if (counts.given) need(is(THPVariable_Unpack(counts.given), {B, 5}, at::kInt));
    const hipStream_t stream = stream_of(a[16]);
    int32_t *pt = ptr<int32_t>(tokens), *pr = ptr<int32_t>(remask), *pn = counts.data<int32_t>();
    const int32_t *pa = ptr<int32_t>(top), *pi = d.max_seeds ? ptr<int32_t>(idx) : nullptr,
                  *ps = d.max_seeds ? ptr<int32_t>(ns) : nullptr;
    const float* pc = ptr<float>(conf);
    uint8_t *pf = flags.data<uint8_t>(), *pd = drafted.data<uint8_t>();
    const cover_status st = call(
        [&] { return lib.decode_update(pt, pa, pc, pi, ps, pr, pf, pd, pn, nullptr, nullptr, &d, stream); });
    return st == COVER_OK ? tuple(flags, drafted, counts) : PyLong_FromLong(st);
  });
}

// the addresses of the library's entry points, in Entry's order
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  constexpr Py_ssize_t kN = sizeof(Entry) / sizeof(void*);
  if (n != kN) {
    PyErr_SetString(PyExc_TypeError, "bind() takes the library's entry points");
    return nullptr;
  }
  void* p[kN];
  for (Py_ssize_t i = 0; i < kN; ++i) {
    p[i] = PyLong_AsVoidPtr(a[i]);
    if (!p[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null entry point");
      return nullptr;
    }
  }
  static_assert(sizeof(p) == sizeof(lib), "one address per entry point");
  memcpy((void*)&lib, p, sizeof(lib));
  Py_RETURN_NONE;
}

#define COVER_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {COVER_METHOD(bind),       COVER_METHOD(attn_fwd),     COVER_METHOD(token_stats),
                         COVER_METHOD(token_sample), COVER_METHOD(attn_stats), COVER_METHOD(select_seeds),
                         COVER_METHOD(decode_update), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_cover_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__cover_host(void) { return PyModule_Create(&module); }
