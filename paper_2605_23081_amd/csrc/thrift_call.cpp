// Python entry of the calls a serving loop makes for every token or prompt: checks the tensors, allocates what the caller
// left out and calls the C ABI, without a Python object per pointer and shape (ctypes: 20 us of host time for a decode
// call, as long as its kernels take on a short cache; here 2 us).
//
// Every function returns the result, or the C call's status as an int when it is not THRIFT_OK, or None when the
// arguments are not of the plain kind that is served here; the caller then takes its general path, which names what is
// wrong with them.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <initializer_list>

#include "thrift.h"

namespace {

using at::Tensor;

bool tensor(PyObject* o, const Tensor** t) {
  if (!THPVariable_Check(o)) return false;
  *t = &THPVariable_Unpack(o);
  return (*t)->is_cuda() && (*t)->is_contiguous();
}
bool optional(PyObject* o, const Tensor** t) {
  if (o == Py_None) { *t = nullptr; return true; }
  return tensor(o, t);
}
bool is(const Tensor& t, at::ScalarType dt, std::initializer_list<int64_t> shape) {
  return t.scalar_type() == dt && t.sizes() == at::IntArrayRef(shape.begin(), shape.size());
}
bool dtype16(const Tensor& t, thrift_dtype* dt) {
  if (t.scalar_type() == at::kHalf) *dt = THRIFT_F16;
  else if (t.scalar_type() == at::kBFloat16) *dt = THRIFT_BF16;
  else return false;
  return true;
}
bool dtype_out(const Tensor& t, thrift_dtype* dt) {
  if (t.scalar_type() == at::kFloat) { *dt = THRIFT_F32; return true; }
  return dtype16(t, dt);
}
// small sizes only: what does not fit an int takes the general path
bool integer(PyObject* o, int* x) {
  int overflow = 0;
  const long v = PyLong_Check(o) ? PyLong_AsLongAndOverflow(o, &overflow) : (overflow = 1, 0);
  *x = (int)v;
  return overflow == 0 && v == (long)*x;
}
bool real(PyObject* o, double* x) {
  if (PyFloat_Check(o)) { *x = PyFloat_AS_DOUBLE(o); return true; }
  if (!PyLong_Check(o)) return false;
  *x = PyLong_AsDouble(o);
  if (*x == -1.0 && PyErr_Occurred()) { PyErr_Clear(); return false; }
  return true;
}
bool stream_of(PyObject* o, void** s) {
  *s = PyLong_AsVoidPtr(o);
  if (*s == nullptr && PyErr_Occurred()) { PyErr_Clear(); return false; }
  return true;
}
void* ptr(const Tensor* t) { return t ? t->data_ptr() : nullptr; }
template <typename P>
P* ptr_as(const Tensor* t) { return static_cast<P*>(ptr(t)); }

PyObject* answer(thrift_status s, const Tensor& out) {
  if (s != THRIFT_OK) return PyLong_FromLong((long)s);
  return THPVariable_Wrap(out);
}
// The interpreter lock, given up while this lives; also taken back when an exception passes (a tensor without storage has no
// data pointer).
struct Unlocked {
  PyThreadState* state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};
Tensor bytes_like(const Tensor& t, size_t n) { return at::empty({(int64_t)std::max<size_t>(n, 256)}, t.options().dtype(at::kByte)); }

// the tensors of a cache: k16 v16 k4 ks v4 vs kmean
struct Cache {
  const Tensor *k16, *v16, *k4, *ks, *v4, *vs, *kmean;
  thrift_dtype dt;
  int B, Hkv, N, D;
};
bool cache(PyObject* const* a, int Bk, Cache* c) {
  if (!tensor(a[0], &c->k16) || !tensor(a[1], &c->v16) || !tensor(a[2], &c->k4) || !tensor(a[3], &c->ks) || !tensor(a[4], &c->v4) ||
      !tensor(a[5], &c->vs) || !tensor(a[6], &c->kmean) || !dtype16(*c->k16, &c->dt) || c->k16->dim() != 4 || Bk <= 0)
    return false;
  const auto s = c->k16->sizes();
  for (int i = 0; i < 4; ++i) if (s[i] > 0x7fffffff) return false;
  const int64_t B = s[0], H = s[1], N = s[2], D = s[3];
  c->B = (int)B; c->Hkv = (int)H; c->N = (int)N; c->D = (int)D;
  return is(*c->v16, c->k16->scalar_type(), {B, H, N, D}) && is(*c->k4, at::kByte, {B, H, N, D / 2}) && is(*c->ks, at::kByte, {B, H, N, D / 32}) &&
         is(*c->v4, at::kByte, {B, H, N / 64, D, 32}) && is(*c->vs, at::kByte, {B, H, N / 32, D}) && is(*c->kmean, at::kFloat, {B, H, N / Bk, D});
}

// decode(q, k16, v16, k4, ks, v4, vs, kmean, Bk, budget, fixed_k, split_blocks, scale, seqlens, out, workspace, shared, stream)
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n) {
  const Tensor *q, *seqlens, *out_given, *ws_given;
  Cache c;
  int Bk, fixed_k, split, shared;
  double budget, scale;
  void* stream;
  thrift_dtype odt;
  if (n != 18 || !tensor(a[0], &q) || !integer(a[8], &Bk) || !cache(a + 1, Bk, &c) || !real(a[9], &budget) || !integer(a[10], &fixed_k) ||
      !integer(a[11], &split) || !real(a[12], &scale) || !optional(a[13], &seqlens) || !optional(a[14], &out_given) ||
      !optional(a[15], &ws_given) || !integer(a[16], &shared) || !stream_of(a[17], &stream) || q->dim() != 3 || q->size(1) > 0x7fffffff)
    Py_RETURN_NONE;
  const int Hq = (int)q->size(1);
  if (!is(*q, c.k16->scalar_type(), {c.B, Hq, c.D}) || (seqlens && !is(*seqlens, at::kInt, {c.B})) ||
      (out_given && !is(*out_given, out_given->scalar_type(), {c.B, Hq, c.D})))
    Py_RETURN_NONE;
  const Tensor out = out_given ? *out_given : at::empty({c.B, Hq, c.D}, q->options());
  if (!dtype_out(out, &odt)) Py_RETURN_NONE;
  const Tensor ws = ws_given ? *ws_given : bytes_like(*q, thrift_attn_decode_workspace(c.B, Hq, c.Hkv, c.N, c.D, Bk, split));
  const size_t ws_bytes = (size_t)ws.numel();
  thrift_status s;
  {
    const Unlocked unlocked;
    s = (shared ? thrift_attn_decode_shared : thrift_attn_decode)(
        ptr(q), c.dt, ptr(c.k16), ptr(c.v16), ptr_as<uint8_t>(c.k4), ptr_as<uint8_t>(c.ks), ptr_as<uint8_t>(c.v4), ptr_as<uint8_t>(c.vs),
        ptr_as<float>(c.kmean), ptr_as<int32_t>(seqlens), c.B, Hq, c.Hkv, c.N, c.D, Bk, budget, fixed_k, split, (float)scale,
        out.data_ptr(), odt, nullptr, nullptr, 0, ws.data_ptr(), ws_bytes, stream);
  }
  return answer(s, out);
}

// append(k_new, v_new, seqlens, new_lens, k16, v16, k4, ks, v4, vs, kmean, Bk, stream): the lengths after the call
PyObject* append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  const Tensor *k_new, *v_new, *seqlens, *new_lens;
  Cache c;
  int Bk;
  void* stream;
  if (n != 13 || !tensor(a[0], &k_new) || !tensor(a[1], &v_new) || !tensor(a[2], &seqlens) || !optional(a[3], &new_lens) ||
      !integer(a[11], &Bk) || !cache(a + 4, Bk, &c) || !stream_of(a[12], &stream) || k_new->dim() != 4 || k_new->size(2) > 0x7fffffff)
    Py_RETURN_NONE;
  const int n_new = (int)k_new->size(2);
  const auto st = c.k16->scalar_type();
  if (!is(*k_new, st, {c.B, c.Hkv, n_new, c.D}) || !is(*v_new, st, {c.B, c.Hkv, n_new, c.D}) || !is(*seqlens, at::kInt, {c.B}) ||
      (new_lens && !is(*new_lens, at::kInt, {c.B})))
    Py_RETURN_NONE;
  const Tensor after = at::empty({c.B}, seqlens->options());
  thrift_status s;
  {
    const Unlocked unlocked;
    s = thrift_kv_cache_append_advance(ptr(k_new), ptr(v_new), c.dt, n_new, ptr_as<int32_t>(seqlens), ptr_as<int32_t>(new_lens),
                                       after.data_ptr<int32_t>(), ptr(c.k16), ptr(c.v16), ptr_as<uint8_t>(c.k4), ptr_as<uint8_t>(c.ks),
                                       ptr_as<uint8_t>(c.v4), ptr_as<uint8_t>(c.vs), ptr_as<float>(c.kmean), c.B, c.Hkv, c.N, c.D, Bk, stream);
  }
  return answer(s, after);
}

// attention(q, k, v, causal, Bq, Bk, budget, fixed_k, scale, workspace, out, lse, tile_order, stream)
PyObject* attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
  const Tensor *q, *k, *v, *ws_given, *out_given, *lse;
  int causal, Bq, Bk, fixed_k, order;
  double budget, scale;
  void* stream;
  thrift_dtype dt, odt;
  if (n != 14 || !tensor(a[0], &q) || !tensor(a[1], &k) || !tensor(a[2], &v) || !integer(a[3], &causal) || !integer(a[4], &Bq) ||
      !integer(a[5], &Bk) || !real(a[6], &budget) || !integer(a[7], &fixed_k) || !real(a[8], &scale) || !optional(a[9], &ws_given) ||
      !optional(a[10], &out_given) || !optional(a[11], &lse) || !integer(a[12], &order) || !stream_of(a[13], &stream) ||
      !dtype16(*q, &dt) || q->dim() != 4 || k->dim() != 4)
    Py_RETURN_NONE;
  const auto s = q->sizes();
  const int64_t Hkv = k->size(1);
  for (int i = 0; i < 4; ++i) if (s[i] > 0x7fffffff || k->size(i) > 0x7fffffff) Py_RETURN_NONE;
  if (!is(*k, q->scalar_type(), {s[0], Hkv, s[2], s[3]}) || !is(*v, q->scalar_type(), {s[0], Hkv, s[2], s[3]})) Py_RETURN_NONE;
  // what the C call would write past, were it of another shape or type, takes the general path
  if ((out_given && !is(*out_given, out_given->scalar_type(), {s[0], s[1], s[2], s[3]})) || (lse && !is(*lse, at::kFloat, {s[0], s[1], s[2]})) ||
      (ws_given && ws_given->scalar_type() != at::kByte))
    Py_RETURN_NONE;
  const Tensor out = out_given ? *out_given : at::empty(s, q->options());
  if (!dtype_out(out, &odt)) Py_RETURN_NONE;
  const int B = (int)s[0], Hq = (int)s[1], N = (int)s[2], D = (int)s[3];
  const Tensor ws = ws_given ? *ws_given
                             : bytes_like(*q, thrift_attention_forward_workspace(B, Hq, (int)Hkv, N, D, Bq, Bk, causal, budget, fixed_k));
  const size_t ws_bytes = (size_t)ws.numel();
  thrift_status st;
  {
    const Unlocked unlocked;
    st = thrift_attention_forward(ptr(q), ptr(k), ptr(v), dt, B, Hq, (int)Hkv, N, D, Bq, Bk, causal, budget, fixed_k, order, (float)scale,
                                  out.data_ptr(), odt, ptr_as<float>(lse), ws.data_ptr(), ws_bytes, stream);
  }
  return answer(st, out);
}

// A tensor whose sizes or storage cannot be asked for (a fake one, one under a transform) throws: not a plain argument.
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  try {
    return F(self, a, n);
  } catch (const std::exception&) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

PyMethodDef methods[] = {
    {"decode", (PyCFunction)(void (*)(void))guarded<decode>, METH_FASTCALL, nullptr},
    {"append", (PyCFunction)(void (*)(void))guarded<append>, METH_FASTCALL, nullptr},
    {"attention", (PyCFunction)(void (*)(void))guarded<attention>, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call(void) { return PyModule_Create(&module); }
