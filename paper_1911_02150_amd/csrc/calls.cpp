// The calls of a decoding loop from Python without the interpreter's share of them: checks of the tensors, their addresses,
// the current stream and the call into libmqa_decode.so in one native function each (a CPython extension over torch's own tensor
// type).  They take what the binding's general path takes in its plainest form only, torch tensors on the current GPU, contiguous, of the
// right types and shapes, with no mode of torch active; for anything else they return None, nothing has happened, and the general path accepts it or says
// what is wrong.
// Measured (us a call among others, general path through ctypes / here; GPU alone, from a graph): one attention 7.1 / 4.5 (4.3), a layer's
// three calls 21.7 / 17.3 (16.9), a memory and its step 15.3 / 9.4 (9.0), a beam step and its reorder 18.8 / 12.7 (11.5).  The launch
// itself is 3.2 of a call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/mqa.h"

namespace {

// Addresses of the library's functions (binding.py loads the library and hands them over), and the error to raise.
struct Functions {
  decltype(&mqa_decode_step) mqa_decode, mha_decode;
  decltype(&mqa_decode_step_window) mqa_window, mha_window;
  decltype(&mqa_project_append_qkv) append_qkv;
  decltype(&mqa_project_qkvo_ex) project;
  decltype(&mqa_project_add_layernorm) add_layernorm;
  decltype(&mqa_project_memory_kv) memory_kv;
  decltype(&mqa_project_memory_kv_ws) memory_kv_ws;
  decltype(&mqa_memory_decode_step) memory_decode;
  decltype(&mqa_decode_step_beams) beams;
  decltype(&mqa_beam_reorder_kv) reorder;
  decltype(&mqa_prefill_attention) mqa_prefill, mha_prefill;
} fn;
PyObject* error_class = nullptr;
PyObject* parameter_class = nullptr;

const uint64_t kPlainKeys = (c10::DispatchKeySet(c10::DispatchKey::CUDA) | c10::DispatchKeySet(c10::DispatchKey::AutogradCUDA) |
                             c10::DispatchKeySet(c10::DispatchKey::ADInplaceOrView) | c10::DispatchKeySet(c10::DispatchKey::AutocastCUDA)).raw_repr();

// Nobody looks on: the output is made without a word to a function mode or a dispatch mode.
bool no_modes() { return !at::impl::torch_function_mode_enabled() && !c10::impl::TorchDispatchModeTLS::any_modes_set(); }

thread_local c10::DeviceIndex device = 0;      // the current one, of a call

// A tensor that is no more than memory on that GPU (no subclass, no wrapper of a transform), contiguous, of this type; else null.
const at::Tensor* plain(PyObject* o) {
  if (reinterpret_cast<PyObject*>(Py_TYPE(o)) != THPVariableClass && reinterpret_cast<PyObject*>(Py_TYPE(o)) != parameter_class) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || (t.unsafeGetTensorImpl()->key_set().raw_repr() & ~kPlainKeys) || !t.is_cuda() || t.device().index() != device || !t.is_contiguous()) return nullptr;
  return &t;
}
const at::Tensor* plain(PyObject* o, at::ScalarType type) {
  const at::Tensor* t = plain(o);
  return t && t->scalar_type() == type ? t : nullptr;
}
const at::Tensor* f32(PyObject* o) { return plain(o, at::kFloat); }
const at::Tensor* i32(PyObject* o) { return plain(o, at::kInt); }

bool shape_is(const at::Tensor& t, std::initializer_list<int64_t> s) { return t.sizes() == at::IntArrayRef(s); }
bool fits(const at::Tensor& t) {               // sizes as the library's ints
  for (int64_t s : t.sizes())
    if (s > INT32_MAX) return false;
  return true;
}
int cache_type(const at::Tensor& K) { return K.scalar_type() == at::kBFloat16 ? MQA_BF16 : K.scalar_type() == at::kFloat ? MQA_F32 : -1; }
size_t bytes_of(const at::Tensor& t) { return (size_t)t.numel() * t.element_size(); }
void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }      // (of the current device)

template <typename T> T* at_of(const at::Tensor* t) { return t ? static_cast<T*>(t->data_ptr()) : nullptr; }

// The output: the caller's, or a new one of this shape like `like`.  Returns a new reference, or null.
PyObject* output(PyObject* given, const at::Tensor& like, std::initializer_list<int64_t> shape, const at::Tensor** t, at::Tensor* own) {
  if (given == Py_None) {
    *own = at::empty(at::IntArrayRef(shape), like.options().requires_grad(false));
    *t = own;
    return THPVariable_Wrap(*own);
  }
  *t = f32(given);
  if (!*t || !shape_is(**t, shape)) return nullptr;
  Py_INCREF(given);
  return given;
}

PyObject* result(int status, const char* name, PyObject* value) {
  if (status == MQA_OK) return value;
  Py_DECREF(value);
  PyObject* e = PyObject_CallFunction(error_class, "si", name, status);
  if (e) {
    PyErr_SetObject(error_class, e);
    Py_DECREF(e);
  }
  return nullptr;
}

struct Held {                                  // a reference that goes with an exception
  PyObject* p;
  ~Held() { Py_XDECREF(p); }
  PyObject* take() { PyObject* const q = p; p = nullptr; return q; }
};

#define NOT_HERE return PyErr_Occurred() ? nullptr : (Py_INCREF(Py_None), Py_None)
// C++ exceptions (an allocation that fails, memory that a tensor does not have) stay here: the general path meets them again
#define MQA_CALL(NAME, COUNT)                                                             \
  PyObject* NAME##_body(PyObject* const* a);                                              \
  PyObject* NAME(PyObject*, PyObject* const* a, Py_ssize_t n) {                           \
    if (n != COUNT) { PyErr_SetString(PyExc_TypeError, #NAME ": " #COUNT " arguments"); return nullptr; } \
    try { if (!no_modes()) NOT_HERE; device = c10::hip::current_device(); return NAME##_body(a); } catch (const std::exception&) { NOT_HERE; }            \
  }                                                                                       \
  PyObject* NAME##_body(PyObject* const* a)
#define WITHOUT_GIL(EXPR) [&] { int rc_; Py_BEGIN_ALLOW_THREADS rc_ = (EXPR); Py_END_ALLOW_THREADS return rc_; }()

bool number(PyObject* o, float* x) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) { PyErr_Clear(); return false; }
  *x = (float)v;
  return true;
}
bool integer(PyObject* o, int* x) {
  if (!PyLong_Check(o)) return false;
  const long v = PyLong_AsLong(o);
  if ((v == -1 && PyErr_Occurred()) || v < INT32_MIN || v > INT32_MAX) { PyErr_Clear(); return false; }
  *x = (int)v;
  return true;
}

// (multi_head, q, K, V, lens, o, scale, workspace, window or None)
MQA_CALL(decode, 9) {
  const bool mh = a[0] == Py_True;
  const at::Tensor *q = f32(a[1]), *K = plain(a[2]), *V = plain(a[3]), *lens = i32(a[4]), *ws = plain(a[7]), *o;
  float scale;
  int window = 0;
  if (!q || !K || !V || !lens || !ws || q->dim() != 3 || V->dim() < 2 || !number(a[6], &scale) || (a[8] != Py_None && !integer(a[8], &window))) NOT_HERE;
  const int64_t b = q->size(0), h = q->size(1), k = q->size(2), cap = V->size(-2), v = V->size(-1);
  const int dt = cache_type(*K);
  if (dt < 0 || K->scalar_type() != V->scalar_type() || lens->numel() != b || !fits(*q) || !fits(*V) ||
      !(mh ? shape_is(*K, {b, h, cap, k}) && shape_is(*V, {b, h, cap, v}) : shape_is(*K, {b, cap, k}) && shape_is(*V, {b, cap, v})))
    NOT_HERE;
  at::Tensor own;
  Held out{output(a[5], *q, {b, h, v}, &o, &own)};
  if (!out.p) NOT_HERE;
  const float *qp = at_of<float>(q);
  const void *Kp = K->data_ptr(), *Vp = V->data_ptr();
  const int32_t* lp = at_of<int32_t>(lens);
  float* op = at_of<float>(o);
  void *wp = ws->data_ptr(), *st = current_stream();
  const size_t nbytes = bytes_of(*ws);
  if (a[8] == Py_None)
    return result(WITHOUT_GIL((mh ? fn.mha_decode : fn.mqa_decode)(qp, Kp, Vp, lp, op, b, h, cap, k, v, (mqa_dtype)dt, scale, wp, nbytes, st)),
                  mh ? "mha_decode_step" : "mqa_decode_step", out.take());
  return result(WITHOUT_GIL((mh ? fn.mha_window : fn.mqa_window)(qp, Kp, Vp, lp, op, b, h, cap, k, v, (mqa_dtype)dt, scale, window, wp, nbytes, st)),
                mh ? "mha_decode_step_window" : "mqa_decode_step_window", out.take());
}

// (x, P_q, P_k, P_v, K, V, lens_in, lens_out, q)
MQA_CALL(append_qkv, 9) {
  const at::Tensor *x = f32(a[0]), *Pq = f32(a[1]), *Pk = f32(a[2]), *Pv = f32(a[3]), *K = plain(a[4]), *V = plain(a[5]), *in = i32(a[6]), *out = i32(a[7]), *q;
  if (!x || !Pq || !Pk || !Pv || !K || !V || !in || !out || x->dim() != 2 || Pq->dim() != 3 || Pk->dim() < 2 || Pk->dim() > 3 || Pv->dim() != Pk->dim() ||
      K->dim() < 2)
    NOT_HERE;
  const int64_t b = x->size(0), d = x->size(1), h = Pq->size(0), k = Pq->size(2), v = Pv->size(-1), cap = K->size(-2);
  const bool one = Pk->dim() == 2;
  const int64_t h_kv = one ? 1 : Pk->size(0);
  const int dt = cache_type(*K);
  if (dt < 0 || K->scalar_type() != V->scalar_type() || Pq->size(1) != d || Pk->size(-2) != d || Pk->size(-1) != k || Pv->size(-2) != d ||
      (!one && Pv->size(0) != h_kv) || in->numel() != b || out->numel() != b || !fits(*x) || !fits(*Pq) || !fits(*Pv) || !fits(*K) ||
      !(one ? shape_is(*K, {b, cap, k}) && shape_is(*V, {b, cap, v}) : shape_is(*K, {b, h_kv, cap, k}) && shape_is(*V, {b, h_kv, cap, v})))
    NOT_HERE;
  at::Tensor own;
  Held res{output(a[8], *x, {b, h, k}, &q, &own)};
  if (!res.p) NOT_HERE;
  const float *xp = at_of<float>(x), *Pqp = at_of<float>(Pq), *Pkp = at_of<float>(Pk), *Pvp = at_of<float>(Pv);
  float* qp = at_of<float>(q);
  void *Kp = K->data_ptr(), *Vp = V->data_ptr(), *st = current_stream();
  int32_t *ip = at_of<int32_t>(in), *lp = at_of<int32_t>(out);
  return result(WITHOUT_GIL(fn.append_qkv(xp, Pqp, Pkp, Pvp, qp, Kp, Vp, ip, lp, b, d, h, h_kv, cap, k, v, (mqa_dtype)dt, st)), "mqa_project_append_qkv", res.take());
}

// The sizes of a projection; false: not these
struct Product { int64_t rows, d, h, kv; };
bool product_of(int mode, const at::Tensor& x, const at::Tensor& P, Product* s) {
  const bool two = mode == MQA_PROJ_KV || mode == MQA_PROJ_LINEAR;
  if (mode < 0 || mode > 4 || P.dim() != (two ? 2 : 3) || x.dim() != (mode == MQA_PROJ_O ? 3 : 2) || !fits(x) || !fits(P)) return false;
  *s = Product{x.size(0), P.size(-2), two ? 1 : P.size(0), P.size(-1)};
  return mode == MQA_PROJ_O ? x.size(1) == s->h && x.size(2) == s->kv : x.size(1) == s->d;
}

// (mode, x, P, out, epilogue or None)
MQA_CALL(project, 5) {
  int mode, epilogue = MQA_EPI_STORE;
  const at::Tensor *x = f32(a[1]), *P = f32(a[2]), *out;
  Product s;
  if (!x || !P || !integer(a[0], &mode) || (a[4] != Py_None && !integer(a[4], &epilogue)) || !product_of(mode, *x, *P, &s) || (epilogue == MQA_EPI_ADD && a[3] == Py_None)) NOT_HERE;
  at::Tensor own;
  Held res{mode == MQA_PROJ_O ? output(a[3], *x, {s.rows, s.d}, &out, &own)
                              : mode == MQA_PROJ_Q || mode == MQA_PROJ_KV_MH ? output(a[3], *x, {s.rows, s.h, s.kv}, &out, &own)
                                                                             : output(a[3], *x, {s.rows, s.kv}, &out, &own)};
  if (!res.p) NOT_HERE;
  const float *xp = at_of<float>(x), *Pp = at_of<float>(P);
  float* op = at_of<float>(out);
  void* st = current_stream();
  return result(WITHOUT_GIL(fn.project((mqa_proj_mode)mode, xp, Pp, op, s.rows, s.d, s.h, s.kv, (mqa_proj_epilogue)epilogue, st)),
                a[4] == Py_None ? "mqa_project_qkvo" : "mqa_project_qkvo_ex", res.take());
}

// (mode, x, P, acc, out, eps, workspace)
MQA_CALL(add_layernorm, 7) {
  int mode;
  float eps;
  const at::Tensor *x = f32(a[1]), *P = f32(a[2]), *acc = f32(a[3]), *ws = plain(a[6]), *out;
  Product s;
  if (!x || !P || !acc || !ws || !integer(a[0], &mode) || (mode != MQA_PROJ_O && mode != MQA_PROJ_LINEAR) || !number(a[5], &eps) || !product_of(mode, *x, *P, &s) ||
      !shape_is(*acc, {s.rows, mode == MQA_PROJ_O ? s.d : s.kv}))
    NOT_HERE;
  at::Tensor own;
  Held res{output(a[4], *acc, {acc->size(0), acc->size(1)}, &out, &own)};
  if (!res.p) NOT_HERE;
  const float *xp = at_of<float>(x), *Pp = at_of<float>(P);
  float *ap = at_of<float>(acc), *op = at_of<float>(out);
  void *wp = ws->data_ptr(), *st = current_stream();
  const size_t nbytes = bytes_of(*ws);
  return result(WITHOUT_GIL(fn.add_layernorm((mqa_proj_mode)mode, xp, Pp, ap, op, s.rows, s.d, s.h, s.kv, eps, wp, nbytes, st)), "mqa_project_add_layernorm", res.take());
}

// (M, P_k, P_v, K, V, lens, mem_lens, workspace, products from which a call asks for a workspace)
MQA_CALL(memory_kv, 9) {
  const at::Tensor *M = f32(a[0]), *Pk = f32(a[1]), *Pv = f32(a[2]), *K = plain(a[3]), *V = plain(a[4]), *lens = i32(a[5]);
  const at::Tensor *valid = a[6] == Py_None ? nullptr : i32(a[6]), *ws = a[7] == Py_None ? nullptr : plain(a[7]);
  if (!M || !Pk || !Pv || !K || !V || !lens || (a[6] != Py_None && !valid) || (a[7] != Py_None && !ws) || M->dim() != 3 || Pk->dim() < 2 || Pk->dim() > 3 ||
      Pv->dim() != Pk->dim() || K->dim() != Pk->dim() + 1)
    NOT_HERE;
  const int64_t b = M->size(0), m = M->size(1), d = M->size(2), k = Pk->size(-1), v = Pv->size(-1), cap = K->size(-2);
  const bool one = Pk->dim() == 2;
  const int64_t h_kv = one ? 1 : Pk->size(0);
  const int dt = cache_type(*K);
  int small;
  if (!integer(a[8], &small) || (!ws && (double)b * m * d * h_kv * (k + v) >= small)) NOT_HERE;
  if (dt < 0 || K->scalar_type() != V->scalar_type() || Pk->size(-2) != d || Pv->size(-2) != d || (!one && Pv->size(0) != h_kv) || lens->numel() != b ||
      (valid && valid->numel() != b) || !fits(*M) || !fits(*Pk) || !fits(*Pv) || !fits(*K) ||
      !(one ? shape_is(*K, {b, cap, k}) && shape_is(*V, {b, cap, v}) : shape_is(*K, {b, h_kv, cap, k}) && shape_is(*V, {b, h_kv, cap, v})))
    NOT_HERE;
  const float *Mp = at_of<float>(M), *Pkp = at_of<float>(Pk), *Pvp = at_of<float>(Pv);
  void *Kp = K->data_ptr(), *Vp = V->data_ptr(), *wp = at_of<void>(ws), *st = current_stream();
  int32_t *vp = at_of<int32_t>(valid), *lp = at_of<int32_t>(lens);
  const size_t nbytes = ws ? bytes_of(*ws) : 0;
  Py_INCREF(Py_True);
  return result(WITHOUT_GIL(ws ? fn.memory_kv_ws(Mp, Pkp, Pvp, Kp, Vp, vp, lp, b, m, d, h_kv, cap, k, v, (mqa_dtype)dt, wp, nbytes, st)
                               : fn.memory_kv(Mp, Pkp, Pvp, Kp, Vp, vp, lp, b, m, d, h_kv, cap, k, v, (mqa_dtype)dt, st)),
                "mqa_project_memory_kv", Py_True);
}

// (which: 0 a memory's step, q [b,queries,h,k]; 1 a prompt, q [b,n,h,k]; 2 a multi-head one, q [b,h,n,k]; q, K, V, lens, o, scale, workspace)
MQA_CALL(attend_rows, 8) {
  int which;
  float scale;
  const at::Tensor *q = f32(a[1]), *K = plain(a[2]), *V = plain(a[3]), *lens = i32(a[4]), *ws = plain(a[7]), *o;
  if (!q || !K || !V || !lens || !ws || q->dim() != 4 || V->dim() < 2 || !integer(a[0], &which) || !number(a[6], &scale)) NOT_HERE;
  const bool mh = which == 2;
  const int64_t b = q->size(0), n = q->size(mh ? 2 : 1), h = q->size(mh ? 1 : 2), k = q->size(3), cap = V->size(-2), v = V->size(-1);
  const int dt = cache_type(*K);
  if (dt < 0 || K->scalar_type() != V->scalar_type() || lens->numel() != b || !fits(*q) || !fits(*V) ||
      !(mh ? shape_is(*K, {b, h, cap, k}) && shape_is(*V, {b, h, cap, v}) : shape_is(*K, {b, cap, k}) && shape_is(*V, {b, cap, v})))
    NOT_HERE;
  at::Tensor own;
  Held out{output(a[5], *q, {b, q->size(1), q->size(2), v}, &o, &own)};
  if (!out.p) NOT_HERE;
  const float* qp = at_of<float>(q);
  const void *Kp = K->data_ptr(), *Vp = V->data_ptr();
  const int32_t* lp = at_of<int32_t>(lens);
  float* op = at_of<float>(o);
  void *wp = ws->data_ptr(), *st = current_stream();
  const size_t nbytes = bytes_of(*ws);
  static const char* const names[] = {"mqa_memory_decode_step", "mqa_prefill_attention", "mha_prefill_attention"};
  const auto call = which == 0 ? fn.memory_decode : which == 1 ? fn.mqa_prefill : fn.mha_prefill;
  return result(WITHOUT_GIL(call(qp, Kp, Vp, lp, op, b, n, h, cap, k, v, (mqa_dtype)dt, scale, wp, nbytes, st)), names[which], out.take());
}

// (q, K_src, V_src, lens_src, K_own, V_own, lens_own, o, scale, workspace)
MQA_CALL(beams, 10) {
  float scale;
  const at::Tensor *q = f32(a[0]), *Ks = plain(a[1]), *Vs = plain(a[2]), *ls = i32(a[3]), *Ko = plain(a[4]), *Vo = plain(a[5]), *lo = i32(a[6]), *ws = plain(a[9]), *o;
  if (!q || !Ks || !Vs || !ls || !Ko || !Vo || !lo || !ws || q->dim() != 4 || Vs->dim() != 3 || Vo->dim() != 4 || !number(a[8], &scale)) NOT_HERE;
  const int64_t b = q->size(0), e = q->size(1), h = q->size(2), k = q->size(3), cs = Vs->size(1), co = Vo->size(2), v = Vs->size(2);
  const int dt = cache_type(*Ks);
  if (dt < 0 || Ks->scalar_type() != Ko->scalar_type() || Ks->scalar_type() != Vs->scalar_type() || Ks->scalar_type() != Vo->scalar_type() ||
      !shape_is(*Ks, {b, cs, k}) || !shape_is(*Vs, {b, cs, v}) || !shape_is(*Ko, {b, e, co, k}) || !shape_is(*Vo, {b, e, co, v}) || ls->numel() != b ||
      lo->numel() != b * e || !fits(*q) || !fits(*Vs) || !fits(*Vo))
    NOT_HERE;
  at::Tensor own;
  Held out{output(a[7], *q, {b, e, h, v}, &o, &own)};
  if (!out.p) NOT_HERE;
  const float* qp = at_of<float>(q);
  const void *Ksp = Ks->data_ptr(), *Vsp = Vs->data_ptr(), *Kop = Ko->data_ptr(), *Vop = Vo->data_ptr();
  const int32_t *lsp = at_of<int32_t>(ls), *lop = at_of<int32_t>(lo);
  float* op = at_of<float>(o);
  void *wp = ws->data_ptr(), *st = current_stream();
  const size_t nbytes = bytes_of(*ws);
  return result(WITHOUT_GIL(fn.beams(qp, Ksp, Vsp, lsp, Kop, Vop, lop, op, b, e, h, cs, co, k, v, (mqa_dtype)dt, scale, wp, nbytes, st)), "mqa_decode_step_beams", out.take());
}

// (K_src, V_src, lens_src, parent, K_dst, V_dst, lens_dst)
MQA_CALL(reorder, 7) {
  const at::Tensor *Ks = plain(a[0]), *Vs = plain(a[1]), *ls = i32(a[2]), *parent = i32(a[3]), *Kd = plain(a[4]), *Vd = plain(a[5]), *ld = i32(a[6]);
  if (!Ks || !Vs || !ls || !parent || !Kd || !Vd || !ld || Ks->dim() < 3 || Ks->dim() > 4 || Vs->dim() != Ks->dim()) NOT_HERE;
  const int64_t n = Ks->size(0), cap = Ks->size(-2), k = Ks->size(-1), v = Vs->size(-1), h_kv = Ks->dim() == 4 ? Ks->size(1) : 1;
  const int dt = cache_type(*Ks);
  if (dt < 0 || Vs->scalar_type() != Ks->scalar_type() || Kd->scalar_type() != Ks->scalar_type() || Vd->scalar_type() != Ks->scalar_type() ||
      Kd->sizes() != Ks->sizes() || Vd->sizes() != Vs->sizes() || Vs->sizes().slice(0, Vs->dim() - 1) != Ks->sizes().slice(0, Ks->dim() - 1) ||
      ls->numel() != n || parent->numel() != n || ld->numel() != n || !fits(*Ks) || !fits(*Vs))
    NOT_HERE;
  const void *Ksp = Ks->data_ptr(), *Vsp = Vs->data_ptr();
  void *Kdp = Kd->data_ptr(), *Vdp = Vd->data_ptr(), *st = current_stream();
  const int32_t *lsp = at_of<int32_t>(ls), *pp = at_of<int32_t>(parent);
  int32_t* ldp = at_of<int32_t>(ld);
  Py_INCREF(Py_True);
  return result(WITHOUT_GIL(fn.reorder(Ksp, Vsp, lsp, pp, Kdp, Vdp, ldp, n, h_kv, cap, k, v, (mqa_dtype)dt, st)), "mqa_beam_reorder_kv", Py_True);
}

// (the error's class, torch.nn.Parameter, addresses in the order of Functions)
PyObject* init(PyObject*, PyObject* const* a, Py_ssize_t n) {
  constexpr Py_ssize_t count = sizeof(Functions) / sizeof(void*);
  if (n != 2 + count) { PyErr_SetString(PyExc_TypeError, "init: a class, a class and the functions' addresses"); return nullptr; }
  void* at[count];
  for (Py_ssize_t i = 0; i < count; ++i) {
    at[i] = PyLong_AsVoidPtr(a[2 + i]);
    if (!at[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "init: no address");
      return nullptr;
    }
  }
  memcpy(&fn, at, sizeof fn);
  Py_INCREF(a[0]), Py_INCREF(a[1]);
  Py_XSETREF(error_class, a[0]);
  Py_XSETREF(parameter_class, a[1]);
  Py_RETURN_NONE;
}

// of the torch whose tensors these functions know from within
PyObject* torch_version(PyObject*, PyObject* const*, Py_ssize_t) { return PyUnicode_FromString(MQA_TORCH_VERSION); }

#define ENTRY(NAME) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(NAME)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ENTRY(init), ENTRY(torch_version), ENTRY(decode), ENTRY(append_qkv), ENTRY(project), ENTRY(add_layernorm), ENTRY(memory_kv), ENTRY(attend_rows), ENTRY(beams),
                         ENTRY(reorder), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", "Native argument marshalling of binding.py", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() { return PyModule_Create(&module); }
