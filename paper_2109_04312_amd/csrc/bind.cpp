// The tensor-level calls of mate.py: checks the tensors, allocates what the caller did not pass,
// looks up the current stream and calls the C ABI.  Host code only, no arithmetic.
//
// A step on a short sequence is a handful of 5-10 us kernels, so the host path bounds it: with
// the same marshalling in Python and ctypes a forward cost 10 us and a backward 14 us on the host,
// most of it attribute look-ups, torch.empty_like and argument conversion (a training step of
// three launches at B = 32, N = 128 enqueued in 35 us; its kernels need less).
//
// The C ABI arrives as addresses (bind()), so that this module follows whatever library mate.py
// has loaded and links against torch alone.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <cstring>

#include "../../include/mate.h"

namespace {

// ---- the C ABI, bound at import --------------------------------------------------------------
#define MATE_FUNCTIONS(X)                                                                         \
  X(mate_segments_bytes) X(mate_workspace_bytes) X(mate_build_segments)                           \
  X(mate_build_segments_bucketed) X(mate_cell_positions) X(mate_attn_fwd) X(mate_attn_bwd)        \
  X(mate_dense_workspace_bytes) X(mate_attn_fwd_dense) X(mate_attn_bwd_dense) X(mate_qkv_project) \
  X(mate_out_project) X(mate_project_bwd_workspace_bytes) X(mate_qkv_project_bwd)                 \
  X(mate_out_project_bwd)
struct Abi {
#define X(name) decltype(&::name) name;
  MATE_FUNCTIONS(X)
#undef X
} abi;
PyObject* mate_error;                    // mate.MateError
PyObject* to_head_kinds;                 // mate._head_kind_host
PyObject *s_buf, *s_B, *s_N;             // attribute names of mate.Segments

// ---- errors: thrown as C++ exceptions below, turned into Python ones in guarded() --------------
struct PyFailure {};                     // a Python exception is already set
[[noreturn]] void fail(PyObject* type, const char* text) {
  PyErr_SetString(type, text);
  throw PyFailure();
}
#define MATE_ASSERT(cond)                                  \
  do {                                                     \
    if (!(cond)) fail(PyExc_AssertionError, #cond);        \
  } while (0)
void check(int status, const char* where) {
  if (status == MATE_OK) return;
  if (PyObject* e = PyObject_CallFunction(mate_error, "is", status, where)) {
    PyErr_SetObject(mate_error, e);
    Py_DECREF(e);
  }
  throw PyFailure();
}

// The C call itself runs without the GIL (a launch can block when the queue is full).
template <class F>
void call(const char* where, F&& f) {
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = f();
  Py_END_ALLOW_THREADS
  check(status, where);
}

// ---- arguments -------------------------------------------------------------------------------
const at::Tensor& tensor(PyObject* o, const char* name) {
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_TypeError, "%s must be a tensor", name);
    throw PyFailure();
  }
  return THPVariable_Unpack(o);
}
void* dev(const at::Tensor& t, const char* name) {
  if (!(t.is_cuda() && t.is_contiguous())) {
    PyErr_Format(PyExc_ValueError, "%s must be a contiguous device tensor", name);
    throw PyFailure();
  }
  return t.data_ptr();
}
void* dev(PyObject* o, const char* name) { return dev(tensor(o, name), name); }
void* dev_or_null(PyObject* o, const char* name) { return o == Py_None ? nullptr : dev(o, name); }
bool has_shape(const at::Tensor& t, std::initializer_list<int64_t> s) {
  return t.sizes() == at::IntArrayRef(s.begin(), s.size());
}
int integer(PyObject* o) {
  const long v = PyLong_AsLong(o);
  if (v == -1 && PyErr_Occurred()) throw PyFailure();
  return (int)std::max(-2147483647L, std::min(2147483647L, v));
}
float real(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw PyFailure();
  return (float)v;
}
bool truth(PyObject* o) {
  const int v = PyObject_IsTrue(o);
  if (v < 0) throw PyFailure();
  return v != 0;
}
mate_dtype dtype_code(const at::Tensor& t) {
  if (t.scalar_type() == at::kFloat) return MATE_F32;
  if (t.scalar_type() == at::kBFloat16) return MATE_BF16;
  PyErr_Format(PyExc_TypeError, "unsupported dtype %s", c10::toString(t.scalar_type()));
  throw PyFailure();
}
struct Shape4 { int B, H, N, D; };
Shape4 shape4(const at::Tensor& t) {
  if (t.dim() != 4) fail(PyExc_ValueError, "expected a tensor of shape [B, H, N, D]");
  return {(int)t.size(0), (int)t.size(1), (int)t.size(2), (int)t.size(3)};
}
void* stream() { return c10::hip::getCurrentHIPStreamMasqueradingAsCUDA().stream(); }

// Head kinds on the host: a one-dimensional contiguous array of H unsigned bytes is read in place, anything
// else (a list, an array of another type or shape, a tensor) goes through mate.py's conversion, which
// accepts or refuses it.  (A bytes object is text to that conversion, not an array.)
struct HeadKinds {
  Py_buffer view;
  HeadKinds(PyObject* o, int H) {
    if (!PyBytes_Check(o) && PyObject_CheckBuffer(o)) {
      if (PyObject_GetBuffer(o, &view, PyBUF_ND | PyBUF_FORMAT) == 0) {
        if (view.ndim == 1 && view.len == H && view.itemsize == 1 && view.format && !std::strcmp(view.format, "B")) return;
        PyBuffer_Release(&view);
      } else {
        PyErr_Clear();
      }
    }
    PyObject* converted = PyObject_CallFunction(to_head_kinds, "Oi", o, H);
    if (!converted) throw PyFailure();
    const int bad = PyObject_GetBuffer(converted, &view, PyBUF_SIMPLE);  // (the view keeps it alive)
    Py_DECREF(converted);
    if (bad) throw PyFailure();
  }
  ~HeadKinds() { PyBuffer_Release(&view); }
  HeadKinds(const HeadKinds&) = delete;
  HeadKinds& operator=(const HeadKinds&) = delete;
  const uint8_t* get() const { return static_cast<const uint8_t*>(view.buf); }
};

// ---- outputs ---------------------------------------------------------------------------------
at::Tensor given_or_like(PyObject* o, const at::Tensor& like, const char* name) {
  return o == Py_None ? at::empty_like(like) : tensor(o, name);
}
at::Tensor new_tensor(std::initializer_list<int64_t> s, at::ScalarType t, const at::Tensor& like) {
  return at::empty(at::IntArrayRef(s.begin(), s.size()), at::TensorOptions(like.device()).dtype(t));
}
// Workspace: the caller's, or bytes that live until the call is enqueued (the caching allocator
// hands them on in stream order).
struct Workspace {
  at::Tensor t;
  void* ptr;
  size_t bytes;
  Workspace(PyObject* o, size_t need, const at::Tensor& like) {
    t = o == Py_None ? new_tensor({(int64_t)std::max<size_t>(need, 16)}, at::kByte, like) : tensor(o, "ws");
    ptr = t.data_ptr();
    bytes = (size_t)t.numel();
  }
};
PyObject* pack(std::initializer_list<at::Tensor> ts) {
  PyObject* r = PyTuple_New((Py_ssize_t)ts.size());
  if (!r) throw PyFailure();
  Py_ssize_t i = 0;
  for (const at::Tensor& t : ts) {
    PyObject* o = nullptr;
    if (t.defined()) {
      o = THPVariable_Wrap(t);
    } else {
      Py_INCREF(Py_None);
      o = Py_None;
    }
    if (!o) {
      Py_DECREF(r);
      throw PyFailure();
    }
    PyTuple_SET_ITEM(r, i++, o);
  }
  return r;
}

struct Ids { void *row, *col, *flags; int B, N; };
Ids ids(PyObject* row, PyObject* col, PyObject* flags) {
  const at::Tensor &r = tensor(row, "row_ids"), &c = tensor(col, "col_ids"), &f = tensor(flags, "flags");
  if (f.dim() != 2) fail(PyExc_ValueError, "flags must have shape [B, N]");
  MATE_ASSERT(r.scalar_type() == at::kInt && c.scalar_type() == at::kInt && f.scalar_type() == at::kByte);
  MATE_ASSERT(r.sizes() == f.sizes() && c.sizes() == f.sizes());
  return {dev(r, "row_ids"), dev(c, "col_ids"), dev(f, "flags"), (int)f.size(0), (int)f.size(1)};
}

// The table buffer of a mate.Segments, checked against the tensors' (B, N).
void* tables(PyObject* seg, int B, int N) {
  PyObject *buf = PyObject_GetAttr(seg, s_buf), *b = PyObject_GetAttr(seg, s_B), *n = PyObject_GetAttr(seg, s_N);
  Py_XDECREF(buf);  // the Segments object keeps them alive
  Py_XDECREF(b);
  Py_XDECREF(n);
  if (!buf || !b || !n) throw PyFailure();
  const at::Tensor& t = tensor(buf, "segments");
  if (integer(b) != B || integer(n) != N || (size_t)t.numel() < abi.mate_segments_bytes(B, N))
    check(MATE_ERR_SHAPE, "segment tables are for another (B, N) than the tensors");
  return t.data_ptr();
}

// ---- entry points ----------------------------------------------------------------------------
using Args = PyObject* const*;

PyObject* build_segments(Args a) {  // row, col, flags, buffer, global_length | None, radius
  const Ids i = ids(a[0], a[1], a[2]);
  void* buf = tensor(a[3], "out").data_ptr();
  void* s = stream();
  if (a[4] == Py_None) {
    call("mate_build_segments", [&] {
      return abi.mate_build_segments((int32_t*)i.row, (int32_t*)i.col, (uint8_t*)i.flags, i.B, i.N, buf, s);
    });
  } else {
    const int G = integer(a[4]), R = integer(a[5]);
    call("mate_build_segments_bucketed", [&] {
      return abi.mate_build_segments_bucketed((int32_t*)i.row, (int32_t*)i.col, (uint8_t*)i.flags, i.B, i.N, G, R,
                                              buf, s);
    });
  }
  Py_RETURN_NONE;
}

PyObject* segments_buffer(Args a) {  // flags -> uninitialised table buffer
  const at::Tensor& f = tensor(a[0], "flags");
  if (f.dim() != 2) fail(PyExc_ValueError, "flags must have shape [B, N]");
  const size_t n = abi.mate_segments_bytes((int)f.size(0), (int)f.size(1));
  if (n == 0) check(MATE_ERR_SHAPE, "mate_segments_bytes");
  return THPVariable_Wrap(new_tensor({(int64_t)n}, at::kByte, f));
}

PyObject* cell_positions(Args a) {  // row, col, flags, out | None
  const Ids i = ids(a[0], a[1], a[2]);
  at::Tensor out = a[3] == Py_None ? new_tensor({i.B, i.N}, at::kInt, tensor(a[2], "flags")) : tensor(a[3], "positions");
  MATE_ASSERT(out.scalar_type() == at::kInt && has_shape(out, {i.B, i.N}));
  void *p = dev(out, "positions"), *s = stream();
  call("mate_cell_positions", [&] {
    return abi.mate_cell_positions((int32_t*)i.row, (int32_t*)i.col, (uint8_t*)i.flags, i.B, i.N, (int32_t*)p, s);
  });
  return THPVariable_Wrap(std::move(out));
}

PyObject* attn_fwd(Args a) {  // q, k, v, seg, head_kind, scale, out, lse, ws
  const at::Tensor& q = tensor(a[0], "q");
  const Shape4 x = shape4(q);
  void* seg = tables(a[3], x.B, x.N);
  const HeadKinds hk(a[4], x.H);
  const mate_dtype t = dtype_code(q);
  const float scale = real(a[5]);
  at::Tensor out = given_or_like(a[6], q, "out");
  at::Tensor lse = a[7] == Py_None ? new_tensor({x.B, x.H, x.N}, at::kFloat, q) : tensor(a[7], "lse");
  const Workspace ws(a[8], abi.mate_workspace_bytes(x.B, x.H, x.N, x.D, t, 0), q);
  void *pq = dev(q, "q"), *pk = dev(a[1], "k"), *pv = dev(a[2], "v"), *po = dev(out, "out"), *pl = dev(lse, "lse");
  void* s = stream();
  call("mate_attn_fwd", [&] {
    return abi.mate_attn_fwd(pq, pk, pv, seg, hk.get(), x.B, x.H, x.N, x.D, t, scale, po, (float*)pl, ws.ptr,
                             ws.bytes, s);
  });
  return pack({out, lse});
}

PyObject* attn_bwd(Args a) {  // q, k, v, out, lse, dout, seg, head_kind, scale, dq, dk, dv, ws
  const at::Tensor& q = tensor(a[0], "q");
  const Shape4 x = shape4(q);
  void* seg = tables(a[6], x.B, x.N);
  const HeadKinds hk(a[7], x.H);
  const mate_dtype t = dtype_code(q);
  const float scale = real(a[8]);
  at::Tensor dq = given_or_like(a[9], q, "dq"), dk = given_or_like(a[10], q, "dk"), dv = given_or_like(a[11], q, "dv");
  const Workspace ws(a[12], abi.mate_workspace_bytes(x.B, x.H, x.N, x.D, t, 1), q);
  void *pq = dev(q, "q"), *pk = dev(a[1], "k"), *pv = dev(a[2], "v"), *po = dev(a[3], "out"), *pl = dev(a[4], "lse"),
       *pg = dev(a[5], "dout"), *pdq = dev(dq, "dq"), *pdk = dev(dk, "dk"), *pdv = dev(dv, "dv");
  void* s = stream();
  call("mate_attn_bwd", [&] {
    return abi.mate_attn_bwd(pq, pk, pv, po, (const float*)pl, pg, seg, hk.get(), x.B, x.H, x.N, x.D, t, scale, pdq,
                             pdk, pdv, ws.ptr, ws.bytes, s);
  });
  return pack({dq, dk, dv});
}

PyObject* attn_fwd_dense(Args a) {  // q, k, v, row, col, flags, head_kind, scale, out, lse
  const at::Tensor& q = tensor(a[0], "q");
  const Shape4 x = shape4(q);
  const HeadKinds hk(a[6], x.H);
  const mate_dtype t = dtype_code(q);
  const float scale = real(a[7]);
  at::Tensor out = given_or_like(a[8], q, "out");
  at::Tensor lse = a[9] == Py_None ? new_tensor({x.B, x.H, x.N}, at::kFloat, q) : tensor(a[9], "lse");
  void *pq = dev(q, "q"), *pk = dev(a[1], "k"), *pv = dev(a[2], "v"), *r = dev(a[3], "row_ids"),
       *c = dev(a[4], "col_ids"), *f = dev(a[5], "flags"), *po = dev(out, "out"), *pl = dev(lse, "lse");
  void* s = stream();
  call("mate_attn_fwd_dense", [&] {
    return abi.mate_attn_fwd_dense(pq, pk, pv, (int32_t*)r, (int32_t*)c, (uint8_t*)f, hk.get(), x.B, x.H, x.N, x.D,
                                   t, scale, po, (float*)pl, s);
  });
  return pack({out, lse});
}

PyObject* attn_bwd_dense(Args a) {  // q, k, v, out, lse, dout, row, col, flags, head_kind, scale, dq, dk, dv, ws
  const at::Tensor& q = tensor(a[0], "q");
  const Shape4 x = shape4(q);
  const HeadKinds hk(a[9], x.H);
  const mate_dtype t = dtype_code(q);
  const float scale = real(a[10]);
  at::Tensor dq = given_or_like(a[11], q, "dq"), dk = given_or_like(a[12], q, "dk"), dv = given_or_like(a[13], q, "dv");
  const Workspace ws(a[14], abi.mate_dense_workspace_bytes(x.B, x.H, x.N), q);
  void *pq = dev(q, "q"), *pk = dev(a[1], "k"), *pv = dev(a[2], "v"), *po = dev(a[3], "out"), *pl = dev(a[4], "lse"),
       *pg = dev(a[5], "dout"), *r = dev(a[6], "row_ids"), *c = dev(a[7], "col_ids"), *f = dev(a[8], "flags"),
       *pdq = dev(dq, "dq"), *pdk = dev(dk, "dk"), *pdv = dev(dv, "dv");
  void* s = stream();
  call("mate_attn_bwd_dense", [&] {
    return abi.mate_attn_bwd_dense(pq, pk, pv, po, (const float*)pl, pg, (int32_t*)r, (int32_t*)c, (uint8_t*)f,
                                   hk.get(), x.B, x.H, x.N, x.D, t, scale, pdq, pdk, pdv, ws.ptr, ws.bytes, s);
  });
  return pack({dq, dk, dv});
}

PyObject* qkv_project(Args a) {  // x, w_qkv, bias, flags, H, q, k, v
  const at::Tensor &x = tensor(a[0], "x"), &w = tensor(a[1], "w_qkv"), &flags = tensor(a[3], "flags");
  if (x.dim() != 3) fail(PyExc_ValueError, "x must have shape [B, N, E]");
  const int B = (int)x.size(0), N = (int)x.size(1), E = (int)x.size(2), H = integer(a[4]);
  MATE_ASSERT(x.scalar_type() == at::kBFloat16 && w.scalar_type() == at::kBFloat16 && has_shape(w, {3 * H * 64, E}));
  MATE_ASSERT(flags.scalar_type() == at::kByte && has_shape(flags, {B, N}));
  if (a[2] != Py_None) {
    const at::Tensor& bias = tensor(a[2], "bias");
    MATE_ASSERT(bias.scalar_type() == at::kFloat && has_shape(bias, {3 * H * 64}));
  }
  at::Tensor out[3];
  void* po[3];
  for (int i = 0; i < 3; ++i) {
    out[i] = a[5 + i] == Py_None ? new_tensor({B, H, N, 64}, at::kBFloat16, x) : tensor(a[5 + i], "out");
    MATE_ASSERT(out[i].scalar_type() == at::kBFloat16 && has_shape(out[i], {B, H, N, 64}));
    po[i] = dev(out[i], "out");
  }
  void *px = dev(x, "x"), *pw = dev(w, "w_qkv"), *pb = dev_or_null(a[2], "bias"), *pf = dev(flags, "flags"), *s = stream();
  call("mate_qkv_project", [&] {
    return abi.mate_qkv_project(px, pw, (const float*)pb, (uint8_t*)pf, B, N, H, E, MATE_BF16, po[0], po[1], po[2], s);
  });
  return pack({out[0], out[1], out[2]});
}

PyObject* out_project(Args a) {  // o, w_o, bias, flags, y
  const at::Tensor &o = tensor(a[0], "o"), &w = tensor(a[1], "w_o"), &flags = tensor(a[3], "flags");
  const Shape4 x = shape4(o);
  if (w.dim() != 2) fail(PyExc_ValueError, "w_o must have shape [E, H * 64]");
  const int E = (int)w.size(0);
  MATE_ASSERT(o.scalar_type() == at::kBFloat16 && w.scalar_type() == at::kBFloat16 && has_shape(w, {E, x.H * 64}) && x.D == 64);
  MATE_ASSERT(flags.scalar_type() == at::kByte && has_shape(flags, {x.B, x.N}));
  if (a[2] != Py_None) {
    const at::Tensor& bias = tensor(a[2], "bias");
    MATE_ASSERT(bias.scalar_type() == at::kFloat && has_shape(bias, {E}));
  }
  at::Tensor y = a[4] == Py_None ? new_tensor({x.B, x.N, E}, at::kBFloat16, o) : tensor(a[4], "y");
  MATE_ASSERT(y.scalar_type() == at::kBFloat16 && has_shape(y, {x.B, x.N, E}));
  void *po = dev(o, "o"), *pw = dev(w, "w_o"), *pb = dev_or_null(a[2], "bias"), *pf = dev(flags, "flags"),
       *py = dev(y, "y"), *s = stream();
  call("mate_out_project", [&] {
    return abi.mate_out_project(po, pw, (const float*)pb, (uint8_t*)pf, x.B, x.N, x.H, E, MATE_BF16, py, s);
  });
  return THPVariable_Wrap(std::move(y));
}

Workspace project_workspace(PyObject* o, int B, int N, int H, int E, const at::Tensor& like) {
  const size_t n = o == Py_None ? abi.mate_project_bwd_workspace_bytes(B, N, H, E) : 1;
  if (n == 0) check(MATE_ERR_UNSUPPORTED, "mate_project_bwd_workspace_bytes");
  return Workspace(o, n, like);
}

PyObject* qkv_project_bwd(Args a) {  // x, w_qkv, flags, dq, dk, dv, want_dx, want_dw, want_dbias, ws
  const at::Tensor &x = tensor(a[0], "x"), &w = tensor(a[1], "w_qkv"), &flags = tensor(a[2], "flags"),
                   &dq = tensor(a[3], "dq"), &dk = tensor(a[4], "dk"), &dv = tensor(a[5], "dv");
  if (x.dim() != 3) fail(PyExc_ValueError, "x must have shape [B, N, E]");
  if (dq.dim() != 4) fail(PyExc_ValueError, "dq must have shape [B, H, N, 64]");
  const int B = (int)x.size(0), N = (int)x.size(1), E = (int)x.size(2), H = (int)dq.size(1);
  MATE_ASSERT(x.scalar_type() == at::kBFloat16 && has_shape(w, {3 * H * 64, E}) && has_shape(dq, {B, H, N, 64}));
  MATE_ASSERT(dk.sizes() == dq.sizes() && dv.sizes() == dq.sizes() && has_shape(flags, {B, N}));
  at::Tensor dx, dw, db;
  if (truth(a[6])) dx = at::empty_like(x);
  if (truth(a[7])) dw = new_tensor({3 * H * 64, E}, at::kFloat, x);
  if (truth(a[8])) db = new_tensor({3 * H * 64}, at::kFloat, x);
  const Workspace ws = project_workspace(a[9], B, N, H, E, x);
  void *px = dev(x, "x"), *pw = dev(w, "w_qkv"), *pf = dev(flags, "flags"), *pq = dev(dq, "dq"), *pk = dev(dk, "dk"),
       *pv = dev(dv, "dv"), *pdx = dx.defined() ? dx.data_ptr() : nullptr, *pdw = dw.defined() ? dw.data_ptr() : nullptr,
       *pdb = db.defined() ? db.data_ptr() : nullptr, *s = stream();
  call("mate_qkv_project_bwd", [&] {
    return abi.mate_qkv_project_bwd(px, pw, (uint8_t*)pf, pq, pk, pv, B, N, H, E, MATE_BF16, pdx, (float*)pdw,
                                    (float*)pdb, ws.ptr, ws.bytes, s);
  });
  return pack({dx, dw, db});
}

PyObject* out_project_bwd(Args a) {  // o, w_o, flags, dy, want_do, want_dw, want_dbias, ws
  const at::Tensor &o = tensor(a[0], "o"), &w = tensor(a[1], "w_o"), &flags = tensor(a[2], "flags"), &dy = tensor(a[3], "dy");
  const Shape4 x = shape4(o);
  if (w.dim() != 2) fail(PyExc_ValueError, "w_o must have shape [E, H * 64]");
  const int E = (int)w.size(0);
  MATE_ASSERT(o.scalar_type() == at::kBFloat16 && has_shape(w, {E, x.H * 64}) && has_shape(dy, {x.B, x.N, E}) && x.D == 64);
  at::Tensor d_o, dw, db;
  if (truth(a[4])) d_o = at::empty_like(o);
  if (truth(a[5])) dw = new_tensor({E, x.H * 64}, at::kFloat, o);
  if (truth(a[6])) db = new_tensor({E}, at::kFloat, o);
  const Workspace ws = project_workspace(a[7], x.B, x.N, x.H, E, o);
  void *po = dev(o, "o"), *pw = dev(w, "w_o"), *pf = dev(flags, "flags"), *py = dev(dy, "dy"),
       *pdo = d_o.defined() ? d_o.data_ptr() : nullptr, *pdw = dw.defined() ? dw.data_ptr() : nullptr,
       *pdb = db.defined() ? db.data_ptr() : nullptr, *s = stream();
  call("mate_out_project_bwd", [&] {
    return abi.mate_out_project_bwd(po, pw, (uint8_t*)pf, py, x.B, x.N, x.H, E, MATE_BF16, pdo, (float*)pdw,
                                    (float*)pdb, ws.ptr, ws.bytes, s);
  });
  return pack({d_o, dw, db});
}

PyObject* bind(Args a) {  // {name: address}, MateError, _head_kind_host
#define X(name)                                                              \
  {                                                                          \
    PyObject* v = PyDict_GetItemString(a[0], #name);                         \
    if (!v) fail(PyExc_KeyError, #name);                                     \
    void* p = PyLong_AsVoidPtr(v);                                           \
    if (!p) fail(PyExc_ValueError, #name);                                   \
    std::memcpy(&abi.name, &p, sizeof(p));                                   \
  }
  MATE_FUNCTIONS(X)
#undef X
  Py_INCREF(a[1]);
  mate_error = a[1];
  Py_INCREF(a[2]);
  to_head_kinds = a[2];
  Py_RETURN_NONE;
}

template <PyObject* (*F)(Args), int kArgs>
PyObject* guarded(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != kArgs) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  try {
    return F(args);
  } catch (const PyFailure&) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}

#define METHOD(name, n) {#name, (PyCFunction)(void (*)())guarded<name, n>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(bind, 3),           METHOD(build_segments, 6),  METHOD(segments_buffer, 1),
                         METHOD(cell_positions, 4), METHOD(attn_fwd, 9),        METHOD(attn_bwd, 13),
                         METHOD(attn_fwd_dense, 10), METHOD(attn_bwd_dense, 15), METHOD(qkv_project, 8),
                         METHOD(out_project, 5),    METHOD(qkv_project_bwd, 10), METHOD(out_project_bwd, 8),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "Tensor-level calls of the C ABI (see mate.py).", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__native() {
  s_buf = PyUnicode_InternFromString("buf");
  s_B = PyUnicode_InternFromString("B");
  s_N = PyUnicode_InternFromString("N");
  return PyModule_Create(&module);
}
