// Native fast path of the Python binding (module _coxbind).
//
// A small call's time is the host's: a launch takes about 3 us and torch
// allocations, argument checks and ctypes marshalling in Python took another
// 4 to 6.  The functions below do the same work for the ordinary case -- plain
// contiguous tensors of the expected type, the default schedule, a cached
// workspace that is large enough -- and return None for everything else,
// which the Python functions in cox.py then handle with their own checks and
// messages.  A nonzero status of the C entry point comes back as an int.
//
// The entry points are called through the addresses that cox.py hands to
// init(), so this module is linked against neither libcox.so nor HIP.
#include <ATen/ATen.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/cox.h"

namespace {

decltype(&cox_warp_reduce_blocks_i32) p_reduce_blocks;
decltype(&cox_warp_reduce) p_reduce;
decltype(&cox_warp_dot) p_dot;
decltype(&cox_warp_scan) p_scan;
decltype(&cox_ballot_compact) p_compact;
decltype(&cox_tile_sort) p_sort;
decltype(&cox_tile_reduce) p_tile_reduce;
decltype(&cox_warp_masked) p_masked;
decltype(&cox_segmented) p_segmented;
decltype(&cox_integral_image) p_image;

// the tensor behind o if it is a plain contiguous device tensor of type dt
const at::Tensor *tensor(PyObject *o, at::ScalarType dt) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor &t = THPVariable_Unpack(o);
  return t.is_cuda() && t.scalar_type() == dt && t.is_contiguous() ? &t : nullptr;
}

at::Tensor make(at::IntArrayRef sizes, at::ScalarType dt, const at::Tensor &like) {
  return at::empty(sizes, at::TensorOptions().dtype(dt).device(like.device()));
}

// the caller's output, or a new one in its place; false: not handled here
bool output(PyObject *o, at::IntArrayRef sizes, at::ScalarType dt, const at::Tensor &like, at::Tensor &out) {
  if (o == Py_None) {
    out = make(sizes, dt, like);
    return true;
  }
  if (!THPVariable_CheckExact(o)) return false;
  out = THPVariable_Unpack(o);
  return true;
}

void *ptr_arg(PyObject *o) { return PyLong_AsVoidPtr(o); }
int64_t int_arg(PyObject *o) { return PyLong_AsLongLong(o); }
// a caller's own number; false: not a C int (as ctypes takes it), not handled here
bool user_int(PyObject *o, int &v) {
  int over = 0;
  const long long w = PyLong_AsLongLongAndOverflow(o, &over);
  if (PyErr_Occurred()) PyErr_Clear();
  v = (int)w;
  return !over && w == v;
}

// a status that is not 0, as the value the Python side raises from
PyObject *status(cox_status s) { return PyLong_FromLong((long)s); }

PyObject *pack(std::initializer_list<at::Tensor> ts) {
  PyObject *r = PyTuple_New((Py_ssize_t)ts.size());
  if (!r) return nullptr;
  Py_ssize_t i = 0;
  for (const at::Tensor &t : ts) {
    PyObject *w = nullptr;
    if (t.defined()) {
      w = THPVariable_Wrap(t);
    } else {
      Py_INCREF(Py_None);
      w = Py_None;
    }
    PyTuple_SET_ITEM(r, i++, w);
  }
  return r;
}

// the data of a tensor, or of none.  Throws for a tensor without storage (inside a
// vmap or grad transform), so the pointers are taken before COX_CALL gives up the
// lock that raising needs.
template <class T>
T *data(const at::Tensor &t) { return t.defined() ? (T *)t.data_ptr() : nullptr; }

// the C call without the interpreter's lock, as ctypes makes it; nothing in it
// may throw
#define COX_CALL(r, call)    \
  cox_status r;              \
  Py_BEGIN_ALLOW_THREADS;    \
  r = call;                  \
  Py_END_ALLOW_THREADS;      \
  if (r != COX_OK) return status(r)

#define COX_ARGS(count)                                                             \
  if (n_args != count) {                                                            \
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");                  \
    return nullptr;                                                                 \
  }

// (x, block_sums, warp_pos_count, stream)
PyObject *reduce_blocks(PyObject *, PyObject *const *a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  COX_ARGS(4)
  const at::Tensor *x = tensor(a[0], at::kInt);
  if (!x) Py_RETURN_NONE;
  const int64_t n = x->numel();
  at::Tensor sums, pos;
  if (!output(a[1], {(n + 255) / 256}, at::kInt, *x, sums) || !output(a[2], {(n + 31) / 32}, at::kInt, *x, pos))
    Py_RETURN_NONE;
  void *st = ptr_arg(a[3]);
  const int32_t *xp = data<int32_t>(*x);
  int32_t *sp = data<int32_t>(sums), *pp = data<int32_t>(pos);
  COX_CALL(r, p_reduce_blocks(xp, n, sp, pp, st));
  return pack({sums, pos});
  END_HANDLE_TH_ERRORS
}

// (x, y or None, acc, chunk elements or 0 (no partials), workspace, its
// bytes, stream) under the default schedule
PyObject *reduce(PyObject *, PyObject *const *a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  COX_ARGS(7)
  if (!THPVariable_CheckExact(a[0])) Py_RETURN_NONE;
  const at::ScalarType dt = THPVariable_Unpack(a[0]).scalar_type();
  const cox_dtype code = dt == at::kInt ? COX_I32 : dt == at::kFloat ? COX_F32 : COX_BF16;
  if (dt != at::kInt && dt != at::kFloat && dt != at::kBFloat16) Py_RETURN_NONE;
  const at::Tensor *x = tensor(a[0], dt), *y = nullptr;
  if (!x) Py_RETURN_NONE;
  if (a[1] != Py_None) {
    y = tensor(a[1], dt);
    if (!y || y->numel() != x->numel()) Py_RETURN_NONE;
  }
  const int64_t n = x->numel(), acc = int_arg(a[2]), S = int_arg(a[3]);
  void *ws = ptr_arg(a[4]);
  const size_t wsb = (size_t)int_arg(a[5]);
  void *st = ptr_arg(a[6]);
  at::Tensor total = make({1}, y || dt != at::kInt ? at::kDouble : at::kLong, *x), part;
  if (S > 0) {
    const int64_t nch = (n + S - 1) / S;
    const at::ScalarType pt = y || dt != at::kInt ? at::kFloat : at::kInt;
    part = acc == COX_ACC_TWOSUM ? make({nch, 2}, pt, *x) : make({nch}, pt, *x);
  }
  const void *xp = data<void>(*x), *yp = y ? data<void>(*y) : nullptr;
  void *pp = data<void>(part), *tp = data<void>(total);
  if (y) {
    COX_CALL(r, p_dot(xp, yp, code, n, (cox_acc)acc, nullptr, pp, (double *)tp, ws, wsb, st));
  } else {
    COX_CALL(r, p_reduce(xp, code, n, (cox_acc)acc, nullptr, pp, tp, ws, wsb, st));
  }
  return pack({total, part});
  END_HANDLE_TH_ERRORS
}

// (x, out, workspace, its bytes, stream)
PyObject *scan(PyObject *, PyObject *const *a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  COX_ARGS(5)
  const at::Tensor *x = tensor(a[0], at::kInt);
  at::Tensor y;
  if (!x || !output(a[1], x->sizes(), at::kInt, *x, y)) Py_RETURN_NONE;
  void *ws = ptr_arg(a[2]), *st = ptr_arg(a[4]);
  const size_t wsb = (size_t)int_arg(a[3]);
  const int64_t n = x->numel();
  const int32_t *xp = data<int32_t>(*x);
  int32_t *yp = data<int32_t>(y);
  COX_CALL(r, p_scan(xp, yp, n, nullptr, ws, wsb, st));
  return THPVariable_Wrap(y);
  END_HANDLE_TH_ERRORS
}

// (x, out, count, workspace, its bytes, stream)
PyObject *compact(PyObject *, PyObject *const *a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  COX_ARGS(6)
  const at::Tensor *x = tensor(a[0], at::kInt);
  at::Tensor out, count;
  if (!x || !output(a[1], x->sizes(), at::kInt, *x, out) || !output(a[2], {1}, at::kLong, *x, count)) Py_RETURN_NONE;
  void *ws = ptr_arg(a[3]), *st = ptr_arg(a[5]);
  const size_t wsb = (size_t)int_arg(a[4]);
  const int64_t n = x->numel();
  const int32_t *xp = data<int32_t>(*x);
  int32_t *op = data<int32_t>(out);
  int64_t *cp = data<int64_t>(count);
  COX_CALL(r, p_compact(xp, n, op, cp, nullptr, ws, wsb, st));
  return pack({out, count});
  END_HANDLE_TH_ERRORS
}

// (keys, tile, out, stream)
PyObject *sort(PyObject *, PyObject *const *a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  COX_ARGS(4)
  const at::Tensor *x = tensor(a[0], at::kInt);
  at::Tensor out;
  int tile;
  if (!x || !user_int(a[1], tile) || !output(a[2], x->sizes(), at::kInt, *x, out)) Py_RETURN_NONE;
  void *st = ptr_arg(a[3]);
  const int64_t n = x->numel();
  const uint32_t *xp = data<uint32_t>(*x);
  uint32_t *op = data<uint32_t>(out);
  COX_CALL(r, p_sort(xp, op, n, tile, nullptr, st));
  return THPVariable_Wrap(out);
  END_HANDLE_TH_ERRORS
}

// (x, tile, out, stream), tile > 0
PyObject *tile_reduce(PyObject *, PyObject *const *a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  COX_ARGS(4)
  const at::Tensor *x = tensor(a[0], at::kInt);
  int tile;
  if (!x || !user_int(a[1], tile) || tile <= 0) Py_RETURN_NONE;
  const int64_t n = x->numel();
  at::Tensor out;
  if (!output(a[2], {(n + tile - 1) / tile}, at::kInt, *x, out)) Py_RETURN_NONE;
  void *st = ptr_arg(a[3]);
  const int32_t *xp = data<int32_t>(*x);
  int32_t *op = data<int32_t>(out);
  COX_CALL(r, p_tile_reduce(xp, n, tile, op, st));
  return THPVariable_Wrap(out);
  END_HANDLE_TH_ERRORS
}

// (x, density, out, rec, stream)
PyObject *masked(PyObject *, PyObject *const *a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  COX_ARGS(5)
  const at::Tensor *x = tensor(a[0], at::kInt);
  int density;
  if (!x || !user_int(a[1], density)) Py_RETURN_NONE;
  const int64_t n = x->numel();
  at::Tensor out, rec;
  if (!output(a[2], x->sizes(), at::kInt, *x, out) || !output(a[3], {n / 32, 4}, at::kInt, *x, rec)) Py_RETURN_NONE;
  void *st = ptr_arg(a[4]);
  const int32_t *xp = data<int32_t>(*x);
  int32_t *op = data<int32_t>(out);
  uint32_t *rp = data<uint32_t>(rec);
  COX_CALL(r, p_masked(xp, n, density, op, rp, st));
  return pack({out, rec});
  END_HANDLE_TH_ERRORS
}

// (x, offsets, which, seg_total, y, out, seg_count, workspace, its bytes, stream)
PyObject *segmented(PyObject *, PyObject *const *a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  COX_ARGS(10)
  if (!THPVariable_CheckExact(a[0])) Py_RETURN_NONE;
  const at::ScalarType dt = THPVariable_Unpack(a[0]).scalar_type();
  if (dt != at::kInt && dt != at::kFloat) Py_RETURN_NONE;
  const at::Tensor *x = tensor(a[0], dt), *off = tensor(a[1], at::kLong);
  int which;
  if (!x || !off || off->numel() < 1 || !user_int(a[2], which) || which <= 0 || which > 7) Py_RETURN_NONE;
  const int64_t nseg = off->numel() - 1, n = x->numel();
  // an output that was not asked for stays what the caller gave
  at::Tensor total, y, out, count;
  const at::Tensor none;
  auto given = [](PyObject *o, at::Tensor &t) {
    if (o == Py_None) return true;
    if (!THPVariable_CheckExact(o)) return false;
    t = THPVariable_Unpack(o);
    return true;
  };
  if (!given(a[3], total) || !given(a[4], y) || !given(a[5], out) || !given(a[6], count)) Py_RETURN_NONE;
  if ((which & 1) && !total.defined()) total = make({nseg}, dt == at::kInt ? at::kLong : at::kDouble, *x);
  if ((which & 2) && !y.defined()) y = make(x->sizes(), dt, *x);
  if ((which & 4) && !out.defined()) out = at::zeros(x->sizes(), x->options().requires_grad(false));
  if ((which & 4) && !count.defined()) count = make({nseg}, at::kLong, *x);
  void *ws = ptr_arg(a[7]), *st = ptr_arg(a[9]);
  const size_t wsb = (size_t)int_arg(a[8]);
  const void *xp = data<void>(*x);
  const int64_t *ofp = data<int64_t>(*off);
  void *tp = data<void>(total), *yp = data<void>(y), *op = data<void>(out);
  int64_t *cp = data<int64_t>(count);
  COX_CALL(r, p_segmented(xp, dt == at::kInt ? COX_I32 : COX_F32, ofp, nseg, n, tp, yp, op, cp, which, nullptr, ws, wsb,
                          st));
  return pack({total, y, out, count});
  END_HANDLE_TH_ERRORS
}

// (img, out, workspace, its bytes, stream)
PyObject *image(PyObject *, PyObject *const *a, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  COX_ARGS(5)
  const at::Tensor *img = tensor(a[0], at::kByte);
  at::Tensor out;
  if (!img || img->dim() != 2 || !output(a[1], img->sizes(), at::kInt, *img, out)) Py_RETURN_NONE;
  void *ws = ptr_arg(a[2]), *st = ptr_arg(a[4]);
  const size_t wsb = (size_t)int_arg(a[3]);
  const int64_t H = img->size(0), W = img->size(1);
  const uint8_t *ip = data<uint8_t>(*img);
  uint32_t *op = data<uint32_t>(out);
  COX_CALL(r, p_image(ip, H, W, op, ws, wsb, st));
  return THPVariable_Wrap(out);
  END_HANDLE_TH_ERRORS
}

// the entry points' addresses, in the order below
PyObject *init(PyObject *, PyObject *const *a, Py_ssize_t n_args) {
  COX_ARGS(10)
  void *p[10];
  for (int i = 0; i < 10; i++) {
    p[i] = PyLong_AsVoidPtr(a[i]);
    if (!p[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null entry point");
      return nullptr;
    }
  }
  p_reduce_blocks = (decltype(p_reduce_blocks))p[0];
  p_reduce = (decltype(p_reduce))p[1];
  p_dot = (decltype(p_dot))p[2];
  p_scan = (decltype(p_scan))p[3];
  p_compact = (decltype(p_compact))p[4];
  p_sort = (decltype(p_sort))p[5];
  p_tile_reduce = (decltype(p_tile_reduce))p[6];
  p_masked = (decltype(p_masked))p[7];
  p_segmented = (decltype(p_segmented))p[8];
  p_image = (decltype(p_image))p[9];
  Py_RETURN_NONE;
}

#define COX_FN(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {COX_FN(init),    COX_FN(reduce_blocks), COX_FN(reduce),    COX_FN(scan),
                         COX_FN(compact), COX_FN(sort),          COX_FN(tile_reduce), COX_FN(masked),
                         COX_FN(segmented), COX_FN(image),       {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_coxbind", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__coxbind() { return PyModule_Create(&module); }
