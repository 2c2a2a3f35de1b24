// Native half of the Python binding (tq.py): the argument checks and the C-ABI call of the
// entry points that a serving loop makes, in one C call. The checks through Python
// attributes and the ctypes conversion cost about 7 us a call, more than the smaller kernels
// take (2048 x 4096, one token: 4.4 us a call, 9.8 through Python).
//
// Every function returns the C status, or None if an argument is not exactly what the call
// needs: the caller then takes the Python path, which names the fault. Nothing is cached:
// each call checks its own arguments.
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include "../../include/tq.h"

namespace {

struct Api {
  decltype(&tq_quantize_act) quantize_act;
  decltype(&tq_gemv) gemv;
  decltype(&tq_gemv_f32) gemv_f32;
  decltype(&tq_gemv2) gemv2;
  decltype(&tq_gemv_mx) gemv_mx;
  decltype(&tq_moe_grouped) moe_grouped;
} api;

// A plain contiguous device tensor of this type and shape (dims: its nd sizes; dev_any: of any).
struct Arg {
  void* ptr = nullptr;
  bool ok = false;
};

Arg dev_sizes(PyObject* o, at::ScalarType dt, int nd, const int64_t* dims) {
  Arg a;
  if (!THPVariable_CheckExact(o)) return a;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda() || t.scalar_type() != dt || !t.is_contiguous()) return a;
  if (nd >= 0) {
    if (t.dim() != nd) return a;
    for (int i = 0; i < nd; ++i)
      if (t.size(i) != dims[i]) return a;
  }
  a.ptr = t.data_ptr();
  a.ok = true;
  return a;
}

template <typename... D>
Arg dev(PyObject* o, at::ScalarType dt, D... d) {
  const int64_t dims[] = {(int64_t)d...};
  return dev_sizes(o, dt, (int)sizeof...(d), dims);
}

Arg dev_any(PyObject* o, at::ScalarType dt) { return dev_sizes(o, dt, -1, nullptr); }

bool to_i64(PyObject* o, int64_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  int over = 0;
  *v = PyLong_AsLongLongAndOverflow(o, &over);
  return over == 0;
}
bool to_i32(PyObject* o, int64_t* v) { return to_i64(o, v) && *v >= INT32_MIN && *v <= INT32_MAX; }

// sizes of a plain 2-D tensor
bool sizes2(PyObject* o, int64_t* a, int64_t* b) {
  if (!THPVariable_CheckExact(o)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (t.dim() != 2) return false;
  *a = t.size(0);
  *b = t.size(1);
  return true;
}

// C++ exceptions (a tensor without storage, say) also mean the Python path.
template <typename F>
PyObject* call(F f) {
  int64_t st = 0;
  bool ok = false;
  try {
    ok = f(&st);
  } catch (...) {
    ok = false;
  }
  if (PyErr_Occurred()) PyErr_Clear();
  if (!ok) Py_RETURN_NONE;
  return PyLong_FromLongLong(st);
}

template <typename F>
int64_t unlocked(F f) {
  PyThreadState* s = PyEval_SaveThread();
  const int64_t st = f();
  PyEval_RestoreThread(s);
  return st;
}

constexpr auto kF32 = at::kFloat, kI8 = at::kChar, kU8 = at::kByte, kI16 = at::kShort, kI32 = at::kInt;

// (x, q, d, bsum, stream)
PyObject* py_quantize_act(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return call([&](int64_t* st) {
    int64_t t, k, stream;
    if (n != 5 || !sizes2(a[0], &t, &k) || k > INT32_MAX || !to_i64(a[4], &stream)) return false;
    const Arg x = dev(a[0], kF32, t, k), q = dev(a[1], kI8, t, k), d = dev(a[2], kF32, t, k / 256),
              b = dev(a[3], kI32, t, k / 256);
    if (!x.ok || !q.ok || !d.ok || !b.ok) return false;
    *st = unlocked([&] {
      return api.quantize_act((const float*)x.ptr, t, (int32_t)k, (int8_t*)q.ptr, (float*)d.ptr, (int32_t*)b.ptr, (void*)stream);
    });
    return true;
  });
}

// (n, k, codes, scales, x, y, q, d, bsum, stream)
PyObject* py_gemv_f32(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  return call([&](int64_t* st) {
    int64_t n, k, t, kx, stream;
    if (nargs != 10 || !to_i32(a[0], &n) || !to_i32(a[1], &k) || k < 0 || !sizes2(a[4], &t, &kx) || !to_i64(a[9], &stream))
      return false;
    const int64_t kb = k / 256;
    const Arg c = dev(a[2], kU8, n, kb, 128), s = dev(a[3], kI16, n, kb), x = dev(a[4], kF32, t, k), y = dev(a[5], kF32, t, n),
              q = dev(a[6], kI8, t, k), d = dev(a[7], kF32, t, kb), b = dev(a[8], kI32, t, kb);
    if (!c.ok || !s.ok || !x.ok || !y.ok || !q.ok || !d.ok || !b.ok) return false;
    const tq_mat m = {(int32_t)n, (int32_t)k, (uint8_t*)c.ptr, (uint16_t*)s.ptr};
    *st = unlocked([&] {
      return api.gemv_f32(&m, (const float*)x.ptr, t, (float*)y.ptr, (int8_t*)q.ptr, (float*)d.ptr, (int32_t*)b.ptr, nullptr,
                          (void*)stream);
    });
    return true;
  });
}

// (n, k, codes, scales, q, d, bsum, y, stream)
PyObject* py_gemv(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  return call([&](int64_t* st) {
    int64_t n, k, t, kq, stream;
    if (nargs != 9 || !to_i32(a[0], &n) || !to_i32(a[1], &k) || k < 0 || !sizes2(a[4], &t, &kq) || !to_i64(a[8], &stream))
      return false;
    const int64_t kb = k / 256;
    const Arg c = dev(a[2], kU8, n, kb, 128), s = dev(a[3], kI16, n, kb), q = dev(a[4], kI8, t, k), d = dev(a[5], kF32, t, kb),
              b = dev(a[6], kI32, t, kb), y = dev(a[7], kF32, t, n);
    if (!c.ok || !s.ok || !q.ok || !d.ok || !b.ok || !y.ok) return false;
    const tq_mat m = {(int32_t)n, (int32_t)k, (uint8_t*)c.ptr, (uint16_t*)s.ptr};
    *st = unlocked([&] {
      return api.gemv(&m, (const int8_t*)q.ptr, (const float*)d.ptr, (const int32_t*)b.ptr, t, (float*)y.ptr, nullptr,
                      (void*)stream);
    });
    return true;
  });
}

// (n, k, codes, scales, q, d, y, stream)
template <typename Mat, typename Scale>
PyObject* gemv_planes(PyObject* const* a, Py_ssize_t nargs, tq_status (*fn)(const Mat*, const int8_t*, const float*, int64_t, float*, int32_t*, void*),
                      Arg (*scales)(PyObject*, int64_t, int64_t)) {
  return call([&](int64_t* st) {
    int64_t n, k, t, kq, stream;
    if (nargs != 8 || !to_i32(a[0], &n) || !to_i32(a[1], &k) || k < 0 || !sizes2(a[4], &t, &kq) || !to_i64(a[7], &stream))
      return false;
    const int64_t kb = k / 256;
    const Arg c = dev(a[2], kU8, n, kb, 128), s = scales(a[3], n, k), q = dev(a[4], kI8, t, k), d = dev(a[5], kF32, t, kb),
              y = dev(a[6], kF32, t, n);
    if (!c.ok || !s.ok || !q.ok || !d.ok || !y.ok) return false;
    const Mat m = {(int32_t)n, (int32_t)k, (uint8_t*)c.ptr, (Scale*)s.ptr};
    *st = unlocked([&] {
      return fn(&m, (const int8_t*)q.ptr, (const float*)d.ptr, t, (float*)y.ptr, nullptr, (void*)stream);
    });
    return true;
  });
}
PyObject* py_gemv2(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return gemv_planes<tq_mat2, uint16_t>(a, n, api.gemv2,
                                        [](PyObject* o, int64_t r, int64_t k) { return dev(o, kI16, r, k / 256, (int64_t)2); });
}
PyObject* py_gemv_mx(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return gemv_planes<tq_mat_mx, uint8_t>(a, n, api.gemv_mx,
                                         [](PyObject* o, int64_t r, int64_t k) { return dev(o, kU8, r, k / 32); });
}

// (n_experts, hidden, inter, codes tuple, scales tuple, x, topk_idx, topk_w, out, ws, flags, stream)
PyObject* py_moe_grouped(PyObject*, PyObject* const* a, Py_ssize_t nargs) {
  return call([&](int64_t* st) {
    int64_t E, H, I, t, h, t2, topk, flags, stream;
    if (nargs != 12 || !to_i32(a[0], &E) || !to_i32(a[1], &H) || !to_i32(a[2], &I) || H < 0 || I < 0 || !sizes2(a[5], &t, &h) ||
        h != H || !sizes2(a[6], &t2, &topk) || t2 != t || topk > INT32_MAX || !to_i32(a[10], &flags) || !to_i64(a[11], &stream))
      return false;
    if (!PyTuple_CheckExact(a[3]) || !PyTuple_CheckExact(a[4]) || PyTuple_GET_SIZE(a[3]) != 3 || PyTuple_GET_SIZE(a[4]) != 3)
      return false;
    const int64_t rows[3] = {I, I, H}, kbs[3] = {H / 256, H / 256, I / 256};
    Arg c[3], s[3];
    for (int p = 0; p < 3; ++p) {
      c[p] = dev(PyTuple_GET_ITEM(a[3], p), kU8, E, rows[p], kbs[p], (int64_t)128);
      s[p] = dev(PyTuple_GET_ITEM(a[4], p), kI16, E, rows[p], kbs[p]);
      if (!c[p].ok || !s[p].ok) return false;
    }
    const Arg x = dev(a[5], kF32, t, H), idx = dev(a[6], kI32, t, topk), w = dev(a[7], kF32, t, topk), out = dev(a[8], kF32, t, H),
              ws = dev_any(a[9], kU8);
    if (!x.ok || !idx.ok || !w.ok || !out.ok || !ws.ok) return false;
    tq_experts ex{};
    ex.n_experts = (int32_t)E;
    ex.hidden = (int32_t)H;
    ex.inter = (int32_t)I;
    ex.gate_codes = (uint8_t*)c[0].ptr;
    ex.gate_scales = (uint16_t*)s[0].ptr;
    ex.up_codes = (uint8_t*)c[1].ptr;
    ex.up_scales = (uint16_t*)s[1].ptr;
    ex.down_codes = (uint8_t*)c[2].ptr;
    ex.down_scales = (uint16_t*)s[2].ptr;
    for (int p = 0; p < 3; ++p) {
      ex.stride_codes[p] = rows[p] * kbs[p] * 128;
      ex.stride_scales[p] = rows[p] * kbs[p];
    }
    const size_t wsn = (size_t)THPVariable_Unpack(a[9]).numel();
    *st = unlocked([&] {
      return api.moe_grouped(&ex, (const float*)x.ptr, t, (const int32_t*)idx.ptr, (const float*)w.ptr, (int32_t)topk,
                             (float*)out.ptr, ws.ptr, wsn, (int32_t)flags, (void*)stream);
    });
    return true;
  });
}

// bind(addresses of the C entry points, in the order of Api)
PyObject* py_bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  int64_t v[6];
  if (n != 6) {
    PyErr_SetString(PyExc_TypeError, "bind: six addresses");
    return nullptr;
  }
  for (int i = 0; i < 6; ++i)
    if (!to_i64(a[i], &v[i])) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "bind: an address is not an int");
      return nullptr;
    }
  api.quantize_act = reinterpret_cast<decltype(api.quantize_act)>(v[0]);
  api.gemv = reinterpret_cast<decltype(api.gemv)>(v[1]);
  api.gemv_f32 = reinterpret_cast<decltype(api.gemv_f32)>(v[2]);
  api.gemv2 = reinterpret_cast<decltype(api.gemv2)>(v[3]);
  api.gemv_mx = reinterpret_cast<decltype(api.gemv_mx)>(v[4]);
  api.moe_grouped = reinterpret_cast<decltype(api.moe_grouped)>(v[5]);
  Py_RETURN_NONE;
}

#define TQ_PY(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_##name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {TQ_PY(bind),  TQ_PY(quantize_act), TQ_PY(gemv),        TQ_PY(gemv_f32),
                         TQ_PY(gemv2), TQ_PY(gemv_mx),      TQ_PY(moe_grouped), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tqpy", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__tqpy() { return PyModule_Create(&module); }
