// Argument marshalling of the four entry points that a program calls once or more for every layer (routing with and without the
// normalisation, forward, backward), for binding.py: the checks and addresses of up to thirty tensors and the call itself.  In
// Python these are 0.2 us a tensor and 0.1 us an argument, 7 us of a call that launches two kernels.  Nothing is kept from one call
// for the next but the addresses of the library's functions.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <dlfcn.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <exception>
#include <type_traits>

#include "btx_moe.h"

namespace {

struct Library {
  decltype(&btx_moe_route_workspace_bytes) route_bytes;
  decltype(&btx_moe_route) route;
  decltype(&btx_moe_norm_route) norm_route;
  decltype(&btx_moe_ff_forward_workspace_bytes) forward_bytes;
  decltype(&btx_moe_ff_forward) forward;
  decltype(&btx_moe_ff_backward_workspace_bytes) backward_bytes;
  decltype(&btx_moe_ff_backward) backward;
} lib{};

struct PyError {};                       // a Python exception has been set
[[noreturn]] void fail(PyObject* type, const char* what) {
  PyErr_SetString(type, what);
  throw PyError{};
}
void require(bool ok, const char* what) {
  if (!ok) fail(PyExc_AssertionError, what);
}

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) fail(PyExc_TypeError, "a tensor is expected");
  return THPVariable_Unpack(o);
}
// stacked expert matrices: each [rows, cols] matrix contiguous, the experts any distance apart
bool is_stacked(const at::Tensor& w) {
  return w.dim() == 3 && w.stride(2) == 1 && w.stride(1) == w.size(2) && w.stride(0) >= w.size(1) * w.size(2);
}
int64_t stacked(const at::Tensor& w) {
  require(is_stacked(w), "stacked expert matrices only");
  return w.stride(0);
}
// device address (None: NULL)
void* address(PyObject* o, bool or_stacked = false) {
  if (o == Py_None) return nullptr;
  const at::Tensor& t = tensor(o);
  require(t.is_cuda() && (t.is_contiguous() || (or_stacked && is_stacked(t))), "device-resident contiguous tensors only");
  return t.data_ptr();
}
template <typename T> T* address_of(PyObject* o) { return static_cast<T*>(address(o)); }
int dtype_code(const at::Tensor& t) {
  if (t.scalar_type() == at::kFloat) return BTX_F32;
  if (t.scalar_type() == at::kBFloat16) return BTX_BF16;
  fail(PyExc_TypeError, "unsupported dtype");
}
const at::Tensor& matrix(PyObject* o) {
  const at::Tensor& t = tensor(o);
  if (t.dim() != 2) fail(PyExc_ValueError, "a matrix is expected");
  return t;
}
// Shapes and strides of the experts that x goes through.  The library takes one expert stride for W1 and W3, and one dtype
struct Experts {
  int64_t T, d, E, f, s13, s2;
  Experts(const at::Tensor& x, const at::Tensor& W1, const at::Tensor& W3, const at::Tensor& W2)
      : T(x.size(0)), d(x.size(1)), E(0), f(0), s13(stacked(W1)), s2(stacked(W2)) {
    E = W1.size(0);
    f = W1.size(2);
    require(W1.size(1) == d && W3.sizes() == W1.sizes() && W2.size(0) == E && W2.size(1) == f && W2.size(2) == d &&
                W1.scalar_type() == x.scalar_type() && W3.scalar_type() == x.scalar_type() && W2.scalar_type() == x.scalar_type(),
            "W1, W3 [E, d, f] and W2 [E, f, d] of x's dtype");
    require(E == 1 || (is_stacked(W3) && W3.stride(0) == s13), "W3 is stacked like W1");
  }
};
int64_t integer(PyObject* o) {
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw PyError{};
  return v;
}
int int32(PyObject* o) { return (int)integer(o); }
float real(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw PyError{};
  return (float)v;
}
// out: attributes of a Routing
struct RoutingPtrs {
  void* at[10];
  int k;
  RoutingPtrs(PyObject* r, const char* const* names, int n) : k(0) {
    for (int i = 0; i < n; ++i) {
      PyObject* o = PyObject_GetAttrString(r, names[i]);
      if (!o) throw PyError{};
      try {
        at[i] = address(o);
        if (i == 0) k = (int)matrix(o).size(1);          // topk_idx
      } catch (...) {
        Py_DECREF(o);
        throw;
      }
      Py_DECREF(o);                                      // the Routing holds on to it
    }
  }
};

// The call with this workspace, or, where it is too small or there is none, minus the bytes that one has to have
template <typename Call> PyObject* with_workspace(PyObject* workspace, size_t bytes, Call call) {
  if (workspace != Py_None) {
    const at::Tensor& w = tensor(workspace);
    if ((size_t)w.numel() * w.element_size() >= bytes) {
      void* const at = address(workspace);
      const size_t numel = (size_t)w.numel();
      int status;
      Py_BEGIN_ALLOW_THREADS
      status = call(at, numel);
      Py_END_ALLOW_THREADS
      return PyLong_FromLong(status);
    }
  }
  return PyLong_FromLongLong(-(long long)std::max<size_t>(bytes, 256));
}

// arguments by position; Python exceptions and C++ ones end here
template <typename Body> PyObject* guarded(Py_ssize_t n, Py_ssize_t expected, Body body) {
  try {
    if (!lib.route) fail(PyExc_RuntimeError, "the library is not loaded");
    if (n != expected) fail(PyExc_TypeError, "wrong number of arguments");
    return body();
  } catch (const PyError&) {
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
  }
  return nullptr;
}

const char* const kRouting[10] = {"topk_idx", "gates", "probs", "counts", "offsets", "perm", "inv_pos", "gate_sum", "prob_sum", "lb_loss"};

// x, W_router, b_router, U, k, route_mode, lb_mode, lb_alpha, tau, capacity_factor, routing, workspace, stream
PyObject* route(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 13, [&] {
    const at::Tensor &x = matrix(a[0]), &W = matrix(a[1]);
    const int T = (int)x.size(0), d = (int)x.size(1), E = (int)W.size(1), k = int32(a[4]);
    require(W.size(0) == d && W.scalar_type() == at::kFloat, "W_router is [d, E] fp32");
    const int dt = dtype_code(x), mode = int32(a[5]), lb_mode = int32(a[6]);
    const float alpha = real(a[7]), tau = real(a[8]), cf = real(a[9]);
    const RoutingPtrs r(a[10], kRouting, 10);
    const void* const xp = address(a[0]);
    const float *Wp = address_of<float>(a[1]), *bp = address_of<float>(a[2]), *Up = address_of<float>(a[3]);
    void* const stream = reinterpret_cast<void*>(integer(a[12]));
    return with_workspace(a[11], lib.route_bytes(T, d, E, k), [&](void* ws, size_t bytes) {
      return lib.route(xp, dt, Wp, bp, Up, T, d, E, k, mode, lb_mode, alpha, tau, cf, (int32_t*)r.at[0], (float*)r.at[1], (float*)r.at[2],
                       (int32_t*)r.at[3], (int32_t*)r.at[4], (int32_t*)r.at[5], (int32_t*)r.at[6], (float*)r.at[7], (float*)r.at[8],
                       (float*)r.at[9], ws, bytes, stream);
    });
  });
}

// h, gain, eps, xn, rstd, and route()'s from W_router on
PyObject* norm_route(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 17, [&] {
    const at::Tensor &h = matrix(a[0]), &gain = tensor(a[1]), &W = matrix(a[5]);
    const int T = (int)h.size(0), d = (int)h.size(1), E = (int)W.size(1), k = int32(a[8]);
    require(W.size(0) == d && W.scalar_type() == at::kFloat, "W_router is [d, E] fp32");
    require(gain.dim() == 1 && gain.size(0) == d && gain.scalar_type() == at::kFloat, "gain is [d] fp32");
    const int dt = dtype_code(h), mode = int32(a[9]), lb_mode = int32(a[10]);
    const float eps = real(a[2]), alpha = real(a[11]), tau = real(a[12]), cf = real(a[13]);
    const RoutingPtrs r(a[14], kRouting, 10);
    const void* const hp = address(a[0]);
    void* const xn = address(a[3]);
    float* const rstd = address_of<float>(a[4]);
    const float *gp = address_of<float>(a[1]), *Wp = address_of<float>(a[5]), *bp = address_of<float>(a[6]), *Up = address_of<float>(a[7]);
    void* const stream = reinterpret_cast<void*>(integer(a[16]));
    return with_workspace(a[15], lib.route_bytes(T, d, E, k), [&](void* ws, size_t bytes) {
      return lib.norm_route(hp, dt, gp, eps, xn, rstd, Wp, bp, Up, T, d, E, k, mode, lb_mode, alpha, tau, cf, (int32_t*)r.at[0],
                            (float*)r.at[1], (float*)r.at[2], (int32_t*)r.at[3], (int32_t*)r.at[4], (int32_t*)r.at[5], (int32_t*)r.at[6],
                            (float*)r.at[7], (float*)r.at[8], (float*)r.at[9], ws, bytes, stream);
    });
  });
}

// x, W1, W3, W2, routing, residual, out, h1, h3, workspace, stream
PyObject* forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 11, [&] {
    const at::Tensor &x = matrix(a[0]), &W1 = tensor(a[1]), &W3 = tensor(a[2]), &W2 = tensor(a[3]);
    const Experts w(x, W1, W3, W2);
    static const char* const names[] = {"topk_idx", "gates", "offsets", "perm", "inv_pos"};
    const RoutingPtrs r(a[4], names, 5);
    const int dt = dtype_code(x), k = r.k;
    const void *xp = address(a[0]), *w1 = address(a[1], true), *w3 = address(a[2], true), *w2 = address(a[3], true), *res = address(a[5]);
    void *out = address(a[6]), *h1 = address(a[7]), *h3 = address(a[8]);
    void* const stream = reinterpret_cast<void*>(integer(a[10]));
    return with_workspace(a[9], lib.forward_bytes((int)w.T, (int)w.d, (int)w.f, (int)w.E, k, dt), [&](void* ws, size_t bytes) {
      return lib.forward(xp, w1, w3, w2, dt, w.s13, w.s2, (int)w.T, (int)w.d, (int)w.f, (int)w.E, k, (const float*)r.at[1], (const int32_t*)r.at[2],
                         (const int32_t*)r.at[3], (const int32_t*)r.at[4], res, out, h1, h3, ws, bytes, stream);
    });
  });
}

// dY, x, W_router, W1, W3, W2, routing, h1, h3, route_mode, lb_mode, lb_alpha, lb_grad_scale, flags, noise, tau, dX, dW_router, db_router,
// dW1, dW3, dW2, weight gradients in fp32, workspace, stream
PyObject* backward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 25, [&] {
    const at::Tensor &x = matrix(a[1]), &W1 = tensor(a[3]), &W3 = tensor(a[4]), &W2 = tensor(a[5]);
    const Experts w(x, W1, W3, W2);
    const bool dw_f32 = PyObject_IsTrue(a[22]) == 1;
    for (int i = 0; i < 3; ++i) {
      if (a[19 + i] == Py_None) continue;
      const at::Tensor &dW = tensor(a[19 + i]), &W = tensor(a[3 + i]);
      require(dW.sizes() == W.sizes() && stacked(dW) == stacked(W), "dW is stacked like W");
      require(dW.scalar_type() == (dw_f32 ? at::kFloat : at::kBFloat16), "dW is of dW_dtype");
    }
    static const char* const names[] = {"topk_idx", "gates", "probs", "offsets", "perm", "inv_pos", "gate_sum", "prob_sum", "counts"};
    const RoutingPtrs r(a[6], names, 9);
    const int dt = dtype_code(x), k = r.k, mode = int32(a[9]), lb_mode = int32(a[10]), dw_dt = dw_f32 ? BTX_F32 : BTX_BF16;
    const float alpha = real(a[11]), scale = real(a[12]), tau = real(a[15]);
    const unsigned flags = (unsigned)integer(a[13]);
    const void *dY = address(a[0]), *xp = address(a[1]), *w1 = address(a[3], true), *w3 = address(a[4], true), *w2 = address(a[5], true);
    const void *h1 = address(a[7]), *h3 = address(a[8]);
    const float *Wr = address_of<float>(a[2]), *noise = address_of<float>(a[14]);
    void *dX = address(a[16]), *dW1 = address(a[19], true), *dW3 = address(a[20], true), *dW2 = address(a[21], true);
    float *dWr = address_of<float>(a[17]), *dbr = address_of<float>(a[18]);
    void* const stream = reinterpret_cast<void*>(integer(a[24]));
    return with_workspace(a[23], lib.backward_bytes((int)w.T, (int)w.d, (int)w.f, (int)w.E, k, dt), [&](void* ws, size_t bytes) {
      return lib.backward(dY, xp, Wr, w1, w3, w2, dt, w.s13, w.s2, (int)w.T, (int)w.d, (int)w.f, (int)w.E, k, mode, lb_mode, alpha, scale, flags, noise,
                          tau, (const int32_t*)r.at[0], (const float*)r.at[1], (const float*)r.at[2], (const int32_t*)r.at[3],
                          (const int32_t*)r.at[4], (const int32_t*)r.at[5], (const float*)r.at[6], (const float*)r.at[7],
                          (const int32_t*)r.at[8], h1, h3, dX, dWr, dbr, dW1, dW3, dW2, dw_dt, ws, bytes, stream);
    });
  });
}

// path of the library, which is loaded already
PyObject* bind(PyObject*, PyObject* path) {
  const char* p = PyUnicode_AsUTF8(path);
  if (!p) return nullptr;
  void* const handle = dlopen(p, RTLD_NOW | RTLD_NOLOAD);
  Library l{};
  auto find = [&](auto& to, const char* name) {
    to = handle ? reinterpret_cast<std::remove_reference_t<decltype(to)>>(dlsym(handle, name)) : nullptr;
    return to != nullptr;
  };
  if (!find(l.route_bytes, "btx_moe_route_workspace_bytes") || !find(l.route, "btx_moe_route") || !find(l.norm_route, "btx_moe_norm_route") ||
      !find(l.forward_bytes, "btx_moe_ff_forward_workspace_bytes") || !find(l.forward, "btx_moe_ff_forward") ||
      !find(l.backward_bytes, "btx_moe_ff_backward_workspace_bytes") || !find(l.backward, "btx_moe_ff_backward")) {
    PyErr_Format(PyExc_RuntimeError, "%s does not have the library's entry points", p);
    return nullptr;
  }
  lib = l;
  Py_RETURN_NONE;
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"bind", bind, METH_O, nullptr}, FAST(route), FAST(norm_route), FAST(forward), FAST(backward), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
