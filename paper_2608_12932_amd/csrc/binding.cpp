// Native fast path of the Python binding: the hot entry points of w4a8.h on
// torch tensors, on the current stream.
//
// The calls of the decode and verify steps run for 2 - 10 us on the GPU, and
// argument checks, the stream lookup, the output's allocation and the
// foreign-function call took 9 - 18 us of interpreted Python per call, so
// consecutive calls were bound by the host.  Here they take about 1 us
// beyond the launches.
//
// Each function returns None for anything but the plain case (a tensor
// subclass, another stream's workspace, a wrong type or shape ...): the
// interpreted path in __init__.py then takes the call, grows the workspace
// or raises the error.  An int is a nonzero status of the library call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/zeros.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "w4a8.h"

namespace {

// a plain, contiguous device tensor of the given type; nullptr otherwise
const at::Tensor* plain(PyObject* o, at::ScalarType type) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  return t.is_cuda() && t.scalar_type() == type && t.is_contiguous() ? &t : nullptr;
}

bool is_int(PyObject* o) { return PyLong_CheckExact(o); }
int64_t as_int(PyObject* o) { return PyLong_AsLongLong(o); }  // -1 with an error set past 64 bits

hipStream_t current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// Runs f without the interpreter's lock, also where it throws: launches may
// wait for room in the queue, allocations for the allocator's lock, whose
// holder may itself be waiting for the interpreter's.
template <class F>
w4a8_status without_gil(F f) {
  struct Released {
    PyThreadState* state = PyEval_SaveThread();
    ~Released() { PyEval_RestoreThread(state); }
  } released;
  return f();
}

// linear(swiglu, x, w_packed, w_scale, N, x_scale, scale_mode, out_kind, out,
//        workspace, workspace_stream, is_workspace)
// workspace_stream: the stream that a Workspace's buffer (is_workspace)
// belongs to, None while it is empty or that is not known (a copy's).  A
// negative int is the size that an
// otherwise plain call's Workspace has to grow to.
PyObject* linear(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 12 || !is_int(a[0]) || !is_int(a[4]) || !is_int(a[6]) || !is_int(a[7])) Py_RETURN_NONE;
  const bool swiglu = as_int(a[0]) != 0;
  const int64_t N = as_int(a[4]), mode = as_int(a[6]), kind = as_int(a[7]);
  if (PyErr_Occurred()) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  if (mode < 0 || mode > 1 || kind < 0 || kind > 2 || N <= 0) Py_RETURN_NONE;
  const at::Tensor* x = plain(a[1], at::kBFloat16);
  const at::Tensor* xs = nullptr;
  int in_kind = W4A8_IN_BF16;
  if (!x) {
    x = plain(a[1], at::kChar);
    xs = x ? plain(a[5], at::kFloat) : nullptr;
    if (!xs) Py_RETURN_NONE;
    in_kind = W4A8_IN_I8;
  }
  const at::Tensor* wp = plain(a[2], at::kByte);
  if (!wp || x->dim() != 2) Py_RETURN_NONE;
  const at::Tensor* ws = nullptr;
  if (a[3] != Py_None && !(ws = plain(a[3], mode == W4A8_SCALE_CHANNEL_F32 ? at::kFloat : at::kHalf))) Py_RETURN_NONE;
  const int64_t M = x->size(0), K = x->size(1), cols = swiglu ? N / 2 : N;
  const at::ScalarType out_type = kind == W4A8_OUT_BF16 ? at::kBFloat16 : kind == W4A8_OUT_F32 ? at::kFloat : at::kInt;

  const at::Tensor* out = nullptr;
  if (a[8] != Py_None) {
    out = plain(a[8], out_type);
    if (!out || out->dim() != 2 || out->size(0) != M || out->size(1) != cols) Py_RETURN_NONE;
  }

  const size_t need = swiglu ? w4a8_linear_swiglu_workspace_bytes(M, N, K, (int)mode, in_kind)
                             : w4a8_linear_workspace_bytes(M, N, K, (int)mode, in_kind);
  const hipStream_t stream = current_stream();
  void* wk = nullptr;
  size_t wk_bytes = 0;
  const bool temporary = need && a[9] == Py_None && a[11] != Py_True;
  if (need && !temporary) {
    const at::Tensor* buf = plain(a[9], at::kByte);
    if (!buf) Py_RETURN_NONE;
    if (a[11] == Py_True) {  // a Workspace: of this stream (its memory is ordered on it), and large enough
      if (a[10] != Py_None && (!is_int(a[10]) || PyLong_AsVoidPtr(a[10]) != (void*)stream)) {
        PyErr_Clear();
        Py_RETURN_NONE;
      }
      if ((size_t)buf->numel() < need) return PyLong_FromLongLong(-(long long)need);
      if (a[10] == Py_None) Py_RETURN_NONE;
    }
    wk = buf->data_ptr();
    wk_bytes = (size_t)buf->numel();
  }

  const void *xp = x->data_ptr(), *sp = ws ? ws->data_ptr() : nullptr;
  const float* xsp = xs ? static_cast<const float*>(xs->data_ptr()) : nullptr;
  const uint8_t* wpp = static_cast<const uint8_t*>(wp->data_ptr());
  at::Tensor y;
  const w4a8_status s = without_gil([&] {
    y = out ? *out : at::empty({M, cols}, x->options().dtype(out_type));
    at::Tensor tmp;  // released to the allocator on this stream, which orders its next use
    if (temporary) {
      tmp = at::zeros({(int64_t)need}, x->options().dtype(at::kByte));
      wk = tmp.data_ptr();
      wk_bytes = need;
    }
    return (swiglu ? w4a8_linear_swiglu : w4a8_linear)(xp, in_kind, xsp, M, K, wpp, sp, (int)mode, N, y.data_ptr(), (int)kind,
                                                       wk, wk_bytes, stream);
  });
  if (s != W4A8_OK) return PyLong_FromLong(s);
  if (out) return Py_NewRef(a[8]);
  return THPVariable_Wrap(std::move(y));
  END_HANDLE_TH_ERRORS
}

PyObject* pair(at::Tensor q, at::Tensor s) {
  PyObject* t = PyTuple_New(2);
  if (!t) return nullptr;
  PyTuple_SET_ITEM(t, 0, THPVariable_Wrap(std::move(q)));
  PyTuple_SET_ITEM(t, 1, THPVariable_Wrap(std::move(s)));
  return t;
}

// quantize(x) / rmsnorm_quantize(x, gamma, eps)
PyObject* quantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  const at::Tensor* x = n == 1 || n == 3 ? plain(a[0], at::kBFloat16) : nullptr;
  if (!x || x->dim() != 2) Py_RETURN_NONE;
  const int64_t M = x->size(0), K = x->size(1);
  const at::Tensor* g = nullptr;
  float eps = 0.0f;
  if (n == 3) {
    g = plain(a[1], at::kBFloat16);
    if (!g || g->dim() != 1 || g->size(0) != K || !PyFloat_CheckExact(a[2])) Py_RETURN_NONE;
    eps = (float)PyFloat_AS_DOUBLE(a[2]);
  }
  at::Tensor q, s;
  const uint16_t *xp = static_cast<const uint16_t*>(x->data_ptr()), *gp = g ? static_cast<const uint16_t*>(g->data_ptr()) : nullptr;
  const hipStream_t stream = current_stream();
  const w4a8_status st = without_gil([&] {
    q = at::empty({M, K}, x->options().dtype(at::kChar));
    s = at::empty({M}, x->options().dtype(at::kFloat));
    int8_t* qp = static_cast<int8_t*>(q.data_ptr());
    float* sp = static_cast<float*>(s.data_ptr());
    return g ? w4a8_rmsnorm_quantize_act(xp, gp, eps, M, K, qp, sp, stream) : w4a8_quantize_act(xp, M, K, qp, sp, stream);
  });
  if (st != W4A8_OK) return PyLong_FromLong(st);
  return pair(std::move(q), std::move(s));
  END_HANDLE_TH_ERRORS
}

// flow_step(x, v_new, v_cache, dt, stats, repeat) -> the stats tensor, True
// without stats
PyObject* flow_step(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 6 || !PyFloat_CheckExact(a[3]) || !PyBool_Check(a[4]) || !is_int(a[5])) Py_RETURN_NONE;
  const at::Tensor *x = plain(a[0], at::kFloat), *c = plain(a[2], at::kBFloat16), *v = nullptr;
  if (!x || !c || x->dim() != 2) Py_RETURN_NONE;
  const int64_t B = x->size(0), len = x->size(1), repeat = as_int(a[5]);
  if (PyErr_Occurred()) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  auto fits = [&](const at::Tensor& t) { return t.dim() == 2 && t.size(0) == B && t.size(1) == len; };
  if (!fits(*c)) Py_RETURN_NONE;
  if (a[1] != Py_None) {
    v = plain(a[1], at::kBFloat16);
    if (!v || !fits(*v)) Py_RETURN_NONE;
  }
  const bool stats = a[4] == Py_True;
  at::Tensor st;
  float* xp = static_cast<float*>(x->data_ptr());
  const uint16_t* vp = v ? static_cast<const uint16_t*>(v->data_ptr()) : nullptr;
  uint16_t* cp = static_cast<uint16_t*>(c->data_ptr());
  const float dt = (float)PyFloat_AS_DOUBLE(a[3]);
  const hipStream_t stream = current_stream();
  const w4a8_status s = without_gil([&] {
    if (stats) st = at::empty({B, 4}, x->options().dtype(at::kDouble));
    double* stp = stats ? static_cast<double*>(st.data_ptr()) : nullptr;
    return w4a8_flow_step(xp, vp, cp, B, len, dt, repeat, stp, stream);
  });
  if (s != W4A8_OK) return PyLong_FromLong(s);
  if (!stats) Py_RETURN_TRUE;
  return THPVariable_Wrap(std::move(st));
  END_HANDLE_TH_ERRORS
}

#define FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL
PyMethodDef methods[] = {{"linear", FAST(linear), nullptr},
                         {"quantize", FAST(quantize), nullptr},
                         {"flow_step", FAST(flow_step), nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&module); }
