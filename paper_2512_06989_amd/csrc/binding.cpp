// Host side of the Python binding: from tensors to a call of the C ABI, as a CPython module.
//
// A decoding step lasts about 17 us on the GPU; checking six tensors and filling a descriptor
// through ctypes took 26 us on the host, so the calls of a serving or training loop are
// marshalled here (6.5 us with the two launches; forward + backward 85 -> 25, a module step
// 148 -> 70).  Each function checks its arguments, allocates what the caller left
// out, calls the library on the current (or given) stream and returns
//   the result      where all went well,
//   an int          where the library refused (its status),
//   None            where an argument is not what the kernels assume: mhffn.py then runs its
//                   own checks, which say what is wrong.
// Nothing is kept between calls.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>

#include <optional>
#include <vector>

#include "../../include/mhffn.h"

namespace {

// Thrown by a check; becomes None.
struct Refused {};

inline void require(bool ok) {
  if (!ok) throw Refused{};
}

const at::Tensor& tensor(PyObject* o) {
  require(THPVariable_Check(o));
  return THPVariable_Unpack(o);
}

bool same_kind(const at::Tensor& t, const at::Tensor& like) {
  return t.scalar_type() == like.scalar_type() && t.device() == like.device();
}

void dense(const at::Tensor& t, at::IntArrayRef shape, at::ScalarType type, at::Device device) {
  require(t.sizes() == shape && t.scalar_type() == type && t.device() == device && t.is_contiguous());
}

// Row tensor [N, d_model] like X: its row stride in elements (d_model for fewer than two rows)
int64_t rows(const at::Tensor& t, const at::Tensor& x) {
  require(t.dim() == 2 && t.size(0) == x.size(0) && t.size(1) == x.size(1) && same_kind(t, x));
  if (t.size(0) < 2) {
    require(t.size(0) == 0 || t.stride(1) == 1);
    return t.size(1);
  }
  require(t.stride(1) == 1 && t.stride(0) >= t.size(1));
  return t.stride(0);
}

// Uninitialised [N, d_model] with X's row stride (the kernels index dX with ld_x)
at::Tensor empty_rows_like(const at::Tensor& x) {
  if (x.size(0) < 2 || x.is_contiguous()) return at::empty(x.sizes(), x.options());
  return at::empty_strided(x.sizes(), x.strides(), x.options());
}

void* data(const at::Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }

// The tensors every call shares, and the descriptor they give (ld_y still d_model)
struct Problem {
  at::Tensor x, wg, wu, wd, route;
  mhffn_desc d;

  Problem(PyObject* X, PyObject* Wg, PyObject* Wu, PyObject* Wd, PyObject* R, double eps, long mode)
      : x(tensor(X)), wg(tensor(Wg)), wu(tensor(Wu)), wd(tensor(Wd)), route(tensor(R)) {
    require(wg.dim() == 4 && x.dim() == 2);
    const int64_t H = wg.size(0), E = wg.size(1), de = wg.size(2), dh = wg.size(3);
    require(x.size(1) == H * dh);
    const auto type = x.scalar_type();
    require(type == at::kBFloat16 || type == at::kFloat);
    for (const at::Tensor* w : {&wg, &wu, &wd}) dense(*w, wg.sizes(), type, x.device());
    if (mode == MHFFN_ROUTE_PARAMS) dense(route, {H, dh, E}, type, x.device());
    else dense(route, {x.size(0), H, E}, at::kFloat, x.device());
    d.n_tokens = x.size(0);
    d.n_heads = (int32_t)H;
    d.d_head = (int32_t)dh;
    d.n_sub = (int32_t)E;
    d.d_sub = (int32_t)de;
    d.ld_x = rows(x, x);
    d.ld_y = H * dh;
    d.dtype = type == at::kBFloat16 ? MHFFN_BF16 : MHFFN_F32;
    d.route_mode = (int32_t)mode;
    d.eps = (float)eps;
  }
};

// None: the current stream of the current device
hipStream_t stream_of(PyObject* stream) {
  if (stream != Py_None) {
    void* s = PyLong_AsVoidPtr(stream);
    require(!PyErr_Occurred());
    return static_cast<hipStream_t>(s);
  }
  return c10::hip::getCurrentHIPStream().stream();
}

// Makes a stream the current one of the tensors' device for as long as it lives
struct OnStream {
  c10::hip::HIPStream before;
  OnStream(hipStream_t stream, const at::Tensor& x) : before(c10::hip::getCurrentHIPStream(x.device().index())) {
    c10::hip::setCurrentHIPStream(c10::hip::getStreamFromExternal(stream, x.device().index()));
  }
  ~OnStream() { c10::hip::setCurrentHIPStream(before); }
  OnStream(const OnStream&) = delete;
  OnStream& operator=(const OnStream&) = delete;
};

// The caller's workspace, or a fresh one of the size the library asks for.  It is given back when
// the call returns, so it has to belong to the stream the kernels run on: only what follows
// them there may get its memory.
struct Workspace {
  at::Tensor t;
  size_t bytes = 0;
  Workspace(const Problem& p, int op, PyObject* given, PyObject* stream) {
    if (given != Py_None) {
      t = tensor(given);
    } else if (const size_t need = mhffn_workspace_bytes(&p.d, op)) {
      std::optional<OnStream> guard;
      if (stream != Py_None && p.x.is_cuda()) guard.emplace(stream_of(stream), p.x);
      t = at::empty({(int64_t)need}, p.x.options().dtype(at::kByte));
    }
    if (t.defined()) bytes = (size_t)t.numel() * t.element_size();
  }
  void* ptr() const { return data(t); }
};

double number(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  require(!(v == -1.0 && PyErr_Occurred()));
  return v;
}
long integer(PyObject* o) {
  const long v = PyLong_AsLong(o);
  require(!(v == -1 && PyErr_Occurred()));
  return v;
}

PyObject* status(int rc) { return PyLong_FromLong(rc); }

// Runs `body`, which throws Refused for None; any other exception becomes the Python exception
// that torch itself raises for it (a failed allocation: torch.OutOfMemoryError)
template <typename F>
PyObject* guarded(F&& body) {
  HANDLE_TH_ERRORS
  try {
    return body();
  } catch (const Refused&) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  END_HANDLE_TH_ERRORS
}

// Named outputs of a call: a copy of the caller's dict (or an empty one)
struct Outputs {
  PyObject* dict;
  explicit Outputs(PyObject* given) : dict(given == Py_None ? PyDict_New() : PyDict_Copy(given)) {
    if (!dict) throw Refused{};
  }
  ~Outputs() { Py_XDECREF(dict); }
  Outputs(const Outputs&) = delete;
  Outputs& operator=(const Outputs&) = delete;
  // what the caller gave under `key`: undefined where nothing or None
  at::Tensor get(const char* key) const {
    PyObject* o = PyDict_GetItemString(dict, key);
    return o && o != Py_None ? tensor(o) : at::Tensor();
  }
  bool has(const char* key) const { return PyDict_GetItemString(dict, key) != nullptr; }
  void set(const char* key, const at::Tensor& t) {
    PyObject* o = THPVariable_Wrap(t);
    require(o && PyDict_SetItemString(dict, key, o) == 0);
    Py_DECREF(o);
  }
  PyObject* release() {
    PyObject* o = dict;
    dict = nullptr;
    return o;
  }
};

// One gradient: its name, the parameter it belongs to (undefined: dX, row-strided like X)
struct Grad {
  const char* key;
  const at::Tensor* like;
};

// The gradient tensors of a backward call: the caller's, checked against what the kernels
// assume, and fresh ones for the rest of `want`
template <size_t G>
void gradients(const Problem& p, PyObject* want, Outputs& out, const Grad (&grads)[G], at::Tensor (&t)[G]) {
  require(PyTuple_Check(want) || PyList_Check(want));
  for (Py_ssize_t i = 0; i < PySequence_Fast_GET_SIZE(want); ++i) {
    PyObject* k = PySequence_Fast_GET_ITEM(want, i);
    size_t j = 0;
    while (j < G && !(PyUnicode_Check(k) && PyUnicode_CompareWithASCIIString(k, grads[j].key) == 0)) ++j;
    if (j == G) {   // not a gradient of this call: what the caller gave under that name, if anything
      require(PyDict_Contains(out.dict, k) == 1);
      continue;
    }
    if (out.has(grads[j].key)) continue;
    out.set(grads[j].key, grads[j].like ? at::empty(grads[j].like->sizes(), grads[j].like->options())
                                        : empty_rows_like(p.x));
  }
  for (size_t j = 0; j < G; ++j) {
    t[j] = out.get(grads[j].key);
    if (!t[j].defined()) continue;
    if (grads[j].like) dense(t[j], grads[j].like->sizes(), grads[j].like->scalar_type(), grads[j].like->device());
    else require(rows(t[j], p.x) == p.d.ld_x || p.d.n_tokens < 2);
  }
}

// The interpreter lock, released for as long as it lives
struct Unlocked {
  PyThreadState* state = PyEval_SaveThread();
  Unlocked() = default;
  ~Unlocked() { PyEval_RestoreThread(state); }
  Unlocked(const Unlocked&) = delete;
  Unlocked& operator=(const Unlocked&) = delete;
};
// Calls the library with the lock released, as a foreign call would.  The arguments are plain
// values by then: a tensor without memory of its own (inside torch.func) throws when asked for
// its address.
template <typename... P, typename... A>
int unlocked(int (*call)(P...), A... args) {
  const Unlocked released;
  return call(args...);
}

// forward(X, W_gate, W_up, W_down, route, eps, mode, out, stream, workspace)
PyObject* forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    require(n == 10);
    Problem p(a[0], a[1], a[2], a[3], a[4], number(a[5]), integer(a[6]));
    const at::Tensor y = a[7] == Py_None ? at::empty(p.x.sizes(), p.x.options()) : tensor(a[7]);
    p.d.ld_y = rows(y, p.x);
    const Workspace ws(p, MHFFN_OP_FORWARD, a[9], a[8]);
    void* const stream = stream_of(a[8]);
    const int rc = unlocked(mhffn_forward, &p.d, data(p.x), data(p.wg), data(p.wu), data(p.wd), data(p.route),
                            data(y), ws.ptr(), ws.bytes, stream);
    return rc ? status(rc) : THPVariable_Wrap(y);
  });
}

// forward_static(X, W_gate, W_up, W_down, route, out, eps, mode, stream)
PyObject* forward_static(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    require(n == 9);
    Problem p(a[0], a[1], a[2], a[3], a[4], number(a[6]), integer(a[7]));
    const at::Tensor y = tensor(a[5]);
    p.d.ld_y = rows(y, p.x);
    void* const stream = stream_of(a[8]);
    const int rc = unlocked(mhffn_forward_static, &p.d, data(p.x), data(p.wg), data(p.wu), data(p.wd),
                            data(p.route), data(y), stream);
    return rc ? status(rc) : THPVariable_Wrap(y);
  });
}

// backward(X, W_gate, W_up, W_down, route, dY, eps, mode, want, workspace, out, stream, phase_events)
PyObject* backward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    require(n == 13);
    Problem p(a[0], a[1], a[2], a[3], a[4], number(a[6]), integer(a[7]));
    const at::Tensor dy = tensor(a[5]);
    p.d.ld_y = rows(dy, p.x);
    std::vector<void*> events;
    if (a[12] != Py_None) {
      require(PyList_Check(a[12]) || PyTuple_Check(a[12]));
      for (Py_ssize_t i = 0; i < PySequence_Fast_GET_SIZE(a[12]); ++i) {
        events.push_back(PyLong_AsVoidPtr(PySequence_Fast_GET_ITEM(a[12], i)));
        require(!PyErr_Occurred());
      }
    }
    Outputs out(a[10]);
    const Grad grads[5] = {{"dX", nullptr}, {"dW_gate", &p.wg}, {"dW_up", &p.wu}, {"dW_down", &p.wd}, {"d_route", &p.route}};
    at::Tensor t[5];
    gradients(p, a[8], out, grads, t);
    const Workspace ws(p, MHFFN_OP_BACKWARD, a[9], a[11]);
    void* const stream = stream_of(a[11]);
    const int rc = unlocked(mhffn_backward_phases, &p.d, data(p.x), data(p.wg), data(p.wu), data(p.wd),
                            data(p.route), data(dy), data(t[0]), data(t[1]), data(t[2]), data(t[3]), data(t[4]),
                            ws.ptr(), ws.bytes, stream, events.empty() ? nullptr : events.data(),
                            (int)events.size());
    return rc ? status(rc) : out.release();
  });
}

// module_forward(X, W_in, W_gate, W_up, W_down, W_r, W_out, eps, out, stream, workspace) -> (O, Q, S)
PyObject* module_forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    require(n == 11);
    Problem p(a[0], a[2], a[3], a[4], a[5], number(a[7]), MHFFN_ROUTE_PARAMS);
    const int64_t N = p.x.size(0), dm = p.x.size(1);
    const at::Tensor w_in = tensor(a[1]), w_out = tensor(a[6]);
    dense(w_in, {dm, dm}, p.x.scalar_type(), p.x.device());
    dense(w_out, {dm, dm}, p.x.scalar_type(), p.x.device());
    const char* keys[3] = {"O", "Q", "S"};
    at::Tensor t[3];
    for (int i = 0; i < 3; ++i) {
      PyObject* o = a[8] == Py_None ? nullptr : PyDict_GetItemString(a[8], keys[i]);
      t[i] = o ? tensor(o) : at::empty({N, dm}, p.x.options());
      if (i > 0) dense(t[i], {N, dm}, p.x.scalar_type(), p.x.device());
    }
    p.d.ld_y = rows(t[0], p.x);
    const Workspace ws(p, MHFFN_OP_MODULE_FORWARD, a[10], a[9]);
    void* const stream = stream_of(a[9]);
    const int rc = unlocked(mhffn_module_forward, &p.d, data(p.x), data(w_in), data(p.wg), data(p.wu),
                            data(p.wd), data(p.route), data(w_out), data(t[0]), data(t[1]), data(t[2]),
                            ws.ptr(), ws.bytes, stream);
    if (rc) return status(rc);
    PyObject* r = PyTuple_New(3);
    if (!r) return nullptr;
    for (int i = 0; i < 3; ++i) PyTuple_SET_ITEM(r, i, THPVariable_Wrap(t[i]));
    return r;
  });
}

// module_backward(X, W_in, W_gate, W_up, W_down, W_r, W_out, Q, S, dO, eps, want, out, stream, workspace)
PyObject* module_backward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    require(n == 15);
    Problem p(a[0], a[2], a[3], a[4], a[5], number(a[10]), MHFFN_ROUTE_PARAMS);
    const int64_t N = p.x.size(0), dm = p.x.size(1);
    const at::Tensor w_in = tensor(a[1]), w_out = tensor(a[6]), q = tensor(a[7]), s = tensor(a[8]), d_o = tensor(a[9]);
    for (const at::Tensor* w : {&w_in, &w_out}) dense(*w, {dm, dm}, p.x.scalar_type(), p.x.device());
    for (const at::Tensor* t : {&q, &s}) dense(*t, {N, dm}, p.x.scalar_type(), p.x.device());
    p.d.ld_y = rows(d_o, p.x);
    Outputs out(a[12]);
    const Grad grads[7] = {{"dX", nullptr}, {"dW_in", &w_in}, {"dW_gate", &p.wg}, {"dW_up", &p.wu},
                           {"dW_down", &p.wd}, {"dW_r", &p.route}, {"dW_out", &w_out}};
    at::Tensor t[7];
    gradients(p, a[11], out, grads, t);
    const Workspace ws(p, MHFFN_OP_MODULE_BACKWARD, a[14], a[13]);
    void* const stream = stream_of(a[13]);
    const int rc = unlocked(mhffn_module_backward, &p.d, data(p.x), data(w_in), data(p.wg), data(p.wu),
                            data(p.wd), data(p.route), data(w_out), data(q), data(s), data(d_o), data(t[0]),
                            data(t[1]), data(t[2]), data(t[3]), data(t[4]), data(t[5]), data(t[6]), ws.ptr(),
                            ws.bytes, stream);
    return rc ? status(rc) : out.release();
  });
}

#define MHFFN_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {MHFFN_METHOD(forward), MHFFN_METHOD(forward_static), MHFFN_METHOD(backward),
                         MHFFN_METHOD(module_forward), MHFFN_METHOD(module_backward), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host", "Argument marshalling of the mhffn binding.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host(void) { return PyModule_Create(&module); }
