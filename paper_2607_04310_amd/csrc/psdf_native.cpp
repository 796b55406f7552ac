// The Python calls of api.py in native code: argument checks, output and
// workspace tensors, and the C ABI call.  A call against a small map is over
// on the GPU in 8 us, less than the interpreter needs for its tensors and
// ctypes conversions (15 to 20 us a call), so it was the host that bounded
// it.  Nothing is kept between calls; an argument in any other form than the
// plain one (a float32 array, a contiguous float32 device tensor) goes through
// the conversions of api.py.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/device_lazy_init.h>

#include <cmath>
#include <cstring>
#include <exception>
#include <string>
#include <utility>

#include "psdf.h"

namespace {

struct PyError {};   // a Python exception is set

// Owned reference.
class Ref {
 public:
  explicit Ref(PyObject* p = nullptr) : p_(p) {}
  Ref(Ref&& o) noexcept : p_(o.p_) { o.p_ = nullptr; }
  Ref(const Ref&) = delete;
  Ref& operator=(Ref&& o) noexcept {
    std::swap(p_, o.p_);
    return *this;
  }
  ~Ref() { Py_XDECREF(p_); }
  PyObject* get() const { return p_; }
  PyObject* release() {
    PyObject* p = p_;
    p_ = nullptr;
    return p;
  }

 private:
  PyObject* p_;
};

Ref own(PyObject* p) {
  if (!p) throw PyError();
  return Ref(p);
}

PyObject* g_api = nullptr;   // the api module (its conversions and PsdfError)

// Interned attribute names.
struct Names {
  PyObject *ax, *ay, *bx, *by, *obst_off, *E, *M, *mbar, *staged, *eps, *eps_sat, *eta;
} g_n;

Ref attr(PyObject* o, PyObject* name) { return own(PyObject_GetAttr(o, name)); }

long as_long(PyObject* o) {
  const long v = PyLong_AsLong(o);
  if (v == -1 && PyErr_Occurred()) throw PyError();
  return v;
}
double as_double(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw PyError();
  return v;
}

// int(o) as a C int32 argument, float(o)
int32_t int_of(PyObject* o) {
  const Ref r = own(PyNumber_Long(o));
  const unsigned long v = PyLong_AsUnsignedLongMask(r.get());
  if (PyErr_Occurred()) throw PyError();
  return (int32_t)v;
}
float float_of(PyObject* o) { return (float)as_double(own(PyNumber_Float(o)).get()); }

// api.<name>(o)
Ref convert(const char* name, PyObject* o) {
  Ref f = own(PyObject_GetAttrString(g_api, name));
  return own(PyObject_CallOneArg(f.get(), o));
}

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_AttributeError, "'%s' object has no attribute 'data_ptr'",
                 Py_TYPE(o)->tp_name);
    throw PyError();
  }
  return THPVariable_Unpack(o);
}

template <class T>
T* data(const at::Tensor& t) {
  return static_cast<T*>(const_cast<void*>(static_cast<const void*>(t.data_ptr())));
}

// The footprint's vertices: a C-contiguous float32 buffer of 2 m values as it
// is, anything else through api._fp_array.
class Footprint {
 public:
  explicit Footprint(PyObject* o) {
    if (take(o)) return;
    const Ref conv = convert("_fp_array", o);   // the buffer keeps it alive
    if (!take(conv.get())) {
      PyErr_SetString(PyExc_TypeError, "footprint: not an array of float32 vertices");
      throw PyError();
    }
  }
  ~Footprint() {
    if (held_) PyBuffer_Release(&b_);
  }
  const float* xy() const { return static_cast<const float*>(b_.buf); }
  int m() const { return (int)(b_.len / (Py_ssize_t)(2 * sizeof(float))); }

 private:
  bool take(PyObject* o) {
    if (PyObject_GetBuffer(o, &b_, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT) != 0) {
      PyErr_Clear();
      return false;
    }
    held_ = true;
    const bool ok = b_.itemsize == (Py_ssize_t)sizeof(float) && b_.format &&
                    std::strcmp(b_.format, "f") == 0 &&
                    b_.len % (Py_ssize_t)(2 * sizeof(float)) == 0;
    if (!ok) {
      PyBuffer_Release(&b_);
      held_ = false;
    }
    return ok;
  }
  Py_buffer b_{};
  bool held_ = false;
};

// The poses (N, 3), float32, on the device, contiguous.
at::Tensor poses_of(PyObject* o) {
  if (THPVariable_Check(o)) {
    const at::Tensor& t = THPVariable_Unpack(o);
    if (t.scalar_type() == at::kFloat && t.is_cuda() && t.dim() == 2 && t.size(1) == 3)
      return t.contiguous();
  }
  Ref r = convert("_poses", o);   // raises, as it does there
  return tensor(r.get());
}

// psdf_edges of an api.EdgeSet; holds the tensors and the staged record.
class Edges {
 public:
  Edges(PyObject* es, bool with_staged) {
    PyObject* names[5] = {g_n.ax, g_n.ay, g_n.bx, g_n.by, g_n.obst_off};
    const void* p[5];
    for (int k = 0; k < 5; ++k) {
      Ref r = attr(es, names[k]);
      t_[k] = tensor(r.get());
      p[k] = t_[k].data_ptr();
    }
    c.ax = static_cast<const float*>(p[0]);
    c.ay = static_cast<const float*>(p[1]);
    c.bx = static_cast<const float*>(p[2]);
    c.by = static_cast<const float*>(p[3]);
    c.obst_off = static_cast<const int32_t*>(p[4]);
    c.E = (int32_t)as_long(attr(es, g_n.E).get());
    c.M = (int32_t)as_long(attr(es, g_n.M).get());
    c.mbar = (int32_t)as_long(attr(es, g_n.mbar).get());
    c.staged = nullptr;
    if (!with_staged) return;
    Ref s = attr(es, g_n.staged);
    if (s.get() == Py_None) return;
    if (PyObject_GetBuffer(s.get(), &b_, PyBUF_SIMPLE) != 0) throw PyError();
    if (b_.len != (Py_ssize_t)sizeof(psdf_staged)) {
      PyBuffer_Release(&b_);
      b_.obj = nullptr;
      PyErr_SetString(PyExc_TypeError, "staged: not a PsdfStaged record");
      throw PyError();
    }
    c.staged = static_cast<const psdf_staged*>(b_.buf);
  }
  ~Edges() {
    if (b_.obj) PyBuffer_Release(&b_);
  }
  psdf_edges c{};

 private:
  at::Tensor t_[5];
  Py_buffer b_{};
};

psdf_params params_of(PyObject* o) {
  psdf_params p = {1e-12f, 1e-6f, 1000.0f};
  if (o != Py_None) {
    p.eps = (float)as_double(attr(o, g_n.eps).get());
    p.eps_sat = (float)as_double(attr(o, g_n.eps_sat).get());
    p.eta = (float)as_double(attr(o, g_n.eta).get());
  }
  return p;
}

// torch's current stream.  A call on host tensors may be the process's first
// use of the device: without it getCurrentHIPStream indexes per-device tables
// that do not exist where there is no usable GPU (torch raises here).
hipStream_t stream() {
  torch::utils::device_lazy_init(at::kCUDA);
  return c10::hip::getCurrentHIPStream().stream();
}

void check(int rc) {
  if (rc == PSDF_OK) return;
  Ref cls = own(PyObject_GetAttrString(g_api, "PsdfError"));
  Ref e = own(PyObject_CallFunction(cls.get(), "is", rc, psdf_last_error()));
  PyErr_SetObject(cls.get(), e.get());
  throw PyError();
}

// The interpreter lock, released in a scope; back also when an exception (a
// tensor without storage, an error of the device) leaves it.
class Unlocked {
 public:
  Unlocked() : s_(PyEval_SaveThread()) {}
  Unlocked(const Unlocked&) = delete;
  Unlocked& operator=(const Unlocked&) = delete;
  ~Unlocked() { PyEval_RestoreThread(s_); }

 private:
  PyThreadState* s_;
};

// The call on torch's current stream, with the interpreter lock released; the
// message of an error is the thread's own, so it is read after the lock is back.
template <class F>
void call(F f) {
  const hipStream_t st = stream();
  int rc;
  {
    const Unlocked unlocked;
    rc = f(st);
  }
  check(rc);
}

at::Tensor empty(const at::Tensor& like, at::ScalarType t, std::initializer_list<int64_t> n) {
  return at::empty(at::IntArrayRef(n.begin(), n.size()),
                   at::TensorOptions().dtype(t).device(like.device()));
}

at::Tensor workspace(PyObject* ws, const at::Tensor& poses, int32_t N, int32_t M) {
  if (ws != Py_None) return tensor(ws);
  const size_t n = psdf_workspace_bytes(N, M);
  return empty(poses, at::kByte, {(int64_t)(n > 8 ? n : 8)});
}

PyObject* tuple(std::initializer_list<at::Tensor> ts) {
  Ref r = own(PyTuple_New((Py_ssize_t)ts.size()));
  Py_ssize_t k = 0;
  for (const at::Tensor& t : ts) {
    PyObject* o = THPVariable_Wrap(t);
    if (!o) throw PyError();
    PyTuple_SET_ITEM(r.get(), k++, o);
  }
  return r.release();
}

// ---- the entry points: positional arguments, as api.py passes them

PyObject* eval(PyObject* const* a) {   // footprint, poses, edges, params, ws
  const at::Tensor poses = poses_of(a[1]);
  const int32_t N = (int32_t)poses.size(0);
  const psdf_params pr = params_of(a[3]);
  const Edges e(a[2], true);
  const Footprint fp(a[0]);
  const at::Tensor d = empty(poses, at::kFloat, {N}), edge = empty(poses, at::kInt, {N}),
                   obst = empty(poses, at::kInt, {N}), keys = empty(poses, at::kLong, {N}),
                   ws = workspace(a[4], poses, N, e.c.M);
  call([&](hipStream_t st) {
    return psdf_eval(fp.xy(), fp.m(), data<float>(poses), N, &e.c, &pr, data<float>(d),
                     data<int32_t>(edge), data<int32_t>(obst), data<uint64_t>(keys),
                     data<void>(ws), (size_t)ws.numel(), st);
  });
  return tuple({d, edge, obst, keys});
}

PyObject* grad(PyObject* const* a) {   // footprint, poses, edges, params, out, ws
  const at::Tensor poses = poses_of(a[1]);
  const int32_t N = (int32_t)poses.size(0);
  const psdf_params pr = params_of(a[3]);
  const Edges e(a[2], true);
  const Footprint fp(a[0]);
  at::Tensor o[5];   // d, edge, obst, grad, keys
  Ref given;         // the caller's tensors themselves, read once: out may be an iterator
  if (a[4] == Py_None) {
    o[0] = empty(poses, at::kFloat, {N});
    o[1] = empty(poses, at::kInt, {N});
    o[2] = empty(poses, at::kInt, {N});
    o[3] = empty(poses, at::kFloat, {N, 3});
    o[4] = empty(poses, at::kLong, {N});
  } else {
    given = own(PySequence_Tuple(a[4]));
    if (PyTuple_GET_SIZE(given.get()) != 5) {
      PyErr_Format(PyExc_ValueError, "out holds %zd tensors, 5 wanted (d, edge, obst, grad, keys)",
                   PyTuple_GET_SIZE(given.get()));
      throw PyError();
    }
    for (int k = 0; k < 5; ++k) o[k] = tensor(PyTuple_GET_ITEM(given.get(), k));
  }
  const at::Tensor ws = workspace(a[5], poses, N, e.c.M);
  call([&](hipStream_t st) {
    return psdf_grad(fp.xy(), fp.m(), data<float>(poses), N, &e.c, &pr, data<float>(o[0]),
                     data<int32_t>(o[1]), data<int32_t>(o[2]), data<float>(o[3]),
                     data<uint64_t>(o[4]), data<void>(ws), (size_t)ws.numel(), st);
  });
  return given.get() ? given.release() : tuple({o[0], o[1], o[2], o[3], o[4]});
}

PyObject* bwd(PyObject* const* a) {   // footprint, poses, edges, keys, gout, params
  const at::Tensor poses = poses_of(a[1]);
  const int32_t N = (int32_t)poses.size(0);
  const at::Tensor g = tensor(a[4]).contiguous().to(at::kFloat);
  const at::Tensor keys = tensor(a[3]);
  const psdf_params pr = params_of(a[5]);
  const Edges e(a[2], true);
  const Footprint fp(a[0]);
  const at::Tensor gpose = empty(poses, at::kFloat, {N, 3});
  call([&](hipStream_t st) {
    return psdf_bwd(fp.xy(), fp.m(), data<float>(poses), N, &e.c, &pr, data<uint64_t>(keys),
                    data<float>(g), data<float>(gpose), st);
  });
  return THPVariable_Wrap(gpose);
}

PyObject* constraints(PyObject* const* a) {   // footprint, poses, edges, d_min, params, host, ws
  const at::Tensor poses = poses_of(a[1]);
  const int32_t N = (int32_t)poses.size(0);
  const float d_min = float_of(a[3]);
  const psdf_params pr = params_of(a[4]);
  float* host = nullptr;
  at::Tensor h;
  if (a[5] != Py_None) {
    const bool is_tensor = THPVariable_Check(a[5]);
    if (is_tensor) h = tensor(a[5]);
    else own(PyObject_GetAttrString(a[5], "dtype"));   // an array is a value error, as below
    if (!is_tensor || h.scalar_type() != at::kFloat || h.dim() != 2 || h.size(0) != N || h.size(1) != 4 ||
        !h.is_contiguous() || h.is_cuda()) {
      PyErr_SetString(PyExc_ValueError,
                      "host must be a contiguous CPU float32 tensor of shape (N, 4)");
      throw PyError();
    }
    host = data<float>(h);
  }
  const Edges e(a[2], true);
  const Footprint fp(a[0]);
  const at::Tensor hj = empty(poses, at::kFloat, {N, 4}), keys = empty(poses, at::kLong, {N}),
                   ws = workspace(a[6], poses, N, e.c.M);
  call([&](hipStream_t st) {
    return psdf_constraints(fp.xy(), fp.m(), data<float>(poses), N, &e.c, &pr, d_min,
                            data<float>(hj), host, data<uint64_t>(keys), data<void>(ws),
                            (size_t)ws.numel(), st);
  });
  return tuple({hj, keys});
}

PyObject* bwd_geometry(PyObject* const* a) {   // footprint, poses, edges, keys, gout, params
  const at::Tensor poses = poses_of(a[1]);
  const int32_t N = (int32_t)poses.size(0);
  const at::Tensor g = tensor(a[4]).contiguous().to(at::kFloat);
  const at::Tensor keys = tensor(a[3]);
  const psdf_params pr = params_of(a[5]);
  const Edges e(a[2], true);
  const Footprint fp(a[0]);
  const at::Tensor gedges = empty(poses, at::kFloat, {e.c.E, 4}),
                   gfp = empty(poses, at::kFloat, {fp.m(), 2});
  call([&](hipStream_t st) {
    return psdf_bwd_geometry(fp.xy(), fp.m(), data<float>(poses), N, &e.c, &pr,
                             data<uint64_t>(keys), data<float>(g), data<float>(gedges),
                             data<float>(gfp), st);
  });
  return tuple({gedges, gfp});
}

PyObject* sd_matrix(PyObject* const* a) {   // footprint, poses, edges, params, out
  const at::Tensor poses = poses_of(a[1]);
  const int32_t N = (int32_t)poses.size(0);
  const psdf_params pr = params_of(a[3]);
  const Edges e(a[2], true);
  const Footprint fp(a[0]);
  const at::Tensor sd = a[4] == Py_None ? empty(poses, at::kFloat, {N, e.c.M}) : tensor(a[4]);
  call([&](hipStream_t st) {
    return psdf_sd_matrix(fp.xy(), fp.m(), data<float>(poses), N, &e.c, &pr, data<float>(sd),
                          st);
  });
  if (a[4] == Py_None) return THPVariable_Wrap(sd);
  Py_INCREF(a[4]);
  return a[4];
}

PyObject* encode_padded(PyObject* const* a) {   // A, B, S -> (ax, ay, bx, by, off)
  const at::Tensor s0 = tensor(a[2]);
  if (s0.dim() < 2) {
    PyErr_SetString(PyExc_IndexError, "S must be of shape (Mbar, mbar)");
    throw PyError();
  }
  const int32_t Mbar = (int32_t)s0.size(0), mbar = (int32_t)s0.size(1);
  const at::Tensor A = tensor(a[0]).contiguous().to(at::kFloat);
  const at::Tensor B = tensor(a[1]).contiguous().to(at::kFloat);
  // a mask of bools is one of bytes
  const at::Tensor S = s0.scalar_type() == at::kBool ? s0.contiguous()
                                                     : s0.contiguous().to(at::kByte);
  const int64_t n = (int64_t)Mbar * mbar, cap = n > 1 ? n : 1;
  const at::Tensor ax = empty(S, at::kFloat, {cap}), ay = empty(S, at::kFloat, {cap}),
                   bx = empty(S, at::kFloat, {cap}), by = empty(S, at::kFloat, {cap}),
                   off = empty(S, at::kInt, {(int64_t)Mbar + 1});
  const size_t wsb = psdf_encode_ws_bytes(Mbar);
  const at::Tensor ws = empty(S, at::kByte, {(int64_t)(wsb > 1 ? wsb : 1)});
  call([&](hipStream_t st) {
    return psdf_encode_padded(data<float>(A), data<float>(B), data<uint8_t>(S), Mbar, mbar,
                              data<float>(ax), data<float>(ay), data<float>(bx), data<float>(by),
                              data<int32_t>(off), data<void>(ws), wsb, st);
  });
  int64_t E = 0;
  if (Mbar > 0) {
    const Unlocked unlocked;
    E = off.select(0, Mbar).item<int32_t>();
  }
  return tuple({ax.slice(0, 0, E), ay.slice(0, 0, E), bx.slice(0, 0, E), by.slice(0, 0, E), off});
}

PyObject* stage_edges(PyObject* const* a) {   // edges, params, table, PsdfStaged record
  const psdf_params pr = params_of(a[1]);
  const Edges e(a[0], false);
  const at::Tensor table = tensor(a[2]);
  struct Record {
    Py_buffer b{};
    ~Record() {
      if (b.obj) PyBuffer_Release(&b);
    }
  } r;
  if (PyObject_GetBuffer(a[3], &r.b, PyBUF_WRITABLE) != 0) throw PyError();
  if (r.b.len != (Py_ssize_t)sizeof(psdf_staged)) {
    PyErr_SetString(PyExc_TypeError, "not a PsdfStaged record");
    throw PyError();
  }
  psdf_staged* rec = static_cast<psdf_staged*>(r.b.buf);
  psdf_staged out = *rec;
  call([&](hipStream_t st) {
    return psdf_stage_edges(&e.c, &pr, table.data_ptr(), (size_t)table.numel(), &out, st);
  });
  *rec = out;
  Py_RETURN_NONE;
}

// theta, m, v, step, lr, X, T, loss, ws
PyObject* mlp_train_step(PyObject* const* a) {
  const at::Tensor th = tensor(a[0]), m = tensor(a[1]), v = tensor(a[2]), X = tensor(a[5]),
                   T = tensor(a[6]);
  const int32_t step = int_of(a[3]);
  const float lr = float_of(a[4]);
  const int32_t B = (int32_t)X.size(0);
  at::Tensor loss, ws;
  if (a[7] != Py_None) loss = tensor(a[7]);
  if (a[8] != Py_None) {
    ws = tensor(a[8]);
  } else {
    const size_t n = psdf_mlp_ws_bytes(B);
    ws = empty(X, at::kByte, {(int64_t)(n > 4 ? n : 4)});
  }
  call([&](hipStream_t st) {
    return psdf_mlp_train_step(data<float>(th), data<float>(m), data<float>(v), step, lr,
                               data<float>(X), data<float>(T), B,
                               loss.defined() ? data<float>(loss) : nullptr, data<void>(ws),
                               (size_t)ws.numel(), st);
  });
  Py_RETURN_NONE;
}

// No C++ exception leaves an entry point.
template <PyObject* (*F)(PyObject* const*), int NARGS>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != NARGS) {
    PyErr_Format(PyExc_TypeError, "%d arguments wanted, got %zd", NARGS, n);
    return nullptr;
  }
  try {
    return F(args);
  } catch (const PyError&) {
  } catch (...) {   // as torch's own calls raise it (OutOfMemoryError, IndexError, ...)
    torch::translate_exception_to_python(std::current_exception());
  }
  return nullptr;
}

PyObject* bind(PyObject*, PyObject* api) {
  Py_INCREF(api);
  Py_XDECREF(g_api);
  g_api = api;
  Py_RETURN_NONE;
}

#define PSDF_ENTRY(name, n) \
  {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(&entry<name, n>)), METH_FASTCALL, nullptr}

PyMethodDef methods[] = {PSDF_ENTRY(eval, 5),
                         PSDF_ENTRY(grad, 6),
                         PSDF_ENTRY(bwd, 6),
                         PSDF_ENTRY(constraints, 7),
                         PSDF_ENTRY(bwd_geometry, 6),
                         PSDF_ENTRY(sd_matrix, 5),
                         PSDF_ENTRY(encode_padded, 3),
                         PSDF_ENTRY(stage_edges, 4),
                         PSDF_ENTRY(mlp_train_step, 9),
                         {"bind", bind, METH_O, nullptr},
                         {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "Native calls of api.py.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
  const char* names[] = {"ax", "ay", "bx", "by", "obst_off", "E", "M", "mbar", "_staged",
                         "eps", "eps_sat", "eta"};
  PyObject** to[] = {&g_n.ax, &g_n.ay, &g_n.bx, &g_n.by, &g_n.obst_off, &g_n.E, &g_n.M,
                     &g_n.mbar, &g_n.staged, &g_n.eps, &g_n.eps_sat, &g_n.eta};
  for (size_t k = 0; k < sizeof(names) / sizeof(names[0]); ++k) {
    *to[k] = PyUnicode_InternFromString(names[k]);
    if (!*to[k]) return nullptr;
  }
  return PyModule_Create(&module);
}
