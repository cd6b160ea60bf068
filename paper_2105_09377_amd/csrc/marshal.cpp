// Native half of the Python binding: torch tensors -> `gs_ap` descriptors -> C entry point.
//
// A call through ctypes cost 8 us on the host for a product and 10 for a convolution, of which the
// entry point itself (checks and one launch) is 3: for small problems the descriptors, built
// field by field in Python, were what a pass waited for.  Here a call reads the tensors directly.
// No arithmetic, no fallback; the entry points are those that binding.py has loaded (`bind`).
#include <Python.h>

#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <utility>
#include <vector>

#include "../../include/glenside.h"

namespace {

struct Failed {};   // a Python error is set

struct Api {
  decltype(&glenside_windows_out_shape) windows_out_shape;
  decltype(&glenside_access_windows) access_windows;
  decltype(&glenside_cartesian_dot) cartesian_dot;
  decltype(&glenside_conv2d_direct) conv2d_direct, conv2d_im2col, conv2d_direct_packed;
  decltype(&glenside_conv2d_direct_packed_with_projection) conv2d_direct_packed_with_projection;
  decltype(&glenside_conv2d_direct_workspace) conv2d_direct_workspace, conv2d_im2col_workspace;
  decltype(&glenside_reduce) reduce;
  decltype(&glenside_windows_reduce) windows_reduce;
  decltype(&glenside_pair_reduce) pair_reduce;
  decltype(&glenside_depthwise_conv2d) depthwise_conv2d;
  decltype(&glenside_transpose) transpose;
  decltype(&glenside_program_shape) program_shape;
  decltype(&glenside_program_workspace) program_workspace;
  decltype(&glenside_program_eval) program_eval;
} api;
PyObject* error_class;

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_AttributeError, "'%.100s' object is no tensor", Py_TYPE(o)->tp_name);
    throw Failed{};
  }
  return THPVariable_Unpack(o);
}

int dtype_code(at::ScalarType t) {
  switch (t) {
    case at::kChar: return GS_I8;
    case at::kInt: return GS_I32;
    case at::kBFloat16: return GS_BF16;
    case at::kFloat: return GS_F32;
    case at::kFloat8_e4m3fn: return GS_F8;
    default: PyErr_SetString(PyExc_KeyError, c10::toString(t)); throw Failed{};
  }
}

// Descriptor of a contiguous tensor with n_access access dimensions (the library refuses impossible ones).
gs_ap describe(const at::Tensor& t, int64_t n_access) {
  gs_ap a{};
  if (!t.is_contiguous()) {
    PyErr_SetString(PyExc_ValueError, "access patterns are dense row-major tensors");
    throw Failed{};
  }
  const auto sizes = t.sizes();
  if (sizes.size() > GS_MAX_RANK) {
    PyErr_SetString(PyExc_ValueError, "rank above GS_MAX_RANK");
    throw Failed{};
  }
  a.data = t.data_ptr();
  a.dtype = dtype_code(t.scalar_type());
  a.rank = int32_t(sizes.size());
  a.n_access = int32_t(n_access);
  for (size_t i = 0; i < sizes.size(); ++i) a.shape[i] = sizes[i];
  return a;
}
// Every dimension an access dimension: results and element-wise operands.
gs_ap describe_all(const at::Tensor& t) { return describe(t, t.dim()); }

int64_t integer(PyObject* o) {
  if (PyLong_CheckExact(o)) {
    const int64_t v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw Failed{};
    return v;
  }
  PyObject* l = PyNumber_Long(o);
  if (!l) throw Failed{};
  const int64_t v = PyLong_AsLongLong(l);
  Py_DECREF(l);
  if (v == -1 && PyErr_Occurred()) throw Failed{};
  return v;
}

// An operator or activation code: integers only, a float is no code.
int code(PyObject* o) {
  PyObject* l = PyNumber_Index(o);
  if (!l) throw Failed{};
  const int v = int(PyLong_AsUnsignedLongMask(l));
  Py_DECREF(l);
  return v;
}

// A new reference, held until the end of the scope.
struct Owned {
  PyObject* object;
  explicit Owned(PyObject* o) : object(o) {
    if (!o) throw Failed{};
  }
  ~Owned() { Py_DECREF(object); }
  Owned(const Owned&) = delete;
};

// The items of a mapping, held until the end of the scope: all of them are taken before any is converted, which
// may run any code.  Twice cheaper than a copy of the dict, which only other mappings need.
struct Items {
  std::vector<std::pair<PyObject*, PyObject*>> items;
  explicit Items(PyObject* mapping) {
    if (PyDict_CheckExact(mapping)) {
      take(mapping);
      return;
    }
    const Owned copy(PyDict_New());
    if (PyDict_Update(copy.object, mapping)) throw Failed{};
    take(copy.object);
  }
  ~Items() {
    for (const auto& i : items) {
      Py_DECREF(i.first);
      Py_DECREF(i.second);
    }
  }
  Items(const Items&) = delete;

 private:
  void take(PyObject* dict) {
    items.reserve(size_t(PyDict_GET_SIZE(dict)));
    PyObject *key, *value;
    for (Py_ssize_t pos = 0; PyDict_Next(dict, &pos, &key, &value);) {
      Py_INCREF(key);
      Py_INCREF(value);
      items.push_back({key, value});
    }
  }
};

// A sequence of integers; None = absent (a null pointer at the C boundary).
struct Ints {
  int64_t v[2 * GS_MAX_RANK] = {};
  int n = 0;
  bool present = false;
  explicit Ints(PyObject* o) {
    if (o == Py_None) return;
    present = true;
    // sized, as a generator is not; a tuple of its own, for the conversions may run any code
    if (PyObject_Size(o) < 0) throw Failed{};
    const Owned seq(PySequence_Tuple(o));
    const Py_ssize_t len = PyTuple_GET_SIZE(seq.object);
    if (len > 2 * GS_MAX_RANK) {
      PyErr_SetString(PyExc_ValueError, "too many integers");
      throw Failed{};
    }
    for (Py_ssize_t i = 0; i < len; ++i) v[i] = integer(PyTuple_GET_ITEM(seq.object, i));
    n = int(len);
  }
  const int64_t* get() const { return present ? v : nullptr; }
};

void* stream_of(const at::Tensor& t) {
  return t.is_cuda() ? static_cast<void*>(c10::hip::getCurrentHIPStream(t.get_device()).stream()) : nullptr;
}

[[noreturn]] void refuse(int status, const char* where) {
  PyObject* args = Py_BuildValue("(is)", status, where);
  if (args) {
    PyErr_SetObject(error_class, args);
    Py_DECREF(args);
  }
  throw Failed{};
}

// The interpreter lock released until the end of the scope, also where that is left by an exception.
struct Unlocked {
  PyThreadState* const state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};

// Runs an entry point without the interpreter lock; a status other than GS_OK becomes GlensideError.
template <typename F>
void call(const char* where, F&& f) {
  int status;
  {
    const Unlocked unlocked;
    status = f();
  }
  if (status != GS_OK) refuse(status, where);
}

// The result: `out` as given, or a new tensor of this shape, of `dtype` (a torch dtype, None = `otherwise`).
struct Result {
  PyObject* object;      // a new reference
  at::Tensor value;
  Result(PyObject* out, PyObject* dtype, at::ScalarType otherwise, const int64_t* shape, int rank, const at::Tensor& like) {
    if (out != Py_None) {
      value = tensor(out);
      object = out;
      Py_INCREF(out);
      return;
    }
    at::ScalarType st = otherwise;
    if (dtype != Py_None) {
      if (!THPDtype_Check(dtype)) {
        PyErr_SetString(PyExc_TypeError, "out_dtype is a torch dtype");
        throw Failed{};
      }
      st = reinterpret_cast<THPDtype*>(dtype)->scalar_type;
    }
    value = at::empty(at::IntArrayRef(shape, rank), at::TensorOptions().dtype(st).device(like.device()));
    object = THPVariable_Wrap(value);
    if (!object) throw Failed{};
  }
};

template <typename F>
PyObject* guarded(Py_ssize_t got, Py_ssize_t want, F&& f) {
  if (got != want) {
    PyErr_Format(PyExc_TypeError, "%zd arguments are wanted", want);
    return nullptr;
  }
  PyObject* r = nullptr;       // set as soon as there is a result, so that a failed call releases it
  try {
    f(r);
    return r;
  } catch (const Failed&) {
  } catch (...) {       // torch's own classes: torch.OutOfMemoryError stays what it is
    torch::translate_exception_to_python(std::current_exception());
  }
  Py_XDECREF(r);
  return nullptr;
}

at::ScalarType sum_type(const at::Tensor& x) { return x.scalar_type() == at::kChar ? at::kInt : at::kFloat; }

// cartesian_dot(a0, a1, n_access0, n_access1, out_dtype, act, out)
PyObject* py_cartesian_dot(PyObject*, PyObject* const* p, Py_ssize_t n) {
  return guarded(n, 7, [&](PyObject*& r) {
    const at::Tensor &a0 = tensor(p[0]), &a1 = tensor(p[1]);
    const int64_t n0 = integer(p[2]), n1 = integer(p[3]);
    const int act = code(p[5]);
    int64_t shape[2 * GS_MAX_RANK];
    int rank = 0;
    if (p[6] == Py_None) {
      for (int64_t i = 0; i < n0 && i < a0.dim() && i < GS_MAX_RANK; ++i) shape[rank++] = a0.size(i);
      for (int64_t i = 0; i < n1 && i < a1.dim() && i < GS_MAX_RANK; ++i) shape[rank++] = a1.size(i);
    }
    Result out(p[6], p[4], sum_type(a0), shape, rank, a0);
    r = out.object;
    gs_ap x = describe(a0, n0), y = describe(a1, n1), o = describe_all(out.value);
    void* s = stream_of(a0);
    call("cartesian_dot", [&] { return api.cartesian_dot(&x, &y, &o, act, nullptr, 0, s); });
  });
}

// conv(form, x, w, stride, pad, residual, act, out_dtype, out, workspace); form 0 direct, 1 packed, 2 im2col
PyObject* py_conv(PyObject*, PyObject* const* p, Py_ssize_t n) {
  return guarded(n, 10, [&](PyObject*& r) {
    const int64_t form = integer(p[0]);
    const at::Tensor &x = tensor(p[1]), &w = tensor(p[2]);
    const Ints stride(p[3]), pad(p[4]);
    const int act = code(p[6]);
    gs_ap xa = describe(x, 1), wa = describe(w, 1);
    int64_t shape[4] = {0, 0, 0, 0};
    if (p[8] == Py_None) {
      // H', W' from the shape rule of `windows` (window (C,Kh,Kw), strides (1,Sh,Sw))
      if (x.dim() < 2 || w.dim() != 4 || stride.n < 2 || pad.n < 2) {
        PyErr_SetString(PyExc_IndexError, "activations (N,C,H,W), weights (O,C,Kh,Kw), two strides and pads are wanted");
        throw Failed{};
      }
      const int64_t window[3] = {x.size(1), w.size(2), w.size(3)}, st[3] = {1, stride.v[0], stride.v[1]}, pd[3] = {0, pad.v[0], pad.v[1]};
      gs_ap want{};
      if (x.dim() != 4) {
        PyErr_SetString(PyExc_IndexError, "activations (N,C,H,W) are wanted");
        throw Failed{};
      }
      call("windows_out_shape", [&] { return api.windows_out_shape(&xa, window, st, pd, pd, &want); });
      shape[0] = x.size(0);
      shape[1] = w.size(0);
      shape[2] = want.shape[2];
      shape[3] = want.shape[3];
    }
    Result out(p[8], p[7], sum_type(x), shape, 4, x);
    r = out.object;
    at::Tensor ws;
    if (p[9] != Py_None) {
      ws = tensor(p[9]);
    } else {
      const size_t need = form == 2 ? api.conv2d_im2col_workspace(&xa, &wa, stride.get(), pad.get())
                                    : api.conv2d_direct_workspace(&xa, &wa, stride.get(), pad.get());
      ws = at::empty({int64_t(need > 16 ? need : 16)}, at::TensorOptions().dtype(at::kByte).device(x.device()));
    }
    gs_ap oa = describe(out.value, 4), ra{};
    if (p[5] != Py_None) ra = describe_all(tensor(p[5]));
    const gs_ap* res = p[5] != Py_None ? &ra : nullptr;
    void *wsp = ws.data_ptr(), *s = stream_of(x);
    const size_t bytes = size_t(ws.numel());
    const auto fn = form == 0 ? api.conv2d_direct : form == 1 ? api.conv2d_direct_packed : api.conv2d_im2col;
    call(form == 0 ? "glenside_conv2d_direct" : form == 1 ? "glenside_conv2d_direct_packed" : "glenside_conv2d_im2col",
         [&] { return fn(&xa, &wa, stride.get(), pad.get(), res, act, &oa, wsp, bytes, s); });
  });
}

// conv_with_projection(x, w, packed, w_proj, packed_proj, stride, pad, act, out, out_proj)
PyObject* py_conv_with_projection(PyObject*, PyObject* const* p, Py_ssize_t n) {
  return guarded(n, 10, [&](PyObject*& r) {
    const at::Tensor &x = tensor(p[0]), &packed = tensor(p[2]), &packed_proj = tensor(p[4]);
    const Ints stride(p[5]), pad(p[6]);
    const int act = code(p[7]);
    const gs_ap xa = describe(x, 1), wa = describe(tensor(p[1]), 1), pa = describe(tensor(p[3]), 1);
    gs_ap oa = describe(tensor(p[8]), 4), qa = describe(tensor(p[9]), 4);
    void* s = stream_of(x);
    call("glenside_conv2d_direct_packed_with_projection", [&] {
      return api.conv2d_direct_packed_with_projection(&xa, &wa, stride.get(), pad.get(), act, &oa, packed.data_ptr(), size_t(packed.numel()),
                                                      &pa, &qa, packed_proj.data_ptr(), size_t(packed_proj.numel()), s);
    });
    Py_INCREF(p[8]);
    r = p[8];
  });
}

at::ScalarType reduce_type(const at::Tensor& x, int op) {
  if (x.scalar_type() == at::kChar) return op == GS_SUM ? at::kInt : at::kChar;
  return x.scalar_type();
}

// reduce(x, n_access, op, scale, out_dtype, out)
PyObject* py_reduce(PyObject*, PyObject* const* p, Py_ssize_t n) {
  return guarded(n, 6, [&](PyObject*& r) {
    const at::Tensor& x = tensor(p[0]);
    const int64_t na = integer(p[1]);
    const int op = code(p[2]);
    const double scale = PyFloat_AsDouble(p[3]);
    if (scale == -1.0 && PyErr_Occurred()) throw Failed{};
    const auto sizes = x.sizes();
    // a leading slice as Python takes it: a negative end counts from the back
    const int64_t dims = x.dim(), lead = na < 0 ? (na + dims > 0 ? na + dims : 0) : na < dims ? na : dims;
    Result out(p[5], p[4], reduce_type(x, op), sizes.data(), int(lead), x);
    r = out.object;
    gs_ap xa = describe(x, 0), oa = describe_all(out.value);
    xa.n_access = int32_t(na);
    void* s = stream_of(x);
    call("reduce", [&] { return api.reduce(&xa, op, float(scale), &oa, s); });
  });
}

// windows_reduce(x, n_access, window, stride, pad_lo, pad_hi, op, scale, out_dtype, out)
PyObject* py_windows_reduce(PyObject*, PyObject* const* p, Py_ssize_t n) {
  return guarded(n, 10, [&](PyObject*& r) {
    const at::Tensor& x = tensor(p[0]);
    const int64_t na = integer(p[1]);
    const Ints window(p[2]), stride(p[3]), lo(p[4]), hi(p[5]);
    const int op = code(p[6]);
    const double scale = PyFloat_AsDouble(p[7]);
    if (scale == -1.0 && PyErr_Occurred()) throw Failed{};
    gs_ap xa = describe(x, 0), want{};
    xa.n_access = int32_t(na);
    if (p[9] == Py_None)
      call("windows_out_shape", [&] { return api.windows_out_shape(&xa, window.get(), stride.get(), lo.get(), hi.get(), &want); });
    Result out(p[9], p[8], reduce_type(x, op), want.shape, want.n_access, x);
    r = out.object;
    gs_ap oa = describe_all(out.value);
    void* s = stream_of(x);
    call("windows_reduce", [&] {
      return api.windows_reduce(&xa, window.get(), stride.get(), lo.get(), hi.get(), op, float(scale), &oa, s);
    });
  });
}

// access_windows(x, n_access, window, stride, pad_lo, pad_hi, pad_mode, out)
PyObject* py_access_windows(PyObject*, PyObject* const* p, Py_ssize_t n) {
  return guarded(n, 8, [&](PyObject*& r) {
    const at::Tensor& x = tensor(p[0]);
    const int64_t na = integer(p[1]);
    const Ints window(p[2]), stride(p[3]), lo(p[4]), hi(p[5]);
    const int mode = code(p[6]);
    gs_ap xa = describe(x, 0), want{};
    xa.n_access = int32_t(na);
    call("windows_out_shape", [&] { return api.windows_out_shape(&xa, window.get(), stride.get(), lo.get(), hi.get(), &want); });
    Result out(p[7], Py_None, x.scalar_type(), want.shape, want.rank, x);
    r = out.object;
    gs_ap oa = describe(out.value, na + window.n);
    void* s = stream_of(x);
    call("access_windows", [&] {
      return api.access_windows(&xa, window.get(), stride.get(), lo.get(), hi.get(), mode, &oa, s);
    });
  });
}

// depthwise_conv2d(x, w, stride, pad, act, out_dtype, out)
PyObject* py_depthwise(PyObject*, PyObject* const* p, Py_ssize_t n) {
  return guarded(n, 7, [&](PyObject*& r) {
    const at::Tensor &x = tensor(p[0]), &w = tensor(p[1]);
    const Ints stride(p[2]), pad(p[3]);
    const int act = code(p[4]);
    gs_ap xa = describe(x, 1), wa = describe(w, 1), want{};
    if (p[6] == Py_None) {
      if (w.dim() < 3) {
        PyErr_SetString(PyExc_IndexError, "weights (C,Kh,Kw) are wanted");
        throw Failed{};
      }
      const int64_t window[2] = {w.size(1), w.size(2)};
      gs_ap planes = xa;
      planes.n_access = 2;
      call("windows_out_shape", [&] { return api.windows_out_shape(&planes, window, stride.get(), pad.get(), pad.get(), &want); });
    }
    Result out(p[6], p[5], sum_type(x), want.shape, 4, x);
    r = out.object;
    gs_ap oa = describe(out.value, 4);
    void* s = stream_of(x);
    call("depthwise_conv2d", [&] { return api.depthwise_conv2d(&xa, &wa, stride.get(), pad.get(), act, &oa, s); });
  });
}

// pair_reduce(a, b, op, act, out)
PyObject* py_pair_reduce(PyObject*, PyObject* const* p, Py_ssize_t n) {
  return guarded(n, 5, [&](PyObject*& r) {
    const at::Tensor &a = tensor(p[0]), &b = tensor(p[1]);
    const int op = code(p[2]), act = code(p[3]);
    Result out(p[4], Py_None, a.scalar_type(), a.sizes().data(), int(a.dim()), a);
    r = out.object;
    gs_ap xa = describe_all(a), ya = describe_all(b), oa = describe_all(out.value);
    void* s = stream_of(a);
    call("pair_reduce", [&] { return api.pair_reduce(&xa, &ya, op, act, &oa, s); });
  });
}

// transpose(x, n_access, perm, out)
PyObject* py_transpose(PyObject*, PyObject* const* p, Py_ssize_t n) {
  return guarded(n, 4, [&](PyObject*& r) {
    const at::Tensor& x = tensor(p[0]);
    const int64_t na = integer(p[1]);
    const Ints perm(p[2]);
    int64_t shape[2 * GS_MAX_RANK];
    if (p[3] == Py_None)
      for (int i = 0; i < perm.n; ++i) {
        const int64_t d = perm.v[i] < 0 ? perm.v[i] + x.dim() : perm.v[i];
        if (d < 0 || d >= x.dim()) {
          PyErr_SetString(PyExc_IndexError, "tuple index out of range");
          throw Failed{};
        }
        shape[i] = x.size(d);
      }
    Result out(p[3], Py_None, x.scalar_type(), shape, perm.n, x);
    r = out.object;
    gs_ap xa = describe(x, 0), oa = describe(out.value, 0);
    xa.n_access = oa.n_access = int32_t(na);
    void* s = stream_of(x);
    call("transpose", [&] { return api.transpose(&xa, perm.get(), &oa, s); });
  });
}

// program_eval(text, tensors by name, integers by name, out_dtype, out, workspace)
PyObject* py_program_eval(PyObject*, PyObject* const* p, Py_ssize_t n) {
  return guarded(n, 6, [&](PyObject*& r) {
    const char* text = PyUnicode_AsUTF8(p[0]);
    if (!text) throw Failed{};
    // Names and tensors are held: the caller's mappings may change meanwhile, from another thread while the
    // interpreter lock is released, or from the conversion of an integer.
    const Items named(p[1]), numbers(p[2]);
    auto name_of = [](PyObject* key) {
      const char* s = PyUnicode_AsUTF8(key);
      if (!s) throw Failed{};
      return s;
    };
    std::vector<gs_named_ap> tensors;
    std::vector<gs_named_int> ints;
    const at::Tensor* first = nullptr;
    for (const auto& [key, value] : named.items) {
      const at::Tensor& t = tensor(value);
      if (!first) first = &t;
      tensors.push_back({name_of(key), describe(t, 0)});
    }
    for (const auto& [key, value] : numbers.items) ints.push_back({name_of(key), integer(value)});
    if (!first) {
      PyErr_SetString(PyExc_StopIteration, "a program needs a tensor");
      throw Failed{};
    }
    const int nt = int(tensors.size()), ni = int(ints.size());
    gs_ap want{};
    call("program_shape", [&] { return api.program_shape(text, tensors.data(), nt, ints.data(), ni, &want); });
    constexpr at::ScalarType types[5] = {at::kChar, at::kInt, at::kBFloat16, at::kFloat, at::kFloat8_e4m3fn};   // by gs_dtype
    Result out(p[4], p[3], types[want.dtype], want.shape, want.rank, *first);
    r = out.object;
    at::Tensor ws;
    if (p[5] != Py_None) {
      ws = tensor(p[5]);
    } else {
      const size_t need = api.program_workspace(text, tensors.data(), nt, ints.data(), ni);
      ws = at::empty({int64_t(need > 16 ? need : 16)}, at::TensorOptions().dtype(at::kByte).device(first->device()));
    }
    // the result as the program's access pattern, whatever shape its tensor has: as many elements, at least
    gs_ap oa = describe(out.value, 0);
    int64_t elements = 1;
    for (int i = 0; i < want.rank; ++i) elements *= want.shape[i];
    if (out.value.numel() < elements) refuse(GS_ERR_SHAPE, "program_eval");
    oa.rank = want.rank;
    oa.n_access = want.n_access;
    for (int i = 0; i < want.rank; ++i) oa.shape[i] = want.shape[i];
    void *wsp = ws.data_ptr(), *s = stream_of(*first);
    const size_t bytes = size_t(ws.numel());
    call("program_eval", [&] { return api.program_eval(text, tensors.data(), nt, ints.data(), ni, &oa, wsp, bytes, s); });
  });
}

// bind(addresses by entry point name, GlensideError)
PyObject* py_bind(PyObject*, PyObject* const* p, Py_ssize_t n) {
  return guarded(n, 2, [&](PyObject*& r) {
    auto get = [&](const char* name, auto& fn) {
      PyObject* v = PyDict_GetItemString(p[0], name);
      if (!v) {
        PyErr_SetString(PyExc_KeyError, name);
        throw Failed{};
      }
      fn = reinterpret_cast<std::decay_t<decltype(fn)>>(PyLong_AsVoidPtr(v));
      if (!fn) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, name);
        throw Failed{};
      }
    };
    get("glenside_windows_out_shape", api.windows_out_shape);
    get("glenside_access_windows", api.access_windows);
    get("glenside_cartesian_dot", api.cartesian_dot);
    get("glenside_conv2d_direct", api.conv2d_direct);
    get("glenside_conv2d_im2col", api.conv2d_im2col);
    get("glenside_conv2d_direct_packed", api.conv2d_direct_packed);
    get("glenside_conv2d_direct_packed_with_projection", api.conv2d_direct_packed_with_projection);
    get("glenside_conv2d_direct_workspace", api.conv2d_direct_workspace);
    get("glenside_conv2d_im2col_workspace", api.conv2d_im2col_workspace);
    get("glenside_reduce", api.reduce);
    get("glenside_windows_reduce", api.windows_reduce);
    get("glenside_pair_reduce", api.pair_reduce);
    get("glenside_depthwise_conv2d", api.depthwise_conv2d);
    get("glenside_transpose", api.transpose);
    get("glenside_program_shape", api.program_shape);
    get("glenside_program_workspace", api.program_workspace);
    get("glenside_program_eval", api.program_eval);
    Py_INCREF(p[1]);
    Py_XDECREF(error_class);
    error_class = p[1];
    Py_INCREF(Py_None);
    r = Py_None;
  });
}

#define GS_FN(name, fn) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fn)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    GS_FN("bind", py_bind), GS_FN("cartesian_dot", py_cartesian_dot), GS_FN("conv", py_conv), GS_FN("conv_with_projection", py_conv_with_projection), GS_FN("reduce", py_reduce),
    GS_FN("windows_reduce", py_windows_reduce), GS_FN("access_windows", py_access_windows),
    GS_FN("depthwise_conv2d", py_depthwise), GS_FN("pair_reduce", py_pair_reduce), GS_FN("transpose", py_transpose),
    GS_FN("program_eval", py_program_eval),
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
