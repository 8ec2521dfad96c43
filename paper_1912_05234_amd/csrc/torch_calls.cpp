// The calls of binding.py in native code: reads the tensors, allocates the results and calls the C ABI of
// include/cnn.h on the current stream.
//
// A call of the library with small tensors is over in about 5 us on the GPU, less than Python needed to make it: 10.5 us
// for a convolution, of which 3.4 are the launch itself, 2.9 the lookup of the current stream, 1.7 each allocation and
// the rest the conversion of a dozen arguments by ctypes.  Here the same call takes 4.2 us, or 5 to 6 where the host's
// processor runs slower (both occur on one machine).  A network made of single operations at batch 100 (18 calls, 21
// launches, 67 us of kernels) is still limited by the host: 98 to 107 us a pass, 211 before.
// Arguments arrive positionally from the wrappers in binding.py, which hold the names, the defaults and the
// descriptions.  The interpreter lock is released around each call of the library, as ctypes does.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>

#include "cnn.h"

namespace {

struct Raised {};  // a Python exception is set

PyObject* check = nullptr;  // binding._check: raises CnnError for a code other than 0

template <class FN>
PyObject* guarded(FN fn) {
  try {
    return fn();
  } catch (const Raised&) {
  } catch (const c10::Error& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
  }
  return nullptr;
}

[[noreturn]] void raise(PyObject* type, const char* text) {
  PyErr_SetString(type, text);
  throw Raised();
}

const at::Tensor& tensor(PyObject* o, at::ScalarType type = at::kFloat) {
  if (!THPVariable_Check(o)) {
    if (PyObject* a = PyObject_GetAttrString(o, "is_cuda")) {  // None and other objects: AttributeError
      Py_DECREF(a);
      raise(PyExc_TypeError, "expected a tensor");
    }
    throw Raised();
  }
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda() || t.scalar_type() != type || !t.is_contiguous())
    raise(PyExc_ValueError, type == at::kInt ? "expected a contiguous torch.int32 tensor on the GPU"
                                             : "expected a contiguous torch.float32 tensor on the GPU");
  return t;
}

const at::Tensor& tensor(PyObject* o, int dims) {
  const at::Tensor& t = tensor(o);
  if (t.dim() != dims) {
    PyErr_Format(PyExc_ValueError, "expected %d dimensions, got %d", dims, (int)t.dim());
    throw Raised();
  }
  return t;
}

template <class T = float>
T* data(const at::Tensor& t) {
  return static_cast<T*>(t.data_ptr());
}

template <class T = float>
T* data_or_null(PyObject* o, at::ScalarType type = at::kFloat) {
  return o == Py_None ? nullptr : data<T>(tensor(o, type));
}

int size(const at::Tensor& t, int i) { return (int)t.sizes()[i]; }

int first_size(const at::Tensor& t) {
  if (t.dim() < 1) raise(PyExc_IndexError, "tuple index out of range");
  return size(t, 0);
}

long integer(PyObject* o) {
  const long v = PyLong_AsLong(o);
  if (v == -1 && PyErr_Occurred()) throw Raised();
  return v;
}

double number(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw Raised();
  return v;
}

at::Tensor empty(at::IntArrayRef sizes, at::Device device, at::ScalarType type = at::kFloat) {
  return at::empty(sizes, at::TensorOptions().dtype(type).device(device));
}

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

template <class FN>
void call(const char* name, FN fn) {
  int code;
  Py_BEGIN_ALLOW_THREADS;
  code = fn();
  Py_END_ALLOW_THREADS;
  if (code == 0) return;
  if (PyObject* r = PyObject_CallFunction(check, "is", code, name)) Py_DECREF(r);
  if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, name);
  throw Raised();
}

PyObject* wrap(at::Tensor t) { return THPVariable_Wrap(std::move(t)); }

PyObject* pair(PyObject* a, PyObject* b) {
  PyObject* r = a && b ? PyTuple_Pack(2, a, b) : nullptr;
  Py_XDECREF(a);
  Py_XDECREF(b);
  return r;
}

void* context(PyObject* o) {
  if (o == Py_None) return nullptr;  // closed: the library refuses it
  void* p = PyLong_AsVoidPtr(o);
  if (!p && PyErr_Occurred()) throw Raised();
  return p;
}

at::Device device_at(PyObject* index) { return at::Device(at::kCUDA, (c10::DeviceIndex)integer(index)); }

#define CALL(name, count)                                                                      \
  PyObject* name(PyObject*, PyObject* const* a, Py_ssize_t n) {                                \
    if (n != count) return PyErr_Format(PyExc_TypeError, #name " takes %d arguments", count);  \
    return guarded([&]() -> PyObject* {
#define END \
  });       \
  }

// ---- the network: ctx, ..., device index -------------------------------------------------------------------
CALL(forward, 4)  // ctx, images, yhat or None, device
  const at::Tensor& x = tensor(a[1]);
  const int B = first_size(x);
  at::Tensor made;
  if (a[2] == Py_None) made = empty({B, 10}, device_at(a[3]));
  float* y = a[2] == Py_None ? data(made) : data(tensor(a[2]));
  void* ctx = context(a[0]);
  call("cnn_forward", [&] { return cnn_forward(static_cast<cnn_ctx*>(ctx), data(x), B, y); });
  if (a[2] == Py_None) return wrap(std::move(made));
  Py_INCREF(a[2]);
  return a[2];
END

CALL(gradient, 4)  // ctx, images, labels, device
  const at::Tensor& x = tensor(a[1]);
  const int32_t* labels = data_or_null<int32_t>(a[2], at::kInt);
  const int B = first_size(x);
  at::Tensor grad = empty({CNN_NPARAM}, device_at(a[3])), loss = empty({1}, device_at(a[3]));
  void* ctx = context(a[0]);
  call("cnn_gradient", [&] { return cnn_gradient(static_cast<cnn_ctx*>(ctx), data(x), labels, B, data(grad), data(loss)); });
  return pair(wrap(std::move(grad)), wrap(std::move(loss)));
END

CALL(train_batch, 5)  // ctx, images, labels, rate, loss or None
  const at::Tensor& x = tensor(a[1]);
  const int32_t* labels = data_or_null<int32_t>(a[2], at::kInt);
  const int B = first_size(x);
  const float rate = (float)number(a[3]);
  float* loss = data_or_null(a[4]);
  void* ctx = context(a[0]);
  call("cnn_train_batch", [&] { return cnn_train_batch(static_cast<cnn_ctx*>(ctx), data(x), labels, B, rate, loss); });
  Py_INCREF(a[4]);
  return a[4];
END

CALL(evaluate, 4)  // ctx, images, labels, device
  const at::Tensor& x = tensor(a[1]);
  const int32_t* labels = data_or_null<int32_t>(a[2], at::kInt);
  const int B = first_size(x);
  at::Tensor right = empty({1}, device_at(a[3]), at::kLong), loss = empty({1}, device_at(a[3]));
  void* ctx = context(a[0]);
  call("cnn_evaluate", [&] {
    return cnn_evaluate(static_cast<cnn_ctx*>(ctx), data(x), labels, B, data<int64_t>(right), data(loss));
  });
  return pair(wrap(std::move(right)), wrap(std::move(loss)));
END

// ---- single operations -------------------------------------------------------------------------------------
CALL(conv_fwd, 4)  // in, k, bias or None, form: 0 fp32, 1 bf16, 2 plain
  const at::Tensor &x = tensor(a[0], 4), &k = tensor(a[1], 4);
  const float* bias = data_or_null(a[2]);
  const int B = size(x, 0), Cin = size(x, 1), H = size(x, 2), W = size(x, 3), Cout = size(k, 0), KH = size(k, 2), KW = size(k, 3);
  at::Tensor out = empty({B, Cout, H - KH + 1, W - KW + 1}, x.device());
  const long form = integer(a[3]);
  const auto fn = form == 1 ? cnn_conv_fwd_bf16 : form == 2 ? cnn_conv_fwd_valu : cnn_conv_fwd;
  call(form == 1 ? "cnn_conv_fwd_bf16" : form == 2 ? "cnn_conv_fwd_valu" : "cnn_conv_fwd",
       [&] { return fn(data(x), data(k), bias, data(out), B, Cin, H, W, Cout, KH, KW, stream()); });
  return wrap(std::move(out));
END

CALL(conv_bwd_input, 5)  // d_out, k, H, W, form
  const at::Tensor &d = tensor(a[0]), &k = tensor(a[1], 4);
  const int B = first_size(d), Cout = size(k, 0), Cin = size(k, 1), KH = size(k, 2), KW = size(k, 3);
  const long H = integer(a[2]), W = integer(a[3]), form = integer(a[4]);
  at::Tensor out = empty({B, Cin, H, W}, d.device());
  const auto fn = form == 1 ? cnn_conv_bwd_input_bf16 : form == 2 ? cnn_conv_bwd_input_valu : cnn_conv_bwd_input;
  call(form == 1 ? "cnn_conv_bwd_input_bf16" : form == 2 ? "cnn_conv_bwd_input_valu" : "cnn_conv_bwd_input",
       [&] { return fn(data(d), data(k), data(out), B, Cin, (int)H, (int)W, Cout, KH, KW, stream()); });
  return wrap(std::move(out));
END

CALL(conv_bwd_weight, 5)  // in, d_out, want_bias, workspace, bf16
  const at::Tensor &x = tensor(a[0], 4), &d = tensor(a[1], 4);
  const int B = size(x, 0), Cin = size(x, 1), H = size(x, 2), W = size(x, 3), Cout = size(d, 1);
  const int KH = H - size(d, 2) + 1, KW = W - size(d, 3) + 1;
  const bool bf16 = integer(a[4]);
  at::Tensor d_k = empty({Cout, Cin, KH, KW}, x.device()), d_b, ws;
  if (integer(a[2])) d_b = empty({Cout}, x.device());
  size_t bytes = 0;
  if (integer(a[3])) {
    bytes = (bf16 ? cnn_conv_bwd_weight_bf16_workspace_bytes : cnn_conv_bwd_weight_workspace_bytes)(B, Cin, H, W, Cout, KH, KW);
    if (bytes) ws = empty({(int64_t)bytes}, x.device(), at::kByte);
  }
  const auto fn = bf16 ? cnn_conv_bwd_weight_bf16 : cnn_conv_bwd_weight;
  call(bf16 ? "cnn_conv_bwd_weight_bf16" : "cnn_conv_bwd_weight", [&] {
    return fn(data(x), data(d), data(d_k), d_b.defined() ? data(d_b) : nullptr, B, Cin, H, W, Cout, KH, KW,
              bytes ? ws.data_ptr() : nullptr, bytes, stream());
  });
  return pair(wrap(std::move(d_k)), d_b.defined() ? wrap(std::move(d_b)) : (Py_INCREF(Py_None), Py_None));
END

CALL(avgpool_fwd, 1)
  const at::Tensor& x = tensor(a[0], 4);
  const int B = size(x, 0), C = size(x, 1), H = size(x, 2), W = size(x, 3);
  at::Tensor out = empty({B, C, H / 2, W / 2}, x.device());
  call("cnn_avgpool_fwd", [&] { return cnn_avgpool_fwd(data(x), data(out), B, C, H, W, stream()); });
  return wrap(std::move(out));
END

CALL(avgpool_bwd, 1)
  const at::Tensor& d = tensor(a[0], 4);
  const int B = size(d, 0), C = size(d, 1), Ho = size(d, 2), Wo = size(d, 3);
  at::Tensor out = empty({B, C, 2 * Ho, 2 * Wo}, d.device());
  call("cnn_avgpool_bwd", [&] { return cnn_avgpool_bwd(data(d), data(out), B, C, Ho, Wo, stream()); });
  return wrap(std::move(out));
END

CALL(fc_fwd, 3)  // in, w, bias or None
  const at::Tensor &x = tensor(a[0], 2), &w = tensor(a[1]);
  const float* bias = data_or_null(a[2]);
  const int B = size(x, 0), I = size(x, 1), O = first_size(w);
  at::Tensor out = empty({B, O}, x.device());
  call("cnn_fc_fwd", [&] { return cnn_fc_fwd(data(x), data(w), bias, data(out), B, I, O, stream()); });
  return wrap(std::move(out));
END

CALL(fc_bwd_input, 2)  // d_out, w
  const at::Tensor &d = tensor(a[0], 2), &w = tensor(a[1]);
  if (w.dim() < 2) raise(PyExc_IndexError, "tuple index out of range");
  const int B = size(d, 0), O = size(d, 1), I = size(w, 1);
  at::Tensor out = empty({B, I}, d.device());
  call("cnn_fc_bwd_input", [&] { return cnn_fc_bwd_input(data(d), data(w), data(out), B, I, O, stream()); });
  return wrap(std::move(out));
END

CALL(fc_bwd_weight, 4)  // in, d_out, want_bias, workspace
  const at::Tensor &x = tensor(a[0], 2), &d = tensor(a[1]);
  if (d.dim() < 2) raise(PyExc_IndexError, "tuple index out of range");
  const int B = size(x, 0), I = size(x, 1), O = size(d, 1);
  at::Tensor d_w = empty({O, I}, x.device()), d_b, ws;
  if (integer(a[2])) d_b = empty({O}, x.device());
  size_t bytes = 0;
  if (integer(a[3])) {
    bytes = cnn_fc_bwd_weight_workspace_bytes(B, I, O);
    if (bytes) ws = empty({(int64_t)bytes}, x.device(), at::kByte);
  }
  call("cnn_fc_bwd_weight", [&] {
    return cnn_fc_bwd_weight(data(x), data(d), data(d_w), d_b.defined() ? data(d_b) : nullptr, B, I, O,
                             bytes ? ws.data_ptr() : nullptr, bytes, stream());
  });
  return pair(wrap(std::move(d_w)), d_b.defined() ? wrap(std::move(d_b)) : (Py_INCREF(Py_None), Py_None));
END

CALL(logistic_fwd, 1)
  const at::Tensor& x = tensor(a[0]);
  at::Tensor y = empty(x.sizes(), x.device());
  call("cnn_logistic_fwd", [&] { return cnn_logistic_fwd(data(x), data(y), (size_t)x.numel(), stream()); });
  return wrap(std::move(y));
END

CALL(logistic_bwd, 2)  // y, d_y
  const at::Tensor& y = tensor(a[0]);
  const float* d_y = data_or_null(a[1]);
  at::Tensor d_x = empty(y.sizes(), y.device());
  call("cnn_logistic_bwd", [&] { return cnn_logistic_bwd(data(y), d_y, data(d_x), (size_t)y.numel(), stream()); });
  return wrap(std::move(d_x));
END

PyObject* raise_through(PyObject*, PyObject* fn) {  // binding._check
  Py_INCREF(fn);
  Py_XSETREF(check, fn);
  Py_RETURN_NONE;
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(forward), FAST(gradient), FAST(train_batch), FAST(evaluate), FAST(conv_fwd), FAST(conv_bwd_input),
                         FAST(conv_bwd_weight), FAST(avgpool_fwd), FAST(avgpool_bwd), FAST(fc_fwd), FAST(fc_bwd_input),
                         FAST(fc_bwd_weight), FAST(logistic_fwd), FAST(logistic_bwd),
                         {"raise_through", raise_through, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() { return PyModule_Create(&module); }
