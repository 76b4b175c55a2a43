// Host side of the Python entry points that run once per request: argument checks, descriptor
// tables, output and workspace tensors, and the call into the C-ABI (include/kan.h), without a trip
// through the interpreter for each of them.
//
// What bounds a small call is this path and not the GPU: a launch costs the host 2.0-2.5 us on this
// stack, and the ctypes form of the binding (a descriptor array built in Python, the stream looked up as a
// torch.cuda.Stream object, one ctypes conversion per argument, torch.full for the output) added 5.4 us
// to a call with buffers of its own and 14 us to one without (2 x 17 us for the descriptors of fifty
// heads), where its two launches themselves take 5-6 us.  Host time per call, ctypes form and this one: a
// two-layer head at batch 1 with kept buffers 11.3 and 6.8 us; one 64 x 32 layer with neither workspace nor
// output given 20.0 and 9.0 (its GPU work 7.7); fifty two-layer heads 33.5 and 18.8.
//
// The functions take the objects of the binding (VQLayer, tensors) as they are and return the output,
// or the kan_status as an int when the call was refused.

#include <ATen/ops/empty.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <c10/util/SmallVector.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/kan.h"

namespace {

PyObject* g_desc_name = nullptr;        // "desc": the attribute that holds a layer's C descriptor
PyObject* g_raw_stream = nullptr;       // torch._C._cuda_getCurrentRawStream

typedef c10::SmallVector<kan_vq_layer, 8> Table;

// Copies the descriptor of one VQLayer; false with a Python error set.
bool read_desc(PyObject* layer, kan_vq_layer* out) {
  PyObject* desc = PyObject_GetAttr(layer, g_desc_name);
  if (!desc) return false;
  Py_buffer view;
  const int got = PyObject_GetBuffer(desc, &view, PyBUF_SIMPLE);
  Py_DECREF(desc);
  if (got != 0) return false;
  const bool fits = view.len == (Py_ssize_t)sizeof(kan_vq_layer);
  if (fits) memcpy(out, view.buf, sizeof(kan_vq_layer));
  PyBuffer_Release(&view);
  if (!fits) PyErr_SetString(PyExc_TypeError, "desc is not a kan_vq_layer");
  return fits;
}

// heads: sequence (heads) of sequences (layers) of VQLayer -> table [n_heads][n_layers].
bool read_heads(PyObject* heads, Table* table, int32_t* n_layers, int32_t* n_heads) {
  PyObject* hs = PySequence_Fast(heads, "heads: a list of heads, each a list of VQLayer");
  if (!hs) return false;
  const Py_ssize_t H = PySequence_Fast_GET_SIZE(hs);
  Py_ssize_t N = 0;
  bool ok = true;
  for (Py_ssize_t h = 0; ok && h < H; ++h) {
    PyObject* ls = PySequence_Fast(PySequence_Fast_GET_ITEM(hs, h), "a head is a list of VQLayer");
    if (!ls) {
      ok = false;
      break;
    }
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(ls);
    if (h == 0) {
      N = n;
      table->reserve((size_t)(H * N));
    }
    if (n != N) {
      PyErr_SetString(PyExc_AssertionError, "every head has the same number of layers");
      ok = false;
    }
    for (Py_ssize_t l = 0; ok && l < n; ++l) {
      table->emplace_back();
      ok = read_desc(PySequence_Fast_GET_ITEM(ls, l), &table->back());
    }
    Py_DECREF(ls);
  }
  Py_DECREF(hs);
  if (ok && (H == 0 || N == 0)) {
    PyErr_SetString(PyExc_IndexError, "no heads or no layers");
    ok = false;
  }
  *n_layers = (int32_t)N;
  *n_heads = (int32_t)H;
  return ok;
}

const at::Tensor* tensor_of(PyObject* o, const char* what) {
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_TypeError, "%s: a tensor is expected", what);
    return nullptr;
  }
  return &THPVariable_Unpack(o);
}

// Like the rest of the binding, calls go to the current stream of the current device.
bool current_stream(void** out) {
  const c10::Device dev = c10::impl::VirtualGuardImpl(c10::DeviceType::CUDA).getDevice();
  PyObject* index = PyLong_FromLong(dev.index());
  PyObject* raw = index ? PyObject_CallFunctionObjArgs(g_raw_stream, index, nullptr) : nullptr;
  Py_XDECREF(index);
  if (!raw) return false;
  *out = PyLong_AsVoidPtr(raw);
  Py_DECREF(raw);
  return !(*out == nullptr && PyErr_Occurred());
}

bool check_floats(const at::Tensor& t, const char* what) {
  if (t.scalar_type() == at::kFloat && t.is_contiguous()) return true;
  PyErr_Format(PyExc_AssertionError, "%s: float32 and contiguous", what);
  return false;
}

// Workspace and output of one call: the caller's tensors, or tensors of its own.
struct Buffers {
  at::Tensor ws_own, y_own;
  void* ws = nullptr;
  size_t ws_bytes = 0;
  void* y = nullptr;
  PyObject* y_obj = nullptr;        // borrowed: the caller's output

  bool use_ws(PyObject* o, size_t need, const at::Tensor& like) {
    if (o != Py_None) {
      const at::Tensor* t = tensor_of(o, "ws");
      if (!t) return false;
      ws = t->data_ptr();
      ws_bytes = (size_t)t->numel();
    } else if (need > 0) {
      ws_own = at::empty({(int64_t)need}, like.options().dtype(at::kByte));
      ws = ws_own.data_ptr();
      ws_bytes = need;
    }
    return true;
  }
  bool use_y(PyObject* o, at::IntArrayRef shape, const at::Tensor& like) {
    if (o != Py_None) {
      const at::Tensor* t = tensor_of(o, "y");
      if (!t) return false;
      y = t->data_ptr();
      y_obj = o;
    } else {
      y_own = at::empty(shape, like.options());
      y = y_own.data_ptr();
    }
    return true;
  }
  PyObject* result(kan_status st) {
    if (st != KAN_OK) return PyLong_FromLong(st);
    if (y_obj) {
      Py_INCREF(y_obj);
      return y_obj;
    }
    return THPVariable_Wrap(std::move(y_own));
  }
};

PyObject* forward(const Table& table, int32_t n_layers, int32_t n_heads, const at::Tensor& x, long path, PyObject* ws,
                  PyObject* y, bool is_static, bool one_layer) {
  const int64_t B = x.size(0);
  Buffers b;
  if (!is_static) {
    size_t need = 0;
    if (ws == Py_None) {
      need = kan_vq_workspace_bytes(table.data(), n_layers, n_heads, B, (int32_t)path);
      if (need == (size_t)-1) need = 0;        // the forward call reports the precise status
    }
    if (!b.use_ws(ws, need, x)) return nullptr;
  }
  const int64_t out = table[n_layers - 1].out;
  if (!(one_layer ? b.use_y(y, {B, out}, x) : b.use_y(y, {n_heads, B, out}, x))) return nullptr;
  void* stream;
  if (!current_stream(&stream)) return nullptr;
  const float* xp = (const float*)x.data_ptr();
  kan_status st;
  Py_BEGIN_ALLOW_THREADS
  st = is_static ? kan_vq_head_forward_static(table.data(), n_layers, n_heads, xp, B, (float*)b.y, (int32_t)path, stream)
                 : kan_vq_head_forward(table.data(), n_layers, n_heads, xp, B, (float*)b.y, b.ws, b.ws_bytes, (int32_t)path,
                                       stream);
  Py_END_ALLOW_THREADS
  return b.result(st);
}

bool arity(Py_ssize_t n, Py_ssize_t want) {
  if (n == want) return true;
  PyErr_Format(PyExc_TypeError, "%zd arguments, got %zd", want, n);
  return false;
}

// layer_forward(layer, x, path, ws, y)
PyObject* layer_forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (!arity(n, 5)) return nullptr;
  const at::Tensor* x = tensor_of(a[1], "x");
  if (!x || !check_floats(*x, "x")) return nullptr;
  Table table(1);
  if (!read_desc(a[0], &table[0])) return nullptr;
  if (x->dim() != 2 || x->size(1) != table[0].in) {
    PyErr_SetString(PyExc_AssertionError, "x: [batch][inputs of the layer]");
    return nullptr;
  }
  const long path = PyLong_AsLong(a[2]);
  if (path == -1 && PyErr_Occurred()) return nullptr;
  return forward(table, 1, 1, *x, path, a[3], a[4], false, true);
  END_HANDLE_TH_ERRORS
}

PyObject* heads_call(PyObject* heads, PyObject* xo, PyObject* patho, PyObject* ws, PyObject* y, bool is_static) {
  const at::Tensor* x = tensor_of(xo, "x");
  if (!x || !check_floats(*x, "x")) return nullptr;
  if (x->dim() < 1) {
    PyErr_SetString(PyExc_IndexError, "x: [batch][inputs]");
    return nullptr;
  }
  Table table;
  int32_t n_layers, n_heads;
  if (!read_heads(heads, &table, &n_layers, &n_heads)) return nullptr;
  const long path = PyLong_AsLong(patho);
  if (path == -1 && PyErr_Occurred()) return nullptr;
  return forward(table, n_layers, n_heads, *x, path, ws, y, is_static, false);
}

// head_forward(heads, x, path, ws, y)
PyObject* head_forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  return arity(n, 5) ? heads_call(a[0], a[1], a[2], a[3], a[4], false) : nullptr;
  END_HANDLE_TH_ERRORS
}

// head_forward_static(heads, x, path, y)
PyObject* head_forward_static(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  return arity(n, 4) ? heads_call(a[0], a[1], a[2], Py_None, a[3], true) : nullptr;
  END_HANDLE_TH_ERRORS
}

// dense_layer_forward(coef, x, ws, y)
PyObject* dense_layer_forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (!arity(n, 4)) return nullptr;
  const at::Tensor* coef = tensor_of(a[0], "coef");
  const at::Tensor* x = coef ? tensor_of(a[1], "x") : nullptr;
  if (!x || !check_floats(*coef, "coef")) return nullptr;
  if (!x->is_contiguous()) {
    PyErr_SetString(PyExc_AssertionError, "x: contiguous");
    return nullptr;
  }
  if (coef->dim() != 3 || x->dim() < 1) {
    PyErr_SetString(PyExc_ValueError, "coef: [in][out][10], x: [batch][in]");
    return nullptr;
  }
  const int64_t n_in = coef->size(0), n_out = coef->size(1), g = coef->size(2), B = x->size(0);
  Buffers b;
  size_t need = 0;
  if (a[2] == Py_None) {
    need = kan_dense_workspace_bytes((int32_t)n_in, (int32_t)n_out, B);
    if (need == (size_t)-1) return PyLong_FromLong(KAN_ERR_SHAPE);
  }
  if (!b.use_ws(a[2], need, *x) || !b.use_y(a[3], {B, n_out}, *x)) return nullptr;
  void* stream;
  if (!current_stream(&stream)) return nullptr;
  const float *cp = (const float*)coef->data_ptr(), *xp = (const float*)x->data_ptr();
  kan_status st;
  Py_BEGIN_ALLOW_THREADS
  st = kan_dense_layer_forward(cp, (int32_t)n_in, (int32_t)n_out, (int32_t)g, xp, B, (float*)b.y, b.ws, b.ws_bytes, stream);
  Py_END_ALLOW_THREADS
  return b.result(st);
  END_HANDLE_TH_ERRORS
}

// assign(coef, codebook, ws) -> (idx, gain, bias)
PyObject* assign(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (!arity(n, 3)) return nullptr;
  const at::Tensor* coef = tensor_of(a[0], "coef");
  const at::Tensor* cb = coef ? tensor_of(a[1], "codebook") : nullptr;
  if (!cb || !check_floats(*coef, "coef") || !check_floats(*cb, "codebook")) return nullptr;
  if (coef->dim() != 3 || coef->size(2) != 10 || cb->dim() != 2 || cb->size(1) != 10) {
    PyErr_SetString(PyExc_AssertionError, "coef: [in][out][10], codebook: [K][10]");
    return nullptr;
  }
  const int64_t n_in = coef->size(0), n_out = coef->size(1), K = cb->size(0);
  const bool u16 = K <= 65536;
  at::Tensor idx = at::empty({n_in, n_out}, coef->options().dtype(u16 ? at::kShort : at::kInt));
  at::Tensor gain = at::empty({n_in, n_out}, coef->options()), bias = at::empty({n_in, n_out}, coef->options());
  Buffers b;
  size_t need = a[2] == Py_None ? kan_vq_assign_fast_workspace_bytes((int32_t)n_in, (int32_t)n_out, (int32_t)K) : 0;
  if (need == (size_t)-1) return PyLong_FromLong(KAN_ERR_SHAPE);
  if (!b.use_ws(a[2], need, *coef)) return nullptr;
  void* stream;
  if (!current_stream(&stream)) return nullptr;
  const float *cp = (const float*)coef->data_ptr(), *kp = (const float*)cb->data_ptr();
  void* ip = idx.data_ptr();
  float *gp = (float*)gain.data_ptr(), *bp = (float*)bias.data_ptr();
  kan_status st;
  Py_BEGIN_ALLOW_THREADS
  st = kan_vq_assign(cp, (int32_t)n_in, (int32_t)n_out, kp, (int32_t)K, u16 ? KAN_U16 : KAN_U32, ip, gp, bp, b.ws,
                     b.ws_bytes, stream);
  Py_END_ALLOW_THREADS
  if (st != KAN_OK) return PyLong_FromLong(st);
  PyObject* r = PyTuple_New(3);
  if (!r) return nullptr;
  PyTuple_SET_ITEM(r, 0, THPVariable_Wrap(std::move(idx)));
  PyTuple_SET_ITEM(r, 1, THPVariable_Wrap(std::move(gain)));
  PyTuple_SET_ITEM(r, 2, THPVariable_Wrap(std::move(bias)));
  return r;
  END_HANDLE_TH_ERRORS
}

template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyMethodDef method(const char* name) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(F)), METH_FASTCALL, nullptr};
}

PyMethodDef g_methods[] = {method<layer_forward>("layer_forward"),
                           method<head_forward>("head_forward"),
                           method<head_forward_static>("head_forward_static"),
                           method<dense_layer_forward>("dense_layer_forward"),
                           method<assign>("assign"),
                           {nullptr, nullptr, 0, nullptr}};

PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_kan_host", "Per-request entry points of the binding.", -1, g_methods,
                        nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__kan_host(void) {
  g_desc_name = PyUnicode_InternFromString("desc");
  PyObject* c = PyImport_ImportModule("torch._C");
  if (!g_desc_name || !c) return nullptr;
  g_raw_stream = PyObject_GetAttrString(c, "_cuda_getCurrentRawStream");
  Py_DECREF(c);
  if (!g_raw_stream) return nullptr;
  return PyModule_Create(&g_module);
}
