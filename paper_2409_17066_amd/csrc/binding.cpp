// The convenience calls of the Python package over torch tensors, marshalled in C++: a decode-sized kernel takes a few
// microseconds, and checking the tensors, asking for the stream, allocating the result and converting the arguments through
// ctypes took longer than that (256 x 384, one row, calls back to back: 8.9 us against 4.4 us here).  Every function returns
// None when the arguments are not the plain ones it takes -- the Python code then does the call, with its own checks and
// errors --, the status code when the library refused, and the result otherwise.
#include <Python.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/vq.h"
#include "vq_lend.h"

namespace {

decltype(&vq_gemv) p_gemv;
decltype(&vq_gemv_with_workspace) p_gemv_ws;
decltype(&vq_lend_gemv_bytes) p_lend_gemv_bytes;
decltype(&vq_gemv_multi) p_gemv_multi;
decltype(&vq_gemm) p_gemm, p_gemm_default;
decltype(&vq_gemm_workspace_bytes) p_gemm_workspace_bytes, p_gemm_default_workspace_bytes, p_lend_gemm_least_bytes;
decltype(&vq_dequant) p_dequant;
decltype(&vq_lend_assign) p_lend_assign;

PyObject *s_desc, *s_places;

// The layer's descriptor: the memory of the ctypes structure in its attribute `desc`.
struct Desc {
  Py_buffer view;
  bool held = false;
  const vq_layer_desc *get(PyObject *layer) {
    PyObject *d = PyObject_GetAttr(layer, s_desc);
    if (!d) { PyErr_Clear(); return nullptr; }
    held = PyObject_GetBuffer(d, &view, PyBUF_SIMPLE) == 0;
    Py_DECREF(d);
    if (!held) { PyErr_Clear(); return nullptr; }
    return view.len == (Py_ssize_t)sizeof(vq_layer_desc) ? static_cast<const vq_layer_desc *>(view.buf) : nullptr;
  }
  ~Desc() { if (held) PyBuffer_Release(&view); }
};

// A device tensor [rows][columns] of halfs with adjacent columns, else nullptr.
const at::Tensor *half_matrix(PyObject *o) {
  if (!THPVariable_Check(o)) return nullptr;
  const at::Tensor &t = THPVariable_Unpack(o);
  return t.is_cuda() && t.scalar_type() == at::kHalf && t.dim() == 2 && t.stride(1) == 1 ? &t : nullptr;
}

at::TensorBase empty(at::IntArrayRef size, at::ScalarType type) {
  return at::detail::empty_cuda(size, type, c10::Device(c10::kCUDA, c10::hip::current_device()), std::nullopt);
}

void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

template <typename Call>
int released(Call call) {                       // the library call, without the interpreter's lock as ctypes makes it
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = call();
  Py_END_ALLOW_THREADS
  return rc;
}

PyObject *tensor_or_status(int rc, at::TensorBase &&fresh, PyObject *given) {
  if (rc != VQ_OK) return PyLong_FromLong(rc);
  if (given != Py_None) { Py_INCREF(given); return given; }
  return THPVariable_Wrap(std::move(fresh));
}

// Workspace for one call, from torch's allocator, or nullptr: there is a route without.  On a full card the allocator would first give
// all its unused memory back and wait for the GPU, in every call: beyond the size of small results it is asked only for what it has
// unused or the device has free.
void *borrow(at::TensorBase &scratch, size_t bytes) {
  try {
    if (bytes > (1u << 20)) {
      using c10::CachingAllocator::StatType;
      const auto stats = c10::hip::HIPCachingAllocator::getDeviceStats(c10::hip::current_device());
      const auto sum = static_cast<size_t>(StatType::AGGREGATE);
      const size_t unused = (size_t)(stats.reserved_bytes[sum].current - stats.allocated_bytes[sum].current);
      size_t free = 0, total = 0;
      if (unused < bytes && hipMemGetInfo(&free, &total) == hipSuccess && free + unused < bytes) return nullptr;
    }
    scratch = empty({(int64_t)bytes}, at::kByte);
    return scratch.data_ptr();
  } catch (const c10::Error &) {
    return nullptr;
  }
}

#define VQ_TRY try {
#define VQ_CATCH                                            \
  } catch (const std::exception &e) {                       \
    PyErr_SetString(PyExc_RuntimeError, e.what());          \
    return nullptr;                                         \
  }

// Whether gemv() without a workspace may borrow one (vq_lend.h says how much): the layers that never do are spared the question.
bool may_borrow(const vq_layer_desc &d) { return (!d.group_vectors && (d.v != 6 || d.k <= 2048 || d.col_perm)) || (d.v == 6 && (d.in_features & 1)); }

// gemv(layer, x, out or None, workspace or None)
PyObject *gemv(PyObject *, PyObject *const *args, Py_ssize_t n) {
  VQ_TRY
  Desc desc;
  const vq_layer_desc *d;
  const at::Tensor *x;
  if (n != 4 || !(x = half_matrix(args[1])) || !(d = desc.get(args[0]))) Py_RETURN_NONE;
  const bool has_ws = args[3] != Py_None;
  if (has_ws && !THPVariable_Check(args[3])) Py_RETURN_NONE;
  at::TensorBase fresh;
  const at::TensorBase *y = &fresh;
  if (args[2] != Py_None) {
    if (!THPVariable_Check(args[2])) Py_RETURN_NONE;
    y = &THPVariable_Unpack(args[2]);
    if (y->dim() != 2) Py_RETURN_NONE;
  } else {
    fresh = empty({x->size(0), d->out_features}, at::kHalf);
  }
  const void *xp = x->data_ptr();
  void *yp = y->data_ptr(), *s = stream();
  const int64_t ldx = x->stride(0), ldy = y->stride(0);
  const int32_t batch = (int32_t)x->size(0);
  int rc;
  if (has_ws) {
    const at::Tensor &ws = THPVariable_Unpack(args[3]);
    void *wp = ws.data_ptr();
    const size_t bytes = (size_t)ws.numel();
    rc = released([&] { return p_gemv_ws(d, xp, ldx, batch, yp, ldy, wp, bytes, s); });
  } else if (const size_t bytes = may_borrow(*d) ? p_lend_gemv_bytes(d, batch) : 0) {
    at::TensorBase scratch;
    void *wp = borrow(scratch, bytes);
    rc = released([&] { return p_gemv_ws(d, xp, ldx, batch, yp, ldy, wp, wp ? bytes : 0, s); });
  } else {
    rc = released([&] { return p_gemv(d, xp, ldx, batch, yp, ldy, s); });
  }
  return tensor_or_status(rc, std::move(fresh), args[2]);
  VQ_CATCH
}

// gemv_multi(list of layers, x)
PyObject *gemv_multi(PyObject *, PyObject *const *args, Py_ssize_t n) {
  VQ_TRY
  constexpr Py_ssize_t MOST = 8;
  const at::Tensor *x;
  if (n != 2 || !PyList_CheckExact(args[0]) || !(x = half_matrix(args[1]))) Py_RETURN_NONE;
  const Py_ssize_t layers = PyList_GET_SIZE(args[0]);
  if (layers < 1 || layers > MOST) Py_RETURN_NONE;
  Desc desc[MOST];
  const vq_layer_desc *d[MOST];
  at::TensorBase y[MOST];
  void *yp[MOST];
  int64_t ldy[MOST];
  for (Py_ssize_t i = 0; i < layers; ++i)
    if (!(d[i] = desc[i].get(PyList_GET_ITEM(args[0], i)))) Py_RETURN_NONE;
  for (Py_ssize_t i = 0; i < layers; ++i) {
    y[i] = empty({x->size(0), d[i]->out_features}, at::kHalf);
    yp[i] = y[i].data_ptr();
    ldy[i] = y[i].stride(0);
  }
  const void *xp = x->data_ptr();
  void *s = stream();
  const int rc = released([&] { return p_gemv_multi(d, (int32_t)layers, xp, x->stride(0), (int32_t)x->size(0), yp, ldy, s); });
  if (rc != VQ_OK) return PyLong_FromLong(rc);
  PyObject *out = PyList_New(layers);
  for (Py_ssize_t i = 0; out && i < layers; ++i) PyList_SET_ITEM(out, i, THPVariable_Wrap(std::move(y[i])));
  return out;
  VQ_CATCH
}

// gemm(layer, X, out or None, workspace or None)
PyObject *gemm(PyObject *, PyObject *const *args, Py_ssize_t n) {
  VQ_TRY
  Desc desc;
  const vq_layer_desc *d;
  const at::Tensor *x;
  if (n != 4 || !(x = half_matrix(args[1])) || !(d = desc.get(args[0]))) Py_RETURN_NONE;
  void *wp = nullptr;
  size_t bytes = 0;
  at::TensorBase scratch;
  auto call = p_gemm;
  const int32_t tokens = (int32_t)x->size(0);
  if (args[3] != Py_None) {
    if (!THPVariable_Check(args[3])) Py_RETURN_NONE;
    const at::Tensor &ws = THPVariable_Unpack(args[3]);
    wp = ws.data_ptr();
    bytes = (size_t)ws.numel() * ws.element_size();
  } else if (tokens > 8) {
    call = p_gemm_default;
    if ((bytes = p_gemm_default_workspace_bytes(d, tokens)) != 0 && !(wp = borrow(scratch, bytes))) {
      const size_t least = p_lend_gemm_least_bytes(d, tokens);
      bytes = least < bytes && (wp = borrow(scratch, least)) ? least : 0;
    }
  }
  if (p_gemm_workspace_bytes(d, tokens) > bytes) Py_RETURN_NONE;
  at::TensorBase fresh;
  const at::TensorBase *y = &fresh;
  if (args[2] != Py_None) {
    if (!THPVariable_Check(args[2])) Py_RETURN_NONE;
    y = &THPVariable_Unpack(args[2]);
    if (y->dim() != 2) Py_RETURN_NONE;
  } else {
    fresh = empty({x->size(0), d->out_features}, at::kHalf);
  }
  const void *xp = x->data_ptr();
  void *yp = y->data_ptr(), *s = stream();
  const int64_t ldx = x->stride(0), ldy = y->stride(0);
  const int rc = released([&] { return call(d, xp, ldx, tokens, yp, ldy, wp, bytes, s); });
  return tensor_or_status(rc, std::move(fresh), args[2]);
  VQ_CATCH
}

// dequant(layer): all of W written, rows in_features apart
PyObject *dequant(PyObject *, PyObject *layer) {
  VQ_TRY
  Desc desc;
  const vq_layer_desc *d = desc.get(layer);
  if (!d) Py_RETURN_NONE;
  PyObject *places = PyObject_GetAttr(layer, s_places);
  if (!places) { PyErr_Clear(); Py_RETURN_NONE; }
  const bool all = places == Py_True;
  Py_DECREF(places);
  if (!all) Py_RETURN_NONE;
  at::TensorBase W = empty({d->out_features, d->in_features}, at::kHalf);
  void *wp = W.data_ptr(), *s = stream();
  const int rc = released([&] { return p_dequant(d, wp, d->in_features, s); });
  return tensor_or_status(rc, std::move(W), Py_None);
  VQ_CATCH
}

// assign(W, codebook, base or None, orientation): all columns of W
PyObject *assign(PyObject *, PyObject *const *args, Py_ssize_t n) {
  VQ_TRY
  const at::Tensor *W, *C, *B = nullptr;
  if (n != 4 || !(W = half_matrix(args[0])) || !(C = half_matrix(args[1])) || !C->is_contiguous() || !PyLong_CheckExact(args[3])) Py_RETURN_NONE;
  if (args[2] != Py_None && (!(B = half_matrix(args[2])) || B->sizes() != W->sizes() || B->strides() != W->strides())) Py_RETURN_NONE;
  const bool down = PyLong_AsLong(args[3]) != 0;
  const int64_t rows = W->size(0), cols = W->size(1), k = C->size(0), v = C->size(1);
  if (rows < 1 || cols < 1 || v < 1 || k < 1) Py_RETURN_NONE;
  int bits = 1;
  while ((int64_t(1) << bits) < k) ++bits;
  const int64_t streams = down ? (rows + v - 1) / v : rows, per_stream = down ? cols : (cols + v - 1) / v;
  const int64_t stride = (per_stream * bits + 127) / 128 * 16;
  at::TensorBase idx = empty({streams, stride}, at::kByte);
  const void *wp = W->data_ptr(), *bp = B ? B->data_ptr() : nullptr, *cp = C->data_ptr();
  void *ip = idx.data_ptr(), *s = stream();
  const int64_t ld = W->stride(0);
  const int rc = released([&] { return p_lend_assign(wp, bp, ld, (int32_t)rows, (int32_t)cols, cp, (int32_t)v, (int32_t)k, ip, stride, down, s); });
  if (rc != VQ_OK) return PyLong_FromLong(rc);
  return THPVariable_Wrap(std::move(idx));
  VQ_CATCH
}

PyMethodDef methods[] = {{"gemv", (PyCFunction)(void *)gemv, METH_FASTCALL, nullptr},
                         {"gemv_multi", (PyCFunction)(void *)gemv_multi, METH_FASTCALL, nullptr},
                         {"gemm", (PyCFunction)(void *)gemm, METH_FASTCALL, nullptr},
                         {"dequant", dequant, METH_O, nullptr},
                         {"assign", (PyCFunction)(void *)assign, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};

// bind(addresses): the library's entry points, which the package has loaded
PyObject *bind(PyObject *, PyObject *addresses) {
  auto at = [&](const char *name, auto &f) {
    PyObject *a = PyDict_GetItemString(addresses, name);
    if (!a) return false;
    f = reinterpret_cast<std::remove_reference_t<decltype(f)>>(PyLong_AsVoidPtr(a));
    return f != nullptr;
  };
  if (!at("vq_gemv", p_gemv) || !at("vq_gemv_with_workspace", p_gemv_ws) || !at("vq_gemv_multi", p_gemv_multi) || !at("vq_gemm", p_gemm) || !at("vq_gemm_default", p_gemm_default) ||
      !at("vq_gemm_workspace_bytes", p_gemm_workspace_bytes) || !at("vq_lend_gemv_bytes", p_lend_gemv_bytes) || !at("vq_gemm_default_workspace_bytes", p_gemm_default_workspace_bytes) ||
      !at("vq_lend_gemm_least_bytes", p_lend_gemm_least_bytes) ||
       !at("vq_dequant", p_dequant) || !at("vq_lend_assign", p_lend_assign)) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "an entry point is missing");
    return nullptr;
  }
  Py_RETURN_NONE;
}
PyMethodDef bind_method = {"bind", bind, METH_O, nullptr};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() {
  PyObject *m = PyModule_Create(&module);
  if (!m) return nullptr;
  s_desc = PyUnicode_InternFromString("desc");
  s_places = PyUnicode_InternFromString("places_every_column");
  PyObject *f = PyCFunction_New(&bind_method, nullptr);
  if (!f || PyModule_AddObject(m, "bind", f) != 0) return nullptr;
  return m;
}
