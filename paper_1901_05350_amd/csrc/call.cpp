// The host path of the Python entry points in native code (module paper_1901_05350_amd._call).
//
// A call of a small op is bound by what the host does around the kernel, not by the kernel: 64x128x64 matMul, 2.4 us
// on the GPU, took 12.7 us per call through ctypes (shape arrays, attribute look-ups on the tensors, the allocation
// and the stream handle through Python), 15.8 us for a convolution with bias.  Here the same checks read the tensors'
// C++ objects, the result comes straight from torch's device allocator and the C ABI is called without a
// foreign-function layer; what is left is the runtime's kernel launch (2.7 us) and about 1.5 us around it.
//
// Every function takes exactly the arguments of its Python wrapper, positionally, and returns the result, or None
// for anything that is not the plain case (other types, layouts, ranks, shapes, a status from the library): the
// wrapper then goes through its own checks, which name the argument at fault.  None never follows an enqueued kernel,
// except after a failed launch.
#include <Python.h>

#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/tfx.h"

namespace {

// The tensor behind `o` if it is a plain contiguous GPU tensor of this type and rank (rank < 0: any), else null.
const at::Tensor* plain(PyObject* o, at::ScalarType type, int rank) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda() || t.scalar_type() != type || t.layout() != at::kStrided || !t.is_contiguous()) return nullptr;
  if (rank >= 0 && t.dim() != rank) return nullptr;
  return &t;
}

bool has_shape(const at::Tensor& t, const int64_t* shape, int rank) {
  if (t.dim() != rank) return false;
  for (int i = 0; i < rank; ++i)
    if (t.size(i) != shape[i]) return false;
  return true;
}

// An optional tensor: null and true for None, null and false if it is not plain or not of that shape.
bool optional_plain(PyObject* o, at::ScalarType type, const int64_t* shape, int rank, const at::Tensor** t) {
  *t = nullptr;
  if (o == Py_None) return true;
  *t = plain(o, type, rank);
  return *t && has_shape(**t, shape, rank);
}

bool as_int(PyObject* o, int* v) {
  if (!PyLong_Check(o)) return false;
  int overflow = 0;
  const long x = PyLong_AsLongAndOverflow(o, &overflow);
  if (overflow || x != (int)x) return false;
  *v = (int)x;
  return true;
}

void* stream_of(const at::Tensor& t) { return c10::hip::getCurrentHIPStream(t.device().index()).stream(); }

// Where the result goes: the caller's `out` (checked) or a new tensor.  `made` owns a new one.
struct Result {
  PyObject* given = nullptr;
  at::Tensor made;
  void* ptr = nullptr;
};
bool result(PyObject* out, at::ScalarType type, const int64_t* shape, int rank, const at::Tensor& like, Result* r) {
  if (out != Py_None) {
    const at::Tensor* t = plain(out, type, rank);
    if (!t || !has_shape(*t, shape, rank)) return false;
    r->given = out;
    r->ptr = t->data_ptr();
    return true;
  }
  r->made = at::Tensor(at::detail::empty_cuda(at::IntArrayRef(shape, rank), type, like.device(), std::nullopt));
  r->ptr = r->made.data_ptr();
  return true;
}
PyObject* answer(int status, Result& r) {
  if (status != TFX_OK) Py_RETURN_NONE;
  if (!r.given) return THPVariable_Wrap(std::move(r.made));
  Py_INCREF(r.given);
  return r.given;
}

template <typename F>
int without_gil(F f) {
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = f();
  Py_END_ALLOW_THREADS
  return status;
}

template <typename T>
T* data(const at::Tensor* t) { return t ? static_cast<T*>(t->data_ptr()) : nullptr; }

// matmul(a, b, transpose_a, transpose_b, out): rank 2 or 3 float32
template <int RANK>
PyObject* matmul(PyObject*, PyObject* const* arg, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n != 5) Py_RETURN_NONE;
  const at::Tensor *a = plain(arg[0], at::kFloat, RANK), *b = plain(arg[1], at::kFloat, RANK);
  if (!a || !b) Py_RETURN_NONE;
  const int ta = PyObject_IsTrue(arg[2]), tb = PyObject_IsTrue(arg[3]);
  if (ta < 0 || tb < 0) return nullptr;
  const int64_t *as = a->sizes().data(), *bs = b->sizes().data();
  int64_t shape[3] = {as[0], 0, 0};
  if (tfx_matmul_out_shape(as + RANK - 2, bs + RANK - 2, ta, tb, shape + RANK - 2) != TFX_OK) Py_RETURN_NONE;
  Result r;
  if (!result(arg[4], at::kFloat, shape, RANK, *a, &r)) Py_RETURN_NONE;
  void* const stream = stream_of(*a);
  const int status = without_gil([&] {
    return (RANK == 2 ? tfx_matmul : tfx_batch_matmul)(data<float>(a), as, data<float>(b), bs, ta, tb,
                                                        static_cast<float*>(r.ptr), stream);
  });
  return answer(status, r);
  END_HANDLE_TH_ERRORS
}

// batch_matmul_f16(a, b, transpose_a, transpose_b, bias, act, out)
PyObject* batch_matmul_f16(PyObject*, PyObject* const* arg, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  int act;
  if (n != 7 || !as_int(arg[5], &act)) Py_RETURN_NONE;
  const at::Tensor *a = plain(arg[0], at::kHalf, 3), *b = plain(arg[1], at::kHalf, 3), *bias;
  if (!a || !b) Py_RETURN_NONE;
  const int ta = PyObject_IsTrue(arg[2]), tb = PyObject_IsTrue(arg[3]);
  if (ta < 0 || tb < 0) return nullptr;
  const int64_t *as = a->sizes().data(), *bs = b->sizes().data();
  int64_t shape[3] = {as[0], 0, 0};
  if (tfx_matmul_out_shape(as + 1, bs + 1, ta, tb, shape + 1) != TFX_OK) Py_RETURN_NONE;
  if (!optional_plain(arg[4], at::kHalf, shape + 2, 1, &bias)) Py_RETURN_NONE;
  Result r;
  if (!result(arg[6], at::kHalf, shape, 3, *a, &r)) Py_RETURN_NONE;
  void* const stream = stream_of(*a);
  const int status = without_gil([&] {
    return tfx_batch_matmul_f16(data<uint16_t>(a), as, data<uint16_t>(b), bs, ta, tb, data<uint16_t>(bias),
                                (tfx_activation)act, static_cast<uint16_t*>(r.ptr), stream);
  });
  return answer(status, r);
  END_HANDLE_TH_ERRORS
}

// conv(x, filter, bias, stride, pad, act, out), of one storage type and kind
template <typename T, bool DEPTHWISE>
PyObject* conv(PyObject*, PyObject* const* arg, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  constexpr at::ScalarType type = sizeof(T) == 4 ? at::kFloat : at::kHalf;
  int sh, sw, pad, act;
  if (n != 7 || !as_int(arg[4], &pad) || !as_int(arg[5], &act)) Py_RETURN_NONE;
  if (PyTuple_Check(arg[3]) && PyTuple_GET_SIZE(arg[3]) == 2) {
    if (!as_int(PyTuple_GET_ITEM(arg[3], 0), &sh) || !as_int(PyTuple_GET_ITEM(arg[3], 1), &sw)) Py_RETURN_NONE;
  } else if (!as_int(arg[3], &sh)) {
    Py_RETURN_NONE;
  } else {
    sw = sh;
  }
  const at::Tensor *x = plain(arg[0], type, 4), *f = plain(arg[1], type, 4), *bias;
  if (!x || !f) Py_RETURN_NONE;
  const int64_t *xs = x->sizes().data(), *fs = f->sizes().data();
  int64_t shape[4], pads[4];
  if ((DEPTHWISE ? tfx_depthwise_conv2d_out_shape : tfx_conv2d_out_shape)(xs, fs, sh, sw, (tfx_padding)pad, shape, pads) != TFX_OK)
    Py_RETURN_NONE;
  if (!optional_plain(arg[2], type, shape + 3, 1, &bias)) Py_RETURN_NONE;
  Result r;
  if (!result(arg[6], type, shape, 4, *x, &r)) Py_RETURN_NONE;
  void* const stream = stream_of(*x);
  const int status = without_gil([&] {
    if constexpr (sizeof(T) == 4)
      return (DEPTHWISE ? tfx_depthwise_conv2d : tfx_conv2d)(data<T>(x), xs, data<T>(f), fs, data<T>(bias), sh, sw,
                                                             (tfx_padding)pad, (tfx_activation)act, static_cast<T*>(r.ptr), stream);
    else
      return (DEPTHWISE ? tfx_depthwise_conv2d_f16 : tfx_conv2d_f16)(data<T>(x), xs, data<T>(f), fs, data<T>(bias), sh, sw,
                                                                     (tfx_padding)pad, (tfx_activation)act, static_cast<T*>(r.ptr), stream);
  });
  return answer(status, r);
  END_HANDLE_TH_ERRORS
}

// add(a, b, out) of one storage type
template <typename T>
PyObject* add(PyObject*, PyObject* const* arg, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  constexpr at::ScalarType type = sizeof(T) == 4 ? at::kFloat : at::kHalf;
  if (n != 3) Py_RETURN_NONE;
  const at::Tensor *a = plain(arg[0], type, -1), *b = plain(arg[1], type, -1);
  if (!a || !b || a->sizes() != b->sizes()) Py_RETURN_NONE;
  Result r;
  if (!result(arg[2], type, a->sizes().data(), (int)a->dim(), *a, &r)) Py_RETURN_NONE;
  void* const stream = stream_of(*a);
  const int status = without_gil([&] {
    if constexpr (sizeof(T) == 4) return tfx_add(data<T>(a), data<T>(b), a->numel(), static_cast<T*>(r.ptr), stream);
    else return tfx_add_f16(data<T>(a), data<T>(b), a->numel(), static_cast<T*>(r.ptr), stream);
  });
  return answer(status, r);
  END_HANDLE_TH_ERRORS
}

// net(image, variant address, weights address, workspace, probs, logits): one forward pass of one storage type;
// returns True, or None for the plain path's checks.  Batch, image size and class count are held against the
// variant here: the library reads as much of every buffer as they say.
template <typename T>
PyObject* net(PyObject*, PyObject* const* arg, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  constexpr at::ScalarType type = sizeof(T) == 4 ? at::kFloat : at::kHalf;
  if (n != 6 || !PyLong_Check(arg[1]) || !PyLong_Check(arg[2])) Py_RETURN_NONE;
  const auto* variant = static_cast<const tfx_mobilenet_v1_variant*>(PyLong_AsVoidPtr(arg[1]));
  const void* weights = PyLong_AsVoidPtr(arg[2]);
  if (!variant || !weights) Py_RETURN_NONE;
  const at::Tensor* image = plain(arg[0], type, 4);
  const at::Tensor* ws = plain(arg[3], at::kByte, 1);
  const at::Tensor *probs = plain(arg[4], type, 2), *logits = plain(arg[5], type, 2);
  if (!image || !ws || !probs || !logits) Py_RETURN_NONE;
  const int64_t batch = probs->size(0);
  const int64_t in[4] = {batch, variant->image_size, variant->image_size, 3}, out[2] = {batch, variant->classes};
  if (!has_shape(*image, in, 4) || !has_shape(*probs, out, 2) || !has_shape(*logits, out, 2)) Py_RETURN_NONE;
  void* const stream = stream_of(*image);
  const int status = without_gil([&] {
    if constexpr (sizeof(T) == 4)
      return tfx_mobilenet_v1_variant_forward(variant, data<T>(image), batch, static_cast<const tfx_mobilenet_v1_weights*>(weights),
                                              ws->data_ptr(), (size_t)ws->numel(), data<T>(probs), data<T>(logits), stream);
    else
      return tfx_mobilenet_v1_forward_f16(variant, data<T>(image), batch, static_cast<const tfx_mobilenet_v1_weights_f16*>(weights),
                                          ws->data_ptr(), (size_t)ws->numel(), data<T>(probs), data<T>(logits), stream);
  });
  if (status != TFX_OK) Py_RETURN_NONE;
  Py_RETURN_TRUE;
  END_HANDLE_TH_ERRORS
}

#define FAST(f) (PyCFunction)(void (*)(void))static_cast<PyObject* (*)(PyObject*, PyObject* const*, Py_ssize_t)>(f), METH_FASTCALL, nullptr
PyMethodDef methods[] = {
    {"matmul", FAST(matmul<2>)},
    {"batch_matmul", FAST(matmul<3>)},
    {"batch_matmul_f16", FAST(batch_matmul_f16)},
    {"conv2d", FAST((conv<float, false>))},
    {"conv2d_f16", FAST((conv<uint16_t, false>))},
    {"depthwise_conv2d", FAST((conv<float, true>))},
    {"depthwise_conv2d_f16", FAST((conv<uint16_t, true>))},
    {"add", FAST(add<float>)},
    {"add_f16", FAST(add<uint16_t>)},
    {"net", FAST(net<float>)},
    {"net_f16", FAST(net<uint16_t>)},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", "Host path of the entry points.", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call(void) { return PyModule_Create(&module); }
