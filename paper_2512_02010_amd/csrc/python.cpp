// Python's way to the C ABI (include/nvfp4_46.h): output allocation, argument marshalling and the call in
// one C function per entry point.  binding.py hands in the entry points of the library that it loaded and the
// exception for statuses other than NVFP4_OK.
//
// Through ctypes and torch.empty a call spent more time in the interpreter than in the launch (per call
// among others, 256 x 1024: quantize with its three outputs 12.5 us, of which launch 3.6, three torch.empty 4.8;
// three calls of a round trip 26.4; here 7.2, of which launch 4, and 16.4).  Nothing is kept between calls.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstring>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/DynamicTypes.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "gemm_shapes.hpp"
#include "layer.hpp"
#include "nvfp4_46.h"
#include "nvfp4_46_fused.h"

namespace {

// The library's entry points, in the order of binding.py's NATIVE_ENTRY_POINTS.
struct EntryPoints {
  decltype(&nvfp4_46_tensor_scale) tensor_scale;
  decltype(&nvfp4_46_tensor_scale_ws) tensor_scale_ws;
  decltype(&nvfp4_46_quantize) quantize;
  decltype(&nvfp4_46_scale_quantize) scale_quantize;
  decltype(&nvfp4_46_dequantize) dequantize;
  decltype(&nvfp4_46_fake_quant) fake_quant;
  decltype(&nvfp4_46_gemm) gemm;
};
EntryPoints entry;
// ... and of binding.py's LAYER_ENTRY_POINTS.
struct LayerEntryPoints {
  decltype(&nvfp4_46_few_rows) few_rows;
  decltype(&nvfp4_46_wgrad_operands) wgrad_operands;
};
LayerEntryPoints layer;
PyObject *error_class;     // Nvfp4Error(status, name of the entry point)
PyObject *empty;           // (shape, dtype, device) -> tensor

struct Failed {};          // a Python exception is set

[[noreturn]] void fail(PyObject *type, const char *text) {
  PyErr_SetString(type, text);
  throw Failed{};
}

// ---- arguments, as ctypes takes them: whatever is an integer by __index__ (NumPy's among them), wrapped to its width

uint64_t word(PyObject *o) {
  const uint64_t w = PyLong_AsUnsignedLongLongMask(o);
  if (w == ~(uint64_t)0 && PyErr_Occurred()) throw Failed{};
  return w;
}
float number(PyObject *o) {
  const double d = PyFloat_AsDouble(o);
  if (d == -1.0 && PyErr_Occurred()) throw Failed{};
  return (float)d;
}
// A reference that is given up unless it is released.
struct Owned {
  PyObject *o;
  explicit Owned(PyObject *p) : o(p) {
    if (!o) throw Failed{};
  }
  Owned(const Owned &) = delete;
  ~Owned() { Py_XDECREF(o); }
  PyObject *release() {
    PyObject *r = o;
    o = nullptr;
    return r;
  }
};

// A plain tensor is read directly; a subclass of its own mind, or any other object with a tensor's
// attributes, is asked for them in Python.
const at::Tensor *plain(PyObject *o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }
bool truth(const Owned &v) {
  const int t = PyObject_IsTrue(v.o);
  if (t < 0) throw Failed{};
  return t;
}
c10::SmallVector<int64_t, 4> shape_of(PyObject *o) {
  if (const at::Tensor *t = plain(o)) return {t->sizes().begin(), t->sizes().end()};
  const Owned attribute(PyObject_GetAttrString(o, "shape")), shape(PySequence_Tuple(attribute.o));
  c10::SmallVector<int64_t, 4> sizes;
  for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(shape.o); ++i) sizes.push_back((int64_t)word(PyTuple_GET_ITEM(shape.o, i)));
  return sizes;
}
size_t numel(PyObject *o) {
  if (const at::Tensor *t = plain(o)) return (size_t)t->numel();
  return (size_t)word(Owned(PyObject_CallMethod(o, "numel", nullptr)).o);
}
// None, an address, or a contiguous device tensor
void *pointer(PyObject *o) {
  if (o == Py_None) return nullptr;
  if (PyLong_Check(o)) return reinterpret_cast<void *>(PyLong_AsUnsignedLongLongMask(o));
  const at::Tensor *t = plain(o);
  if (t ? !t->is_cuda() || !t->is_contiguous()
        : !truth(Owned(PyObject_GetAttrString(o, "is_cuda"))) ||
              !truth(Owned(PyObject_CallMethod(o, "is_contiguous", nullptr))))
    fail(PyExc_AssertionError, "tensors must be contiguous device tensors");
  if (t) return t->data_ptr();
  const Owned address(PyObject_CallMethod(o, "data_ptr", nullptr));
  return address.o == Py_None ? nullptr : reinterpret_cast<void *>(word(address.o));
}
// None: the current stream of the current device
void *stream(PyObject *o) {
  if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
  return reinterpret_cast<void *>(word(o));
}

// Other threads of the interpreter run while this lives, also when an exception ends it.
struct WithoutLock {
  PyThreadState *const state = PyEval_SaveThread();
  ~WithoutLock() { PyEval_RestoreThread(state); }
};

// (an allocation may wait for the device, so it is made without the interpreter's lock, as torch.empty does)
PyObject *new_tensor(at::IntArrayRef shape, at::ScalarType type, PyObject *like, PyObject *allocate = Py_None) {
  if (const at::Tensor *l = allocate == Py_None ? plain(like) : nullptr) {
    at::Tensor t;
    {
      WithoutLock others;
      t = at::empty(shape, at::TensorOptions().dtype(type).device(l->device()));
    }
    return THPVariable_Wrap(t);
  }
  const Owned device(PyObject_GetAttrString(like, "device")), sizes(PyTuple_New((Py_ssize_t)shape.size()));
  for (size_t i = 0; i < shape.size(); ++i)
    PyTuple_SET_ITEM(sizes.o, (Py_ssize_t)i, Owned(PyLong_FromLongLong(shape[i])).release());
  return PyObject_CallFunctionObjArgs(allocate == Py_None ? empty : allocate, sizes.o, torch::getTHPDtype(type), device.o,
                                      nullptr);
}

Owned given_or_new(PyObject *given, at::IntArrayRef shape, at::ScalarType type, PyObject *like) {
  if (given == Py_None) return Owned(new_tensor(shape, type, like));
  Py_INCREF(given);
  return Owned(given);
}

// x [rows][cols], BF16 or fp32
void set_shape(nvfp4_46_params &p, PyObject *x) {
  int64_t dims, rows = 0, cols = 0;
  at::ScalarType type = at::kByte;
  if (const at::Tensor *t = plain(x)) {
    dims = t->dim();
    type = t->scalar_type();
    if (dims == 2) {
      rows = t->size(0);
      cols = t->size(1);
    }
  } else {
    dims = (int64_t)word(Owned(PyObject_CallMethod(x, "dim", nullptr)).o);
    const Owned dtype(PyObject_GetAttrString(x, "dtype"));
    if (THPDtype_Check(dtype.o)) type = reinterpret_cast<THPDtype *>(dtype.o)->scalar_type;
    if (dims == 2) {
      const auto shape = shape_of(x);
      if (shape.size() < 2) fail(PyExc_IndexError, "tuple index out of range");
      rows = shape[0];
      cols = shape[1];
    }
  }
  if (dims != 2 || !(type == at::kFloat || type == at::kBFloat16))
    fail(PyExc_AssertionError, "x must be a matrix of BF16 or fp32");
  p.rows = rows;
  p.cols = cols;
  p.x_dtype = type == at::kFloat ? NVFP4_X_F32 : NVFP4_X_BF16;
}
// layout, rounding, select, rht, sr_seed, rht_seed, fp8_max, block2d
nvfp4_46_params params_of(PyObject *x, PyObject *const *a) {
  nvfp4_46_params p{};
  set_shape(p, x);
  p.layout = (uint32_t)word(a[0]);
  p.rounding = (uint32_t)word(a[1]);
  p.select = (uint32_t)word(a[2]);
  p.rht = (uint32_t)word(a[3]);
  p.sr_seed = word(a[4]);
  p.rht_seed = word(a[5]);
  p.fp8_max = number(a[6]);
  p.block2d = (uint32_t)word(a[7]);
  return p;
}

// The call itself, without the interpreter's lock.
template <typename Call>
void run(const char *where, Call &&call) {
  int rc;
  {
    WithoutLock others;
    rc = call();
  }
  if (rc == NVFP4_OK) return;
  PyObject *e = PyObject_CallFunction(error_class, "is", rc, where);
  if (e) {
    PyErr_SetObject(error_class, e);
    Py_DECREF(e);
  }
  throw Failed{};
}

const char *const kCodeNames[6] = {"codes_row", "scales_row", "choice_row", "codes_col", "scales_col", "choice_col"};

// The dictionary of a quantizer's outputs: those that its layout has as new tensors, None for the others.
PyObject *new_codes(PyObject *x, const nvfp4_46_params &p, bool want_choice) {
  Owned d(PyDict_New());
  for (int i = 0; i < 6; ++i) {
    const bool col = i >= 3, codes = i % 3 == 0, choice = i % 3 == 2;
    Owned v(Py_NewRef(Py_None));
    if ((p.layout & (col ? NVFP4_COLWISE : NVFP4_ROWWISE)) && (!choice || want_choice)) {
      const int64_t lines = col ? p.cols : p.rows, along = col ? p.rows : p.cols;
      const int64_t shape[2] = {codes || !p.block2d ? lines : lines / 16, codes ? along / 2 : along / 16};
      Owned t(new_tensor(shape, at::kByte, x));
      std::swap(v.o, t.o);
    }
    if (PyDict_SetItemString(d.o, kCodeNames[i], v.o) < 0) throw Failed{};
  }
  return d.release();
}
// Their addresses; what a mapping returned is held as long, for nothing else may (an allocator would hand the
// memory of an output that is gone before its launch to the next).
struct CodePointers {
  void *p[6];
  PyObject *held[6] = {};
  explicit CodePointers(PyObject *codes) {
    try {
      for (int i = 0; i < 6; ++i) {
        const Owned key(PyUnicode_FromString(kCodeNames[i]));
        Owned v(PyObject_GetItem(codes, key.o));          // (any mapping)
        p[i] = pointer(v.o);
        held[i] = v.release();
      }
    } catch (...) {
      let_go();
      throw;
    }
  }
  CodePointers(const CodePointers &) = delete;
  ~CodePointers() { let_go(); }
  void let_go() {
    for (PyObject *&v : held) Py_CLEAR(v);
  }
};

void expect(Py_ssize_t n, Py_ssize_t want) {
  if (n != want) fail(PyExc_TypeError, "wrong number of arguments");
}

template <PyObject *(*F)(PyObject *const *, Py_ssize_t)>
PyObject *guarded(PyObject *, PyObject *const *a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  try {
    return F(a, n);
  } catch (const Failed &) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}

// ---- one function per entry point; None stands for an output to be allocated

// x, out, stream, then params
PyObject *tensor_scale(PyObject *const *a, Py_ssize_t n) {
  expect(n, 11);
  PyObject *const x = a[0];
  const nvfp4_46_params p = params_of(x, a + 3);
  Owned alpha = given_or_new(a[1], {1}, at::kFloat, x);
  void *const px = pointer(a[0]), *const s = stream(a[2]);
  float *const pa = static_cast<float *>(pointer(alpha.o));
  run("nvfp4_46_tensor_scale", [&] { return entry.tensor_scale(px, &p, pa, s); });
  return alpha.release();
}

// x, workspace, out, stream, then params
PyObject *tensor_scale_ws(PyObject *const *a, Py_ssize_t n) {
  expect(n, 12);
  PyObject *const x = a[0];
  const nvfp4_46_params p = params_of(x, a + 4);
  Owned alpha = given_or_new(a[2], {1}, at::kFloat, x);
  const size_t bytes = numel(a[1]);
  void *const px = pointer(a[0]), *const w = pointer(a[1]), *const s = stream(a[3]);
  float *const pa = static_cast<float *>(pointer(alpha.o));
  run("nvfp4_46_tensor_scale_ws", [&] { return entry.tensor_scale_ws(px, &p, pa, w, bytes, s); });
  return alpha.release();
}

// x, alpha, out, want_choice, stream, then params
PyObject *quantize(PyObject *const *a, Py_ssize_t n) {
  expect(n, 13);
  PyObject *const x = a[0];
  const nvfp4_46_params p = params_of(x, a + 5);
  const int choice = PyObject_IsTrue(a[3]);
  if (choice < 0) return nullptr;
  Owned codes(a[2] == Py_None ? new_codes(x, p, choice) : Py_NewRef(a[2]));
  const CodePointers c(codes.o);
  void *const px = pointer(a[0]), *const s = stream(a[4]);
  const float *const pa = static_cast<const float *>(pointer(a[1]));
  run("nvfp4_46_quantize", [&] { return entry.quantize(px, &p, pa, c.p[0], c.p[1], c.p[3], c.p[4], c.p[2], c.p[5], s); });
  return codes.release();
}

// x, workspace or None, alpha, out, want_choice, stream, then params; alpha joins the dictionary
PyObject *scale_quantize(PyObject *const *a, Py_ssize_t n) {
  expect(n, 14);
  PyObject *const x = a[0];
  const nvfp4_46_params p = params_of(x, a + 6);
  const int choice = PyObject_IsTrue(a[4]);
  if (choice < 0) return nullptr;
  Owned alpha = given_or_new(a[2], {1}, at::kFloat, x);
  Owned codes(a[3] == Py_None ? new_codes(x, p, choice) : Py_NewRef(a[3]));
  const CodePointers c(codes.o);
  void *const px = pointer(a[0]), *const w = pointer(a[1]), *const s = stream(a[5]);
  const size_t bytes = a[1] == Py_None ? 0 : numel(a[1]);
  float *const pa = static_cast<float *>(pointer(alpha.o));
  run("nvfp4_46_scale_quantize", [&] {
    return entry.scale_quantize(px, &p, pa, w, bytes, c.p[0], c.p[1], c.p[3], c.p[4], c.p[2], c.p[5], s);
  });
  if (PyObject_SetItem(codes.o, Owned(PyUnicode_FromString("alpha")).o, alpha.o) < 0) return nullptr;
  return codes.release();
}

// codes, scales, alpha, rows, cols, layout, out, stream
PyObject *dequantize(PyObject *const *a, Py_ssize_t n) {
  expect(n, 8);
  const int64_t rows = (int64_t)word(a[3]), cols = (int64_t)word(a[4]);
  const uint32_t layout = (uint32_t)word(a[5]);
  Owned out = a[6] == Py_None ? Owned(new_tensor({rows, cols}, at::kBFloat16, a[0]))
                              : Owned(Py_NewRef(a[6]));
  void *const c = pointer(a[0]), *const sc = pointer(a[1]), *const o = pointer(out.o), *const s = stream(a[7]);
  const float *const pa = static_cast<const float *>(pointer(a[2]));
  run("nvfp4_46_dequantize", [&] { return entry.dequantize(c, sc, pa, rows, cols, layout, o, s); });
  return out.release();
}

// x, alpha, out, stream, then params
PyObject *fake_quant(PyObject *const *a, Py_ssize_t n) {
  expect(n, 12);
  PyObject *const x = a[0];
  const nvfp4_46_params p = params_of(x, a + 4);
  Owned out = given_or_new(a[2], {p.rows, p.cols}, at::kBFloat16, x);
  void *const px = pointer(a[0]), *const o = pointer(out.o), *const s = stream(a[3]);
  const float *const pa = static_cast<const float *>(pointer(a[1]));
  run("nvfp4_46_fake_quant", [&] { return entry.fake_quant(px, &p, pa, o, s); });
  return out.release();
}

// codes_a, scales_a, alpha_a, codes_b, scales_b, alpha_b, out_dtype, out, stream, flags
PyObject *gemm(PyObject *const *a, Py_ssize_t n) {
  expect(n, 10);
  const auto ca = shape_of(a[0]), sa = shape_of(a[1]), cb = shape_of(a[3]), sb = shape_of(a[4]);
  const uint32_t out_dtype = (uint32_t)word(a[6]), flags = (uint32_t)word(a[9]);
  if (ca.size() < 2 || cb.size() < 2) fail(PyExc_IndexError, "tuple index out of range");
  const int64_t M = ca[0], N = cb[0], K = ca[1] * 2;
  auto is = [](const auto &shape, int64_t rows, int64_t cols) {
    return shape.size() == 2 && shape[0] == rows && shape[1] == cols;
  };
  if (cb[1] * 2 != K || !is(sa, flags & NVFP4_GEMM_A_TILE_SCALES ? M / 16 : M, K / 16) ||
      !is(sb, flags & NVFP4_GEMM_B_TILE_SCALES ? N / 16 : N, K / 16))
    fail(PyExc_AssertionError, "operands that do not fit together");
  Owned out = given_or_new(a[7], {M, N}, out_dtype == NVFP4_OUT_F32 ? at::kFloat : at::kBFloat16, a[0]);
  void *const pca = pointer(a[0]), *const psa = pointer(a[1]), *const pcb = pointer(a[3]), *const psb = pointer(a[4]);
  const float *const paa = static_cast<const float *>(pointer(a[2])), *const pab = static_cast<const float *>(pointer(a[5]));
  void *const o = pointer(out.o), *const s = stream(a[8]);
  run("nvfp4_46_gemm", [&] { return entry.gemm(pca, psa, paa, pcb, psb, pab, M, N, K, out_dtype, flags, o, s); });
  return out.release();
}

// ---- the products of a linear layer (linear.py), each in one call: the operands that it quantizes on the way live in
// one buffer that is never a Python object.  They work on plain contiguous device tensors that fit together, on the
// current stream; for anything else, also for what the calls one by one refuse, they return None and linear.py makes
// those calls.  `allocate` makes buffers and outputs, as binding.py's OUTPUT_ALLOCATOR (None: as torch.empty).

bool ready(const at::Tensor *t) {
  return t && t->is_cuda() && t->is_contiguous() && reinterpret_cast<uintptr_t>(t->data_ptr()) % 16 == 0;
}
bool ready_matrix(const at::Tensor *t) {
  return ready(t) && t->dim() == 2 && t->size(0) > 0 && t->size(1) > 0 &&
         (t->scalar_type() == at::kBFloat16 || t->scalar_type() == at::kFloat);
}
// a workspace that the calls one by one would take, or none
struct Workspace {
  bool fits;
  void *p = nullptr;
  size_t bytes = 0;
  explicit Workspace(PyObject *o) : fits(o == Py_None) {
    if (fits) return;
    const at::Tensor *t = plain(o);
    fits = ready(t) && t->numel() >= NVFP4_46_TENSOR_SCALE_WS_BYTES;
    if (fits) {
      p = t->data_ptr();
      bytes = (size_t)t->numel();
    }
  }
};
// Device memory for operands, `bytes` of it; parts of it begin at multiples of 256 bytes.
constexpr int64_t round_up(int64_t bytes) { return (bytes + 255) / 256 * 256; }
struct Buffer {
  at::Tensor own;
  PyObject *given = nullptr;
  char *p;
  Buffer(int64_t bytes, PyObject *like, PyObject *allocate) {
    if (allocate == Py_None) {
      WithoutLock others;
      own = at::empty({bytes}, at::TensorOptions().dtype(at::kByte).device(plain(like)->device()));
      p = static_cast<char *>(own.data_ptr());
    } else {
      Owned t(new_tensor({bytes}, at::kByte, like, allocate));
      p = static_cast<char *>(pointer(t.o));
      given = t.release();
    }
  }
  Buffer(const Buffer &) = delete;
  ~Buffer() { Py_XDECREF(given); }
};
// One quantized operand of `lines` lines of K values in a buffer.
struct Operand {
  int64_t lines, K;
  int64_t bytes() const { return round_up(lines * K / 2) + round_up(lines * K / 16) + 256; }
  char *codes(char *p) const { return p; }
  char *scales(char *p) const { return p + round_up(lines * K / 2); }
  float *alpha(char *p) const { return reinterpret_cast<float *>(scales(p) + round_up(lines * K / 16)); }
};

// x, codes_b, scales_b, alpha_b, allocate, workspace, flags, rounding, select, sr_seed: x quantized rowwise, times B^T, BF16
PyObject *product_of_rows(PyObject *const *a, Py_ssize_t n) {
  expect(n, 10);
  const at::Tensor *x = plain(a[0]), *cb = plain(a[1]), *sb = plain(a[2]), *alpha = plain(a[3]);
  const Workspace ws(a[5]);
  if (!ready_matrix(x) || !ready(cb) || !ready(sb) || !alpha || !alpha->is_cuda() || !alpha->is_contiguous() || !ws.fits ||
      cb->dim() != 2 || sb->dim() != 2)
    Py_RETURN_NONE;
  const int64_t M = x->size(0), K = x->size(1), N = cb->size(0);
  const uint32_t flags = (uint32_t)word(a[6]), rounding = (uint32_t)word(a[7]), select = (uint32_t)word(a[8]);
  const uint64_t sr_seed = word(a[9]);
  const bool tiles = flags & NVFP4_GEMM_B_TILE_SCALES;
  if (N <= 0 || K % 32 != 0 || cb->size(1) * 2 != K || (tiles && N % 16 != 0) || sb->size(0) != (tiles ? N / 16 : N) ||
      sb->size(1) != K / 16)
    Py_RETURN_NONE;
  const void *const px = x->data_ptr(), *const pc = cb->data_ptr(), *const ps = sb->data_ptr();
  const float *const pa = static_cast<const float *>(alpha->data_ptr());
  void *const s = stream(Py_None);
  if (x->scalar_type() == at::kBFloat16 && rounding == NVFP4_RTN && select == NVFP4_SEL_46_MSE &&
      nvfp4_46::few_rows_in_one_launch(M, N, K)) {
    Owned out(new_tensor({M, N}, at::kBFloat16, a[0], a[4]));
    void *const o = pointer(out.o);
    run("nvfp4_46_few_rows", [&] { return layer.few_rows(px, 256.0f, pc, ps, pa, M, N, K, flags, o, s); });
    return out.release();
  }
  nvfp4_46_params p{};
  set_shape(p, a[0]);
  p.layout = NVFP4_ROWWISE;
  p.rounding = rounding;
  p.select = select;
  p.sr_seed = sr_seed;
  p.fp8_max = 256.0f;
  const Operand q{M, K};
  const Buffer buffer(q.bytes(), a[0], a[4]);
  char *const b = buffer.p;
  run("nvfp4_46_scale_quantize", [&] {
    return entry.scale_quantize(px, &p, q.alpha(b), ws.p, ws.bytes, q.codes(b), q.scales(b), nullptr, nullptr, nullptr, nullptr,
                                s);
  });
  Owned out(new_tensor({M, N}, at::kBFloat16, a[0], a[4]));
  void *const o = pointer(out.o);
  run("nvfp4_46_gemm", [&] {
    return entry.gemm(q.codes(b), q.scales(b), q.alpha(b), pc, ps, pa, M, N, K, NVFP4_OUT_BF16, flags, o, s);
  });
  return out.release();
}

// dy, x, allocate, workspace, select, sr_seed, rht_seed: dy^T x, fp32, both operands transformed along the rows
PyObject *product_of_columns(PyObject *const *a, Py_ssize_t n) {
  expect(n, 7);
  const at::Tensor *dy = plain(a[0]), *x = plain(a[1]);
  const Workspace ws(a[3]);
  if (!ready_matrix(dy) || !ready_matrix(x) || !ws.fits || dy->scalar_type() != at::kBFloat16 ||
      x->scalar_type() != at::kBFloat16 || dy->device() != x->device())
    Py_RETURN_NONE;
  const int64_t T = dy->size(0), N = dy->size(1), K = x->size(1);
  if (x->size(0) != T || T % 32 != 0 || N % 8 != 0 || K % 8 != 0) Py_RETURN_NONE;
  const uint32_t select = (uint32_t)word(a[4]);
  const uint64_t sr_seed = word(a[5]), rht_seed = word(a[6]);
  const Operand qd{N, T}, qx{K, T};
  const Buffer buffer(qd.bytes() + qx.bytes(), a[0], a[2]);
  char *const bd = buffer.p, *const bx = buffer.p + qd.bytes();
  const void *const pd = dy->data_ptr(), *const px = x->data_ptr();
  void *const s = stream(Py_None);
  run("nvfp4_46_scale_quantize", [&] {
    return layer.wgrad_operands(pd, px, T, N, K, select, sr_seed, rht_seed, qd.alpha(bd), qd.codes(bd), qd.scales(bd),
                                qx.alpha(bx), qx.codes(bx), qx.scales(bx), ws.p, ws.bytes, s);
  });
  Owned out(new_tensor({N, K}, at::kFloat, a[0], a[2]));
  void *const o = pointer(out.o);
  run("nvfp4_46_gemm", [&] {
    return entry.gemm(qd.codes(bd), qd.scales(bd), qd.alpha(bd), qx.codes(bx), qx.scales(bx), qx.alpha(bx), N, K, T,
                      NVFP4_OUT_F32, 0, o, s);
  });
  return out.release();
}

template <typename Points>
void take_addresses(Points &points, PyObject *const *a, Py_ssize_t n) {
  constexpr Py_ssize_t kEntries = sizeof(Points) / sizeof(void *);
  expect(n, kEntries);
  void *to[kEntries];
  for (Py_ssize_t i = 0; i < kEntries; ++i) to[i] = reinterpret_cast<void *>(word(a[i]));
  std::memcpy(&points, to, sizeof points);
}
// The exception class, torch.empty as (shape, dtype, device), then the addresses of the entry points, one integer
// each.
PyObject *connect(PyObject *const *a, Py_ssize_t n) {
  expect(n < 2 ? n : 2, 2);
  take_addresses(entry, a + 2, n - 2);
  error_class = Py_NewRef(a[0]);
  empty = Py_NewRef(a[1]);
  Py_RETURN_NONE;
}
PyObject *connect_layer(PyObject *const *a, Py_ssize_t n) {
  take_addresses(layer, a, n);
  Py_RETURN_NONE;
}

#define NV_METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(guarded<f>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {NV_METHOD(connect), NV_METHOD(connect_layer),
                           NV_METHOD(tensor_scale), NV_METHOD(tensor_scale_ws), NV_METHOD(quantize),
                         NV_METHOD(scale_quantize), NV_METHOD(dequantize), NV_METHOD(fake_quant), NV_METHOD(gemm),
                         NV_METHOD(product_of_rows), NV_METHOD(product_of_columns),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "nvfp4_46_python", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_nvfp4_46_python() { return PyModule_Create(&module); }
