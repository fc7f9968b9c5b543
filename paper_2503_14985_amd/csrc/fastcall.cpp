// The entry points' usual case in native code: what binding.py does with the tensors of a call (their sizes, strides, types and
// addresses, the current stream) took 3.5 of the 7.3 us of a small one, as much as the library and the runtime; here 0.4.
// A function looks at its arguments as binding.py passes them on. Where they are plain tensors on the current GPU of the shapes and types that
// the entry point takes, with an output tensor given and no stream, it makes the call and returns the output, or raises what
// the library's status stands for: the call is made once (a second one could succeed after a launch error that an
// earlier call had left, and an accumulating GEMM would have added twice). Everything else returns None: binding.py then goes
// through it step by step, allocates, or raises.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/mlt.h"

namespace {

// the library's functions, as binding.py has loaded them
decltype(&mlt_gemm) call_gemm;
decltype(&mlt_gemm_bias_act) call_gemm_bias_act;
decltype(&mlt_gemm_acc) call_gemm_acc;
decltype(&mlt_mha_fwd) call_mha_fwd;
decltype(&mlt_paged_attn_decode) call_paged;
PyObject* error_class;      // binding.MltError(status, where)

// A plain tensor with memory of its own kind on GPU `device` (-1: the first one sets it), or null
const at::Tensor* plain(PyObject* o, int& device) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || !t.has_storage() || t.layout() != at::kStrided) return nullptr;
  if (device < 0) device = t.device().index();
  return t.device().index() == device ? &t : nullptr;
}

int dtype_code(const at::Tensor& t) {
  const auto s = t.scalar_type();
  return s == at::kBFloat16 ? MLT_BF16 : s == at::kHalf ? MLT_FP16 : -1;
}

// leading dimension of a matrix with contiguous rows, or -1
int64_t row_stride(const at::Tensor& t) {
  if (t.dim() != 2 || (t.size(1) > 1 && t.stride(1) != 1)) return -1;
  return t.size(0) > 1 ? t.stride(0) : t.size(1) > 1 ? t.size(1) : 1;
}

struct Gemm {
  int64_t M, N, K, lda, ldb, ldc;
  int dtype, device = -1;
  void *a, *b, *c, *stream;
};

bool on_current_device(int device, void** stream) {
  if (c10::hip::current_device() != device) return false;
  *stream = c10::hip::getCurrentHIPStream((c10::DeviceIndex)device).stream();
  return true;
}

bool gemm_operands(PyObject* A, PyObject* B, PyObject* C, bool transB, bool c_is_fp32, Gemm& g) {
  const at::Tensor *a = plain(A, g.device), *b = a ? plain(B, g.device) : nullptr, *c = b ? plain(C, g.device) : nullptr;
  if (!c) return false;
  g.dtype = dtype_code(*a);
  if (g.dtype < 0 || b->scalar_type() != a->scalar_type()) return false;
  if (c->scalar_type() != (c_is_fp32 ? at::kFloat : a->scalar_type())) return false;
  g.lda = row_stride(*a);
  g.ldb = row_stride(*b);
  g.ldc = row_stride(*c);
  if (g.lda < 0 || g.ldb < 0 || g.ldc < 0) return false;
  g.M = a->size(0);
  g.K = a->size(1);
  g.N = transB ? b->size(0) : b->size(1);
  if ((transB ? b->size(1) : b->size(0)) != g.K || c->size(0) != g.M || c->size(1) != g.N) return false;
  if (!on_current_device(g.device, &g.stream)) return false;
  g.a = a->data_ptr();
  g.b = b->data_ptr();
  g.c = c->data_ptr();
  return true;
}

PyObject* result(int rc, PyObject* out, const char* where) {
  if (rc != MLT_OK) {
    if (PyObject* e = PyObject_CallFunction(error_class, "is", rc, where)) {
      PyErr_SetObject(error_class, e);
      Py_DECREF(e);
    }
    return nullptr;
  }
  Py_INCREF(out);
  return out;
}

// gemm(A, B, C, transB, stream)
PyObject* py_gemm(PyObject*, PyObject* const* v, Py_ssize_t n) {
  Gemm g;
  if (n != 5 || v[4] != Py_None || !PyBool_Check(v[3]) || !gemm_operands(v[0], v[1], v[2], v[3] == Py_True, false, g)) Py_RETURN_NONE;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = call_gemm(g.M, g.N, g.K, g.a, g.lda, g.b, g.ldb, v[3] == Py_True, g.c, g.ldc, g.dtype, g.stream);
  Py_END_ALLOW_THREADS
  return result(rc, v[2], "mlt_gemm");
}

// gemm_acc(A, B, C, transB, stream)
PyObject* py_gemm_acc(PyObject*, PyObject* const* v, Py_ssize_t n) {
  Gemm g;
  if (n != 5 || v[4] != Py_None || !PyBool_Check(v[3]) || !gemm_operands(v[0], v[1], v[2], v[3] == Py_True, true, g)) Py_RETURN_NONE;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = call_gemm_acc(g.M, g.N, g.K, g.a, g.lda, g.b, g.ldb, v[3] == Py_True, (float*)g.c, g.ldc, g.dtype, g.stream);
  Py_END_ALLOW_THREADS
  return result(rc, v[2], "mlt_gemm_acc");
}

// gemm_bias_act(A, B, bias, act, C, transB, stream)
PyObject* py_gemm_bias_act(PyObject*, PyObject* const* v, Py_ssize_t n) {
  Gemm g;
  if (n != 7 || v[6] != Py_None || !PyBool_Check(v[5]) || !PyLong_CheckExact(v[3])) Py_RETURN_NONE;
  int overflow = 0;
  const long act = PyLong_AsLongAndOverflow(v[3], &overflow);
  if (overflow || act < 0 || act > 2 || !gemm_operands(v[0], v[1], v[4], v[5] == Py_True, false, g)) Py_RETURN_NONE;
  void* bias = nullptr;
  if (v[2] != Py_None) {
    const at::Tensor* t = plain(v[2], g.device);
    if (!t || dtype_code(*t) != g.dtype || t->dim() != 1 || t->size(0) != g.N || !t->is_contiguous()) Py_RETURN_NONE;
    bias = t->data_ptr();
  }
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = call_gemm_bias_act(g.M, g.N, g.K, g.a, g.lda, g.b, g.ldb, v[5] == Py_True, bias, (int)act, g.c, g.ldc, g.dtype, g.stream);
  Py_END_ALLOW_THREADS
  return result(rc, v[4], "mlt_gemm_bias_act");
}

// mha_fwd(Q, K, V, scale, causal, O, stream)
PyObject* py_mha_fwd(PyObject*, PyObject* const* v, Py_ssize_t n) {
  if (n != 7 || v[6] != Py_None || !PyFloat_CheckExact(v[3]) || !PyBool_Check(v[4])) Py_RETURN_NONE;
  int device = -1;
  const at::Tensor* t[4];
  PyObject* const o[4] = {v[0], v[1], v[2], v[5]};
  for (int i = 0; i < 4; ++i) {
    t[i] = plain(o[i], device);
    if (!t[i] || t[i]->dim() != 4 || !t[i]->is_contiguous() || t[i]->scalar_type() != t[0]->scalar_type()) Py_RETURN_NONE;
  }
  const at::Tensor &q = *t[0], &k = *t[1];
  const int dtype = dtype_code(q);
  if (dtype < 0 || k.size(0) != q.size(0) || k.size(1) != q.size(1) || k.size(3) != q.size(3)) Py_RETURN_NONE;
  if (t[2]->sizes() != k.sizes() || t[3]->sizes() != q.sizes()) Py_RETURN_NONE;
  void* stream;
  if (!on_current_device(device, &stream)) Py_RETURN_NONE;
  const int64_t B = q.size(0), H = q.size(1), Sq = q.size(2), Sk = k.size(2), D = q.size(3);
  void* p[4];
  for (int i = 0; i < 4; ++i) p[i] = t[i]->data_ptr();
  const float scale = (float)PyFloat_AS_DOUBLE(v[3]);
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = call_mha_fwd(B, H, Sq, Sk, D, p[0], p[1], p[2], p[3], scale, v[4] == Py_True, dtype, stream);
  Py_END_ALLOW_THREADS
  return result(rc, v[5], "mlt_mha_fwd");
}

// paged_attn_decode(Q, Kc, Vc, block_table, seq_lens, scale, O)
PyObject* py_paged(PyObject*, PyObject* const* v, Py_ssize_t n) {
  if (n != 7 || !PyFloat_CheckExact(v[5])) Py_RETURN_NONE;
  int device = -1;
  const at::Tensor* t[6];
  PyObject* const o[6] = {v[0], v[1], v[2], v[3], v[4], v[6]};
  for (int i = 0; i < 6; ++i) {
    t[i] = plain(o[i], device);
    if (!t[i] || !t[i]->is_contiguous()) Py_RETURN_NONE;
  }
  const at::Tensor &q = *t[0], &kc = *t[1], &vc = *t[2], &table = *t[3], &lens = *t[4], &out = *t[5];
  const int dtype = dtype_code(q);
  if (dtype < 0 || q.dim() != 3 || kc.dim() != 4 || kc.size(1) != q.size(1) || kc.size(3) != q.size(2)) Py_RETURN_NONE;
  if (vc.sizes() != kc.sizes() || kc.scalar_type() != q.scalar_type() || vc.scalar_type() != q.scalar_type()) Py_RETURN_NONE;
  if (table.scalar_type() != at::kInt || lens.scalar_type() != at::kInt || table.dim() != 2 || lens.dim() != 1) Py_RETURN_NONE;
  if (table.size(0) != q.size(0) || lens.size(0) != q.size(0)) Py_RETURN_NONE;
  if (out.scalar_type() != q.scalar_type() || out.sizes() != q.sizes()) Py_RETURN_NONE;
  void* stream;
  if (!on_current_device(device, &stream)) Py_RETURN_NONE;
  const int64_t B = q.size(0), H = q.size(1), D = q.size(2), block = kc.size(2), blocks = table.size(1), num = kc.size(0);
  void* p[6];
  for (int i = 0; i < 6; ++i) p[i] = t[i]->data_ptr();
  const float scale = (float)PyFloat_AS_DOUBLE(v[5]);
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = call_paged(B, H, D, block, blocks, num, p[0], p[1], p[2], (const int32_t*)p[3], (const int32_t*)p[4], p[5], scale, dtype, stream);
  Py_END_ALLOW_THREADS
  return result(rc, v[6], "mlt_paged_attn_decode");
}

// A torch error in here (a tensor without memory behind it, say) is binding.py's to meet again
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* v, Py_ssize_t n) {
  try {
    return F(self, v, n);
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

// bind(error class, gemm, gemm_bias_act, gemm_acc, mha_fwd, paged_attn_decode): the library functions' addresses
PyObject* py_bind(PyObject*, PyObject* args) {
  Py_ssize_t a[5];
  PyObject* err;
  if (!PyArg_ParseTuple(args, "Onnnnn", &err, &a[0], &a[1], &a[2], &a[3], &a[4])) return nullptr;
  Py_INCREF(err);
  error_class = err;
  call_gemm = reinterpret_cast<decltype(call_gemm)>(a[0]);
  call_gemm_bias_act = reinterpret_cast<decltype(call_gemm_bias_act)>(a[1]);
  call_gemm_acc = reinterpret_cast<decltype(call_gemm_acc)>(a[2]);
  call_mha_fwd = reinterpret_cast<decltype(call_mha_fwd)>(a[3]);
  call_paged = reinterpret_cast<decltype(call_paged)>(a[4]);
  Py_RETURN_NONE;
}

#define MLT_FAST(name, f) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(guarded<f>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {MLT_FAST("gemm", py_gemm),
                         MLT_FAST("gemm_acc", py_gemm_acc),
                         MLT_FAST("gemm_bias_act", py_gemm_bias_act),
                         MLT_FAST("mha_fwd", py_mha_fwd),
                         MLT_FAST("paged_attn_decode", py_paged),
                         {"bind", py_bind, METH_VARARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) {
  PyObject* m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "torch_version", MLT_TORCH_VERSION) != 0) Py_CLEAR(m);   // whose tensors it knows
  return m;
}
