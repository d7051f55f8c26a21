// Argument marshalling of the Python binding's hot entry points, in C++: reads the tensors'
// pointers, shapes and strides, makes the checks the binding makes, and calls the C ABI.
//
// Why: the same work in Python took 6.7 us a call (attribute reads of three tensors, the current
// stream, nineteen ctypes conversions), more than the 4.1 us a 256^3 product takes from end to end
// in a loop on the C side.
//
// Every function returns the C call's status, or None for arguments it does not take as they are;
// the Python code then repeats the checks and raises what it has to say about them.  The functions
// of the library are reached through the addresses init() is given, so that the module holds no
// second copy of it.
#include <torch/csrc/autograd/python_variable.h>

#include <c10/hip/HIPStream.h>

#include <string>

#include "../../include/alcop.h"

namespace {

struct Api {
  decltype(&alcop_gemm_fused) gemm = nullptr;
  decltype(&alcop_bmm_fused) bmm = nullptr;
  decltype(&alcop_bmm_unaligned) bmm_any = nullptr;
  decltype(&alcop_conv2d_igemm_dilated) conv = nullptr;
  decltype(&alcop_conv2d_igemm_unaligned) conv_any = nullptr;
} api;

PyObject* sched_type = nullptr;   // the binding's ctypes mirror of alcop_sched

// Raised to leave a call to the Python code.
struct Unusual {};

// An exception out of the library's call itself, which is not made a second time.
struct Failed {
  std::string what;
};

inline void need(bool ok)
{
  if (!ok) throw Unusual{};
}

const at::Tensor& tensor(PyObject* o)
{
  need(THPVariable_Check(o));
  return THPVariable_Unpack(o);
}

alcop_dtype dtype(const at::Tensor& t)
{
  switch (t.scalar_type()) {
    case at::kHalf: return ALCOP_F16;
    case at::kBFloat16: return ALCOP_BF16;
    case at::kFloat: return ALCOP_F32;
    default: throw Unusual{};
  }
}

int truth(PyObject* o)
{
  need(PyLong_Check(o));            // True and False are integers
  const int v = PyObject_IsTrue(o);
  need(v >= 0);
  return v;
}

int integer(PyObject* o)
{
  const long v = PyLong_Check(o) ? PyLong_AsLong(o) : -1;
  need(PyLong_Check(o) && !(v == -1 && PyErr_Occurred()) && v >= INT32_MIN && v <= INT32_MAX);
  return (int)v;
}

void pair(PyObject* o, int (&v)[2])
{
  need(PyTuple_Check(o) && PyTuple_GET_SIZE(o) == 2);
  v[0] = integer(PyTuple_GET_ITEM(o, 0));
  v[1] = integer(PyTuple_GET_ITEM(o, 1));
}

// None: the current stream of the current device; otherwise an object with a cuda_stream handle.
void* stream_of(PyObject* o)
{
  if (o == Py_None) return (void*)c10::hip::getCurrentHIPStream().stream();
  PyObject* h = PyObject_GetAttrString(o, "cuda_stream");
  need(h != nullptr);
  void* s = PyLong_Check(h) ? PyLong_AsVoidPtr(h) : nullptr;
  const bool ok = PyLong_Check(h) && !PyErr_Occurred();
  Py_DECREF(h);
  need(ok);
  return s;
}

// None, or the ctypes mirror of alcop_sched.
struct Schedule {
  alcop_sched s;
  const alcop_sched* p = nullptr;
  explicit Schedule(PyObject* o)
  {
    if (o == Py_None) return;
    const int is = PyObject_IsInstance(o, sched_type);    // any other buffer is not a schedule
    need(is == 1);
    Py_buffer b;
    need(PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) == 0);
    const bool ok = b.len == (Py_ssize_t)sizeof(s);
    if (ok) memcpy(&s, b.buf, sizeof(s));
    PyBuffer_Release(&b);
    need(ok);
    p = &s;
  }
};

alcop_epilogue epilogue(PyObject* alpha, PyObject* bias, PyObject* act, int64_t n, const at::Tensor& like)
{
  alcop_epilogue e{1.0f, nullptr, 0};
  const double a = PyFloat_AsDouble(alpha);
  need(!(a == -1.0 && PyErr_Occurred()));
  e.alpha = (float)a;
  e.act = integer(act);
  if (bias != Py_None) {
    const at::Tensor& b = tensor(bias);
    need(b.dim() == 1 && b.size(0) == n && b.is_contiguous() && b.scalar_type() == at::kFloat && b.device() == like.device());
    e.bias = b.const_data_ptr();
  }
  return e;
}

struct Mats {
  const at::Tensor &A, &B, &C;
  int batch, M, N, K, tA, tB;
  long ld[3], st[3];
  alcop_dtype in, out;
  Mats(PyObject* a, PyObject* b, PyObject* c, PyObject* ta, PyObject* tb)
      : A(tensor(a)), B(tensor(b)), C(tensor(c)), tA(truth(ta)), tB(truth(tb)), in(dtype(A)), out(dtype(C))
  {
    const int64_t d = A.dim();
    need((d == 2 || d == 3) && B.dim() == d && C.dim() == d && A.scalar_type() == B.scalar_type());
    need(A.device() == B.device() && A.device() == C.device());
    need(A.is_cuda());
    const at::Tensor* t[3] = {&A, &B, &C};
    const int64_t nb = d == 3 ? A.size(0) : 1;
    for (int i = 0; i < 3; i++) {
      need(t[i]->stride(d - 1) == 1 && (d == 2 || t[i]->size(0) == nb));
      ld[i] = t[i]->stride(d - 2);
      st[i] = d == 3 ? t[i]->stride(0) : 0;
    }
    const int64_t m = A.size(tA ? d - 1 : d - 2), k = A.size(tA ? d - 2 : d - 1);
    const int64_t kb = B.size(tB ? d - 1 : d - 2), n = B.size(tB ? d - 2 : d - 1);
    need(kb == k && C.size(d - 2) == m && C.size(d - 1) == n);
    need(nb <= INT32_MAX && m <= INT32_MAX && n <= INT32_MAX && k <= INT32_MAX);
    batch = (int)nb;
    M = (int)m;
    N = (int)n;
    K = (int)k;
  }
};

template <class F>
PyObject* guarded(F&& f)
{
  int rc;
  try {
    rc = f();
  } catch (const Unusual&) {
    PyErr_Clear();
    Py_RETURN_NONE;
  } catch (const Failed& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what.c_str());
    return nullptr;
  } catch (const std::exception&) {   // from the tensor accessors
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  return PyLong_FromLong(rc);
}

// The call itself, without the interpreter lock (as ctypes makes it), which is taken back however the
// call ends.
template <class F>
int unlocked(F&& f)
{
  struct Unlock {
    PyThreadState* state = PyEval_SaveThread();
    ~Unlock() { PyEval_RestoreThread(state); }
  } unlock;
  try {
    return f();
  } catch (const std::exception& e) {
    throw Failed{e.what()};
  }
}

// mm(A, B, C, transA, transB, sched, stream[, alpha, bias, act]): 2-D gemm, 3-D batched
PyObject* mm(PyObject*, PyObject* const* a, Py_ssize_t n)
{
  return guarded([&] {
    need(api.gemm && (n == 7 || n == 10));
    const Mats m(a[0], a[1], a[2], a[3], a[4]);
    const Schedule s(a[5]);
    void* st = stream_of(a[6]);
    alcop_epilogue e{1.0f, nullptr, 0};
    if (n == 10) e = epilogue(a[7], a[8], a[9], m.N, m.A);
    const void *A = m.A.const_data_ptr(), *B = m.B.const_data_ptr();
    void* C = m.C.data_ptr();
    const bool two = m.A.dim() == 2;
    return unlocked([&] {
      return two ? api.gemm(A, B, C, m.M, m.N, m.K, m.ld[0], m.ld[1], m.ld[2], m.tA, m.tB, m.in, m.out, &e, s.p, st)
                 : api.bmm(A, B, C, m.batch, m.M, m.N, m.K, m.ld[0], m.ld[1], m.ld[2], m.st[0], m.st[1], m.st[2],
                           m.tA, m.tB, m.in, m.out, &e, s.p, st);
    });
  });
}

// mm_any(A, B, C, workspace, alpha, bias, act, sched, transA, transB, stream)
PyObject* mm_any(PyObject*, PyObject* const* a, Py_ssize_t n)
{
  return guarded([&] {
    need(api.bmm_any && n == 11);
    const Mats m(a[0], a[1], a[2], a[8], a[9]);
    const at::Tensor& w = tensor(a[3]);
    need(w.is_contiguous() && w.device() == m.A.device());
    const alcop_epilogue e = epilogue(a[4], a[5], a[6], m.N, m.A);
    const Schedule s(a[7]);
    void* st = stream_of(a[10]);
    const void *A = m.A.const_data_ptr(), *B = m.B.const_data_ptr();
    void *C = m.C.data_ptr(), *ws = w.data_ptr();
    const size_t bytes = w.nbytes();
    return unlocked([&] {
      return api.bmm_any(A, B, C, m.batch, m.M, m.N, m.K, m.ld[0], m.ld[1], m.ld[2], m.st[0], m.st[1], m.st[2], m.tA,
                         m.tB, m.in, m.out, &e, s.p, ws, bytes, st);
    });
  });
}

struct Conv {
  const at::Tensor &x, &w, &y;
  int krsc, N, H, W, C, K, R, S, stride[2], pad[2], dil[2];
  alcop_dtype in, out;
  Conv(PyObject* ox, PyObject* ow, PyObject* oy, PyObject* ostride, PyObject* opad, PyObject* odil, int k)
      : x(tensor(ox)), w(tensor(ow)), y(tensor(oy)), krsc(k), in(dtype(x)), out(dtype(y))
  {
    need(x.dim() == 4 && w.dim() == 4 && y.dim() == 4 && x.scalar_type() == w.scalar_type());
    need(x.device() == w.device() && x.device() == y.device());
    need(x.is_cuda() && x.is_contiguous() && w.is_contiguous() && y.is_contiguous());
    pair(ostride, stride);
    pair(opad, pad);
    pair(odil, dil);
    need(stride[0] > 0 && stride[1] > 0 && pad[0] >= 0 && pad[1] >= 0 && dil[0] > 0 && dil[1] > 0);
    const int64_t e[7] = {x.size(0), x.size(1), x.size(2), x.size(3), w.size(krsc ? 0 : 3), w.size(krsc ? 1 : 0),
                          w.size(krsc ? 2 : 1)};
    for (int64_t v : e) need(v >= 1 && v <= INT32_MAX);
    need(w.size(krsc ? 3 : 2) == e[3]);
    const int64_t eh = e[1] + 2 * (int64_t)pad[0] - dil[0] * (e[5] - 1) - 1;
    const int64_t ew = e[2] + 2 * (int64_t)pad[1] - dil[1] * (e[6] - 1) - 1;
    need(eh >= 0 && ew >= 0);
    need(y.size(0) == e[0] && y.size(1) == eh / stride[0] + 1 && y.size(2) == ew / stride[1] + 1 && y.size(3) == e[4]);
    N = (int)e[0];
    H = (int)e[1];
    W = (int)e[2];
    C = (int)e[3];
    K = (int)e[4];
    R = (int)e[5];
    S = (int)e[6];
  }
};

// conv(x, w, y, stride, pad, dilation, krsc, sched, stream, alpha, bias, act)
PyObject* conv(PyObject*, PyObject* const* a, Py_ssize_t n)
{
  return guarded([&] {
    need(api.conv && n == 12);
    const Conv c(a[0], a[1], a[2], a[3], a[4], a[5], truth(a[6]));
    const Schedule s(a[7]);
    void* st = stream_of(a[8]);
    const alcop_epilogue e = epilogue(a[9], a[10], a[11], c.K, c.x);
    const void *x = c.x.const_data_ptr(), *w = c.w.const_data_ptr();
    void* y = c.y.data_ptr();
    return unlocked([&] {
      return api.conv(x, w, y, c.N, c.H, c.W, c.C, c.K, c.R, c.S, c.stride[0], c.stride[1], c.pad[0], c.pad[1],
                      c.dil[0], c.dil[1], c.krsc, c.in, c.out, &e, s.p, st);
    });
  });
}

// conv_any(x, w, y, workspace, stride, pad, dilation, alpha, bias, act, sched, stream)
PyObject* conv_any(PyObject*, PyObject* const* a, Py_ssize_t n)
{
  return guarded([&] {
    need(api.conv_any && n == 12);
    const Conv c(a[0], a[1], a[2], a[4], a[5], a[6], 0);
    const at::Tensor& ws = tensor(a[3]);
    need(ws.is_contiguous() && ws.device() == c.x.device());
    const alcop_epilogue e = epilogue(a[7], a[8], a[9], c.K, c.x);
    const Schedule s(a[10]);
    void* st = stream_of(a[11]);
    const void *x = c.x.const_data_ptr(), *w = c.w.const_data_ptr();
    void *y = c.y.data_ptr(), *wp = ws.data_ptr();
    const size_t bytes = ws.nbytes();
    return unlocked([&] {
      return api.conv_any(x, w, y, c.N, c.H, c.W, c.C, c.K, c.R, c.S, c.stride[0], c.stride[1], c.pad[0], c.pad[1],
                          c.dil[0], c.dil[1], c.in, c.out, &e, s.p, wp, bytes, st);
    });
  });
}

// init(Sched, gemm_fused, bmm_fused, bmm_unaligned, conv_dilated, conv_unaligned): the class of schedules
// and addresses in the library
PyObject* init(PyObject*, PyObject* const* a, Py_ssize_t n)
{
  if (n != 6 || !PyType_Check(a[0])) {
    PyErr_SetString(PyExc_TypeError, "init takes a class and five addresses");
    return nullptr;
  }
  void* f[5];
  for (int i = 0; i < 5; i++) {
    f[i] = PyLong_AsVoidPtr(a[i + 1]);
    if (PyErr_Occurred()) return nullptr;
  }
  Py_INCREF(a[0]);
  Py_XDECREF(sched_type);
  sched_type = a[0];
  api.gemm = (decltype(api.gemm))f[0];
  api.bmm = (decltype(api.bmm))f[1];
  api.bmm_any = (decltype(api.bmm_any))f[2];
  api.conv = (decltype(api.conv))f[3];
  api.conv_any = (decltype(api.conv_any))f[4];
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"init", (PyCFunction)(void*)init, METH_FASTCALL, "set the library's entry points"},
    {"mm", (PyCFunction)(void*)mm, METH_FASTCALL, "matrix product, plain or batched"},
    {"mm_any", (PyCFunction)(void*)mm_any, METH_FASTCALL, "matrix product of unaligned operands"},
    {"conv", (PyCFunction)(void*)conv, METH_FASTCALL, "convolution"},
    {"conv_any", (PyCFunction)(void*)conv_any, METH_FASTCALL, "convolution of unaligned operands"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", "argument marshalling of the hot entry points", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&module); }
