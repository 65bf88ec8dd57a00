// CPython side of binding.py: turns Python arguments (torch tensors, Desc objects, views) into the C arguments of
// maskkv.h and makes the call.  Argument marshalling only.
//
// Why it is native: a layer step is four to five library calls whose kernels take 60 us together at short prompts; with the
// arguments built as ctypes objects the four calls cost 43 us of host time, now 16.5 (4 heads x 512 tokens, fp32, each call
// on a drained queue, median of 500: score 14.3 -> 7.5, select 7.9 -> 2.9, compact 8.9 -> 2.9, attend 12.0 -> 3.2 us; of that
// select and attend have a kernel less to launch than then).  Here a tensor argument is a few loads.
//
// The entry points of the library come in as addresses (bind()), so whichever build of libmaskkv.so binding.py has loaded
// is the one that runs.  The GIL is released around every call, as ctypes does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <vector>

#include "../../include/maskkv.h"

namespace {

struct Fns {
  decltype(&maskkv_score_workspace_bytes) score_ws;
  decltype(&maskkv_select_workspace_bytes) select_ws;
  decltype(&maskkv_attend_workspace_bytes) attend_ws;
  decltype(&maskkv_score) score;
  decltype(&maskkv_score_given_lse) score_given_lse;
  decltype(&maskkv_score_static) score_static;
  decltype(&maskkv_select) select;
  decltype(&maskkv_compact) compact;
  decltype(&maskkv_attend) attend;
  decltype(&maskkv_attend_full) attend_full;
  decltype(&maskkv_head_budgets) head_budgets;
  decltype(&maskkv_layer_importance) layer_importance;
  decltype(&maskkv_value_shift) value_shift;
} fn;

PyObject *kB, *kH, *kd, *kdtype, *kn_resp, *kn_query, *kP_max, *kq_per_kv, *kprompt_len, *kcuda_stream, *kdata_ptr;

struct Error {};  // a Python exception has been set

[[noreturn]] void fail(PyObject* type, const char* text) {
  PyErr_SetString(type, text);
  throw Error{};
}

int64_t as_i64(PyObject* o) {
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw Error{};
  return v;
}

int32_t as_i32(PyObject* o) { return (int32_t)as_i64(o); }

double as_f64(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw Error{};
  return v;
}

struct Ref {  // owned reference
  PyObject* o;
  explicit Ref(PyObject* p) : o(p) {
    if (!o) throw Error{};
  }
  ~Ref() { Py_XDECREF(o); }
  Ref(const Ref&) = delete;
  Ref& operator=(const Ref&) = delete;
};

int32_t attr_i32(PyObject* o, PyObject* name) {
  Ref v(PyObject_GetAttr(o, name));
  return as_i32(v.o);
}

// int(x) of every element of a sequence (numpy arrays and lists of floats included)
struct Ints {
  static constexpr Py_ssize_t kInline = 64;
  int32_t some[kInline];
  std::vector<int32_t> many;
  const int32_t* data = nullptr;
  Py_ssize_t n = 0;
  void read(PyObject* seq) {
    Ref fast(PySequence_Fast(seq, "expected a sequence of integers"));
    n = PySequence_Fast_GET_SIZE(fast.o);
    int32_t* out = some;
    if (n > kInline) {
      many.resize((size_t)n);
      out = many.data();
    }
    PyObject** items = PySequence_Fast_ITEMS(fast.o);
    for (Py_ssize_t i = 0; i < n; ++i) {
      if (PyLong_CheckExact(items[i])) {
        out[i] = as_i32(items[i]);
      } else {
        Ref v(PyNumber_Long(items[i]));
        out[i] = as_i32(v.o);
      }
    }
    data = out;
  }
};

struct DescArg {
  maskkv_desc d;
  Ints lens;
  explicit DescArg(PyObject* o) {
    d.B = attr_i32(o, kB);
    d.H = attr_i32(o, kH);
    d.d = attr_i32(o, kd);
    d.dtype = attr_i32(o, kdtype);
    d.n_resp = attr_i32(o, kn_resp);
    d.P_max = attr_i32(o, kP_max);
    d.q_per_kv = attr_i32(o, kq_per_kv);
    Ref nq(PyObject_GetAttr(o, kn_query));
    d.n_query = nq.o == Py_None ? d.n_resp : as_i32(nq.o);
    d.prompt_len = nullptr;
    Ref pl(PyObject_GetAttr(o, kprompt_len));
    if (pl.o != Py_None) {
      lens.read(pl.o);
      if (d.B <= MASKKV_MAX_BATCH && lens.n < d.B) fail(PyExc_ValueError, "prompt_len has fewer than B entries");
      d.prompt_len = lens.data;
    }
  }
};

// A [B, H, T, d] tensor, or a view made by tensor_view() (a ctypes structure with the layout of maskkv_tensor).
struct ViewArg {
  maskkv_tensor v;
  explicit ViewArg(PyObject* o) {
    if (THPVariable_Check(o)) {
      const at::Tensor& t = THPVariable_Unpack(o);
      if (!t.is_cuda() || t.dim() != 4 || t.stride(3) != 1)
        fail(PyExc_AssertionError, "need a [B,H,T,d] device tensor with contiguous d");
      v.ptr = t.data_ptr();
      v.stride_b = t.stride(0);
      v.stride_h = t.stride(1);
      v.stride_t = t.stride(2);
      v.seq_start = nullptr;
      return;
    }
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) throw Error{};
    const bool fits = b.len == (Py_ssize_t)sizeof(v);
    if (fits) memcpy(&v, b.buf, sizeof(v));
    PyBuffer_Release(&b);
    if (!fits) fail(PyExc_TypeError, "expected a tensor or a view made by tensor_view()");
  }
};

void* as_ptr(PyObject* o) {
  if (o == Py_None) return nullptr;
  if (THPVariable_Check(o)) return THPVariable_Unpack(o).data_ptr();
  Ref v(PyObject_CallMethodNoArgs(o, kdata_ptr));
  void* p = PyLong_AsVoidPtr(v.o);
  if (!p && PyErr_Occurred()) throw Error{};
  return p;
}

template <typename T>
T* ptr(PyObject* o) {
  return static_cast<T*>(as_ptr(o));
}

size_t nbytes(PyObject* o) {
  if (o == Py_None) return 0;
  if (!THPVariable_Check(o)) fail(PyExc_TypeError, "a workspace is a tensor or None");
  const at::Tensor& t = THPVariable_Unpack(o);
  return (size_t)t.numel() * (size_t)t.element_size();
}

void* as_stream(PyObject* o) {
  if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
  PyObject* s = PyObject_GetAttr(o, kcuda_stream);
  if (!s) {
    PyErr_Clear();
    s = PyNumber_Long(o);
  }
  Ref v(s);
  void* p = PyLong_AsVoidPtr(v.o);
  if (!p && PyErr_Occurred()) throw Error{};
  return p;
}

template <typename F>
int without_gil(F f) {
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = f();
  Py_END_ALLOW_THREADS
  return status;
}

// One Python function of N arguments that returns the status of the library call (or what `body` returns).
template <int N, typename F>
PyObject* call(Py_ssize_t n, F body) {
  if (n != N) {
    PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", N, n);
    return nullptr;
  }
  try {
    return PyLong_FromLongLong(body());
  } catch (const Error&) {
    return nullptr;
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

typedef PyObject* const* Args;

// Sizes: the status in the low byte's place is told apart by sign: -status on failure, bytes otherwise.
PyObject* score_ws(PyObject*, Args a, Py_ssize_t n) {
  return call<1>(n, [&]() -> long long {
    DescArg d(a[0]);
    size_t bytes = 0;
    const int s = fn.score_ws(&d.d, &bytes);
    return s ? -s : (long long)bytes;
  });
}
PyObject* select_ws(PyObject*, Args a, Py_ssize_t n) {
  return call<1>(n, [&]() -> long long {
    DescArg d(a[0]);
    size_t bytes = 0;
    const int s = fn.select_ws(&d.d, &bytes);
    return s ? -s : (long long)bytes;
  });
}
PyObject* attend_ws(PyObject*, Args a, Py_ssize_t n) {
  return call<2>(n, [&]() -> long long {
    DescArg d(a[0]);
    const int full = PyObject_IsTrue(a[1]);
    if (full < 0) throw Error{};
    size_t bytes = 0;
    const int s = fn.attend_ws(&d.d, full, &bytes);
    return s ? -s : (long long)bytes;
  });
}

PyObject* score(PyObject*, Args a, Py_ssize_t n) {  // desc, Q, K, scale, scores, stride, mass, workspace, stream
  return call<9>(n, [&] {
    DescArg d(a[0]);
    ViewArg q(a[1]), k(a[2]);
    const float scale = (float)as_f64(a[3]);
    float *scores = ptr<float>(a[4]), *mass = ptr<float>(a[6]);
    const int64_t stride = as_i64(a[5]);
    void *ws = as_ptr(a[7]), *st = as_stream(a[8]);
    const size_t wn = nbytes(a[7]);
    return without_gil([&] { return fn.score(&d.d, &q.v, &k.v, scale, scores, stride, mass, ws, wn, st); });
  });
}
PyObject* score_given_lse(PyObject*, Args a, Py_ssize_t n) {  // desc, Q, K, scale, lse, scores, stride, mass, workspace, stream
  return call<10>(n, [&] {
    DescArg d(a[0]);
    ViewArg q(a[1]), k(a[2]);
    const float scale = (float)as_f64(a[3]);
    float *lse = ptr<float>(a[4]), *scores = ptr<float>(a[5]), *mass = ptr<float>(a[7]);
    const int64_t stride = as_i64(a[6]);
    void *ws = as_ptr(a[8]), *st = as_stream(a[9]);
    const size_t wn = nbytes(a[8]);
    return without_gil([&] { return fn.score_given_lse(&d.d, &q.v, &k.v, scale, lse, scores, stride, mass, ws, wn, st); });
  });
}
PyObject* score_static(PyObject*, Args a, Py_ssize_t n) {  // desc, Q, K, scale, scores, stride, mass, stream
  return call<8>(n, [&] {
    DescArg d(a[0]);
    ViewArg q(a[1]), k(a[2]);
    const float scale = (float)as_f64(a[3]);
    float *scores = ptr<float>(a[4]), *mass = ptr<float>(a[6]);
    const int64_t stride = as_i64(a[5]);
    void* st = as_stream(a[7]);
    return without_gil([&] { return fn.score_static(&d.d, &q.v, &k.v, scale, scores, stride, mass, st); });
  });
}
// desc, scores, stride, window, mode, budgets, budgets_host, idx, cu, capacity, workspace, stream
PyObject* select(PyObject*, Args a, Py_ssize_t n) {
  return call<12>(n, [&] {
    DescArg d(a[0]);
    const float* scores = ptr<float>(a[1]);
    const int64_t stride = as_i64(a[2]);
    const int window = as_i32(a[3]), mode = as_i32(a[4]);
    int32_t *budgets = ptr<int32_t>(a[5]), *idx = ptr<int32_t>(a[7]), *cu = ptr<int32_t>(a[8]);
    Ints host;
    if (a[6] != Py_None) {
      host.read(a[6]);
      if (host.n < (int64_t)d.d.B * d.d.H) fail(PyExc_ValueError, "budgets_host has fewer than B*H entries");
    }
    const int64_t cap = as_i64(a[9]);
    void *ws = as_ptr(a[10]), *st = as_stream(a[11]);
    const size_t wn = nbytes(a[10]);
    return without_gil(
        [&] { return fn.select(&d.d, scores, stride, window, mode, budgets, host.data, idx, cu, cap, ws, wn, st); });
  });
}
PyObject* compact(PyObject*, Args a, Py_ssize_t n) {  // desc, K, V, idx, cu, capacity, Kc, Vc, stream
  return call<9>(n, [&] {
    DescArg d(a[0]);
    ViewArg k(a[1]), v(a[2]);
    int32_t *idx = ptr<int32_t>(a[3]), *cu = ptr<int32_t>(a[4]);
    const int64_t cap = as_i64(a[5]);
    void *kc = as_ptr(a[6]), *vc = as_ptr(a[7]), *st = as_stream(a[8]);
    return without_gil([&] { return fn.compact(&d.d, &k.v, &v.v, idx, cu, cap, kc, vc, st); });
  });
}
PyObject* attend(PyObject*, Args a, Py_ssize_t n) {  // desc, Q, Kc, Vc, cu, capacity, Kr, Vr, scale, O, lse, workspace, stream
  return call<13>(n, [&] {
    DescArg d(a[0]);
    ViewArg q(a[1]), k2(a[6]), v2(a[7]), o(a[9]);
    void *kc = as_ptr(a[2]), *vc = as_ptr(a[3]);
    int32_t* cu = ptr<int32_t>(a[4]);
    const int64_t cap = as_i64(a[5]);
    const float scale = (float)as_f64(a[8]);
    float* lse = ptr<float>(a[10]);
    void *ws = as_ptr(a[11]), *st = as_stream(a[12]);
    const size_t wn = nbytes(a[11]);
    return without_gil(
        [&] { return fn.attend(&d.d, &q.v, kc, vc, cu, cap, &k2.v, &v2.v, scale, &o.v, lse, ws, wn, st); });
  });
}
PyObject* attend_full(PyObject*, Args a, Py_ssize_t n) {  // desc, Q, K, V, scale, O, lse, workspace, stream
  return call<9>(n, [&] {
    DescArg d(a[0]);
    ViewArg q(a[1]), k(a[2]), v(a[3]), o(a[5]);
    const float scale = (float)as_f64(a[4]);
    float* lse = ptr<float>(a[6]);
    void *ws = as_ptr(a[7]), *st = as_stream(a[8]);
    const size_t wn = nbytes(a[7]);
    return without_gil([&] { return fn.attend_full(&d.d, &q.v, &k.v, &v.v, scale, &o.v, lse, ws, wn, st); });
  });
}
PyObject* head_budgets(PyObject*, Args a, Py_ssize_t n) {  // desc, mass, k_l, alpha, budgets, stream
  return call<6>(n, [&] {
    DescArg d(a[0]);
    const float* mass = ptr<float>(a[1]);
    const int32_t k_l = as_i32(a[2]);
    const float alpha = (float)as_f64(a[3]);
    int32_t* budgets = ptr<int32_t>(a[4]);
    void* st = as_stream(a[5]);
    return without_gil([&] { return fn.head_budgets(&d.d, mass, k_l, alpha, budgets, st); });
  });
}

// Two [rows, width] device tensors of one dtype and one row stride.
struct RowsArg {
  const void *a, *b;
  int64_t n, stride;
  int32_t width, dtype;
  RowsArg(PyObject* x, PyObject* y) {
    if (!THPVariable_Check(x) || !THPVariable_Check(y)) fail(PyExc_TypeError, "expected two tensors");
    const at::Tensor &s = THPVariable_Unpack(x), &t = THPVariable_Unpack(y);
    if (!s.is_cuda() || s.dim() != 2 || s.stride(1) != 1 || t.sizes() != s.sizes())
      fail(PyExc_AssertionError, "need two [rows, width] device tensors of one shape with contiguous rows");
    if (t.strides() != s.strides() || t.scalar_type() != s.scalar_type())
      fail(PyExc_AssertionError, "the two tensors differ in strides or dtype");
    if (s.scalar_type() == at::kBFloat16)
      dtype = MASKKV_BF16;
    else if (s.scalar_type() == at::kFloat)
      dtype = MASKKV_F32;
    else
      fail(PyExc_TypeError, "unsupported tensor dtype");
    a = s.data_ptr();
    b = t.data_ptr();
    n = s.size(0);
    width = (int32_t)s.size(1);
    stride = s.stride(0);
  }
};

PyObject* layer_importance(PyObject*, Args a, Py_ssize_t n) {  // h_in, h_out, importance, workspace, stream
  return call<5>(n, [&] {
    RowsArg r(a[0], a[1]);
    float* imp = ptr<float>(a[2]);
    void *ws = as_ptr(a[3]), *st = as_stream(a[4]);
    const size_t wn = nbytes(a[3]);
    return without_gil([&] { return fn.layer_importance(r.a, r.b, r.n, r.width, r.dtype, r.stride, imp, ws, wn, st); });
  });
}
PyObject* value_shift(PyObject*, Args a, Py_ssize_t n) {  // V_now, V_prev, delta, cos, refresh, count, stream
  return call<7>(n, [&] {
    RowsArg r(a[0], a[1]);
    const float delta = (float)as_f64(a[2]);
    auto holds = [](PyObject* o, at::ScalarType type, int64_t least) {
      return THPVariable_Check(o) && THPVariable_Unpack(o).scalar_type() == type && THPVariable_Unpack(o).numel() >= least;
    };
    if (!holds(a[3], at::kFloat, r.n)) fail(PyExc_AssertionError, "cos: float32, at least one entry per row");
    if (!holds(a[4], at::kInt, r.n) || !holds(a[5], at::kInt, 0))
      fail(PyExc_AssertionError, "refresh: int32, at least one entry per row; count: int32");
    float* cos = ptr<float>(a[3]);
    int32_t *refresh = ptr<int32_t>(a[4]), *count = ptr<int32_t>(a[5]);
    void* st = as_stream(a[6]);
    return without_gil(
        [&] { return fn.value_shift(r.a, r.b, r.n, r.width, r.dtype, r.stride, delta, cos, refresh, count, st); });
  });
}

// bind({name: address}): the loaded library's entry points.
PyObject* bind(PyObject*, PyObject* table) {
  const struct {
    const char* name;
    void* to;
  } all[] = {
      {"maskkv_score_workspace_bytes", &fn.score_ws}, {"maskkv_select_workspace_bytes", &fn.select_ws},
      {"maskkv_attend_workspace_bytes", &fn.attend_ws}, {"maskkv_score", &fn.score},
      {"maskkv_score_given_lse", &fn.score_given_lse}, {"maskkv_score_static", &fn.score_static},
      {"maskkv_select", &fn.select}, {"maskkv_compact", &fn.compact}, {"maskkv_attend", &fn.attend},
      {"maskkv_attend_full", &fn.attend_full}, {"maskkv_head_budgets", &fn.head_budgets},
      {"maskkv_layer_importance", &fn.layer_importance}, {"maskkv_value_shift", &fn.value_shift}};
  for (const auto& e : all) {
    PyObject* v = PyDict_GetItemString(table, e.name);
    void* p = v ? PyLong_AsVoidPtr(v) : nullptr;
    if (!p) return PyErr_Format(PyExc_KeyError, "%s", e.name);
    memcpy(e.to, &p, sizeof(p));
  }
  Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(score_ws), FAST(select_ws), FAST(attend_ws), FAST(score), FAST(score_given_lse),
                         FAST(score_static), FAST(select), FAST(compact), FAST(attend), FAST(attend_full),
                         FAST(head_budgets), FAST(layer_importance), FAST(value_shift),
                         {"bind", bind, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) {
  const struct {
    PyObject** to;
    const char* text;
  } names[] = {{&kB, "B"}, {&kH, "H"}, {&kd, "d"}, {&kdtype, "dtype"}, {&kn_resp, "n_resp"}, {&kn_query, "n_query"},
               {&kP_max, "P_max"}, {&kq_per_kv, "q_per_kv"}, {&kprompt_len, "prompt_len"},
               {&kcuda_stream, "cuda_stream"}, {&kdata_ptr, "data_ptr"}};
  for (const auto& n : names) {
    *n.to = PyUnicode_InternFromString(n.text);
    if (!*n.to) return nullptr;
  }
  return PyModule_Create(&module);
}
