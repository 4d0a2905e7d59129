// Argument marshalling of the Python binding's hot calls, in native code.
//
// A call on a small table takes the GPU a few microseconds (tens of thousands of fact rows: 2 to 10 us), so what a
// Python program waits for there is the host path: building the descriptor structs through ctypes, asking for the
// workspace size, allocating outputs and reading the current stream cost 11 to 18 us per call, several times the
// kernel.  Here a call unpacks the tensors, checks them, allocates outputs through torch's caching allocator and
// enters the C interface directly: 1 to 2 us around the launches themselves.  The functions take the arguments of
// their namesakes in binding.py positionally; binding.py holds signatures, defaults and documentation.
//
// No arithmetic happens here, and no HIP: streams and allocations go through torch.
#include <Python.h>
#include <structmember.h>

#include <ATen/EmptyTensor.h>
#include <ATen/core/Tensor.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <exception>
#include <optional>
#include <vector>

#include "lq.h"

namespace {

PyObject* g_error_class = nullptr;   // binding.LQError

// A Python exception is set: unwind to the entry point.
struct PyErrorSet {};

[[noreturn]] void raise(PyObject* type, const char* text) {
  PyErr_SetString(type, text);
  throw PyErrorSet{};
}

void check(int rc) {
  if (rc == LQ_OK) return;
  PyObject* e = PyObject_CallFunction(g_error_class, "is", rc, lq_last_error());
  if (e) {
    PyErr_SetObject(g_error_class, e);
    Py_DECREF(e);
  }
  throw PyErrorSet{};
}


const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_TypeError, "expected a tensor, got %s", Py_TYPE(o)->tp_name);
    throw PyErrorSet{};
  }
  return THPVariable_Unpack(o);
}

// "torch.float32" of a tensor, for messages.
[[noreturn]] void raise_dtype(PyObject* o, const char* format, const char* a, const char* b) {
  PyObject* dt = PyObject_GetAttrString(o, "dtype");
  if (dt) {
    if (a) PyErr_Format(PyExc_TypeError, format, a, b, dt);
    else PyErr_Format(PyExc_TypeError, format, dt);
    Py_DECREF(dt);
  }
  throw PyErrorSet{};
}

int32_t dtype_code(PyObject* o, const at::Tensor& t) {
  if (t.scalar_type() == at::kFloat) return LQ_F32;
  if (t.scalar_type() == at::kBFloat16) return LQ_BF16;
  raise_dtype(o, "unsupported dtype %S (float32 or bfloat16)", nullptr, nullptr);
}

// A column or other typed buffer on the GPU.
const at::Tensor& expect(PyObject* o, at::ScalarType st, const char* dtype_name, const char* what) {
  const at::Tensor& t = tensor(o);
  if (t.scalar_type() != st) raise_dtype(o, "%s must be %s, got %S", what, dtype_name);
  if (!t.is_cuda()) {
    PyErr_Format(PyExc_ValueError, "%s must live on the GPU", what);
    throw PyErrorSet{};
  }
  if (t.dim() == 1 && t.numel() > 1 && t.stride(0) != 1) {
    PyErr_Format(PyExc_ValueError, "%s must be contiguous", what);
    throw PyErrorSet{};
  }
  return t;
}
const at::Tensor& expect_i32(PyObject* o, const char* what) { return expect(o, at::kInt, "torch.int32", what); }
const at::Tensor& expect_u8(PyObject* o, const char* what) { return expect(o, at::kByte, "torch.uint8", what); }
const at::Tensor& expect_i64(PyObject* o, const char* what) { return expect(o, at::kLong, "torch.int64", what); }

// Rows of a column (its first size).
int64_t length(const at::Tensor& t) {
  if (t.dim() < 1) raise(PyExc_ValueError, "columns are 1-D tensors");
  return t.size(0);
}

lq_mat mat(PyObject* o) {
  const at::Tensor& t = tensor(o);
  if (t.dim() != 2) raise(PyExc_ValueError, "matrices are 2-D tensors");
  const int64_t r = t.size(0), c = t.size(1);
  const int32_t dt = dtype_code(o, t);
  if (r == 0 || c == 0) return lq_mat{nullptr, r, static_cast<int32_t>(c), std::max<int64_t>(c, 1), dt};
  const int64_t s0 = t.stride(0), s1 = t.stride(1);
  if (c > 1 && s1 != 1) raise(PyExc_ValueError, "matrix columns must be contiguous (row-major)");
  const int64_t ld = (r > 1 || s0 >= c) ? s0 : std::max<int64_t>(c, 1);
  if (r > 1 && ld < c) raise(PyExc_ValueError, "row stride smaller than the row");
  return lq_mat{t.data_ptr(), r, static_cast<int32_t>(c), ld, dt};
}

lq_mat no_mat(int64_t rows, int32_t cols, int32_t dtype) { return lq_mat{nullptr, rows, cols, std::max(cols, 1), dtype}; }

int64_t integer(PyObject* o) {
  if (PyLong_Check(o)) {
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw PyErrorSet{};
    return v;
  }
  PyObject* n = PyNumber_Long(o);
  if (!n) throw PyErrorSet{};
  const long long v = PyLong_AsLongLong(n);
  Py_DECREF(n);
  if (v == -1 && PyErr_Occurred()) throw PyErrorSet{};
  return v;
}

// Number of values of a grouping attribute, and of groups over several.
int32_t cardinality(PyObject* o) {
  const int64_t v = integer(o);
  if (v != static_cast<int32_t>(v)) raise(PyExc_ValueError, "a group cardinality does not fit 32 bits");
  return static_cast<int32_t>(v);
}
int64_t product(int64_t groups, int32_t card) {
  int64_t r;
  if (__builtin_mul_overflow(groups, static_cast<int64_t>(card), &r)) raise(PyExc_ValueError, "the number of groups does not fit 64 bits");
  return r;
}

bool truth(PyObject* o) {
  const int v = PyObject_IsTrue(o);
  if (v < 0) throw PyErrorSet{};
  return v != 0;
}

// A list or tuple (or any other collection) of Python objects.  An iterator is refused where `any_iterable` is not set:
// most arguments are gone through more than once.
class Seq {
 public:
  explicit Seq(PyObject* o, bool any_iterable = false) {
    if (!any_iterable && PyObject_Size(o) < 0) throw PyErrorSet{};
    s_ = PySequence_Fast(o, "expected a sequence");
    if (!s_) throw PyErrorSet{};
  }
  ~Seq() { Py_DECREF(s_); }
  Seq(const Seq&) = delete;
  Seq& operator=(const Seq&) = delete;
  int size() const { return static_cast<int>(PySequence_Fast_GET_SIZE(s_)); }
  PyObject* operator[](int i) const { return PySequence_Fast_GET_ITEM(s_, i); }

 private:
  PyObject* s_;
};

// Up to N items without an allocation; the library itself refuses more dimensions, layers or measures than it takes.
template <typename T> class Array {
 public:
  explicit Array(int n) : n_(std::max(n, 1)), more_(n_ > N ? new T[n_]() : nullptr) {}
  ~Array() { delete[] more_; }
  Array(const Array&) = delete;
  Array& operator=(const Array&) = delete;
  int size() const { return n_; }
  T* data() { return more_ ? more_ : own_; }
  T& operator[](int i) { return data()[i]; }
  operator T*() { return data(); }

 private:
  static constexpr int N = 8;
  int n_;
  T* more_;
  T own_[N] = {};
};

void mats(const Seq& s, Array<lq_mat>& out) {
  if (s.size() > out.size()) raise(PyExc_ValueError, "more matrices than there is room for");
  for (int j = 0; j < s.size(); ++j) out[j] = mat(s[j]);
}

template <typename T> T* data_of(PyObject* o) {
  return o == Py_None ? nullptr : static_cast<T*>(tensor(o).data_ptr());
}

// The stream a call runs on: the given torch stream, or torch's current one on the current device.
struct Stream {
  PyObject* given;
  explicit Stream(PyObject* o) : given(o) {}
  void* handle() const {
    if (given == Py_None) return c10::hip::getCurrentHIPStream().stream();
    PyObject* h = PyObject_GetAttrString(given, "cuda_stream");
    if (!h) throw PyErrorSet{};
    void* p = PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    if (PyErr_Occurred()) throw PyErrorSet{};
    return p;
  }
};

// The library call itself runs without the interpreter lock (a launch may wait for room in the queue, a checked call
// for the stream).
template <typename F> void call(const Stream& s, F&& f) {
  void* stream = s.handle();
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f(stream);
  Py_END_ALLOW_THREADS
  check(rc);
}

// A new tensor for an output or workspace of a call that runs on `s`.  torch hands a freed block to the next
// allocation on the stream it was allocated on; when the kernels run on another stream the block is marked as in use
// there, so that it is not recycled while they still read or write it.
at::Tensor empty(at::IntArrayRef shape, at::ScalarType st, const at::Device& dev, const Stream& s) {
  at::Tensor t(dev.is_cuda() ? at::detail::empty_cuda(shape, st, dev, std::nullopt)
                             : at::detail::empty_cpu(shape, st, false, std::nullopt));
  if (s.given != Py_None && t.is_cuda() && t.numel() > 0) {
    PyObject* o = THPVariable_Wrap(t);
    PyObject* r = o ? PyObject_CallMethod(o, "record_stream", "O", s.given) : nullptr;
    Py_XDECREF(o);
    Py_XDECREF(r);
    if (!r) throw PyErrorSet{};
  }
  return t;
}

PyObject* wrap(const at::Tensor& t) {
  PyObject* o = THPVariable_Wrap(t);
  if (!o) throw PyErrorSet{};
  return o;
}
PyObject* wrap_or_none(const at::Tensor& t) {
  if (!t.defined()) Py_RETURN_NONE;
  return wrap(t);
}
PyObject* pair(PyObject* a, PyObject* b) {
  PyObject* t = PyTuple_New(2);
  if (!t) throw PyErrorSet{};
  PyTuple_SET_ITEM(t, 0, a);
  PyTuple_SET_ITEM(t, 1, b);
  return t;
}
PyObject* list_of(const std::vector<at::Tensor>& ts) {
  PyObject* l = PyList_New(static_cast<Py_ssize_t>(ts.size()));
  if (!l) throw PyErrorSet{};
  for (size_t j = 0; j < ts.size(); ++j) PyList_SET_ITEM(l, j, wrap(ts[j]));
  return l;
}

at::ScalarType scalar_type(PyObject* dtype, at::ScalarType otherwise) {
  if (dtype == Py_None) return otherwise;
  if (!THPDtype_Check(dtype)) raise(PyExc_TypeError, "expected a torch.dtype");
  return reinterpret_cast<THPDtype*>(dtype)->scalar_type;
}

size_t bytes_of(const at::Tensor& t) { return static_cast<size_t>(t.numel()) * t.element_size(); }

// Fact columns and foreign keys of a star schema.
struct Star {
  Seq fks;
  Array<const int32_t*> keys;
  lq_star c{};
  Star(PyObject* X, PyObject* fks_obj) : fks(fks_obj), keys(fks.size()) {
    for (int k = 0; k < fks.size(); ++k)
      keys[k] = static_cast<const int32_t*>(expect_i32(fks[k], "foreign-key column").data_ptr());
    if (X != Py_None) {
      c.fact = mat(X);
      c.n_fact = tensor(X).size(0);
    } else {
      if (fks.size() == 0) raise(PyExc_ValueError, "need fact columns or at least one foreign-key column");
      c.n_fact = length(tensor(fks[0]));
      c.fact = no_mat(c.n_fact, 0, LQ_F32);
    }
    c.n_dims = fks.size();
    c.fks = keys.data();
  }
};

// Dimension tables only (pre-fusion): no fact rows, no keys.
struct DimStar {
  Seq dims_seq;
  Array<lq_mat> dims;
  Array<const int32_t*> keys;
  lq_star c{};
  DimStar(PyObject* dims_obj, int32_t c_f, int32_t dtype) : dims_seq(dims_obj), dims(dims_seq.size()), keys(dims_seq.size()) {
    mats(dims_seq, dims);
    c.fact = no_mat(0, c_f, dtype);
    c.n_dims = dims_seq.size();
    c.dims = dims;
    c.fks = keys.data();
  }
};

struct Model {
  Seq weights;
  std::optional<Seq> biases;
  Array<lq_mat> W;
  Array<const void*> bias;
  lq_model c{};
  Model(PyObject* w, PyObject* b) : weights(w), W(weights.size()), bias(weights.size()) {
    mats(weights, W);
    if (b != Py_None) {
      const Seq& bs = biases.emplace(b);
      for (int j = 0; j < std::min(bs.size(), weights.size()); ++j) bias[j] = data_of<void>(bs[j]);
    }
    c.n_layers = weights.size();
    c.W = W;
    c.bias = bias.data();
  }
  const at::Tensor& first() const {
    if (weights.size() == 0) raise(PyExc_ValueError, "the model has no layers");
    return tensor(weights[0]);
  }
};

// ------------------------------------------------------------------ prediction ----------

// (dims, W0, c_f, P, p_dtype, stream)
PyObject* project_dims(PyObject* const* a) {
  const at::Tensor& W0 = tensor(a[1]);
  const Stream s(a[5]);
  DimStar star(a[0], static_cast<int32_t>(integer(a[2])), dtype_code(a[1], W0));
  const lq_mat w = mat(a[1]);
  const void* no_bias = nullptr;
  const lq_model model{1, &w, &no_bias};
  const int K = star.dims_seq.size();
  // (a caller's list may be longer than the dimensions: the library reads the first K entries)
  Array<lq_mat> P(a[3] != Py_None ? std::max(K, Seq(a[3]).size()) : K);
  PyObject* out;
  if (a[3] != Py_None) {
    mats(Seq(a[3]), P);
    out = a[3];
    Py_INCREF(out);
  } else {
    // rows start 16 bytes apart at the least (the stride is padded to 4 floats / 8 bf16 values): the fast kernels of
    // the join stage then take any hidden width, the padding is never read as data
    const at::ScalarType pd = scalar_type(a[4], W0.scalar_type());
    const int64_t per16 = pd == at::kFloat ? 4 : 8, l1 = W0.size(1), ld = (l1 + per16 - 1) / per16 * per16;
    std::vector<at::Tensor> made;
    made.reserve(K);
    for (int k = 0; k < K; ++k) {
      const at::Tensor& d = tensor(star.dims_seq[k]);
      at::Tensor t = empty({d.size(0), ld}, pd, d.device(), s);
      made.push_back(ld == l1 ? t : t.narrow(1, 0, l1));
    }
    out = list_of(made);
    try {
      mats(Seq(out), P);
    } catch (...) {
      Py_DECREF(out);
      throw;
    }
  }
  try {
    call(s, [&](void* stream) { return lq_project_dims(&star.c, &model, P, stream); });
  } catch (...) {
    Py_DECREF(out);
    throw;
  }
  return out;
}

// (X, fks, P, weights, biases, Y, y_dtype, flags, ws, stream)
PyObject* fused_join_predict(PyObject* const* a) {
  const Stream s(a[9]);
  Star star(a[0], a[1]);
  Model model(a[3], a[4]);
  const at::Tensor& W0 = model.first();
  const at::Device dev = W0.device();
  const int64_t n = star.c.n_fact;
  const uint32_t flags = static_cast<uint32_t>(integer(a[7]));
  at::Tensor Y = a[5] != Py_None ? tensor(a[5])
                                 : empty({n, model.W[model.c.n_layers - 1].cols}, scalar_type(a[6], W0.scalar_type()), dev, s);
  at::Tensor ws;
  if (a[8] != Py_None) {
    ws = tensor(a[8]);
  } else {
    int32_t widest = 0;
    for (int j = 0; j < model.c.n_layers; ++j) widest = std::max(widest, model.W[j].cols);
    if (n > 0 && model.c.n_layers >= 2 && (widest > 128 || star.c.fact.cols > 16)) {
      // a model that the fused kernels may not take (a layer wider than 128, more than 16 fact columns): room for the
      // layered form (activations of a chunk of rows, at most a quarter of a gigabyte); the library uses it only if
      // it needs to
      const int64_t per_row = static_cast<int64_t>(lq_workspace_bytes(LQ_CALL_FUSED, &star.c, &model.c, 256) - 256) / 256;
      const int64_t rows = std::max<int64_t>(4096, std::min<int64_t>(n, (256ll << 20) / std::max<int64_t>(per_row, 1)));
      ws = empty({static_cast<int64_t>(lq_workspace_bytes(LQ_CALL_FUSED, &star.c, &model.c, rows))}, at::kByte, dev, s);
    } else if (flags & LQ_CHECK_FKS) {
      ws = empty({256}, at::kByte, dev, s);
    }
  }
  Seq Ps(a[2]);
  Array<lq_mat> P(Ps.size());
  mats(Ps, P);
  PyObject* out = a[5] != Py_None ? (Py_INCREF(a[5]), a[5]) : wrap(Y);
  try {
    lq_mat Ym = mat(out);
    void* wp = ws.defined() ? ws.data_ptr() : nullptr;
    const size_t wb = ws.defined() ? bytes_of(ws) : 0;
    call(s, [&](void* stream) { return lq_fused_join_predict(&star.c, &model.c, P, &Ym, wp, wb, flags, stream); });
  } catch (...) {
    Py_DECREF(out);
    throw;
  }
  return out;
}

// (X, dims, fks, weights, biases, Y, y_dtype, ws, chunk_rows, flags, stream)
PyObject* materialized_join_predict(PyObject* const* a) {
  const Stream s(a[10]);
  Star star(a[0], a[2]);
  Model model(a[3], a[4]);
  const at::Tensor& W0 = model.first();
  const at::Device dev = W0.device();
  const int64_t n = star.c.n_fact;
  at::Tensor Y = a[5] != Py_None ? tensor(a[5])
                                 : empty({n, model.W[model.c.n_layers - 1].cols}, scalar_type(a[6], W0.scalar_type()), dev, s);
  at::Tensor ws;
  if (a[7] != Py_None) {
    ws = tensor(a[7]);
  } else {
    int64_t rows = a[8] != Py_None ? integer(a[8]) : 0;
    if (rows == 0) rows = std::min<int64_t>(std::max<int64_t>(n, 256), 1 << 22);
    ws = empty({static_cast<int64_t>(lq_workspace_bytes(LQ_CALL_MATERIALIZED, &star.c, &model.c, rows))}, at::kByte, dev, s);
  }
  Seq dims(a[1]);
  Array<lq_mat> D(dims.size());
  mats(dims, D);
  star.c.dims = D;
  const uint32_t flags = static_cast<uint32_t>(integer(a[9]));
  PyObject* out = a[5] != Py_None ? (Py_INCREF(a[5]), a[5]) : wrap(Y);
  try {
    lq_mat Ym = mat(out);
    void* wp = ws.data_ptr();
    const size_t wb = bytes_of(ws);
    call(s, [&](void* stream) { return lq_materialized_join_predict(&star.c, &model.c, &Ym, wp, wb, flags, stream); });
  } catch (...) {
    Py_DECREF(out);
    throw;
  }
  return out;
}

// ------------------------------------------------------------------ group-by ------------

// Masks or group codes of the dimensions: None, or one tensor or None per dimension.  `keep` holds them until the call is
// made: an iterator's tensors belong to nobody else, and the outputs and workspace allocated after this would be
// given their memory.
template <typename T> void dim_arrays(PyObject* o, int K, const Array<int64_t>* rows, at::ScalarType st, const char* dtype_name,
                                      const char* what, const char* length_error, std::optional<Seq>& keep, const T** out) {
  if (o == Py_None) return;
  const Seq& s = keep.emplace(o, true);
  if (s.size() < K) raise(PyExc_IndexError, "list index out of range");
  for (int k = 0; k < K; ++k) {
    if (s[k] == Py_None) continue;
    if (!rows) {
      out[k] = static_cast<const T*>(tensor(s[k]).data_ptr());
      continue;
    }
    const at::Tensor& t = expect(s[k], st, dtype_name, what);
    if (length(t) != const_cast<Array<int64_t>&>(*rows)[k]) raise(PyExc_ValueError, length_error);
    out[k] = static_cast<const T*>(t.data_ptr());
  }
}

struct GroupShape {
  Array<int64_t> rows;
  Array<int32_t> card, effective;    // effective: 1 where the dimension does not group
  Array<const uint8_t*> mask;
  Array<const int32_t*> code;
  std::optional<Seq> masks, codes;   // what `mask` and `code` point into
  int64_t G = 1;
  GroupShape(int K, PyObject* dim_rows, PyObject* dim_mask, PyObject* dim_code, PyObject* group_card, bool checked)
      : rows(K), card(K), effective(K), mask(K), code(K) {
    Seq r(dim_rows), c(group_card);
    if (r.size() < K || c.size() < K) raise(PyExc_IndexError, "list index out of range");
    // more rows or cardinalities than key columns: a column was forgotten, and the result would not be filtered by it
    if (r.size() > std::max(K, 1) || c.size() > std::max(K, 1))
      raise(PyExc_IndexError, "dim_rows and group_card have an entry for every foreign-key column");
    for (int k = 0; k < K; ++k) {
      rows[k] = integer(r[k]);
      card[k] = cardinality(c[k]);
    }
    dim_arrays(dim_mask, K, checked ? &rows : nullptr, at::kByte, "torch.uint8", "dimension mask", "mask length differs from dim_rows",
               masks, mask.data());
    dim_arrays(dim_code, K, checked ? &rows : nullptr, at::kInt, "torch.int32", "dimension group code",
               "code length differs from dim_rows", codes, code.data());
    for (int k = 0; k < K; ++k) {
      effective[k] = code[k] ? card[k] : 1;
      G = product(G, effective[k]);
    }
  }
};

// (fks, dim_rows, dim_mask, dim_code, group_card, fact_mask, measures, sums, counts, want_counts, ws, flags, stream)
PyObject* masked_groupby_sum(PyObject* const* a) {
  const Stream s(a[12]);
  Seq fks(a[0]), measures(a[6]);
  const int K = fks.size(), M = measures.size();
  if (M == 0) raise(PyExc_IndexError, "list index out of range");
  const at::Tensor& m0 = tensor(measures[0]);
  const int64_t n = length(m0);
  const at::Device dev = m0.device();
  Array<const int32_t*> keys(K), meas(M);
  for (int k = 0; k < K; ++k) {
    const at::Tensor& f = expect_i32(fks[k], "foreign-key column");
    if (length(f) != n) raise(PyExc_ValueError, "foreign-key column length differs from the measures");
    keys[k] = static_cast<const int32_t*>(f.data_ptr());
  }
  for (int m = 0; m < M; ++m) meas[m] = static_cast<const int32_t*>(expect_i32(measures[m], "measure column").data_ptr());
  GroupShape g(K, a[1], a[2], a[3], a[4], true);
  const uint8_t* fact_mask =
      a[5] == Py_None ? nullptr : static_cast<const uint8_t*>(expect_u8(a[5], "fact mask").data_ptr());
  at::Tensor sums = a[7] != Py_None ? tensor(a[7]) : empty({M, g.G}, at::kLong, dev, s), counts;
  if (a[8] != Py_None) counts = tensor(a[8]);
  else if (truth(a[9])) counts = empty({g.G}, at::kLong, dev, s);
  at::Tensor ws;
  if (a[10] != Py_None) {
    ws = tensor(a[10]);
  } else {
    const size_t need = std::max(lq_groupby_workspace_bytes(K, g.rows, g.card, M),
                                 lq_groupby_bucket_workspace_bytes(n, K, g.rows, g.effective, M));
    ws = empty({static_cast<int64_t>(need)}, at::kByte, dev, s);
  }
  const uint32_t flags = static_cast<uint32_t>(integer(a[11]));
  int64_t *sp = static_cast<int64_t*>(sums.data_ptr()), *cp = counts.defined() ? static_cast<int64_t*>(counts.data_ptr()) : nullptr;
  void* wp = ws.data_ptr();
  const size_t wb = bytes_of(ws);
  call(s, [&](void* stream) {
    return lq_masked_groupby_sum(n, K, keys.data(), g.rows, g.mask.data(), g.code.data(), g.card, fact_mask, M, meas.data(), sp, cp,
                                 wp, wb, flags, stream);
  });
  PyObject* so = a[7] != Py_None ? (Py_INCREF(a[7]), a[7]) : wrap(sums);
  return pair(so, a[8] != Py_None ? (Py_INCREF(a[8]), a[8]) : wrap_or_none(counts));
}

// (fks, dim_rows, dim_mask, dim_code, group_card, preds [(col, lo, hi)], measures [(op code, a, b)], want_sum, want_min,
//  want_max, want_count, ws, flags, stream) -> (sums, mins, maxs, counts)
PyObject* groupby_agg(PyObject* const* a) {
  const Stream s(a[13]);
  Seq fks(a[0]), preds(a[5]), measures(a[6]);
  const int K = fks.size(), Q = preds.size(), M = measures.size();
  if (M == 0) raise(PyExc_IndexError, "list index out of range");
  Array<const int32_t*> keys(K);
  for (int k = 0; k < K; ++k) keys[k] = static_cast<const int32_t*>(expect_i32(fks[k], "foreign-key column").data_ptr());
  GroupShape g(K, a[1], a[2], a[3], a[4], false);
  Array<lq_range_pred> pa(Q);
  for (int q = 0; q < Q; ++q) {
    Seq p(preds[q]);
    if (p.size() != 3) raise(PyExc_ValueError, "a predicate is (column, lo, hi)");
    pa[q] = lq_range_pred{static_cast<const int32_t*>(expect_i32(p[0], "predicate column").data_ptr()),
                          static_cast<int32_t>(integer(p[1])), static_cast<int32_t>(integer(p[2]))};
  }
  Array<lq_measure> ma(M);
  int64_t n = 0;
  at::Device dev(at::kCPU);
  for (int m = 0; m < M; ++m) {
    Seq e(measures[m]);
    if (e.size() != 3) raise(PyExc_ValueError, "a measure is (op, a, b)");
    const at::Tensor& ta = expect_i32(e[1], "measure column");
    if (m == 0) {
      n = length(ta);
      dev = ta.device();
    }
    ma[m] = lq_measure{static_cast<int32_t>(integer(e[0])), static_cast<const int32_t*>(ta.data_ptr()),
                       e[2] == Py_None ? nullptr : static_cast<const int32_t*>(expect_i32(e[2], "measure column").data_ptr())};
  }
  const bool w_sum = truth(a[7]), w_min = truth(a[8]), w_max = truth(a[9]), w_count = truth(a[10]);
  at::Tensor sums, mins, maxs, counts, ws;
  if (w_sum) sums = empty({M, g.G}, at::kLong, dev, s);
  if (w_min) mins = empty({M, g.G}, at::kLong, dev, s);
  if (w_max) maxs = empty({M, g.G}, at::kLong, dev, s);
  if (w_count) counts = empty({g.G}, at::kLong, dev, s);
  if (a[11] != Py_None) {
    ws = tensor(a[11]);
  } else {
    size_t need = lq_groupby_agg_workspace_bytes(K, g.rows, g.card, M);
    if (Q == 0 && !w_min && !w_max && w_sum)
      need = std::max(need, lq_groupby_agg_bucket_workspace_bytes(n, K, g.rows, g.effective, M, ma));
    ws = empty({static_cast<int64_t>(need)}, at::kByte, dev, s);
  }
  const uint32_t flags = static_cast<uint32_t>(integer(a[12]));
  auto ptr = [](const at::Tensor& t) { return t.defined() ? static_cast<int64_t*>(t.data_ptr()) : nullptr; };
  void* wp = ws.data_ptr();
  const size_t wb = bytes_of(ws);
  call(s, [&](void* stream) {
    return lq_groupby_agg(n, K, keys.data(), g.rows, g.mask.data(), g.code.data(), g.card, Q, pa, M, ma, ptr(sums), ptr(mins),
                          ptr(maxs), ptr(counts), wp, wb, flags, stream);
  });
  PyObject* t = PyTuple_New(4);
  if (!t) throw PyErrorSet{};
  PyTuple_SET_ITEM(t, 0, wrap_or_none(sums));
  PyTuple_SET_ITEM(t, 1, wrap_or_none(mins));
  PyTuple_SET_ITEM(t, 2, wrap_or_none(maxs));
  PyTuple_SET_ITEM(t, 3, wrap_or_none(counts));
  return t;
}

// (group_card, sums, counts, keys [(kind, index, descending)], order, n_out, stream)
PyObject* order_groups(PyObject* const* a) {
  const Stream s(a[6]);
  const at::Tensor& counts = expect_i64(a[2], "counts");
  const int64_t G = length(counts);
  int32_t M = 0;
  const int64_t* sp = nullptr;
  if (a[1] != Py_None) {
    const at::Tensor& t = expect_i64(a[1], "sums");
    if (t.dim() != 2 || t.size(1) != G || !t.is_contiguous()) raise(PyExc_ValueError, "sums must be a contiguous [n_measures x G] tensor");
    M = static_cast<int32_t>(t.size(0));
    sp = static_cast<const int64_t*>(t.data_ptr());
  }
  Seq cards(a[0]), keys(a[3]);
  Array<int32_t> card(cards.size());
  int64_t prod = 1;
  for (int k = 0; k < cards.size(); ++k) {
    card[k] = cardinality(cards[k]);
    prod = product(prod, card[k]);
  }
  if (prod != G) raise(PyExc_ValueError, "counts length differs from the product of group_card");
  Array<lq_sort_key> ka(keys.size());
  for (int q = 0; q < keys.size(); ++q) {
    Seq e(keys[q]);
    if (e.size() != 3) raise(PyExc_ValueError, "a sort key is (kind, index, descending)");
    ka[q] = lq_sort_key{static_cast<int32_t>(integer(e[0])), static_cast<int32_t>(integer(e[1])), truth(e[2]) ? 1 : 0};
  }
  at::Tensor order = a[4] != Py_None ? expect_i32(a[4], "order") : empty({G}, at::kInt, counts.device(), s);
  at::Tensor n_out = a[5] != Py_None ? expect_i32(a[5], "n_out") : empty({1}, at::kInt, counts.device(), s);
  if (order.numel() < G || n_out.numel() < 1) raise(PyExc_ValueError, "order needs G entries and n_out one");
  const int64_t* cp = static_cast<const int64_t*>(counts.data_ptr());
  int32_t *op = static_cast<int32_t*>(order.data_ptr()), *np = static_cast<int32_t*>(n_out.data_ptr());
  call(s, [&](void* stream) { return lq_order_groups(cards.size(), card, M, sp, cp, keys.size(), ka, op, np, stream); });
  PyObject* oo = a[4] != Py_None ? (Py_INCREF(a[4]), a[4]) : wrap(order);
  return pair(oo, a[5] != Py_None ? (Py_INCREF(a[5]), a[5]) : wrap(n_out));
}

// ------------------------------------------------------------------ trees ---------------

lq_tree tree_of(PyObject* feature, PyObject* threshold, PyObject* H) {
  const at::Tensor& f = expect_i32(feature, "tree feature index");
  const at::Tensor& v = expect(threshold, at::kFloat, "torch.float32", "tree thresholds");
  const at::Tensor& h = tensor(H);
  if (h.scalar_type() != at::kChar || !h.is_cuda() || h.dim() != 2 || !h.is_contiguous())
    raise(PyExc_TypeError, "H must be a contiguous int8 [nodes x leaves] tensor on the GPU");
  if (length(f) != h.size(0) || length(v) != h.size(0))
    raise(PyExc_ValueError, "feature, threshold and H disagree on the number of nodes");
  return lq_tree{static_cast<int32_t>(h.size(0)), static_cast<int32_t>(h.size(1)), static_cast<const int32_t*>(f.data_ptr()),
                 static_cast<const float*>(v.data_ptr()), static_cast<const int8_t*>(h.data_ptr())};
}

// (dims, c_f, feature, threshold, H, stream) -> (tables, target)
PyObject* tree_project_dims(PyObject* const* a) {
  const Stream s(a[5]);
  const lq_tree tree = tree_of(a[2], a[3], a[4]);
  const int64_t ld = lq_tree_table_ld(tree.n_leaves);
  const at::Device dev = tensor(a[4]).device();
  DimStar star(a[0], static_cast<int32_t>(integer(a[1])), LQ_F32);
  const int K = star.dims_seq.size();
  std::vector<at::Tensor> tables;
  Array<void*> ptr(K);
  for (int k = 0; k < K; ++k) {
    tables.push_back(empty({star.dims[k].rows, ld}, at::kByte, dev, s));
    ptr[k] = tables[k].data_ptr();
  }
  at::Tensor target = empty({ld}, at::kByte, dev, s);
  uint8_t* tp = static_cast<uint8_t*>(target.data_ptr());
  call(s, [&](void* stream) { return lq_tree_project_dims(&star.c, &tree, ptr, tp, stream); });
  PyObject* l = list_of(tables);
  return pair(l, wrap(target));
}

// (dims, tables, feature, threshold, H, c_f, stream) -> masks
PyObject* tree_compress_tables(PyObject* const* a) {
  const Stream s(a[6]);
  const lq_tree tree = tree_of(a[2], a[3], a[4]);
  const int64_t words = lq_tree_mask_words(tree.n_leaves);
  const at::Device dev = tensor(a[4]).device();
  DimStar star(a[0], static_cast<int32_t>(integer(a[5])), LQ_F32);
  const int K = star.dims_seq.size();
  Seq tables(a[1]);
  Array<const void*> tp(std::max(K, tables.size()));
  for (int k = 0; k < tables.size(); ++k) tp[k] = tensor(tables[k]).data_ptr();
  std::vector<at::Tensor> masks;
  Array<uint64_t*> mp(K);
  for (int k = 0; k < K; ++k) {
    masks.push_back(empty({star.dims[k].rows, words}, at::kLong, dev, s));
    mp[k] = static_cast<uint64_t*>(masks[k].data_ptr());
  }
  call(s, [&](void* stream) { return lq_tree_compress_tables(&star.c, &tree, tp.data(), mp.data(), stream); });
  return list_of(masks);
}

// (c_f, feature, threshold, H, stream) -> buffer
PyObject* tree_fact_masks(PyObject* const* a) {
  const Stream s(a[4]);
  const lq_tree tree = tree_of(a[1], a[2], a[3]);
  const int32_t c_f = static_cast<int32_t>(integer(a[0]));
  at::Tensor buf = empty({lq_tree_fact_mask_bytes(tree.n_nodes, tree.n_leaves)}, at::kByte, tensor(a[3]).device(), s);
  void* p = buf.data_ptr();
  call(s, [&](void* stream) { return lq_tree_fact_masks(c_f, &tree, p, stream); });
  return wrap(buf);
}

// Outputs of a tree join and the row counts of its tables (as descriptors without data).
struct TreeJoin {
  at::Tensor leaf, onehot;
  Seq tables;
  Array<const void*> ptr;
  Array<lq_mat> rows;
  int32_t* leaf_ptr = nullptr;
  uint8_t* onehot_ptr = nullptr;
  TreeJoin(PyObject* tables_obj, int K, int64_t n, int32_t leaves, const at::Device& dev, bool want_leaf, bool want_onehot, const Stream& s)
      : tables(tables_obj), ptr(std::max(K, tables.size())), rows(std::max(K, tables.size())) {
    if (want_leaf) {
      leaf = empty({n}, at::kInt, dev, s);
      leaf_ptr = static_cast<int32_t*>(leaf.data_ptr());
    }
    if (want_onehot) {
      onehot = empty({n, leaves}, at::kByte, dev, s);
      onehot_ptr = static_cast<uint8_t*>(onehot.data_ptr());
    }
    for (int k = 0; k < tables.size(); ++k) {
      const at::Tensor& t = tensor(tables[k]);
      ptr[k] = t.data_ptr();
      rows[k] = lq_mat{nullptr, length(t), 1, 1, LQ_F32};
    }
  }
};

// (X, fks, tables, target, feature, threshold, H, want_leaf, want_onehot, flags, stream) -> (leaf, onehot)
PyObject* fused_join_tree(PyObject* const* a) {
  const Stream s(a[10]);
  const lq_tree tree = tree_of(a[4], a[5], a[6]);
  Star star(a[0], a[1]);
  const at::Device dev = tensor(a[6]).device();
  const uint32_t flags = static_cast<uint32_t>(integer(a[9]));
  TreeJoin j(a[2], star.c.n_dims, star.c.n_fact, tree.n_leaves, dev, truth(a[7]), truth(a[8]), s);
  at::Tensor ws;
  if (flags & LQ_CHECK_FKS) {
    star.c.dims = j.rows;
    ws = empty({256}, at::kByte, dev, s);
  }
  const uint8_t* target = static_cast<const uint8_t*>(tensor(a[3]).data_ptr());
  void* wp = ws.defined() ? ws.data_ptr() : nullptr;
  const size_t wb = ws.defined() ? bytes_of(ws) : 0;
  call(s, [&](void* stream) {
    return lq_fused_join_tree(&star.c, &tree, j.ptr.data(), target, j.leaf_ptr, j.onehot_ptr, flags, wp, wb, stream);
  });
  return pair(wrap_or_none(j.leaf), wrap_or_none(j.onehot));
}

// (fks, masks, feature, threshold, H, want_leaf, want_onehot, flags, stream, X, fact_masks) -> (leaf, onehot)
PyObject* fused_join_tree_masks(PyObject* const* a) {
  const Stream s(a[8]);
  const lq_tree tree = tree_of(a[2], a[3], a[4]);
  Star star(a[9], a[0]);
  const uint32_t flags = static_cast<uint32_t>(integer(a[7]));
  TreeJoin j(a[1], star.c.n_dims, star.c.n_fact, tree.n_leaves, tensor(a[4]).device(), truth(a[5]), truth(a[6]), s);
  // row counts of the mask tables (the library may then keep small tables in LDS); no data pointers
  star.c.dims = j.rows;
  const void* fact_masks = data_of<void>(a[10]);
  call(s, [&](void* stream) {
    return lq_fused_join_tree_masks(&star.c, &tree, reinterpret_cast<const uint64_t* const*>(j.ptr.data()), fact_masks, j.leaf_ptr,
                                    j.onehot_ptr, flags, stream);
  });
  return pair(wrap_or_none(j.leaf), wrap_or_none(j.onehot));
}

// ------------------------------------------------------------------ key maps ------------

// (keys, max_keys, flags, stream)
template <bool WIDE> PyObject* keymap_build(PyObject* const* a) {
  const Stream s(a[3]);
  const at::Tensor& keys = WIDE ? expect_i64(a[0], "dimension key column") : expect_i32(a[0], "dimension key column");
  const int64_t n = length(keys), cap = std::max(n, a[1] == Py_None ? int64_t{0} : integer(a[1]));
  const size_t bytes = WIDE ? lq_keymap64_bytes(cap) : lq_keymap_bytes(cap);
  const uint32_t flags = static_cast<uint32_t>(integer(a[2]));
  at::Tensor table = empty({static_cast<int64_t>(bytes)}, at::kByte, keys.device(), s);
  void *tp = table.data_ptr(), *kp = keys.data_ptr();
  call(s, [&](void* stream) {
    return WIDE ? lq_keymap64_build(tp, bytes, static_cast<const int64_t*>(kp), n, flags, stream)
                : lq_keymap_build(tp, bytes, static_cast<const int32_t*>(kp), n, flags, stream);
  });
  return wrap(table);
}

// (table, fact_keys, fk, stream)
template <bool WIDE> PyObject* keymap_lookup(PyObject* const* a) {
  const Stream s(a[3]);
  const at::Tensor& table = tensor(a[0]);
  const at::Tensor& keys = WIDE ? expect_i64(a[1], "fact key column") : expect_i32(a[1], "fact key column");
  const int64_t n = length(keys);
  at::Tensor fk = a[2] != Py_None ? tensor(a[2]) : empty(keys.sizes(), at::kInt, keys.device(), s);
  const void *tp = table.data_ptr(), *kp = keys.data_ptr();
  const size_t bytes = static_cast<size_t>(table.numel());
  int32_t* out = static_cast<int32_t*>(fk.data_ptr());
  call(s, [&](void* stream) {
    return WIDE ? lq_keymap64_lookup(tp, bytes, static_cast<const int64_t*>(kp), n, out, stream)
                : lq_keymap_lookup(tp, bytes, static_cast<const int32_t*>(kp), n, out, stream);
  });
  return a[2] != Py_None ? (Py_INCREF(a[2]), a[2]) : wrap(fk);
}

// ------------------------------------------------------------------ module --------------

// The module's functions take a fixed number of positional arguments; C++ exceptions end here.
template <PyObject* (*F)(PyObject* const*), int N> PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != N) {
    PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", N, n);
    return nullptr;
  }
  try {
    return F(args);
  } catch (const PyErrorSet&) {
    return nullptr;
  } catch (const c10::OutOfMemoryError& e) {
    // torch's own class, as its Python API raises it for the same failed allocation
    PyObject* torch = PyImport_ImportModule("torch");
    PyObject* cls = torch ? PyObject_GetAttrString(torch, "OutOfMemoryError") : nullptr;
    PyErr_SetString(cls ? cls : PyExc_MemoryError, e.what_without_backtrace());
    Py_XDECREF(cls);
    Py_XDECREF(torch);
    return nullptr;
  } catch (const c10::Error& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
    return nullptr;
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

// (LQError): the class raised for library errors, called with (code, message).
PyObject* set_error_class(PyObject* const* a) {
  Py_INCREF(a[0]);
  Py_XDECREF(g_error_class);
  g_error_class = a[0];
  Py_RETURN_NONE;
}

#define LQ_PY(name, f, n) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(&entry<f, n>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    LQ_PY("set_error_class", set_error_class, 1),
    LQ_PY("project_dims", project_dims, 6),
    LQ_PY("fused_join_predict", fused_join_predict, 10),
    LQ_PY("materialized_join_predict", materialized_join_predict, 11),
    LQ_PY("masked_groupby_sum", masked_groupby_sum, 13),
    LQ_PY("groupby_agg", groupby_agg, 14),
    LQ_PY("order_groups", order_groups, 7),
    LQ_PY("tree_project_dims", tree_project_dims, 6),
    LQ_PY("tree_compress_tables", tree_compress_tables, 7),
    LQ_PY("tree_fact_masks", tree_fact_masks, 5),
    LQ_PY("fused_join_tree", fused_join_tree, 11),
    LQ_PY("fused_join_tree_masks", fused_join_tree_masks, 11),
    LQ_PY("keymap_build", keymap_build<false>, 4),
    LQ_PY("keymap64_build", keymap_build<true>, 4),
    LQ_PY("keymap_lookup", keymap_lookup<false>, 4),
    LQ_PY("keymap64_lookup", keymap_lookup<true>, 4),
    {nullptr, nullptr, 0, nullptr}};
#undef LQ_PY

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_lqpy", "Native argument marshalling of the lq binding.", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__lqpy(void) { return PyModule_Create(&module); }
