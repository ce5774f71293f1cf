// The binding's way from torch tensors to the C calls of libhiermoe without Python code per argument.
//
// A call of the library takes the host about 2.5 us in the runtime's launch; checking and unpacking its tensors in
// Python and converting a dozen arguments by ctypes took another 2 us (dispatch, combine) and more (the planner's calls, with
// their lists), which is what small layers waited for: plan, dispatch and combine of 1,024 x 256 14.8 -> 8.8 us of host
// time.  Each function here takes the positional arguments of the
// binding's function of that name, checks what the binding checks, calls the library on the current
// stream and returns its status code.  It returns None, having changed nothing, whenever an argument is not the ordinary
// case (a tensor of another type, device, dtype or layout, a missing buffer, a number that is no int): the
// binding's Python code then does the call or says what is wrong with it, so there is one place that words errors.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>

#include "hiermoe.h"

namespace {

// The library's entry points, by address: the binding loads the library, and there is one copy of it.
struct Library {
  decltype(&hm_plan) plan;
  decltype(&hm_plan_mapped) plan_mapped;
  decltype(&hm_dispatch_pack) dispatch_pack;
  decltype(&hm_combine) combine;
  decltype(&hm_combine_f32) combine_f32;
  decltype(&hm_combine_mix) combine_mix;
  decltype(&hm_combine_transpose) combine_transpose;
  decltype(&hm_combine_transpose_bf16) combine_transpose_bf16;
  decltype(&hm_expert_load) expert_load;
  decltype(&hm_group_counts) group_counts;
  decltype(&hm_alltoall_times) alltoall_times;
  decltype(&hm_swap_counts_multi) swap_counts_multi;
  decltype(&hm_swap_select) swap_select;
  decltype(&hm_swap_apply) swap_apply;
} lib;
bool bound = false;

PyObject *name_T, *name_K, *name_c, *name_num_dest, *name_slot_row, *name_slot_keep, *name_rank_mask, *name_node_mask, *name_workspace;

constexpr int kMost = 8;   // entries of a list argument: hierarchies have at most four levels

// Thrown (inside this file only) when the call is left to the Python code.
struct NotOrdinary {};

class Ref {   // owns a reference
 public:
  explicit Ref(PyObject *o) : o_(o) {
    if (!o_) throw NotOrdinary();
  }
  ~Ref() { Py_DECREF(o_); }
  Ref(const Ref &) = delete;
  Ref &operator=(const Ref &) = delete;
  PyObject *get() const { return o_; }

 private:
  PyObject *o_;
};

const at::Tensor &tensor(PyObject *o) {
  if (!THPVariable_CheckExact(o)) throw NotOrdinary();
  return THPVariable_Unpack(o);
}
const at::Tensor &checked(PyObject *o, at::ScalarType type) {
  const at::Tensor &t = tensor(o);
  if (!t.is_cuda() || t.scalar_type() != type || !t.is_contiguous()) throw NotOrdinary();
  return t;
}
template <typename T>
T *pointer(PyObject *o, at::ScalarType type) {
  return static_cast<T *>(checked(o, type).data_ptr());
}
template <typename T>
T *pointer_or_null(PyObject *o, at::ScalarType type) {
  return o == Py_None ? nullptr : pointer<T>(o, type);
}
int32_t size32(int64_t n) {
  if (n < 0 || n > INT32_MAX) throw NotOrdinary();
  return static_cast<int32_t>(n);
}
// Rows and columns of a matrix.
void shape(const at::Tensor &t, int32_t &rows, int32_t &cols) {
  if (t.dim() != 2) throw NotOrdinary();
  rows = size32(t.size(0));
  cols = size32(t.size(1));
}
int64_t length(const at::Tensor &t) {
  if (t.dim() < 1) throw NotOrdinary();
  return t.size(0);
}
int64_t integer(PyObject *o) {
  if (!PyLong_CheckExact(o)) throw NotOrdinary();
  int overflow = 0;
  const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
  if (overflow) throw NotOrdinary();
  return v;
}
int32_t integer32(PyObject *o) {
  const int64_t v = integer(o);
  if (v < INT32_MIN || v > INT32_MAX) throw NotOrdinary();
  return static_cast<int32_t>(v);
}
double real(PyObject *o) {
  if (PyFloat_CheckExact(o)) return PyFloat_AS_DOUBLE(o);
  if (!PyLong_CheckExact(o)) throw NotOrdinary();
  const double v = PyLong_AsDouble(o);
  if (PyErr_Occurred()) throw NotOrdinary();
  return v;
}
// Entries of a list or tuple, borrowed.
int entries(PyObject *o, PyObject **item) {
  if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) throw NotOrdinary();
  const Py_ssize_t n = PySequence_Fast_GET_SIZE(o);
  if (n < 1 || n > kMost) throw NotOrdinary();
  for (Py_ssize_t i = 0; i < n; ++i) item[i] = PySequence_Fast_GET_ITEM(o, i);
  return static_cast<int>(n);
}
int integers(PyObject *o, int32_t *v) {
  PyObject *item[kMost];
  const int n = entries(o, item);
  for (int i = 0; i < n; ++i) v[i] = integer32(item[i]);
  return n;
}
void reals(PyObject *o, int n, double *v) {
  PyObject *item[kMost];
  if (entries(o, item) != n) throw NotOrdinary();
  for (int i = 0; i < n; ++i) v[i] = real(item[i]);
}

// A Plan of the binding: its table's shape and the host struct the C calls take.
class Plan {
 public:
  explicit Plan(PyObject *o) : o_(o) {
    T = integer32(Ref(PyObject_GetAttr(o, name_T)).get());
    K = integer32(Ref(PyObject_GetAttr(o, name_K)).get());
    const Ref c(PyObject_GetAttr(o, name_c));
    if (PyObject_GetBuffer(c.get(), &view_, PyBUF_SIMPLE) != 0) throw NotOrdinary();
    if (view_.len != static_cast<Py_ssize_t>(sizeof(hm_plan_out))) {
      PyBuffer_Release(&view_);
      throw NotOrdinary();
    }
  }
  ~Plan() { PyBuffer_Release(&view_); }
  Plan(const Plan &) = delete;
  Plan &operator=(const Plan &) = delete;
  hm_plan_out *c() const { return static_cast<hm_plan_out *>(view_.buf); }

  // The plan's buffers take another table of `tokens` x `slots` if they are large enough.
  void adopt(int32_t tokens, int32_t slots, const at::Tensor &weights) {
    const int64_t n = static_cast<int64_t>(tokens) * slots;
    if (weights.numel() != n || n > numel(name_slot_row) || n > numel(name_slot_keep)) throw NotOrdinary();
    if (tokens > numel(name_rank_mask) || tokens > numel(name_node_mask)) throw NotOrdinary();
    const Ref workspace(PyObject_GetAttr(o_, name_workspace));
    const at::Tensor &w = tensor(workspace.get());
    workspace_ = w.data_ptr();
    workspace_bytes_ = static_cast<size_t>(w.numel()) * 4;
    set(name_T, T, tokens);
    set(name_K, K, slots);
  }
  // After a plan: as many destinations as the library says.
  void destinations() {
    const Ref now(PyObject_GetAttr(o_, name_num_dest));
    if (!PyLong_CheckExact(now.get()) || PyLong_AsLong(now.get()) != c()->num_dest) {
      const Ref v(PyLong_FromLong(c()->num_dest));
      if (PyObject_SetAttr(o_, name_num_dest, v.get()) != 0) throw NotOrdinary();
    }
  }
  // The row calls take T and K beside the plan and trust them.
  void expect(int32_t tokens, PyObject *weights) const {
    if (tokens != T) throw NotOrdinary();
    if (weights != Py_None && tensor(weights).numel() != static_cast<int64_t>(T) * K) throw NotOrdinary();
  }
  void *workspace() const { return workspace_; }
  size_t workspace_bytes() const { return workspace_bytes_; }

  int32_t T, K;

 private:
  int64_t numel(PyObject *name) const {   // no limit for a buffer that is not asked for
    const Ref t(PyObject_GetAttr(o_, name));
    return t.get() == Py_None ? INT64_MAX : tensor(t.get()).numel();
  }
  void set(PyObject *name, int32_t &have, int32_t v) {
    if (have == v) return;
    const Ref value(PyLong_FromLong(v));
    if (PyObject_SetAttr(o_, name, value.get()) != 0) throw NotOrdinary();
    have = v;
  }
  PyObject *o_;
  Py_buffer view_;
  void *workspace_ = nullptr;
  size_t workspace_bytes_ = 0;
};

// Runs `call` on the current stream without the interpreter's lock.
template <typename Call>
hm_status launched(Call call) {
  void *const stream = c10::hip::getCurrentHIPStream().stream();
  PyThreadState *const state = PyEval_SaveThread();
  const hm_status rc = call(stream);
  PyEval_RestoreThread(state);
  return rc;
}

// The frame of every function: the status as an int, None for calls left to the Python code.
template <typename Body>
PyObject *answer(Py_ssize_t given, Py_ssize_t wanted, Body body) {
  if (bound && given == wanted) {
    try {
      return PyLong_FromLong(body());
    } catch (...) {   // NotOrdinary, or a tensor without storage
      PyErr_Clear();
    }
  }
  Py_RETURN_NONE;
}

PyObject *plan(PyObject *, PyObject *const *a, Py_ssize_t n) {   // ids, weights, expert_to_rank, nodes, ranks_per_node, level, plan
  return answer(n, 7, [&] {
    const at::Tensor &ids = checked(a[0], at::kInt), &weights = checked(a[1], at::kFloat), &e2r = checked(a[2], at::kInt);
    int32_t T, K;
    shape(ids, T, K);
    const int32_t E = size32(length(e2r));
    const hm_topology topo = {integer32(a[3]), integer32(a[4])};
    const auto level = static_cast<hm_dedup_level>(integer32(a[5]));
    const auto *i = static_cast<const int32_t *>(ids.data_ptr()), *e = static_cast<const int32_t *>(e2r.data_ptr());
    const auto *w = static_cast<const float *>(weights.data_ptr());
    Plan p(a[6]);
    p.adopt(T, K, weights);
    const hm_status rc = launched([&](void *s) { return lib.plan(i, w, e, T, K, E, topo, level, p.c(), p.workspace(), p.workspace_bytes(), s); });
    if (rc == HM_OK) p.destinations();
    return rc;
  });
}

PyObject *plan_mapped(PyObject *, PyObject *const *a, Py_ssize_t n) {   // ids, weights, dest_map, num_dest, dedup, plan
  return answer(n, 6, [&] {
    const at::Tensor &ids = checked(a[0], at::kInt), &weights = checked(a[1], at::kFloat), &map = checked(a[2], at::kInt);
    int32_t T, K;
    shape(ids, T, K);
    const int32_t E = size32(length(map)), dests = integer32(a[3]);
    const int dedup = PyObject_IsTrue(a[4]);
    if (dedup < 0) throw NotOrdinary();
    const auto *i = static_cast<const int32_t *>(ids.data_ptr()), *m = static_cast<const int32_t *>(map.data_ptr());
    const auto *w = static_cast<const float *>(weights.data_ptr());
    Plan p(a[5]);
    p.adopt(T, K, weights);
    const hm_status rc = launched([&](void *s) { return lib.plan_mapped(i, w, m, T, K, E, dests, dedup, p.c(), p.workspace(), p.workspace_bytes(), s); });
    if (rc == HM_OK) p.destinations();
    return rc;
  });
}

// in [T, H], plan, out [rows, H]: dispatch and the transposes.
template <typename T, typename Call>
PyObject *spread(PyObject *const *a, Py_ssize_t n, at::ScalarType type, Call call) {
  return answer(n, 3, [&] {
    const at::Tensor &in = checked(a[0], type), &out = checked(a[2], type);
    int32_t tokens, H;
    shape(in, tokens, H);
    const Plan p(a[1]);
    p.expect(tokens, Py_None);
    const int64_t rows = length(out);
    const auto *from = static_cast<const T *>(in.data_ptr());
    auto *to = static_cast<T *>(out.data_ptr());
    return launched([&](void *s) { return call(from, p.T, p.K, H, p.c(), to, rows, s); });
  });
}
PyObject *dispatch_pack(PyObject *, PyObject *const *a, Py_ssize_t n) { return spread<void>(a, n, at::kBFloat16, lib.dispatch_pack); }
PyObject *combine_transpose(PyObject *, PyObject *const *a, Py_ssize_t n) { return spread<float>(a, n, at::kFloat, lib.combine_transpose); }
PyObject *combine_transpose_bf16(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return spread<void>(a, n, at::kBFloat16, lib.combine_transpose_bf16);
}

// y [rows, H], weights or None, plan, out [T, H].
template <typename T, typename Call>
PyObject *merge(PyObject *const *a, Py_ssize_t n, at::ScalarType type, Call call) {
  return answer(n, 4, [&] {
    const at::Tensor &y = checked(a[0], type), &out = checked(a[3], type);
    int32_t tokens, H;
    shape(out, tokens, H);
    const Plan p(a[2]);
    p.expect(tokens, a[1]);
    const auto *w = pointer_or_null<const float>(a[1], at::kFloat);
    const int64_t rows = length(y);
    const auto *from = static_cast<const T *>(y.data_ptr());
    auto *to = static_cast<T *>(out.data_ptr());
    return launched([&](void *s) { return call(from, rows, w, p.T, p.K, H, p.c(), to, s); });
  });
}
PyObject *combine(PyObject *, PyObject *const *a, Py_ssize_t n) { return merge<void>(a, n, at::kBFloat16, lib.combine); }
PyObject *combine_f32(PyObject *, PyObject *const *a, Py_ssize_t n) { return merge<float>(a, n, at::kFloat, lib.combine_f32); }
PyObject *combine_mix(PyObject *, PyObject *const *a, Py_ssize_t n) { return merge<void>(a, n, at::kBFloat16, lib.combine_mix); }

PyObject *expert_load(PyObject *, PyObject *const *a, Py_ssize_t n) {   // ids, expert_to_rank, nodes, ranks_per_node, three loads, status
  return answer(n, 8, [&] {
    int32_t T, K;
    shape(tensor(a[0]), T, K);
    const auto *ids = pointer<const int32_t>(a[0], at::kInt), *e2r = pointer<const int32_t>(a[1], at::kInt);
    const int32_t E = size32(length(tensor(a[1])));
    const hm_topology topo = {integer32(a[2]), integer32(a[3])};
    int32_t *load[3];
    for (int i = 0; i < 3; ++i) load[i] = pointer<int32_t>(a[4 + i], at::kInt);
    auto *status = pointer_or_null<int32_t>(a[7], at::kInt);
    return launched([&](void *s) { return lib.expert_load(ids, e2r, T, K, E, topo, load[0], load[1], load[2], status, s); });
  });
}

PyObject *group_counts(PyObject *, PyObject *const *a, Py_ssize_t n) {   // ids, expert_to_rank, G, groups, counts, status
  return answer(n, 6, [&] {
    int32_t T, K, groups[kMost];
    shape(tensor(a[0]), T, K);
    const auto *ids = pointer<const int32_t>(a[0], at::kInt), *e2r = pointer<const int32_t>(a[1], at::kInt);
    const int32_t E = size32(length(tensor(a[1]))), G = integer32(a[2]);
    const int depth = integers(a[3], groups);
    auto *counts = pointer<int32_t>(a[4], at::kInt), *status = pointer_or_null<int32_t>(a[5], at::kInt);
    return launched([&](void *s) { return lib.group_counts(ids, e2r, T, K, E, G, depth, groups, counts, status, s); });
  });
}

// U, G, M, v, p_inter, p_intra, alpha_inter, beta_inter, alpha_intra, beta_intra, times, best
PyObject *alltoall_times(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return answer(n, 12, [&] {
    int32_t U[kMost];
    double model[4][kMost];
    const int D = integers(a[0], U);
    const int32_t G = integer32(a[1]);
    const double M = real(a[2]), v = real(a[3]);
    const auto *inter = pointer<const int32_t>(a[4], at::kInt), *intra = pointer<const int32_t>(a[5], at::kInt);
    for (int i = 0; i < 4; ++i) reals(a[6 + i], D, model[i]);
    auto *times = pointer<double>(a[10], at::kDouble);
    auto *best = pointer<int32_t>(a[11], at::kInt);
    return launched([&](void *s) {
      return lib.alltoall_times(D, U, G, M, v, inter, intra, model[0], model[1], model[2], model[3], times, best, s);
    });
  });
}

PyObject *swap_counts_multi(PyObject *, PyObject *const *a, Py_ssize_t n) {   // ids, expert_to_rank, G, ng, Z, status, workspace
  return answer(n, 7, [&] {
    int32_t T, K, ng[kMost], *Z[kMost];
    PyObject *item[kMost];
    shape(tensor(a[0]), T, K);
    const auto *ids = pointer<const int32_t>(a[0], at::kInt), *e2r = pointer<const int32_t>(a[1], at::kInt);
    const int32_t E = size32(length(tensor(a[1]))), G = integer32(a[2]);
    const int cuts = integers(a[3], ng);
    if (entries(a[4], item) != cuts) throw NotOrdinary();
    for (int i = 0; i < cuts; ++i) Z[i] = pointer<int32_t>(item[i], at::kInt);
    auto *status = pointer_or_null<int32_t>(a[5], at::kInt);
    const at::Tensor &ws = tensor(a[6]);
    void *const workspace = ws.data_ptr();
    const size_t bytes = static_cast<size_t>(ws.numel()) * 4;
    return launched([&](void *s) { return lib.swap_counts_multi(ids, e2r, T, K, E, G, cuts, ng, Z, status, workspace, bytes, s); });
  });
}

// U, G, M, v, z_inter, z_intra, scale_inter, scale_intra, alpha_inter, beta_inter, alpha_intra, beta_intra, gamma, Q, best_pair,
// best_time, workspace
PyObject *swap_select(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return answer(n, 17, [&] {
    int32_t U[kMost];
    const int32_t *z[kMost] = {};
    double scale[kMost], alpha[kMost], beta[kMost];
    PyObject *item[kMost];
    const int d = integers(a[0], U);
    const int32_t G = integer32(a[1]);
    const double M = real(a[2]), v = real(a[3]);
    if (entries(a[4], item) < d) throw NotOrdinary();
    for (int i = 1; i < d; ++i) z[i] = pointer<const int32_t>(item[i], at::kInt);
    const auto *z_intra = pointer<const int32_t>(a[5], at::kInt);
    const int32_t E = size32(length(tensor(a[5])));
    reals(a[6], d, scale);
    const double scale_intra = real(a[7]);
    reals(a[8], d, alpha);
    reals(a[9], d, beta);
    const double alpha_intra = real(a[10]), beta_intra = real(a[11]), gamma = real(a[12]);
    auto *Q = pointer<double>(a[13], at::kDouble);
    auto *pair = pointer<int32_t>(a[14], at::kInt);
    auto *time = pointer<double>(a[15], at::kDouble);
    const at::Tensor &ws = tensor(a[16]);
    void *const workspace = ws.data_ptr();
    const size_t bytes = static_cast<size_t>(ws.numel()) * 8;
    return launched([&](void *s) {
      return lib.swap_select(d, U, G, E, M, v, z, z_intra, scale, scale_intra, alpha, beta, alpha_intra, beta_intra, gamma, Q, pair,
                             time, workspace, bytes, s);
    });
  });
}

PyObject *swap_apply(PyObject *, PyObject *const *a, Py_ssize_t n) {   // expert_to_rank, best_pair
  return answer(n, 2, [&] {
    auto *e2r = pointer<int32_t>(a[0], at::kInt);
    const int32_t E = size32(length(tensor(a[0])));
    const auto *pair = pointer<const int32_t>(a[1], at::kInt);
    return launched([&](void *s) { return lib.swap_apply(e2r, E, pair, s); });
  });
}

// bind(addresses): the entry points, in the order of Library.
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n) {
  constexpr int kEntries = sizeof(Library) / sizeof(void *);
  void *address[kEntries];
  if (n != kEntries) {
    PyErr_Format(PyExc_TypeError, "%d addresses expected", kEntries);
    return nullptr;
  }
  for (int i = 0; i < kEntries; ++i) {
    address[i] = PyLong_AsVoidPtr(a[i]);
    if (!address[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
      return nullptr;
    }
  }
  std::memcpy(static_cast<void *>(&lib), address, sizeof(lib));
  bound = true;
  Py_RETURN_NONE;
}

#define HM_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {HM_METHOD(plan), HM_METHOD(plan_mapped), HM_METHOD(dispatch_pack), HM_METHOD(combine), HM_METHOD(combine_f32),
                         HM_METHOD(combine_mix), HM_METHOD(combine_transpose), HM_METHOD(combine_transpose_bf16),
                         HM_METHOD(expert_load), HM_METHOD(group_counts), HM_METHOD(alltoall_times), HM_METHOD(swap_counts_multi),
                         HM_METHOD(swap_select), HM_METHOD(swap_apply), HM_METHOD(bind), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_hmcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__hmcall() {
  PyObject **const names[] = {&name_T, &name_K, &name_c, &name_num_dest, &name_slot_row, &name_slot_keep, &name_rank_mask, &name_node_mask,
                              &name_workspace};
  const char *const text[] = {"T", "K", "c", "num_dest", "slot_row", "slot_keep", "rank_mask", "node_mask", "workspace"};
  for (int i = 0; i < 9; ++i)
    if (!(*names[i] = PyUnicode_InternFromString(text[i]))) return nullptr;
  return PyModule_Create(&module);
}
