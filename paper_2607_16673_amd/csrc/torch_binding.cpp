// torch_binding.cpp -- argument marshalling of the device calls for the
// Python binding: torch tensors are checked for device, dtype, shape and
// contiguity and passed to the C ABI of include/sla.h as raw device pointers,
// on the calling thread's current stream.  Each function returns the ABI's
// status code; a bad argument raises TypeError or ValueError before anything
// is launched.
//
// Native because a call's marshalling bounds every launch shorter than it:
// with tensors checked and ctypes structures filled in Python, one eager
// sla_verify took 31 us of host time against 7 us on the GPU for one sequence
// of eight nodes (conv 20 us, commit 21 us, prune 17 us).
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <initializer_list>

#include "sla.h"

namespace {

using Dims = std::initializer_list<int64_t>;

const at::Tensor &tensor(PyObject *o, const char *name) {
  TORCH_CHECK_TYPE(THPVariable_Check(o), name, " must be a torch tensor");
  return THPVariable_Unpack(o);
}

void *device_pointer(const at::Tensor &t, at::ScalarType dtype, Dims shape, const char *name) {
  TORCH_CHECK_VALUE(t.is_cuda(), name, " must live on the GPU");
  TORCH_CHECK_TYPE(t.scalar_type() == dtype, name, " must be ", dtype, ", got ", t.scalar_type());
  const at::IntArrayRef want(shape.begin(), shape.size());
  TORCH_CHECK_VALUE(t.sizes() == want, name, " has shape ", t.sizes(), ", expected ", want);
  TORCH_CHECK_VALUE(t.is_contiguous(), name, " must be contiguous");
  return t.data_ptr();
}

void *pointer(PyObject *o, at::ScalarType dtype, Dims shape, const char *name) {
  return device_pointer(tensor(o, name), dtype, shape, name);
}

void *optional_pointer(PyObject *o, at::ScalarType dtype, Dims shape, const char *name) {
  return o == Py_None ? nullptr : pointer(o, dtype, shape, name);
}

const at::Tensor &sized(PyObject *o, int64_t dims, const char *name) {
  const at::Tensor &t = tensor(o, name);
  TORCH_CHECK_VALUE(t.dim() == dims, name, " must have ", dims, " dimensions, got ", t.dim());
  return t;
}

int activation_code(const at::Tensor &t) {
  TORCH_CHECK_TYPE(t.scalar_type() == at::kBFloat16 || t.scalar_type() == at::kFloat,
                   "q/k/v must be bfloat16 or float32, got ", t.scalar_type());
  return t.scalar_type() == at::kBFloat16 ? SLA_DTYPE_BF16 : SLA_DTYPE_F32;
}

hipStream_t stream_of(const at::Tensor &t) { return c10::hip::getCurrentHIPStream(t.device().index()).stream(); }

long number(PyObject *o) {
  const long v = PyLong_AsLong(o);
  if (v == -1 && PyErr_Occurred()) throw python_error();
  return v;
}

bool truth(PyObject *o) {
  const int v = PyObject_IsTrue(o);
  if (v < 0) throw python_error();
  return v != 0;
}

// other Python threads run while the library enqueues (a launch can wait for
// room in the queue)
template <typename F>
int unlocked(F call) {
  PyThreadState *const ts = PyEval_SaveThread();
  const int code = call();
  PyEval_RestoreThread(ts);
  return code;
}

void count_args(Py_ssize_t got, Py_ssize_t want) {
  TORCH_CHECK_TYPE(got == want, "expected ", want, " arguments, got ", got);
}

// the four tensors of a factor store, from o[0..3]
sla_factors factors(PyObject *const *o, at::ScalarType act, int64_t B, int64_t n, int64_t H, int64_t dk, int64_t dv,
                    bool gates) {
  sla_factors f;
  f.k = pointer(o[0], act, {B, n, H, dk}, "factors.k");
  f.u = static_cast<float *>(pointer(o[1], at::kFloat, {B, n, H, dv}, "factors.u"));
  f.alpha = static_cast<float *>(gates ? pointer(o[2], at::kFloat, {B, n, H, dk}, "factors.alpha")
                                       : pointer(o[2], at::kFloat, {B, n, H}, "factors.alpha"));
  f.parent = static_cast<int32_t *>(pointer(o[3], at::kInt, {B, n}, "factors.parent"));
  return f;
}

// verify(state, q, k, v, alpha, beta, parent_idx, out, f.k, f.u, f.alpha, f.parent,
//        p.k, p.u, p.alpha, p.parent, path, len, pending, status, topology, family, route)
// pending: whether p.k .. len are a pending round's (each is then required)
PyObject *verify(PyObject *, PyObject *const *o, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  count_args(nargs, 23);
  const at::Tensor &q = sized(o[1], 4, "q");
  const at::Tensor &v = tensor(o[3], "v");
  TORCH_CHECK_VALUE(v.dim() > 0, "v has no dimensions");
  const int64_t B = q.size(0), n = q.size(1), H = q.size(2), dk = q.size(3), dv = v.size(-1);
  const at::ScalarType act = q.scalar_type();
  sla_shape shape;
  shape.batch = (int32_t)B;
  shape.heads = (int32_t)H;
  shape.d_k = (int32_t)dk;
  shape.d_v = (int32_t)dv;
  shape.n_nodes = (int32_t)n;
  shape.qkv_dtype = activation_code(q);
  shape.topology = (int32_t)number(o[20]);
  shape.family = (int32_t)number(o[21]);
  shape.route = (int32_t)number(o[22]);
  const bool gates = shape.family == SLA_FAMILY_GLA;
  const sla_factors f = factors(o + 8, act, B, n, H, dk, dv, gates);
  sla_pending pend;
  const bool pending = truth(o[18]);
  if (pending) {
    const int64_t pn = sized(o[15], 2, "pending parent").size(1);
    pend.f = factors(o + 12, act, B, pn, H, dk, dv, gates);
    pend.n_nodes = (int32_t)pn;
    pend.path = static_cast<const int32_t *>(pointer(o[16], at::kInt, {B, pn}, "pending.path"));
    pend.len = static_cast<const int32_t *>(pointer(o[17], at::kInt, {B}, "pending.len"));
  }
  int32_t *status = static_cast<int32_t *>(optional_pointer(o[19], at::kInt, {B}, "status"));
  float *state = static_cast<float *>(pointer(o[0], at::kFloat, {B, H, dk, dv}, "state"));
  const void *qp = device_pointer(q, act, {B, n, H, dk}, "q");
  const void *kp = pointer(o[2], act, {B, n, H, dk}, "k");
  const void *vp = device_pointer(v, act, {B, n, H, dv}, "v");
  const void *alpha = gates ? optional_pointer(o[4], at::kFloat, {B, n, H, dk}, "alpha")
                            : optional_pointer(o[4], at::kFloat, {B, n, H}, "alpha");
  const void *beta = optional_pointer(o[5], at::kFloat, {B, n, H}, "beta");
  const void *parent = pointer(o[6], at::kInt, {B, n}, "parent_idx");
  float *out = static_cast<float *>(pointer(o[7], at::kFloat, {B, n, H, dv}, "out"));
  const hipStream_t stream = stream_of(q);
  return PyLong_FromLong(unlocked([&] {
    return sla_verify(&shape, state, pending ? &pend : nullptr, qp, kp, vp, static_cast<const float *>(alpha),
        static_cast<const float *>(beta), static_cast<const int32_t *>(parent), out, &f, status, stream);
  }));
  END_HANDLE_TH_ERRORS
}

// commit(state, f.k, f.u, f.alpha, f.parent, path, len, status, family)
PyObject *commit(PyObject *, PyObject *const *o, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  count_args(nargs, 9);
  const at::Tensor &k = sized(o[1], 4, "factors.k");
  const at::Tensor &u = tensor(o[2], "factors.u");
  TORCH_CHECK_VALUE(u.dim() > 0, "factors.u has no dimensions");
  const int64_t B = k.size(0), n = k.size(1), H = k.size(2), dk = k.size(3), dv = u.size(-1);
  sla_shape shape;
  shape.batch = (int32_t)B;
  shape.heads = (int32_t)H;
  shape.d_k = (int32_t)dk;
  shape.d_v = (int32_t)dv;
  shape.n_nodes = (int32_t)n;
  shape.qkv_dtype = activation_code(k);
  shape.topology = SLA_TOPO_TREE;
  shape.family = (int32_t)number(o[8]);
  shape.route = SLA_ROUTE_AUTO;
  const sla_factors f = factors(o + 1, k.scalar_type(), B, n, H, dk, dv, shape.family == SLA_FAMILY_GLA);
  int32_t *status = static_cast<int32_t *>(optional_pointer(o[7], at::kInt, {B}, "status"));
  const at::Tensor &state = tensor(o[0], "state");
  float *sp = static_cast<float *>(device_pointer(state, at::kFloat, {B, H, dk, dv}, "state"));
  const void *path = pointer(o[5], at::kInt, {B, n}, "path");
  const void *len = pointer(o[6], at::kInt, {B}, "len");
  const hipStream_t stream = stream_of(state);
  return PyLong_FromLong(unlocked([&] {
    return sla_commit(&shape, sp, &f, static_cast<const int32_t *>(path), static_cast<const int32_t *>(len), status,
        stream);
  }));
  END_HANDLE_TH_ERRORS
}

sla_conv_shape conv_shape(const at::Tensor &x, int64_t K, bool silu) {
  sla_conv_shape s;
  s.batch = (int32_t)x.size(0);
  s.channels = (int32_t)x.size(2);
  s.kernel_size = (int32_t)K;
  s.n_nodes = (int32_t)x.size(1);
  s.x_dtype = activation_code(x);
  s.activation = silu ? SLA_ACT_SILU : SLA_ACT_NONE;
  return s;
}

// conv_verify(conv_state | None, x, weight, parent_idx, y, bias | None,
//             px, pparent, path, len, pending, status, activation)
PyObject *conv_verify(PyObject *, PyObject *const *o, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  count_args(nargs, 13);
  const at::Tensor &x = sized(o[1], 3, "x");
  const at::Tensor &weight = sized(o[2], 2, "weight");
  const int64_t B = x.size(0), n = x.size(1), D = x.size(2), K = weight.size(1);
  const at::ScalarType act = x.scalar_type();
  const sla_conv_shape shape = conv_shape(x, K, truth(o[12]));
  float *cs = static_cast<float *>(optional_pointer(o[0], at::kFloat, {B, K - 1, D}, "conv_state"));
  sla_conv_pending pend;
  const bool pending = truth(o[10]);
  if (pending) {
    const int64_t pn = sized(o[7], 2, "pending parent").size(1);
    pend.x = pointer(o[6], act, {B, pn, D}, "pending.x");
    pend.parent = static_cast<const int32_t *>(pointer(o[7], at::kInt, {B, pn}, "pending.parent"));
    pend.n_nodes = (int32_t)pn;
    pend.path = static_cast<const int32_t *>(pointer(o[8], at::kInt, {B, pn}, "pending.path"));
    pend.len = static_cast<const int32_t *>(pointer(o[9], at::kInt, {B}, "pending.len"));
  }
  const void *bias = optional_pointer(o[5], at::kFloat, {D}, "bias");
  int32_t *status = static_cast<int32_t *>(optional_pointer(o[11], at::kInt, {B}, "status"));
  const void *xp = device_pointer(x, act, {B, n, D}, "x");
  const void *wp = device_pointer(weight, at::kFloat, {D, K}, "weight");
  const void *parent = pointer(o[3], at::kInt, {B, n}, "parent_idx");
  void *y = pointer(o[4], act, {B, n, D}, "y");
  const hipStream_t stream = stream_of(x);
  return PyLong_FromLong(unlocked([&] {
    return sla_conv_verify(&shape, cs, pending ? &pend : nullptr, xp, static_cast<const float *>(wp),
        static_cast<const float *>(bias), static_cast<const int32_t *>(parent), y, status, stream);
  }));
  END_HANDLE_TH_ERRORS
}

// conv_commit(conv_state | None, x, parent_idx, path, len, kernel_size | None, status)
PyObject *conv_commit(PyObject *, PyObject *const *o, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  count_args(nargs, 7);
  const at::Tensor &x = sized(o[1], 3, "x");
  const int64_t B = x.size(0), n = x.size(1), D = x.size(2);
  const int64_t K = o[5] != Py_None ? number(o[5]) : sized(o[0], 3, "conv_state").size(1) + 1;
  const sla_conv_shape shape = conv_shape(x, K, true);
  float *cs = static_cast<float *>(optional_pointer(o[0], at::kFloat, {B, K - 1, D}, "conv_state"));
  int32_t *status = static_cast<int32_t *>(optional_pointer(o[6], at::kInt, {B}, "status"));
  const void *xp = device_pointer(x, x.scalar_type(), {B, n, D}, "x");
  const void *parent = pointer(o[2], at::kInt, {B, n}, "parent_idx");
  const void *path = pointer(o[3], at::kInt, {B, n}, "path");
  const void *len = pointer(o[4], at::kInt, {B}, "len");
  const hipStream_t stream = stream_of(x);
  return PyLong_FromLong(unlocked([&] {
    return sla_conv_commit(&shape, cs, xp, static_cast<const int32_t *>(parent), static_cast<const int32_t *>(path),
        static_cast<const int32_t *>(len), status, stream);
  }));
  END_HANDLE_TH_ERRORS
}

// prune(parent, logp, tau, budget, with_scores) ->
//   (code, packed_parent, index_map, count, status, scores | None)
PyObject *prune(PyObject *, PyObject *const *o, Py_ssize_t nargs) {
  HANDLE_TH_ERRORS
  count_args(nargs, 5);
  const at::Tensor &parent = sized(o[0], 2, "parent");
  const int64_t B = parent.size(0), n = parent.size(1);
  const double tau = PyFloat_AsDouble(o[2]);
  if (tau == -1.0 && PyErr_Occurred()) throw python_error();
  const long budget = number(o[3]);
  const bool scored = truth(o[4]);
  const void *pp = device_pointer(parent, at::kInt, {B, n}, "parent");
  const void *lp = pointer(o[1], at::kFloat, {B, n}, "logp");
  const auto ints = parent.options().dtype(at::kInt);
  const at::Tensor packed = at::empty({B, n}, ints), map = at::empty({B, n}, ints), count = at::empty({B}, ints),
                   status = at::empty({B}, ints);
  at::Tensor scores;
  if (scored) scores = at::empty({B, n}, ints.dtype(at::kFloat));
  const hipStream_t stream = stream_of(parent);
  const int code = unlocked([&] {
    return sla_prune(static_cast<const int32_t *>(pp), static_cast<const float *>(lp), (int32_t)B, (int32_t)n,
        (float)tau, (int32_t)budget, packed.data_ptr<int32_t>(), map.data_ptr<int32_t>(), count.data_ptr<int32_t>(),
            scored ? scores.data_ptr<float>() : nullptr, status.data_ptr<int32_t>(), stream);
  });
  PyObject *r = PyTuple_New(6);
  if (!r) throw python_error();
  PyTuple_SET_ITEM(r, 0, PyLong_FromLong(code));
  PyTuple_SET_ITEM(r, 1, THPVariable_Wrap(packed));
  PyTuple_SET_ITEM(r, 2, THPVariable_Wrap(map));
  PyTuple_SET_ITEM(r, 3, THPVariable_Wrap(count));
  PyTuple_SET_ITEM(r, 4, THPVariable_Wrap(status));
  if (scored) {
    PyTuple_SET_ITEM(r, 5, THPVariable_Wrap(scores));
  } else {
    Py_INCREF(Py_None);
    PyTuple_SET_ITEM(r, 5, Py_None);
  }
  return r;
  END_HANDLE_TH_ERRORS
}

template <PyObject *(*F)(PyObject *, PyObject *const *, Py_ssize_t)>
constexpr PyMethodDef method(const char *name) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(F)), METH_FASTCALL, nullptr};
}

PyMethodDef methods[] = {method<verify>("verify"),           method<commit>("commit"),
    method<conv_verify>("conv_verify"),
                         method<conv_commit>("conv_commit"), method<prune>("prune"),   {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "Argument marshalling of libsla's device calls.", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&module); }
