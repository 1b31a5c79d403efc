// Marshalling of the two calls whose host cost shows (a small forward, the update of one parameter tensor) from torch tensors to the C ABI.
// A call that is anything but plain and right (a rate that is a tuple, a tensor of another shape, type, device or layout, a buffer
// left to the callee) returns None and the Python code takes it, with its checks and its messages: this file decides
// nothing, it only recognises what needs no decision.  HA_BINDING_TAG: the torch and the Python it is compiled for (build.py).
//
// Host time per call, in Python / here: forward of d = 64, H = 2, N = 1024 19 / 8.8 us (three launches), update of one tensor 5.2 / 3.3.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cmath>
#include <limits>

#include "../../include/hybrid_attn.h"

namespace {

typedef ha_status (*forward_fn)(const ha_problem *, const void *, const void *, const void *, const ha_feature_map *, const ha_feature_map *,
                                void *, void *, size_t, void *);
typedef ha_status (*update_fn)(const ha_optimizer *, size_t, float *, const float *, float *, float *, void *, int32_t, void *);

forward_fn g_forward = nullptr;
update_fn g_update = nullptr;
PyObject *g_map_type = nullptr, *g_raw_stream = nullptr;     // the FeatureMap class; device index -> current stream's handle
PyObject *g_w1, *g_b1, *g_w2, *g_b2, *g_w_mid, *g_b_mid, *g_degree, *g_act;

// A reference that is given back on every way out.
struct Ref {
  PyObject *p;
  explicit Ref(PyObject *o) : p(o) {}
  Ref(const Ref &) = delete;
  ~Ref() { Py_XDECREF(p); }
};

const at::Tensor *tensor(PyObject *o) { return THPVariable_Check(o) ? &THPVariable_Unpack(o) : nullptr; }

bool small_int(PyObject *o, int32_t *out) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow = 0;
  const long v = PyLong_AsLongAndOverflow(o, &overflow);
  if (overflow || v < std::numeric_limits<int32_t>::min() || v > std::numeric_limits<int32_t>::max()) return false;
  *out = static_cast<int32_t>(v);
  return true;
}

bool number(PyObject *o, float *out) {
  if (PyFloat_CheckExact(o)) {
    *out = static_cast<float>(PyFloat_AS_DOUBLE(o));
    return true;
  }
  int32_t i;
  if (!small_int(o, &i)) return false;
  *out = static_cast<float>(static_cast<double>(i));
  return true;
}

// The stream's handle: of the given stream object, or the current one of the device.
bool stream_of(PyObject *stream, const at::Tensor &t, void **out) {
  if (stream != Py_None) return false;
  const Ref index(PyLong_FromLong(t.get_device()));
  PyObject *args[] = {index.p};
  const Ref h(PyObject_Vectorcall(g_raw_stream, args, 1, nullptr));
  if (!h.p) {
    PyErr_Clear();
    return false;
  }
  *out = PyLong_AsVoidPtr(h.p);
  if (PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return true;
}

// FeatureMap object -> the C struct, checked against the problem as FeatureMap.check and c_struct do.
bool feature_map(PyObject *o, const at::Tensor &q, ha_feature_map *m) {
  if (reinterpret_cast<PyObject *>(Py_TYPE(o)) != g_map_type) return false;
  const Ref w1(PyObject_GetAttr(o, g_w1)), b1(PyObject_GetAttr(o, g_b1)), w2(PyObject_GetAttr(o, g_w2)), b2(PyObject_GetAttr(o, g_b2)),
      wm(PyObject_GetAttr(o, g_w_mid)), bm(PyObject_GetAttr(o, g_b_mid)), degree(PyObject_GetAttr(o, g_degree)), act(PyObject_GetAttr(o, g_act));
  if (!w1.p || !b1.p || !w2.p || !b2.p || !wm.p || !bm.p || !degree.p || !act.p) {
    PyErr_Clear();
    return false;
  }
  const int64_t H = q.size(1), d = q.size(3);
  auto weight = [&](PyObject *p, int64_t cols) -> const at::Tensor * {        // [H, any, cols]
    const at::Tensor *t = tensor(p);
    if (!t || t->dim() != 3 || t->size(0) != H || t->size(2) != cols || t->scalar_type() != q.scalar_type() || t->device() != q.device() ||
        !t->is_contiguous() || t->size(1) > std::numeric_limits<int32_t>::max())
      return nullptr;
    return t;
  };
  auto bias = [&](PyObject *p, int64_t width, const void **out) {
    *out = nullptr;
    if (p == Py_None) return true;
    const at::Tensor *t = tensor(p);
    if (!t || t->dim() != 2 || t->size(0) != H || t->size(1) != width || t->scalar_type() != at::kFloat || t->device() != q.device() ||
        !t->is_contiguous())
      return false;
    *out = t->data_ptr();
    return true;
  };
  const at::Tensor *t1 = weight(w1.p, d), *tm = nullptr;
  if (!t1) return false;
  int64_t last = t1->size(1);
  if (wm.p != Py_None) {
    if (!(tm = weight(wm.p, last))) return false;
    last = tm->size(1);
  } else if (bm.p != Py_None) {
    return false;
  }
  const at::Tensor *t2 = weight(w2.p, last);
  if (!t2) return false;
  *m = ha_feature_map{};
  const void *v1, *v2, *vm;
  if (!bias(b1.p, t1->size(1), &v1) || !bias(b2.p, t2->size(1), &v2) || !bias(bm.p, last, &vm)) return false;
  int32_t P, A;
  if (!small_int(degree.p, &P) || !small_int(act.p, &A) || P < 1 || t2->size(1) % P != 0) return false;
  m->w1 = t1->data_ptr();
  m->b1 = static_cast<const float *>(v1);
  m->w2 = t2->data_ptr();
  m->b2 = static_cast<const float *>(v2);
  m->d_hidden = static_cast<int32_t>(t1->size(1));
  m->d_out = static_cast<int32_t>(t2->size(1));
  m->poly_degree = P;
  m->out_act = A;
  m->w_mid = tm ? tm->data_ptr() : nullptr;
  m->b_mid = static_cast<const float *>(vm);
  m->d_mid = tm ? static_cast<int32_t>(tm->size(1)) : 0;
  return true;
}

// forward(q, k, v, phi_q, phi_k, hybrid_rate, block_size, softmax_scale, out, workspace, stream) -> status, or None
PyObject *forward(PyObject *, PyObject *const *args, Py_ssize_t n) {
  if (n != 11 || !g_forward) Py_RETURN_NONE;
  try {
    const at::Tensor *q = tensor(args[0]), *k = tensor(args[1]), *v = tensor(args[2]), *out = tensor(args[8]), *ws = tensor(args[9]);
    if (!q || !k || !v || !out || !ws || !q->is_cuda() || q->dim() != 4 || q->stride(3) != 1) Py_RETURN_NONE;
    const bool bf16 = q->scalar_type() == at::kBFloat16;
    if (!bf16 && q->scalar_type() != at::kFloat) Py_RETURN_NONE;
    for (const at::Tensor *t : {k, v, out})
      if (t->scalar_type() != q->scalar_type() || t->device() != q->device() || t->sizes() != q->sizes() || t->strides() != q->strides())
        Py_RETURN_NONE;
    if (ws->device() != q->device()) Py_RETURN_NONE;
    for (int i = 0; i < 4; ++i)
      if (q->size(i) > std::numeric_limits<int32_t>::max()) Py_RETURN_NONE;
    ha_problem p = {};
    if (!small_int(args[5], &p.hybrid_rate) || !small_int(args[6], &p.block_size)) Py_RETURN_NONE;
    if (args[7] == Py_None) p.softmax_scale = static_cast<float>(std::pow(static_cast<double>(q->size(3)), -0.5));
    else if (!number(args[7], &p.softmax_scale)) Py_RETURN_NONE;
    p.B = static_cast<int32_t>(q->size(0));
    p.H = static_cast<int32_t>(q->size(1));
    p.N = static_cast<int32_t>(q->size(2));
    p.d_head = static_cast<int32_t>(q->size(3));
    p.dtype = bf16 ? HA_BF16 : HA_F32;
    p.stride_b = q->stride(0);
    p.stride_h = q->stride(1);
    p.stride_n = q->stride(2);
    ha_feature_map mq, mk;
    const bool has_q = args[3] != Py_None, has_k = args[4] != Py_None;
    if ((has_q && !feature_map(args[3], *q, &mq)) || (has_k && !feature_map(args[4], *q, &mk))) Py_RETURN_NONE;
    void *stream;
    if (!stream_of(args[10], *q, &stream)) Py_RETURN_NONE;
    const void *qp = q->data_ptr(), *kp = k->data_ptr(), *vp = v->data_ptr();
    void *op = out->data_ptr(), *wp = ws->data_ptr();
    const size_t bytes = static_cast<size_t>(ws->numel()) * ws->element_size();
    ha_status st;
    Py_BEGIN_ALLOW_THREADS
    st = g_forward(&p, qp, kp, vp, has_q ? &mq : nullptr, has_k ? &mk : nullptr, op, wp, bytes, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
  } catch (...) {                                        // (a tensor without storage, under some transform)
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

// param_update(master, grad, lr, kind, m, v, step, grad_scale, beta1, beta2, eps, weight_decay, param_io, stream) -> status, or None
PyObject *param_update(PyObject *, PyObject *const *args, Py_ssize_t n) {
  if (n != 14 || !g_update) Py_RETURN_NONE;
  try {
    const at::Tensor *master = tensor(args[0]), *grad = tensor(args[1]);
    if (!master || !master->is_cuda()) Py_RETURN_NONE;
    const int64_t numel = master->numel();
    auto plain = [&](const at::Tensor *t) {
      return t && t->scalar_type() == at::kFloat && t->is_contiguous() && t->numel() == numel && t->device() == master->device();
    };
    if (!plain(master) || !plain(grad)) Py_RETURN_NONE;
    float *moment[2] = {nullptr, nullptr};
    for (int i = 0; i < 2; ++i) {
      if (args[4 + i] == Py_None) continue;
      const at::Tensor *t = tensor(args[4 + i]);
      if (!plain(t)) Py_RETURN_NONE;
      moment[i] = static_cast<float *>(t->data_ptr());
    }
    void *io = nullptr;
    int32_t io_dtype = HA_BF16;
    if (args[12] != Py_None) {
      const at::Tensor *t = tensor(args[12]);
      if (!t || !t->is_contiguous() || t->numel() != numel || t->device() != master->device()) Py_RETURN_NONE;
      if (t->scalar_type() == at::kFloat) io_dtype = HA_F32;
      else if (t->scalar_type() != at::kBFloat16) Py_RETURN_NONE;
      io = t->data_ptr();
    }
    ha_optimizer o = {};
    if (!small_int(args[3], &o.kind) || !small_int(args[6], &o.step) || !number(args[2], &o.lr) || !number(args[7], &o.grad_scale) ||
        !number(args[8], &o.beta1) || !number(args[9], &o.beta2) || !number(args[10], &o.eps) || !number(args[11], &o.weight_decay))
      Py_RETURN_NONE;
    void *stream;
    if (!stream_of(args[13], *master, &stream)) Py_RETURN_NONE;
    float *mp = static_cast<float *>(master->data_ptr());
    const float *gp = static_cast<const float *>(grad->data_ptr());
    ha_status st;
    Py_BEGIN_ALLOW_THREADS
    st = g_update(&o, static_cast<size_t>(numel), mp, gp, moment[0], moment[1], io, io_dtype, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

// bind(address of hybrid_attn_forward, address of hybrid_attn_param_update, FeatureMap, current-raw-stream function)
PyObject *bind(PyObject *, PyObject *args) {
  PyObject *f, *u, *map_type, *raw_stream;
  if (!PyArg_ParseTuple(args, "OOOO", &f, &u, &map_type, &raw_stream)) return nullptr;
  void *fp = PyLong_AsVoidPtr(f), *up = PyLong_AsVoidPtr(u);
  if (PyErr_Occurred()) return nullptr;
  Py_INCREF(map_type);
  Py_INCREF(raw_stream);
  Py_XSETREF(g_map_type, map_type);
  Py_XSETREF(g_raw_stream, raw_stream);
  g_forward = reinterpret_cast<forward_fn>(fp);
  g_update = reinterpret_cast<update_fn>(up);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"forward", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(forward)), METH_FASTCALL, nullptr},
                         {"param_update", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(param_update)), METH_FASTCALL, nullptr},
                         {"bind", bind, METH_VARARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "hybridattn_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_hybridattn_binding() {
  PyObject **names[] = {&g_w1, &g_b1, &g_w2, &g_b2, &g_w_mid, &g_b_mid, &g_degree, &g_act};
  const char *text[] = {"w1", "b1", "w2", "b2", "w_mid", "b_mid", "poly_degree", "out_act"};
  for (int i = 0; i < 8; ++i)
    if (!(*names[i] = PyUnicode_InternFromString(text[i]))) return nullptr;
  PyObject *m = PyModule_Create(&module);
  if (!m) return nullptr;
  // What this file was compiled for: the Python code uses the module only where both are what it finds.
  PyObject *abi = Py_BuildValue("(innn)", HA_ABI_VERSION, static_cast<Py_ssize_t>(sizeof(ha_problem)), static_cast<Py_ssize_t>(sizeof(ha_feature_map)),
                                static_cast<Py_ssize_t>(sizeof(ha_optimizer)));
  if (!abi || PyModule_AddObject(m, "abi", abi) < 0) {
    Py_XDECREF(abi);
    Py_DECREF(m);
    return nullptr;
  }
  if (PyModule_AddStringConstant(m, "tag", HA_BINDING_TAG) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
