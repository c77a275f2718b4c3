// Native half of binding.py: takes tensors apart, allocates outputs and workspaces and calls the C ABI.
//
// A call on a small grid is over in about 10 us on the GPU; marshalling it in Python (five torch.empty of
// 1.5 us, the stream object 2.9 us, a ctypes structure 1.6 us, pointer wrappers) took 14 us of host time
// on top of the launches and set the pace.  Plain CPython entry points on torch's own tensor structs: no
// argument conversion layer, about 3 us.  Nothing is kept between calls.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ATen.h>
#include <cmath>
#include <vector>
#include "../../include/nsattn.h"

namespace {

PyObject *g_error = nullptr;       // binding.NsError
PyObject *g_device = nullptr;      // () -> the current device's number
PyObject *g_stream = nullptr;      // device number -> hipStream_t of its current stream

struct PyFail {};                  // a Python exception is set

[[noreturn]] void value_error(const char *msg) {
  PyErr_SetString(PyExc_ValueError, msg);
  throw PyFail{};
}
void check(int code) {
  if (code == NS_OK) return;
  PyObject *e = PyObject_CallFunction(g_error, "is", code, ns_last_error());
  if (e) {
    PyErr_SetObject(g_error, e);
    Py_DECREF(e);
  }
  throw PyFail{};
}
const at::Tensor &tensor(PyObject *o, const char *name) {
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_TypeError, "%s must be a tensor", name);
    throw PyFail{};
  }
  return THPVariable_Unpack(o);
}
int64_t integer(PyObject *o) {
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw PyFail{};
  return v;
}
double number(PyObject *o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw PyFail{};
  return v;
}
int dtype_code(const at::Tensor &t) {
  const auto s = t.scalar_type();
  if (s == at::kFloat) return NS_F32;
  if (s == at::kBFloat16) return NS_BF16;
  PyErr_Format(PyExc_TypeError, "only float32 and bfloat16 tensors are supported, got torch.%s", c10::toString(s));
  throw PyFail{};
}
void *ptr(const at::Tensor &t) { return t.defined() ? t.data_ptr() : nullptr; }
at::Tensor optional(PyObject *o, const char *name) { return o == Py_None ? at::Tensor() : tensor(o, name); }
at::Tensor empty(at::IntArrayRef sizes, at::ScalarType dt, const at::Tensor &like) {
  return at::empty(sizes, at::TensorOptions().dtype(dt).device(like.device()));
}
// the caller's workspace, or nbytes of device memory (nothing when none are needed)
at::Tensor workspace(PyObject *o, size_t nbytes, const at::Tensor &like) {
  if (o != Py_None) return tensor(o, "workspace");
  return nbytes ? empty({(int64_t)nbytes}, at::kByte, like) : at::Tensor();
}
size_t bytes_of(const at::Tensor &ws) { return ws.defined() ? (size_t)ws.numel() : 0; }
// hipStream_t of a stream object or of the current stream.  Asked for when the arguments have been looked at, so that
// what is wrong with them is reported also where there is no device.
void *stream_of(PyObject *o) {
  PyObject *s;
  if (o == Py_None) {
    PyObject *dev = PyObject_CallNoArgs(g_device);
    if (!dev) throw PyFail{};
    s = PyObject_CallOneArg(g_stream, dev);
    Py_DECREF(dev);
  } else {
    s = PyObject_GetAttrString(o, "cuda_stream");
  }
  if (!s) throw PyFail{};
  const long long v = PyLong_AsLongLong(s);
  Py_DECREF(s);
  if (v == -1 && PyErr_Occurred()) throw PyFail{};
  return reinterpret_cast<void *>((intptr_t)v);
}
bool i32_contiguous(const at::Tensor &t) { return t.scalar_type() == at::kInt && t.is_contiguous(); }

PyObject *wrap(const at::Tensor &t) {
  if (!t.defined()) Py_RETURN_NONE;
  return THPVariable_Wrap(t);
}
template <class... Ts> PyObject *tuple(const Ts &...ts) {
  PyObject *r = PyTuple_New(sizeof...(ts));
  Py_ssize_t i = 0;
  (PyTuple_SET_ITEM(r, i++, wrap(ts)), ...);
  return r;
}
// the C call without the interpreter lock
template <class F> void call(F f) {
  int code;
  Py_BEGIN_ALLOW_THREADS
  code = f();
  Py_END_ALLOW_THREADS
  check(code);
}
template <class F> PyObject *guarded(Py_ssize_t have, Py_ssize_t want, F f) {
  if (have != want) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  try {
    return f();
  } catch (const PyFail &) {
  } catch (...) {                  // torch's own types: OutOfMemoryError, IndexError, ..
    torch::translate_exception_to_python(std::current_exception());
  }
  return nullptr;
}

float scale_of(PyObject *o, int64_t head_dim) { return o == Py_None ? (float)std::pow((double)head_dim, -0.5) : (float)number(o); }

ns_attn_desc make_desc(const at::Tensor &q, int64_t gh, int64_t gw, int64_t block, float scale, const at::Tensor &out,
                       const at::Tensor &coords, int64_t radius, int64_t G) {
  if (q.stride(3) != 1) value_error("head_dim must be contiguous");
  ns_attn_desc d{};
  d.batch = (int32_t)q.size(0); d.heads = (int32_t)q.size(1); d.head_dim = (int32_t)q.size(3);
  d.grid_h = (int32_t)gh; d.grid_w = (int32_t)gw; d.block = (int32_t)block; d.radius = (int32_t)radius;
  d.n_global = (int32_t)G;
  d.dtype = dtype_code(q);
  d.tokens = (int32_t)q.size(2);
  d.scale = scale;
  d.q_stride_b = q.stride(0); d.q_stride_h = q.stride(1); d.q_stride_t = q.stride(2);
  if (out.defined()) {
    d.out_stride_b = out.stride(0); d.out_stride_h = out.stride(1); d.out_stride_t = out.stride(2);
  }
  d.coords = static_cast<const int32_t *>(ptr(coords));
  return d;
}

// attn(q, k, v, grid_h, grid_w, block, scale, coords, out, workspace, stream, radius, n_global, mode)
// mode 0: out; 1: (out, logits, lse); 2: (out, logits, lse, scores)
PyObject *attn(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded(n, 14, [&]() -> PyObject * {
    const at::Tensor &q = tensor(a[0], "q"), &k = tensor(a[1], "k"), &v = tensor(a[2], "v");
    if (q.sizes() != k.sizes() || k.sizes() != v.sizes() || q.strides() != k.strides() || q.strides() != v.strides())
      value_error("q, k, v must have the same shape and strides");
    if (q.scalar_type() != k.scalar_type() || q.scalar_type() != v.scalar_type())
      value_error("q, k, v must have the same dtype");
    if (q.dim() != 4) value_error("q, k, v must be [B,H,T,D]");
    const int64_t B = q.size(0), H = q.size(1), T = q.size(2), D = q.size(3), G = integer(a[12]), mode = integer(a[13]);
    const at::Tensor coords = optional(a[7], "coords");
    at::Tensor out = optional(a[8], "out");
    if (!out.defined()) out = empty({B, H, T, D}, q.scalar_type(), q);
    if (coords.defined() && !i32_contiguous(coords)) value_error("coords must be a contiguous int32 tensor [B, T - n_global]");
    const ns_attn_desc d = make_desc(q, integer(a[3]), integer(a[4]), integer(a[5]), scale_of(a[6], D), out, coords, integer(a[11]), G);
    at::Tensor logits, lse, scores;
    if (mode) {
      logits = G == 1 ? empty({B, H, T}, at::kFloat, q) : empty({B, H, G, T}, at::kFloat, q);
      lse = G == 1 ? empty({B, H}, at::kFloat, q) : empty({B, H, G}, at::kFloat, q);
    }
    if (mode == 2) scores = empty({B, T - G}, at::kFloat, q);
    const at::Tensor ws = workspace(a[9], ns_attn_workspace_bytes(&d), q);
    void *const s = stream_of(a[10]);
    float *const lp = static_cast<float *>(ptr(logits)), *const ep = static_cast<float *>(ptr(lse));
    call([&] {
      return mode == 2 ? ns_attn_forward_scores(&d, ptr(q), ptr(k), ptr(v), ptr(out), lp, ep, static_cast<float *>(ptr(scores)),
                                                ptr(ws), bytes_of(ws), s)
                       : ns_attn_forward(&d, ptr(q), ptr(k), ptr(v), ptr(out), lp, ep, ptr(ws), bytes_of(ws), s);
    });
    if (mode == 0) return wrap(out);
    return mode == 1 ? tuple(out, logits, lse) : tuple(out, logits, lse, scores);
  });
}

// scores(q, k, scale, n_global, scores, workspace, stream)
PyObject *scores(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded(n, 7, [&]() -> PyObject * {
    const at::Tensor &q = tensor(a[0], "q"), &k = tensor(a[1], "k");
    if (q.sizes() != k.sizes() || q.strides() != k.strides() || q.scalar_type() != k.scalar_type())
      value_error("q and k must have the same shape, strides and dtype");
    if (q.dim() != 4) value_error("q and k must be [B,H,T,D]");
    const int64_t G = integer(a[3]), T = q.size(2);
    // the grid fields are not used by scoring; a 1 x (T-G) grid keeps the descriptor valid
    const ns_attn_desc d = make_desc(q, 1, T - G, 1, scale_of(a[2], q.size(3)), at::Tensor(), at::Tensor(), 1, G);
    at::Tensor out = optional(a[4], "scores");
    if (!out.defined()) out = empty({q.size(0), T - G}, at::kFloat, q);
    const at::Tensor ws = workspace(a[5], cls_scores_workspace_bytes(&d), q);
    void *const s = stream_of(a[6]);
    call([&] { return cls_scores(&d, ptr(q), ptr(k), static_cast<float *>(ptr(out)), ptr(ws), bytes_of(ws), s); });
    return wrap(out);
  });
}

// topk(scores, k, x, coords, kept_idx, y, coords_out, workspace, stream, n_global)
PyObject *topk(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded(n, 10, [&]() -> PyObject * {
    const at::Tensor &sc = tensor(a[0], "scores");
    if (sc.scalar_type() != at::kFloat || !sc.is_contiguous()) value_error("scores must be a contiguous float32 tensor");
    if (sc.dim() != 2) value_error("scores must be [B,N]");
    const int64_t B = sc.size(0), N = sc.size(1), k = integer(a[1]), G = integer(a[9]), kk = k > 0 ? k : 0;
    at::Tensor kept = optional(a[4], "kept_idx"), y = optional(a[5], "y"), cout = optional(a[6], "coords_out");
    const at::Tensor x = optional(a[2], "x"), coords = optional(a[3], "coords");
    if (!kept.defined()) kept = empty({B, kk}, at::kInt, sc);
    int32_t C = 0, xdt = NS_BF16;
    if (x.defined()) {
      if (!x.is_contiguous() || x.dim() != 3 || x.size(0) != B || x.size(1) != G + N) value_error("x must be contiguous [B, n_global+N, C]");
      C = (int32_t)x.size(2);
      xdt = dtype_code(x);
      if (!y.defined()) y = empty({B, G + kk, x.size(2)}, x.scalar_type(), sc);
    }
    if (coords.defined()) {
      if (!i32_contiguous(coords)) value_error("coords must be contiguous int32 [B,N]");
      if (!cout.defined()) cout = empty({B, kk}, at::kInt, sc);
    }
    const at::Tensor ws = workspace(a[7], topk_filter_workspace_bytes((int32_t)B, (int32_t)N, (int32_t)k), sc);
    void *const s = stream_of(a[8]);
    call([&] {
      return topk_filter_global((int32_t)B, (int32_t)N, (int32_t)k, (int32_t)G, static_cast<const float *>(ptr(sc)), ptr(x), C, xdt,
                                static_cast<const int32_t *>(ptr(coords)), static_cast<int32_t *>(ptr(kept)), ptr(y),
                                static_cast<int32_t *>(ptr(cout)), ptr(ws), bytes_of(ws), s);
    });
    return tuple(kept, y, cout);
  });
}

// embed(pixels, w_patch, b_patch, cls_token, pos_embed, patch, out, workspace, stream)
PyObject *embed(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded(n, 9, [&]() -> PyObject * {
    static const char *const names[5] = {"pixels", "w_patch", "b_patch", "cls_token", "pos_embed"};
    const at::Tensor *t[5];
    for (int i = 0; i < 5; i++) {
      t[i] = &tensor(a[i], names[i]);
      if (t[i]->scalar_type() != (i == 2 ? at::kFloat : at::kBFloat16) || !t[i]->is_contiguous()) {
        PyErr_Format(PyExc_ValueError, "%s must be a contiguous torch.%s tensor", names[i], i == 2 ? "float32" : "bfloat16");
        throw PyFail{};
      }
    }
    const at::Tensor &px = *t[0], &w = *t[1], &pos = *t[4];
    if (px.dim() != 4) value_error("pixels must be [B,channels,height,width]");
    const int64_t patch = integer(a[5]), B = px.size(0), ch = px.size(1);
    if (patch < 1 || px.size(2) % patch || px.size(3) % patch) value_error("image sides must be multiples of the patch side");
    const int64_t gh = px.size(2) / patch, gw = px.size(3) / patch, dim = w.size(0);
    if (w.dim() != 2 || w.size(1) != ch * patch * patch || pos.dim() != 2 || pos.size(0) != 1 + gh * gw || pos.size(1) != dim)
      value_error("w_patch must be [dim, channels*patch*patch] and pos_embed [1+gh*gw, dim]");
    at::Tensor out = optional(a[6], "out");
    if (!out.defined()) out = empty({B, 1 + gh * gw, dim}, at::kBFloat16, px);
    size_t need = vit_embed_workspace_bytes((int32_t)B, (int32_t)ch, (int32_t)gh, (int32_t)gw, (int32_t)patch, (int32_t)dim);
    const at::Tensor ws = workspace(a[7], need ? need : 1, px);
    void *const s = stream_of(a[8]);
    call([&] {
      return vit_embed((int32_t)B, (int32_t)ch, (int32_t)gh, (int32_t)gw, (int32_t)patch, (int32_t)dim, ptr(px), ptr(w),
                       static_cast<const float *>(ptr(*t[2])), ptr(*t[3]), ptr(pos), ptr(out), ptr(ws), bytes_of(ws), s);
    });
    return wrap(out);
  });
}

// ---- weights: a mapping of the twelve tensors of a block
constexpr int kWeights = 12;
const char *const kNames[kWeights] = {"ln1_g", "ln1_b", "w_qkv", "b_qkv", "w_proj", "b_proj", "ln2_g", "ln2_b",
                                      "w_fc1", "b_fc1", "w_fc2", "b_fc2"};
PyObject *g_names[kWeights];

// What the mappings gave, held until the call has returned: a mapping may make its tensors as they are asked for,
// and another thread may replace a dict's while the interpreter lock is given up.
struct Held {
  std::vector<PyObject *> objects;
  Held() = default;
  Held(const Held &) = delete;
  ~Held() {
    for (PyObject *o : objects) Py_DECREF(o);
  }
  PyObject *item(PyObject *weights, int i) {
    PyObject *o;
    if (PyDict_CheckExact(weights)) {
      o = PyDict_GetItemWithError(weights, g_names[i]);
      if (!o && !PyErr_Occurred()) PyErr_SetObject(PyExc_KeyError, g_names[i]);
      Py_XINCREF(o);
    } else {
      o = PyObject_GetItem(weights, g_names[i]);
    }
    if (!o) throw PyFail{};
    objects.push_back(o);
    return o;
  }
};
ns_vit_block_weights read_weights(Held &held, PyObject *weights, const at::Device &dev, const char *prefix) {
  const void *p[kWeights];
  for (int i = 0; i < kWeights; i++) {
    const at::Tensor &t = tensor(held.item(weights, i), kNames[i]);
    const bool matrix = kNames[i][0] == 'w';
    if (t.scalar_type() != (matrix ? at::kBFloat16 : at::kFloat) || !t.is_contiguous() || t.device() != dev) {
      PyErr_Format(PyExc_ValueError, "%sweight %s must be a contiguous torch.%s tensor on %s", prefix, kNames[i],
                   matrix ? "bfloat16" : "float32", dev.str().c_str());
      throw PyFail{};
    }
    p[i] = t.data_ptr();
  }
  auto f = [&](int i) { return static_cast<const float *>(p[i]); };
  return ns_vit_block_weights{f(0), f(1), p[2], f(3), p[4], f(5), f(6), f(7), p[8], f(9), p[10], f(11)};
}
ns_vit_block_desc block_desc(Held &held, const at::Tensor &x, PyObject *weights, int64_t gh, int64_t gw, int64_t block, int64_t heads,
                             double eps, PyObject *scale, int64_t G) {
  if (x.scalar_type() != at::kBFloat16 || !x.is_contiguous() || x.dim() != 3)
    value_error("x must be a contiguous bfloat16 tensor [B,T,dim]");
  if (heads < 1) value_error("heads must be positive");
  ns_vit_block_desc d{};
  ns_attn_desc &ad = d.attn;
  ad.batch = (int32_t)x.size(0); ad.heads = (int32_t)heads; ad.head_dim = (int32_t)(x.size(2) / heads);
  ad.grid_h = (int32_t)gh; ad.grid_w = (int32_t)gw; ad.block = (int32_t)block; ad.radius = 1; ad.n_global = (int32_t)G;
  ad.dtype = NS_BF16;
  ad.tokens = (int32_t)x.size(1);
  ad.scale = scale_of(scale, x.size(2) / heads);
  d.dim = (int32_t)x.size(2);
  d.mlp_dim = (int32_t)tensor(held.item(weights, 8), "w_fc1").size(0);
  d.ln_eps = (float)eps;
  return d;
}

// block(x, weights, grid_h, grid_w, block, heads, ln_eps, scale, coords, want_scores, out, workspace, stream, n_global)
PyObject *block(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded(n, 14, [&]() -> PyObject * {
    const at::Tensor &x = tensor(a[0], "x");
    const int64_t G = integer(a[13]);
    Held held;
    ns_vit_block_desc d = block_desc(held, x, a[1], integer(a[2]), integer(a[3]), integer(a[4]), integer(a[5]), number(a[6]), a[7], G);
    const ns_vit_block_weights w = read_weights(held, a[1], x.device(), "");
    const at::Tensor coords = optional(a[8], "coords");
    if (coords.defined()) {
      if (!i32_contiguous(coords)) value_error("coords must be a contiguous int32 tensor [B, T-1]");
      d.attn.coords = static_cast<const int32_t *>(ptr(coords));
    }
    const int want = PyObject_IsTrue(a[9]);
    if (want < 0) throw PyFail{};
    at::Tensor out = optional(a[10], "out");
    if (!out.defined()) out = empty(x.sizes(), at::kBFloat16, x);
    at::Tensor sc;
    if (want) sc = empty({x.size(0), x.size(1) - G}, at::kFloat, x);
    const size_t need = vit_block_workspace_bytes(&d);
    const at::Tensor ws = workspace(a[11], need ? need : 1, x);
    void *const s = stream_of(a[12]);
    call([&] { return vit_block_forward(&d, &w, ptr(x), ptr(out), static_cast<float *>(ptr(sc)), ptr(ws), bytes_of(ws), s); });
    return want ? tuple(out, sc) : wrap(out);
  });
}

// stack(x, layer_weights, grid_h, grid_w, block, heads, prune_after, keep_k, ln_eps, scale, out, workspace, stream,
//       n_global, tap_layers)
PyObject *stack(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded(n, 15, [&]() -> PyObject * {
    const at::Tensor &x = tensor(a[0], "x");
    PyObject *layers = PySequence_Fast(a[1], "layer_weights must be a sequence");
    if (!layers) throw PyFail{};
    struct Own { PyObject *o; ~Own() { Py_XDECREF(o); } } own{layers};
    const Py_ssize_t L = PySequence_Fast_GET_SIZE(layers);
    if (L < 1) {
      PyErr_SetString(PyExc_IndexError, "layer_weights is empty");
      throw PyFail{};
    }
    const int64_t gh = integer(a[2]), gw = integer(a[3]), after = integer(a[6]), keep = integer(a[7]), G = integer(a[13]);
    ns_vit_desc d{};
    Held held;
    d.block = block_desc(held, x, PySequence_Fast_GET_ITEM(layers, 0), gh, gw, integer(a[4]), integer(a[5]), number(a[8]), a[9], G);
    d.layers = (int32_t)L;
    d.prune_after = (int32_t)after;
    d.keep_k = (int32_t)keep;
    std::vector<ns_vit_block_weights> w((size_t)L);
    for (Py_ssize_t i = 0; i < L; i++) {
      char prefix[32];
      snprintf(prefix, sizeof(prefix), "layer %d ", (int)i);
      w[(size_t)i] = read_weights(held, PySequence_Fast_GET_ITEM(layers, i), x.device(), prefix);
    }
    const int64_t B = x.size(0), T = x.size(1), dim = x.size(2);
    const bool pruning = after > 0 && keep > 0;
    at::Tensor out = optional(a[10], "out"), kept;
    if (!out.defined()) out = empty({B, pruning ? G + keep : T, dim}, at::kBFloat16, x);
    if (pruning) kept = empty({B, keep}, at::kInt, x);
    const size_t need = vit_workspace_bytes(&d);
    const at::Tensor ws = workspace(a[11], need ? need : 1, x);
    void *const s = stream_of(a[12]);
    int32_t *const kp = static_cast<int32_t *>(ptr(kept));
    if (a[14] == Py_None) {
      call([&] { return vit_forward(&d, w.data(), ptr(x), ptr(out), kp, ptr(ws), bytes_of(ws), s); });
      return tuple(out, kept);
    }
    PyObject *tl = PySequence_Fast(a[14], "tap_layers must be a sequence");
    if (!tl) throw PyFail{};
    Own own2{tl};
    const Py_ssize_t nt = PySequence_Fast_GET_SIZE(tl);
    std::vector<int32_t> at_layer;
    std::vector<at::Tensor> taps;
    std::vector<void *> tp;
    for (Py_ssize_t i = 0; i < nt; i++) {
      at_layer.push_back((int32_t)integer(PySequence_Fast_GET_ITEM(tl, i)));
      taps.push_back(empty({B, gh * gw, dim}, at::kBFloat16, x));
      tp.push_back(ptr(taps.back()));
    }
    call([&] {
      return vit_forward_features(&d, w.data(), ptr(x), ptr(out), kp, (int32_t)nt, at_layer.data(), tp.data(), ptr(ws),
                                  bytes_of(ws), s);
    });
    PyObject *list = PyList_New(nt);
    for (Py_ssize_t i = 0; i < nt; i++) PyList_SET_ITEM(list, i, wrap(taps[(size_t)i]));
    PyObject *r = PyTuple_New(3);
    PyTuple_SET_ITEM(r, 0, wrap(out));
    PyTuple_SET_ITEM(r, 1, wrap(kept));
    PyTuple_SET_ITEM(r, 2, list);
    return r;
  });
}

// setup(error class, function giving the current device, function giving a device's current stream)
PyObject *setup(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded(n, 3, [&]() -> PyObject * {
    PyObject **const to[3] = {&g_error, &g_device, &g_stream};
    for (int i = 0; i < 3; i++) {
      Py_INCREF(a[i]);
      Py_XDECREF(*to[i]);
      *to[i] = a[i];
    }
    Py_RETURN_NONE;
  });
}

#define NS_FAST(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {NS_FAST(attn), NS_FAST(scores), NS_FAST(topk), NS_FAST(embed), NS_FAST(block), NS_FAST(stack),
                         NS_FAST(setup), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_nsbind", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__nsbind(void) {
  for (int i = 0; i < kWeights; i++) g_names[i] = PyUnicode_InternFromString(kNames[i]);
  return PyModule_Create(&module);
}
