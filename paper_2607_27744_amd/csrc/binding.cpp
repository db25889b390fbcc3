// Native call path of ops.py (CPython extension `_binding`).
//
// An operator call from Python spent 14 to 19 us on argument checks, string
// formatting and ctypes conversions (measured without the launches), more than
// the kernels of a small call take. Each function here does the same checks on
// the tensors directly, allocates the outputs and workspace that the caller
// left out and calls the C entry point: 1 to 2 us. It takes exactly the calls
// that ops.py's checks accept; for anything else (other argument types, a
// failed check, an exception from the tensor library) it returns None and
// ops.py's own path runs, which raises the error or handles the call. Nothing
// is kept between calls except the Python callables looked up at import.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/Functions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/rocs.h"

namespace {

PyObject* g_get_device;   // torch._C._cuda_getDevice
PyObject* g_raw_stream;   // torch._C._cuda_getCurrentRawStream
PyObject* g_check;        // _lib.check(status, name): raises RocsError
PyObject* g_cuda_stream;  // "cuda_stream"

struct Refuse {};         // not a call for this path
struct PyError {};        // a Python exception is set

void need(bool ok) {
  if (!ok) throw Refuse();
}

// A tensor argument: plain strided device tensors with storage of their own
// only (not torch.func's wrappers); null for None.
struct Ten {
  const at::Tensor* t = nullptr;
  at::Tensor own;
  explicit operator bool() const { return t != nullptr; }
  const at::Tensor* operator->() const { return t; }
  void* ptr() const { return t == nullptr ? nullptr : t->data_ptr(); }
  const int32_t* i32() const { return static_cast<const int32_t*>(ptr()); }
  const float* f32() const { return static_cast<const float*>(ptr()); }
  size_t bytes() const { return t == nullptr ? 0 : (size_t)t->nbytes(); }
};

// The address in a Python integer (a new reference, or null after an error).
void* address(PyObject* v) {
  if (v == nullptr) throw PyError();
  void* p = PyLong_AsVoidPtr(v);
  Py_DECREF(v);
  if (p == nullptr && PyErr_Occurred()) throw PyError();
  return p;
}

// The current stream of a device (its number, a new reference).
void* current_stream(PyObject* device) {
  if (device == nullptr) throw PyError();
  PyObject* v = PyObject_CallOneArg(g_raw_stream, device);
  Py_DECREF(device);
  return address(v);
}

// The given stream, or the current one of the current device.
void* stream_of(PyObject* o) {
  if (o == Py_None) return current_stream(PyObject_CallNoArgs(g_get_device));
  return address(PyObject_GetAttr(o, g_cuda_stream));
}

struct Call {
  c10::Device dev{c10::DeviceType::CPU};
  bool any = false;
  PyObject* stream;

  explicit Call(PyObject* s) : stream(s) {}

  Ten get(PyObject* o) {
    Ten r;
    if (o == Py_None) return r;
    need(THPVariable_CheckExact(o));
    r.t = &THPVariable_Unpack(o);
    need(r.t->is_cuda() && r.t->layout() == c10::kStrided && r.t->has_storage());
    if (!any) dev = r.t->device();
    any = true;
    need(r.t->device() == dev);
    return r;
  }
  Ten must(PyObject* o) {
    need(o != Py_None);
    return get(o);
  }
  // The caller's output or workspace, or a new one.
  Ten or_new(PyObject* o, c10::IntArrayRef shape, c10::ScalarType type) {
    Ten r = get(o);
    if (!r) {
      // Memory for a call on another stream is that stream's: ops.py takes it.
      need(stream == Py_None || stream_of(stream) == current_stream(PyLong_FromLong(dev.index())));
      r.own = at::empty(shape, c10::TensorOptions().dtype(type).device(dev));
      return r;
    }
    need(r->sizes() == shape && r->scalar_type() == type && r->is_contiguous());
    return r;
  }
};

const at::Tensor& tensor(const Ten& t) { return t.t != nullptr ? *t.t : t.own; }
void* data(const Ten& t) { return t.t != nullptr || t.own.defined() ? tensor(t).data_ptr() : nullptr; }
size_t nbytes(const Ten& t) { return t.t != nullptr || t.own.defined() ? tensor(t).nbytes() : 0; }

int32_t dtype_code(const Ten& t) {
  const c10::ScalarType s = t->scalar_type();
  need(s == c10::kBFloat16 || s == c10::kFloat);
  return s == c10::kBFloat16 ? ROCS_DTYPE_BF16 : ROCS_DTYPE_F32;
}

int32_t activation(PyObject* o) {
  if (o == Py_None) return ROCS_ACT_NONE;
  need(PyUnicode_CheckExact(o));
  if (PyUnicode_CompareWithASCIIString(o, "relu") == 0) return ROCS_ACT_RELU;
  need(PyUnicode_CompareWithASCIIString(o, "none") == 0);
  return ROCS_ACT_NONE;
}

int64_t integer(PyObject* o) {
  need(PyLong_CheckExact(o));
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) {
    PyErr_Clear();
    throw Refuse();
  }
  return v;
}

float scale_of(PyObject* o) {           // float(scale or 0.0)
  if (o == Py_None) return 0.f;
  need(PyFloat_CheckExact(o) || PyLong_CheckExact(o));
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) {
    PyErr_Clear();
    throw Refuse();
  }
  return (float)v;
}

void offsets(const Ten& t, int64_t n_req) {
  need(t->scalar_type() == c10::kInt && t->dim() == 1 && t->is_contiguous() &&
       t->numel() == n_req + 1);
}

void same(const Ten& t, const Ten& as) {          // optional input of the common dtype
  need(!t || (t->scalar_type() == as->scalar_type() && t->is_contiguous()));
}

void shape_is(const Ten& t, c10::IntArrayRef s) { need(t->sizes() == s); }

void bias_of(const Ten& t, int64_t n) {
  need(!t || (t->scalar_type() == c10::kFloat && t->dim() == 1 && t->size(0) == n &&
              t->is_contiguous()));
}

// Without the interpreter lock for its lifetime, however the scope is left.
struct Unlocked {
  PyThreadState* state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};

// Calls the C entry point without the interpreter lock. Every pointer and size
// is an argument here, so it has been taken while the lock was held: data_ptr()
// throws for a tensor without storage (inside torch.vmap or torch.func.grad).
template <typename... P, typename... A>
void run(const char* name, int32_t (*call)(P...), A... args) {
  static_assert(sizeof...(P) == sizeof...(A), "argument count");
  int32_t status;
  {
    Unlocked unlocked;
    status = call(args...);
  }
  if (status == ROCS_OK) return;
  PyObject* r = PyObject_CallFunction(g_check, "is", (int)status, name);
  Py_XDECREF(r);
  if (r == nullptr) throw PyError();
}

// The caller's own object, or the new tensor.
PyObject* result(PyObject* given, const Ten& t) {
  if (given != Py_None) {
    Py_INCREF(given);
    return given;
  }
  return THPVariable_Wrap(t.own);
}

PyObject* pair(PyObject* a, PyObject* b) {
  if (a == nullptr || b == nullptr) {
    Py_XDECREF(a);
    Py_XDECREF(b);
    return nullptr;
  }
  PyObject* r = PyTuple_Pack(2, a, b);
  Py_DECREF(a);
  Py_DECREF(b);
  return r;
}

template <int N, PyObject* (*F)(PyObject* const*)>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != N) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  try {
    return F(args);
  } catch (const PyError&) {
    return nullptr;
  } catch (const Refuse&) {
  } catch (const std::exception&) {
    PyErr_Clear();
  }
  Py_RETURN_NONE;
}

// x_cand, w_cand, x_req, w_req, index, mapped, bias, activation, x_cand_add,
// out, workspace, stream
PyObject* linear(PyObject* const* a) {
  Call c(a[11]);
  const Ten x = c.must(a[0]), w = c.must(a[1]), xr = c.get(a[2]), wr = c.get(a[3]),
            index = c.get(a[4]), bias = c.get(a[6]), add = c.get(a[8]);
  const bool mapped = a[5] == Py_True;
  const int32_t act = activation(a[7]);
  need(x->dim() == 2 && w->dim() == 2);
  const int64_t n = x->size(0), k = x->size(1), d = w->size(0);
  need(w->size(1) == k);
  const int32_t code = dtype_code(x);
  for (const Ten* t : {&x, &w, &xr, &wr, &add}) same(*t, x);
  int64_t r = 0, kr = 0;
  if (xr) {
    need(wr && index && xr->dim() == 2);
    r = xr->size(0);
    kr = xr->size(1);
    shape_is(wr, {d, kr});
  } else {
    need(!wr);
    if (!mapped && index) r = index->numel() - 1;
  }
  if (index) {
    if (mapped) need(index->scalar_type() == c10::kInt && index->dim() == 1 &&
                     index->is_contiguous() && index->numel() == n);
    else offsets(index, r);
  }
  if (add) shape_is(add, x->sizes());
  bias_of(bias, d);
  const Ten out = c.or_new(a[9], {n, d}, x->scalar_type());
  const size_t bytes = rocs_ikbo_linear_workspace_size(r, n, d, kr);
  Ten ws = c.get(a[10]);
  if (!ws && bytes > 0) ws = c.or_new(Py_None, {(int64_t)bytes}, c10::kByte);
  void* s = stream_of(c.stream);
  if (mapped)
    run("rocs_ikbo_linear_mapped", rocs_ikbo_linear_mapped, xr.ptr(), kr, x.ptr(), add.ptr(), k,
        wr.ptr(), w.ptr(), bias.f32(), index.i32(), r, n, d, code, act, data(out), data(ws),
        nbytes(ws), s);
  else
    run("rocs_ikbo_linear", rocs_ikbo_linear, xr.ptr(), kr, x.ptr(), add.ptr(), k, wr.ptr(),
        w.ptr(), bias.f32(), index.i32(), r, n, d, code, act, data(out), data(ws), nbytes(ws), s);
  return result(a[9], out);
}

// x_req, x_cand, w_rr, w_cr, w_cc, cand_offsets, b_req, b_cand, activation,
// x_cand_add, y_req, y_cand, workspace, stream
PyObject* glm_linear(PyObject* const* a) {
  Call c(a[13]);
  const Ten xr = c.must(a[0]), x = c.must(a[1]), wrr = c.must(a[2]), wr = c.must(a[3]),
            w = c.must(a[4]), off = c.must(a[5]), br = c.get(a[6]), bias = c.get(a[7]),
            add = c.get(a[9]);
  const int32_t act = activation(a[8]);
  need(xr->dim() == 2 && x->dim() == 2 && wrr->dim() == 2 && w->dim() == 2);
  const int64_t r = xr->size(0), kr = xr->size(1), n = x->size(0), k = x->size(1),
                dr = wrr->size(0), d = w->size(0);
  shape_is(wrr, {dr, kr});
  shape_is(wr, {d, kr});
  shape_is(w, {d, k});
  const int32_t code = dtype_code(x);
  for (const Ten* t : {&x, &xr, &wrr, &wr, &w, &add}) same(*t, x);
  offsets(off, r);
  if (add) shape_is(add, x->sizes());
  bias_of(br, dr);
  need(!br || br->is_contiguous());
  bias_of(bias, d);
  const Ten yr = c.or_new(a[10], {r, dr}, x->scalar_type());
  const Ten out = c.or_new(a[11], {n, d}, x->scalar_type());
  const size_t bytes = rocs_ikbo_linear_workspace_size(r, n, d, kr);
  Ten ws = c.get(a[12]);
  if (!ws && bytes > 0) ws = c.or_new(Py_None, {(int64_t)bytes}, c10::kByte);
  void* s = stream_of(c.stream);
  run("rocs_glm_linear", rocs_glm_linear, xr.ptr(), kr, x.ptr(), add.ptr(), k, wrr.ptr(), wr.ptr(),
      w.ptr(), br.f32(), bias.f32(), off.i32(), r, n, dr, d, code, act, data(yr), data(out),
      data(ws), nbytes(ws), s);
  return pair(result(a[10], yr), result(a[11], out));
}

// x_cand, w1_cand, w2, x_req, w1_req, cand_offsets, b1, b2, activation1,
// activation2, out, workspace, stream
PyObject* mlp2(PyObject* const* a) {
  Call c(a[12]);
  const Ten x = c.must(a[0]), w1 = c.must(a[1]), w2 = c.must(a[2]), xr = c.get(a[3]),
            wr = c.get(a[4]), off = c.get(a[5]), b1 = c.get(a[6]), b2 = c.get(a[7]);
  const int32_t act1 = activation(a[8]), act2 = activation(a[9]);
  need(x->dim() == 2 && w1->dim() == 2 && w2->dim() == 2);
  const int64_t n = x->size(0), k = x->size(1), dh = w1->size(0), d = w2->size(0);
  need(w1->size(1) == k && w2->size(1) == dh);
  const int32_t code = dtype_code(x);
  for (const Ten* t : {&x, &w1, &w2, &xr, &wr}) same(*t, x);
  int64_t r = 0, kr = 0;
  if (xr) {
    need(wr && off && xr->dim() == 2);
    r = xr->size(0);
    kr = xr->size(1);
    shape_is(wr, {dh, kr});
    offsets(off, r);
  } else {
    need(!wr && !off);
  }
  bias_of(b1, dh);
  bias_of(b2, d);
  const Ten out = c.or_new(a[10], {n, d}, x->scalar_type());
  const size_t bytes = rocs_ikbo_mlp2_workspace_size(r, n, kr, k, dh, d, code);
  Ten ws = c.get(a[11]);
  if (!ws && bytes > 0) ws = c.or_new(Py_None, {(int64_t)bytes}, c10::kByte);
  void* s = stream_of(c.stream);
  run("rocs_ikbo_mlp2", rocs_ikbo_mlp2, xr.ptr(), kr, x.ptr(), k, wr.ptr(), w1.ptr(), b1.f32(),
      w2.ptr(), b2.f32(), off.i32(), r, n, dh, d, code, act1, act2, data(out), data(ws), nbytes(ws),
      s);
  return result(a[10], out);
}

// x_req, x_cand, cand_offsets, w_req, w_cand, bias, activation, out,
// workspace, stream
PyObject* fm_linear(PyObject* const* a) {
  Call c(a[9]);
  const Ten xr = c.must(a[0]), x = c.must(a[1]), off = c.must(a[2]), wr = c.must(a[3]),
            w = c.must(a[4]), bias = c.get(a[5]);
  const int32_t act = activation(a[6]);
  need(xr->dim() == 3 && x->dim() == 3 && xr->size(2) == x->size(2) && w->dim() == 2);
  const int64_t r = xr->size(0), fr = xr->size(1), e = xr->size(2), n = x->size(0),
                fc = x->size(1), d = w->size(0);
  offsets(off, r);
  shape_is(wr, {d, fr * fr});
  shape_is(w, {d, fc * (fr + fc)});
  need(fr <= INT32_MAX && fc <= INT32_MAX && e <= INT32_MAX);
  const int32_t code = dtype_code(x);
  for (const Ten* t : {&x, &xr, &wr, &w}) same(*t, x);
  bias_of(bias, d);
  const Ten out = c.or_new(a[7], {n, d}, x->scalar_type());
  const size_t bytes = rocs_glm_fm_linear_workspace_size(r, n, (int32_t)fr, (int32_t)fc,
                                                         (int32_t)e, d, code);
  Ten ws = c.get(a[8]);
  if (!ws && bytes > 0) ws = c.or_new(Py_None, {(int64_t)bytes}, c10::kByte);
  void* s = stream_of(c.stream);
  run("rocs_glm_fm_linear", rocs_glm_fm_linear, xr.ptr(), x.ptr(), off.i32(), r, n, (int32_t)fr,
      (int32_t)fc, (int32_t)e, wr.ptr(), w.ptr(), bias.f32(), d, code, act, data(out), data(ws),
      nbytes(ws), s);
  return result(a[7], out);
}

// x_req, x_cand, w_rr, w_cr, w_cc, index, mapped, y_req, y_cand, workspace,
// stream
PyObject* lcb(PyObject* const* a) {
  Call c(a[10]);
  const Ten xr = c.must(a[0]), x = c.must(a[1]), wrr = c.get(a[2]), wcr = c.must(a[3]),
            wcc = c.must(a[4]), index = c.must(a[5]);
  const bool mapped = a[6] == Py_True;
  need(xr->dim() == 3 && x->dim() == 3 && xr->size(2) == x->size(2) && wcc->dim() == 2);
  const int64_t r = xr->size(0), fr = xr->size(1), e = xr->size(2), n = x->size(0),
                fc = x->size(1), oc = wcc->size(0);
  shape_is(wcc, {oc, fc});
  shape_is(wcr, {oc, fr});
  int64_t orq = 0;
  if (wrr) {
    need(wrr->dim() == 2);
    orq = wrr->size(0);
    shape_is(wrr, {orq, fr});
  }
  need(orq > 0 || a[7] == Py_None);
  need(fr <= INT32_MAX && fc <= INT32_MAX && e <= INT32_MAX && oc <= INT32_MAX && orq <= INT32_MAX);
  const int32_t code = dtype_code(xr);
  for (const Ten* t : {&xr, &x, &wrr, &wcr, &wcc}) same(*t, xr);
  if (mapped) need(index->scalar_type() == c10::kInt && index->dim() == 1 &&
                   index->is_contiguous() && index->numel() == n);
  else offsets(index, r);
  Ten yr;
  if (orq > 0) yr = c.or_new(a[7], {r, orq, e}, xr->scalar_type());
  const Ten yc = c.or_new(a[8], {n, oc, e}, xr->scalar_type());
  const size_t bytes = rocs_ikbo_lcb_workspace_size(r, oc, e);
  Ten ws = c.get(a[9]);
  if (!ws) ws = c.or_new(Py_None, {(int64_t)(bytes > 0 ? bytes : 1)}, c10::kByte);
  void* s = stream_of(c.stream);
  if (mapped)
    run("rocs_ikbo_lcb_mapped", rocs_ikbo_lcb_mapped, xr.ptr(), x.ptr(), wrr.ptr(), wcr.ptr(),
        wcc.ptr(), index.i32(), r, n, (int32_t)fr, (int32_t)fc, (int32_t)orq, (int32_t)oc,
        (int32_t)e, code, data(yr), data(yc), data(ws), nbytes(ws), s);
  else
    run("rocs_ikbo_lcb", rocs_ikbo_lcb, xr.ptr(), x.ptr(), wrr.ptr(), wcr.ptr(), wcc.ptr(),
        index.i32(), r, n, (int32_t)fr, (int32_t)fc, (int32_t)orq, (int32_t)oc, (int32_t)e, code,
        data(yr), data(yc), data(ws), nbytes(ws), s);
  PyObject* first = Py_None;
  if (orq > 0) first = result(a[7], yr);
  else Py_INCREF(first);
  return pair(first, result(a[8], yc));
}

// cand_offsets, kv_offsets, num_cand, heads, q_len, plan, stream
PyObject* plan(PyObject* const* a) {
  Call c(a[6]);
  const Ten co = c.must(a[0]), ko = c.must(a[1]);
  const int64_t n = integer(a[2]), h = integer(a[3]), q = integer(a[4]);
  need(h >= 0 && h <= INT32_MAX && q >= 0 && q <= INT32_MAX);
  const int64_t r = ko->numel() - 1;
  offsets(ko, r);
  offsets(co, r);
  const int64_t bytes = (int64_t)rocs_dca_attention_plan_size(r);
  Ten p = c.get(a[5]);
  if (p) need(p->scalar_type() == c10::kByte && p->is_contiguous() && p->numel() >= bytes);
  else p = c.or_new(Py_None, {bytes}, c10::kByte);
  void* s = stream_of(c.stream);
  run("rocs_dca_attention_plan", rocs_dca_attention_plan, co.i32(), ko.i32(), r, n, (int32_t)q,
      (int32_t)h, data(p), nbytes(p), s);
  return result(a[5], p);
}

// q (or x), w_q, heads, k, v, cand_offsets, ids, kv_offsets, plan, residual,
// scale, out, out_sum, workspace, stream, ex (the extended entry point)
PyObject* attention(PyObject* const* a) {
  Call c(a[14]);
  const Ten q = c.must(a[0]), wq = c.get(a[1]), k = c.must(a[3]), v = c.must(a[4]),
            co = c.get(a[5]), ids = c.get(a[6]), ko = c.must(a[7]), pl = c.get(a[8]),
            res = c.get(a[9]);
  const float scale = scale_of(a[10]);
  int64_t n, t, h, d, d_in = 0;
  need(q->is_contiguous());
  if (wq) {
    need(q->dim() == 3 && wq->dim() == 2 && wq->is_contiguous() && !ids);
    h = integer(a[2]);
    n = q->size(0);
    t = q->size(1);
    d_in = q->size(2);
    need(h > 0 && wq->size(1) == d_in && wq->size(0) % h == 0 &&
         wq->scalar_type() == q->scalar_type());
    d = wq->size(0) / h;
  } else {
    need(q->dim() == 4);
    n = q->size(0);
    t = q->size(1);
    h = q->size(2);
    d = q->size(3);
  }
  const int32_t code = dtype_code(q);
  need(t <= INT32_MAX && h <= INT32_MAX && d <= INT32_MAX);
  need(k->dim() == 3 && v->dim() == 3 && k->sizes() == v->sizes() && k->size(1) == h &&
       k->size(2) == d);
  need(k->stride(2) == 1 && k->stride(1) == d && v->stride(2) == 1 && v->stride(1) == d &&
       k->stride(0) == v->stride(0));
  need(k->scalar_type() == q->scalar_type() && v->scalar_type() == q->scalar_type());
  const int64_t r = ko->numel() - 1;
  offsets(ko, r);
  if (ids) {
    need(!co && !pl && !res && ids->scalar_type() == c10::kInt && ids->dim() == 1 &&
         ids->is_contiguous() && ids->numel() == n);
  } else {
    need((bool)co);
    offsets(co, r);
  }
  if (pl) need(pl->scalar_type() == c10::kByte && pl->is_contiguous());
  const c10::IntArrayRef shape_q = q->sizes();
  const int64_t full[4] = {n, t, h, d};
  const c10::IntArrayRef shape = wq ? c10::IntArrayRef(full, 4) : shape_q;
  const Ten out = c.or_new(a[11], shape, q->scalar_type());
  Ten sum;
  if (res) {
    need(res->sizes() == shape && res->scalar_type() == q->scalar_type() && res->is_contiguous());
    sum = c.or_new(a[12], shape, q->scalar_type());
  }
  const int64_t stride = k->size(0) > 1 ? k->stride(0) : h * d;
  if (ids) {
    const size_t bytes = rocs_dca_attention_mapped_workspace_size(r, n);
    Ten ws = c.get(a[13]);
    if (!ws && bytes > 0) ws = c.or_new(Py_None, {(int64_t)bytes}, c10::kByte);
    void* s = stream_of(c.stream);
    run("rocs_dca_attention_mapped", rocs_dca_attention_mapped, q.ptr(), k.ptr(), v.ptr(),
        ids.i32(), ko.i32(), r, n, (int32_t)t, (int32_t)h, (int32_t)d, stride, scale, code,
        data(out), data(ws), nbytes(ws), s);
    return result(a[11], out);
  }
  void* s = stream_of(c.stream);
  if (a[15] != Py_True) {
    need(!wq && !pl);
    if (res)
      run("rocs_dca_attention_residual", rocs_dca_attention_residual, q.ptr(), k.ptr(), v.ptr(),
          co.i32(), ko.i32(), r, n, (int32_t)t, (int32_t)h, (int32_t)d, stride, scale, code,
          res.ptr(), data(out), data(sum), s);
    else
      run("rocs_dca_attention", rocs_dca_attention, q.ptr(), k.ptr(), v.ptr(), co.i32(), ko.i32(),
          r, n, (int32_t)t, (int32_t)h, (int32_t)d, stride, scale, code, data(out), s);
    return res ? pair(result(a[11], out), result(a[12], sum)) : result(a[11], out);
  }
  run("rocs_dca_attention_ex", rocs_dca_attention_ex, q.ptr(), d_in, wq.ptr(), k.ptr(), v.ptr(),
      co.i32(), ko.i32(), pl.ptr(), pl.bytes(), r, n, (int32_t)t, (int32_t)h, (int32_t)d, stride,
      scale, code, res.ptr(), data(out), data(sum), s);
  return res ? pair(result(a[11], out), result(a[12], sum)) : result(a[11], out);
}

#define ROCS_ENTRY(name, n) \
  {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(entry<n, name>)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    ROCS_ENTRY(linear, 12),   ROCS_ENTRY(glm_linear, 14), ROCS_ENTRY(mlp2, 13),
    ROCS_ENTRY(fm_linear, 10), ROCS_ENTRY(lcb, 11),        ROCS_ENTRY(plan, 7),
    ROCS_ENTRY(attention, 16), {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, g_methods,
                        nullptr, nullptr, nullptr, nullptr};

PyObject* attribute(const char* module, const char* name) {
  PyObject* m = PyImport_ImportModule(module);
  if (m == nullptr) return nullptr;
  PyObject* v = PyObject_GetAttrString(m, name);
  Py_DECREF(m);
  return v;
}

}  // namespace

PyMODINIT_FUNC PyInit__binding() {
  g_get_device = attribute("torch._C", "_cuda_getDevice");
  g_raw_stream = attribute("torch._C", "_cuda_getCurrentRawStream");
  g_check = attribute("paper_2607_27744_amd._lib", "check");
  g_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  if (!g_get_device || !g_raw_stream || !g_check || !g_cuda_stream) return nullptr;
  return PyModule_Create(&g_module);
}
