// Argument marshalling of the Python binding in native code: torch tensors, ctypes structures and streams to the pointers of the
// C-ABI.  A pass (dispatch and combine) of one token takes the GPU 5.5 us, two launches cost the host 4.7, and reading the arguments
// in Python took half as long again.  Host us per pass, by way of ctypes / here, with 2.3 us of the calling program's own: T = 1 9.85 /
// 8.8; quantised, T = 128 (the plan's structure is built in each call) 11.4 / 8.8; bound calls 8.95 / 8.05.
// Only the plain forms are read here: exact torch.Tensor (or None, or an address), the binding's own structures, the current
// stream.  For anything else a function returns None, and the binding takes its ctypes path, with that path's errors.
// The GIL is released during a call, as ctypes does.
#include <torch/csrc/autograd/python_variable.h>

#include "moe_rbf.h"

namespace {

struct Library {
  int (*plan)(const moe_shape *, const int32_t *, moe_plan_t *, void *);
  int (*plan_static)(const moe_shape *, const int32_t *, moe_plan_t *, void *);
  int (*dispatch)(const moe_shape *, const void *, const int32_t *, moe_plan_t *, void *, void *);
  int (*dispatch_quant)(const moe_shape *, const void *, const int32_t *, moe_plan_t *, void *, float *, void *);
  int (*combine)(const moe_shape *, const void *, const float *, const moe_plan_t *, void *, void *);
} lib;
PyObject *shape_type, *struct_type, *plan_type, *raise_error;      // set once by use()
PyObject *raw_stream, *current_device, *in_bad_fork;               // set by streams(), after the device is up

enum Got { kYes, kOther, kError };   // kOther: not a form that is read here; kError: a Python exception is set

Got address(PyObject *o, void **out) {
  if (o == Py_None) {
    *out = nullptr;
    return kYes;
  }
  if (PyLong_CheckExact(o)) {
    *out = (void *)(uintptr_t)PyLong_AsUnsignedLongLongMask(o);
    return PyErr_Occurred() ? kError : kYes;
  }
  if (!THPVariable_CheckExact(o)) return kOther;
  try {
    const at::Tensor &t = THPVariable_Unpack(o);
    if (t.layout() != at::kStrided) return kOther;
    if (!t.is_contiguous()) {
      PyErr_SetString(PyExc_AssertionError, "tensors must be dense row-major");
      return kError;
    }
    *out = t.data_ptr();
    return kYes;
  } catch (...) {
    return kOther;                   // the ctypes path reports it
  }
}

// The memory of a ctypes structure of exactly this type.  It stays where it is as long as the object lives.
Got structure(PyObject *o, PyObject *type, size_t bytes, void **out) {
  if ((PyObject *)Py_TYPE(o) != type) return kOther;
  Py_buffer view;
  if (PyObject_GetBuffer(o, &view, PyBUF_WRITABLE) != 0) return kError;
  *out = view.buf;
  const bool whole = (size_t)view.len == bytes;
  PyBuffer_Release(&view);
  return whole ? kYes : kOther;
}

// A moe_plan_t from the tensors that a MoePlan holds at the moment.
Got plan_of(PyObject *o, moe_plan_t *p) {
  static const char *const names[] = {"expert_count", "rank_count", "expert_offset", "region_base", "send_idx", "row_map", "status",
                                      "workspace", "source_count", "recv_count", "recv_offset", "dispatch_order", "prefetch"};
  constexpr int kNames = sizeof(names) / sizeof(names[0]);
  void *const into[kNames] = {&p->expert_count, &p->rank_count, &p->expert_offset, &p->region_base, &p->send_idx, &p->row_map,
                              &p->status, &p->workspace, &p->source_count, &p->recv_count, &p->recv_offset, &p->dispatch_order,
                              &p->prefetch};
  static PyObject *keys[kNames];
  p->prefetch_bytes = 0;
  for (int i = 0; i < kNames; ++i) {
    if (!keys[i] && !(keys[i] = PyUnicode_InternFromString(names[i]))) return kError;
    PyObject *t = PyObject_GetAttr(o, keys[i]);
    if (!t) {
      PyErr_Clear();
      return kOther;
    }
    Got got = address(t, (void **)into[i]);
    const bool sized = into[i] == &p->workspace || into[i] == &p->prefetch;
    if (got == kYes && sized && t != Py_None) {
      if (!THPVariable_CheckExact(t)) {
        got = kOther;
      } else {
        const at::Tensor &v = THPVariable_Unpack(t);
        if (into[i] == &p->workspace) p->workspace_bytes = (size_t)v.numel();
        else p->prefetch_bytes = (size_t)v.numel() * v.element_size();
      }
    } else if (got == kYes && into[i] == &p->workspace) {
      got = kOther;
    }
    Py_DECREF(t);
    if (got != kYes) return got;
  }
  return kYes;
}

Got any_plan(PyObject *o, moe_plan_t *room, moe_plan_t **out) {
  if ((PyObject *)Py_TYPE(o) == plan_type) {
    *out = room;
    return plan_of(o, room);
  }
  return structure(o, struct_type, sizeof(moe_plan_t), (void **)out);
}

Got stream_of(PyObject *o, void **out) {
  if (PyLong_CheckExact(o)) return address(o, out);
  if (o != Py_None || !raw_stream) return kOther;
  PyObject *bad = PyObject_CallNoArgs(in_bad_fork);
  if (!bad) return kError;
  const bool forked = bad != Py_False;
  Py_DECREF(bad);
  if (forked) return kOther;
  PyObject *device = PyObject_CallNoArgs(current_device);
  if (!device) return kError;
  PyObject *handle = PyObject_CallOneArg(raw_stream, device);
  Py_DECREF(device);
  if (!handle) return kError;
  const Got got = PyLong_CheckExact(handle) ? address(handle, out) : kOther;
  Py_DECREF(handle);
  return got;
}

#define TRY(call)                    \
  switch (call) {                    \
    case kYes: break;                \
    case kOther: Py_RETURN_NONE;     \
    case kError: return nullptr;     \
  }

// Arguments: shape, `inputs` addresses, plan, `outputs` addresses, stream.
struct Args {
  moe_shape *shape;
  void *in[2], *out[2], *stream;
  moe_plan_t *plan, room;
};
Got read(Args *a, PyObject *const *o, Py_ssize_t n, int inputs, int outputs) {
  if (n != 3 + inputs + outputs || !lib.plan) return kOther;
  Got got = structure(o[0], shape_type, sizeof(moe_shape), (void **)&a->shape);
  for (int i = 0; got == kYes && i < inputs; ++i) got = address(o[1 + i], &a->in[i]);
  if (got == kYes) got = any_plan(o[1 + inputs], &a->room, &a->plan);
  for (int i = 0; got == kYes && i < outputs; ++i) got = address(o[2 + inputs + i], &a->out[i]);
  return got == kYes ? stream_of(o[n - 1], &a->stream) : got;
}

template <typename F>
PyObject *without_gil(F &&call) {
  int code;
  Py_BEGIN_ALLOW_THREADS
  code = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(code);
}

PyObject *plan(PyObject *, PyObject *const *o, Py_ssize_t n) {
  Args a;
  TRY(read(&a, o, n, 1, 0))
  return without_gil([&] { return lib.plan(a.shape, (const int32_t *)a.in[0], a.plan, a.stream); });
}
PyObject *plan_static(PyObject *, PyObject *const *o, Py_ssize_t n) {
  Args a;
  TRY(read(&a, o, n, 1, 0))
  return without_gil([&] { return lib.plan_static(a.shape, (const int32_t *)a.in[0], a.plan, a.stream); });
}
PyObject *dispatch(PyObject *, PyObject *const *o, Py_ssize_t n) {
  Args a;
  TRY(read(&a, o, n, 2, 1))
  return without_gil([&] { return lib.dispatch(a.shape, a.in[0], (const int32_t *)a.in[1], a.plan, a.out[0], a.stream); });
}
PyObject *dispatch_quant(PyObject *, PyObject *const *o, Py_ssize_t n) {
  Args a;
  TRY(read(&a, o, n, 2, 2))
  return without_gil([&] {
    return lib.dispatch_quant(a.shape, a.in[0], (const int32_t *)a.in[1], a.plan, a.out[0], (float *)a.out[1], a.stream);
  });
}
PyObject *combine(PyObject *, PyObject *const *o, Py_ssize_t n) {
  Args a;
  TRY(read(&a, o, n, 2, 1))
  return without_gil([&] { return lib.combine(a.shape, a.in[0], (const float *)a.in[1], a.plan, a.out[0], a.stream); });
}

// A layer's calls on fixed buffers.  The structures are read at every call; they and `buffers`, which owns the memory, are kept alive.
struct Bound {
  PyObject_HEAD
  PyObject *shape, *plan, *buffers;
  const moe_shape *sh;
  moe_plan_t *pl;
  void *x, *ids, *weights, *window, *expert_out, *y, *stream;
  int prefill;
};
void bound_free(PyObject *o) {
  Bound *b = (Bound *)o;
  Py_XDECREF(b->shape);
  Py_XDECREF(b->plan);
  Py_XDECREF(b->buffers);
  Py_TYPE(o)->tp_free(o);
}
PyObject *failed(int code, const char *where) { return PyObject_CallFunction(raise_error, "is", code, where); }

PyObject *bound_dispatch(PyObject *o, PyObject *) {
  const Bound *b = (const Bound *)o;
  int planned = MOE_OK, code = MOE_OK;
  Py_BEGIN_ALLOW_THREADS
  if (b->prefill) planned = lib.plan(b->sh, (const int32_t *)b->ids, b->pl, b->stream);
  if (planned == MOE_OK) code = lib.dispatch(b->sh, b->x, (const int32_t *)b->ids, b->pl, b->window, b->stream);
  Py_END_ALLOW_THREADS
  if (planned != MOE_OK) return failed(planned, "moe_plan");
  if (code != MOE_OK) return failed(code, "moe_dispatch");
  Py_RETURN_NONE;
}
PyObject *bound_combine(PyObject *o, PyObject *) {
  const Bound *b = (const Bound *)o;
  int code;
  Py_BEGIN_ALLOW_THREADS
  code = lib.combine(b->sh, b->expert_out, (const float *)b->weights, b->pl, b->y, b->stream);
  Py_END_ALLOW_THREADS
  if (code != MOE_OK) return failed(code, "moe_combine");
  Py_RETURN_NONE;
}
PyMethodDef bound_methods[] = {{"dispatch", bound_dispatch, METH_NOARGS, "plan (prefill schedule) and dispatch"},
                               {"combine", bound_combine, METH_NOARGS, "combine"},
                               {nullptr, nullptr, 0, nullptr}};
PyTypeObject bound_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

// bind(shape, plan struct, prefill, x, ids, weights, window, expert_out, y, stream, buffers): an object with dispatch() and combine()
PyObject *bind(PyObject *, PyObject *const *o, Py_ssize_t n) {
  if (n != 11 || !lib.plan) Py_RETURN_NONE;
  void *sh, *pl, *at[7];
  TRY(structure(o[0], shape_type, sizeof(moe_shape), &sh))
  TRY(structure(o[1], struct_type, sizeof(moe_plan_t), &pl))
  const int prefill = PyObject_IsTrue(o[2]);
  if (prefill < 0) return nullptr;
  for (int i = 0; i < 7; ++i) TRY(address(o[3 + i], &at[i]))
  Bound *b = (Bound *)bound_type.tp_alloc(&bound_type, 0);
  if (!b) return nullptr;
  Py_INCREF(o[0]);
  Py_INCREF(o[1]);
  Py_INCREF(o[10]);
  b->shape = o[0], b->plan = o[1], b->buffers = o[10], b->sh = (const moe_shape *)sh, b->pl = (moe_plan_t *)pl, b->prefill = prefill;
  b->x = at[0], b->ids = at[1], b->weights = at[2], b->window = at[3], b->expert_out = at[4], b->y = at[5], b->stream = at[6];
  return (PyObject *)b;
}

void keep(PyObject **slot, PyObject *o) {
  Py_INCREF(o);
  PyObject *old = *slot;
  *slot = o;
  Py_XDECREF(old);
}

// use(addresses of the five entry points, MoeShape, _PlanStruct, MoePlan, raise_error)
PyObject *use(PyObject *, PyObject *args) {
  unsigned long long f[5];
  PyObject *types[4];
  if (!PyArg_ParseTuple(args, "KKKKKOOOO", &f[0], &f[1], &f[2], &f[3], &f[4], &types[0], &types[1], &types[2], &types[3]))
    return nullptr;
  keep(&shape_type, types[0]);
  keep(&struct_type, types[1]);
  keep(&plan_type, types[2]);
  keep(&raise_error, types[3]);
  lib.plan_static = (decltype(lib.plan_static))(uintptr_t)f[1];
  lib.dispatch = (decltype(lib.dispatch))(uintptr_t)f[2];
  lib.dispatch_quant = (decltype(lib.dispatch_quant))(uintptr_t)f[3];
  lib.combine = (decltype(lib.combine))(uintptr_t)f[4];
  lib.plan = (decltype(lib.plan))(uintptr_t)f[0];
  Py_RETURN_NONE;
}

// streams(raw stream of a device, current device, in a forked child): torch's own functions
PyObject *streams(PyObject *, PyObject *args) {
  PyObject *f[3];
  if (!PyArg_ParseTuple(args, "OOO", &f[0], &f[1], &f[2])) return nullptr;
  keep(&current_device, f[1]);
  keep(&in_bad_fork, f[2]);
  keep(&raw_stream, f[0]);
  Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(plan), FAST(plan_static), FAST(dispatch), FAST(dispatch_quant), FAST(combine), FAST(bind),
                         {"use", use, METH_VARARGS, nullptr}, {"streams", streams, METH_VARARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", "native argument marshalling", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
  bound_type.tp_name = "paper_2605_06055_amd._marshal.Bound";
  bound_type.tp_basicsize = sizeof(Bound);
  bound_type.tp_flags = Py_TPFLAGS_DEFAULT;
  bound_type.tp_dealloc = bound_free;
  bound_type.tp_methods = bound_methods;
  if (PyType_Ready(&bound_type) < 0) return nullptr;
  PyObject *m = PyModule_Create(&module);
  // the torch and the Python whose objects are read here: the binding leaves the module aside where it finds others
  if (m && PyModule_AddStringConstant(m, "built_for", MOE_BUILT_FOR) < 0) Py_CLEAR(m);
  return m;
}
