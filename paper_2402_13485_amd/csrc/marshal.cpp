// Argument marshalling of the Python binding in native code (host code only): checks of the tensors,
// output tensors and the call of the C entry point, for the calls that a decoding loop makes once
// or several times per step.  Their kernels take 5 to 15 us on small inputs, the same work in Python
// 5 to 20 us per call: a whole step of 1 sequence, 1 head, fp32 took 98 us, most of it here.
//
// Nothing is decided here that binding.py does not say: a function returns None, with nothing enqueued,
// whenever an argument is not what the entry point wants, and binding.py then goes through its own
// checks, which name the argument.  Tensors of other classes than torch.Tensor and Parameter are left to it
// too.  What can fail stands in front of the C call, the Python objects of its results among it: a call
// that has been enqueued returns them and is never made again.  A call that the library refuses returns its
// status.  The interpreter is left to other threads during allocations and the C call, as torch and ctypes
// do.  No state is kept but the addresses of the entry points.
#include <ATen/ATen.h>
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <memory>
#include <vector>

#include "../../include/propd.h"

namespace {

struct Entries {
  decltype(&propd_tree_mask) tree_mask = nullptr;
  decltype(&propd_tree_attention) tree_attention = nullptr;
  decltype(&propd_early_prune) early_prune = nullptr;
  decltype(&propd_early_prune_prob) early_prune_prob = nullptr;
  decltype(&propd_accept_path) accept_path = nullptr;
  decltype(&propd_commit_path) commit_path = nullptr;
  decltype(&propd_workspace_bytes) workspace_bytes = nullptr;
};

struct NotThis {};  // the Python code takes over
struct Raised {};   // a Python error is set
struct Refused {
  propd_status status;
};

const at::Tensor &tensor(PyObject *o) {
  if (!THPVariable_CheckExact(o)) throw NotThis{};
  return THPVariable_Unpack(o);
}

void need(bool ok) {
  if (!ok) throw NotThis{};
}

// Other threads may run Python meanwhile: a launch waits where the queue is full, an allocation where memory has to be
// given back first, and what they wait for may need the interpreter.
struct Unlocked {
  PyThreadState *const state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};

template <class F>
auto unlocked(F &&f) {
  const Unlocked u;
  return f();
}

template <class Entry, class... Args>
void call(Entry entry, Args... args) {
  const propd_status status = unlocked([&] { return entry(args...); });
  if (status != PROPD_OK) throw Refused{status};
}

// a contiguous tensor of this type in GPU memory
const at::Tensor &dev(PyObject *o, at::ScalarType type) {
  const at::Tensor &t = tensor(o);
  need(t.is_cuda() && t.scalar_type() == type && t.is_contiguous());
  return t;
}

propd_dtype type_of(const at::Tensor &t) {
  if (t.scalar_type() == at::kBFloat16) return PROPD_BF16;
  need(t.scalar_type() == at::kFloat);
  return PROPD_F32;
}

void *ptr(PyObject *o) { return o == Py_None ? nullptr : tensor(o).data_ptr(); }

long long whole(PyObject *o) {
  need(PyLong_Check(o));
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) {
    PyErr_Clear();
    throw NotThis{};
  }
  return v;
}

int32_t whole32(PyObject *o) {
  const long long v = whole(o);
  need(v >= INT32_MIN && v <= INT32_MAX);
  return (int32_t)v;
}

int32_t size32(int64_t n) {
  need(n <= INT32_MAX);
  return (int32_t)n;
}

float real(PyObject *o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) {
    PyErr_Clear();
    throw NotThis{};
  }
  return (float)v;
}

bool truth(PyObject *o) {
  const int t = PyObject_IsTrue(o);
  if (t < 0) throw Raised{};
  return t == 1;
}

// binding._stream, called once the arguments have passed
void *stream_of(PyObject *current) {
  PyObject *o = PyObject_CallNoArgs(current);
  void *p = o ? PyLong_AsVoidPtr(o) : nullptr;
  Py_XDECREF(o);
  if (PyErr_Occurred()) throw Raised{};
  return p;
}

// the fields of binding.Tree: n_nodes, parent, token, depth, anc
propd_tree tree_of(PyObject *const *f) {
  const at::Tensor &parent = tensor(f[1]);
  need(parent.dim() >= 2);
  propd_tree t;
  t.B = size32(parent.size(0));
  t.T_max = size32(parent.size(1));
  t.n_nodes = (const int32_t *)ptr(f[0]);
  t.parent = (const int32_t *)parent.data_ptr();
  t.token = (const int32_t *)ptr(f[2]);
  t.depth = (const int32_t *)ptr(f[3]);
  t.anc = (const uint64_t *)ptr(f[4]);
  return t;
}

struct Workspace {
  at::Tensor own;
  void *ptr;
  size_t bytes;
};

Workspace workspace(PyObject *o, size_t need_bytes, const at::Tensor &like) {
  Workspace w;
  if (o != Py_None) {
    const at::Tensor &t = tensor(o);
    w.bytes = t.nbytes();
    need(w.bytes >= need_bytes && t.numel() * t.element_size() == (int64_t)w.bytes);
    w.ptr = t.data_ptr();
  } else {
    w.own = unlocked([&] { return at::empty({(int64_t)(need_bytes > 256 ? need_bytes : 256)}, like.options().dtype(at::kByte)); });
    w.ptr = w.own.data_ptr();
    w.bytes = (size_t)w.own.numel();
  }
  return w;
}

struct Release {
  void operator()(PyObject *o) const { Py_DECREF(o); }
};
using Owned = std::unique_ptr<PyObject, Release>;

Owned owned(PyObject *o) {
  if (!o) throw Raised{};
  return Owned(o);
}

Owned object(const at::Tensor &t) {
  if (t.defined()) return owned(THPVariable_Wrap(t));
  Py_INCREF(Py_None);
  return Owned(Py_None);
}

Owned object(PyObject *o) {
  Py_INCREF(o);
  return Owned(o);
}

template <class... Items>
Owned tuple_of(Items... items) {
  Owned r = owned(PyTuple_New((Py_ssize_t)sizeof...(items)));
  Py_ssize_t n = 0;
  (PyTuple_SET_ITEM(r.get(), n++, items.release()), ...);
  return r;
}

Entries entries;

template <class F>
PyObject *guarded(F &&f) {
  try {
    return f().release();
  } catch (const NotThis &) {
  } catch (const Raised &) {
    return nullptr;
  } catch (const Refused &r) {
    return PyLong_FromLong((long)r.status);
  } catch (const std::exception &e) {  // for instance out of memory: the Python code meets the same and says so
    PyErr_Clear();
  }
  Py_RETURN_NONE;
}

template <class E>
void take(PyObject *o, E &entry) {
  entry = reinterpret_cast<E>(PyLong_AsVoidPtr(o));
}

PyObject *py_init(PyObject *, PyObject *const *a, Py_ssize_t n) {
  if (n != 7) {
    PyErr_SetString(PyExc_TypeError, "init: seven addresses");
    return nullptr;
  }
  take(a[0], entries.tree_mask);
  take(a[1], entries.tree_attention);
  take(a[2], entries.early_prune);
  take(a[3], entries.early_prune_prob);
  take(a[4], entries.accept_path);
  take(a[5], entries.commit_path);
  take(a[6], entries.workspace_bytes);
  if (PyErr_Occurred()) return nullptr;
  Py_RETURN_NONE;
}

// tree_mask(n_nodes, parent, stream) -> (depth, anc)
PyObject *py_tree_mask(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded([&]() -> Owned {
    need(n == 3);
    const at::Tensor &nodes = dev(a[0], at::kInt), &parent = dev(a[1], at::kInt);
    need(parent.dim() == 2);
    const int64_t B = parent.size(0), T = parent.size(1);
    at::Tensor depth, anc;
    {
      const Unlocked u;
      depth = at::empty({B, T}, parent.options());
      anc = at::empty({B, T, 2}, parent.options().dtype(at::kLong));
    }
    Owned result = tuple_of(object(depth), object(anc));
    call(entries.tree_mask, size32(B), size32(T), (const int32_t *)nodes.data_ptr(), (const int32_t *)parent.data_ptr(),
         (int32_t *)depth.data_ptr(), (uint64_t *)anc.data_ptr(), stream_of(a[2]));
    return result;
  });
}

// tree_attention(*tree, q, k_cache, v_cache, k_tree, v_tree, seq_lens, scale, out, workspace, stream) -> out
PyObject *py_tree_attention(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded([&]() -> Owned {
    need(n == 15);
    const propd_tree tree = tree_of(a);
    const at::Tensor &q = tensor(a[5]);
    const propd_dtype dt = type_of(q);
    need(q.dim() == 4);
    const int64_t B = q.size(0), H = q.size(1), T = q.size(2), d = q.size(3);
    const at::Tensor &kc = dev(a[6], q.scalar_type()), &vc = dev(a[7], q.scalar_type());
    const at::Tensor &kt = dev(a[8], q.scalar_type()), &vt = dev(a[9], q.scalar_type()), &seq = dev(a[10], at::kInt);
    need(q.is_cuda() && q.is_contiguous() && kc.dim() == 4);
    const int64_t L = kc.size(2);
    need(kc.sizes() == at::IntArrayRef({B, H, L, d}) && vc.sizes() == kc.sizes() && kt.sizes() == q.sizes() && vt.sizes() == q.sizes());
    need(tree.B == B && tree.T_max == T);
    const at::Tensor out = a[12] == Py_None ? unlocked([&] { return at::empty_like(q); }) : tensor(a[12]);
    const Workspace w = workspace(a[13], entries.workspace_bytes(PROPD_WS_TREE_ATTENTION, tree.B, tree.T_max, size32(H), size32(d),
                                                                 size32(L), 0, 0), q);
    Owned result = a[12] != Py_None ? object(a[12]) : object(out);
    call(entries.tree_attention, &tree, dt, size32(H), size32(d), real(a[11]), q.data_ptr(), L ? kc.data_ptr() : nullptr,
         L ? vc.data_ptr() : nullptr, kt.data_ptr(), vt.data_ptr(), (const int32_t *)seq.data_ptr(),
         size32(L), out.data_ptr(), w.ptr, w.bytes, stream_of(a[14]));
    return result;
  });
}

// early_prune(*tree, hidden, head, mode, value, payloads, payload_out, want_extra, workspace, stream) -> (keep_bits, new_index, orig_index,
// n_kept, cu_nodes, n_nodes, parent, token, depth, anc, rank or log_marginal or None, [payloads]); mode -1: top-k, else propd_prob_mode
PyObject *py_early_prune(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded([&]() -> Owned {
    need(n == 14);
    const propd_tree tree = tree_of(a);
    const at::Tensor &hid = tensor(a[5]);
    const propd_dtype dt = type_of(hid);
    need(hid.dim() == 3 && hid.is_cuda() && hid.is_contiguous());
    const at::Tensor &head = dev(a[6], hid.scalar_type());
    const int64_t B = hid.size(0), T = hid.size(1), hidden = hid.size(2);
    need(head.dim() == 2 && head.size(1) == hidden && tree.B == B && tree.T_max == T);
    const int64_t vocab = head.size(0);
    const long long mode = whole(a[7]);
    const bool top_k = mode < 0, extra = truth(a[11]);
    const int32_t count = top_k || mode == PROPD_PROB_RANK ? whole32(a[8]) : 0;
    const float threshold = mode == PROPD_PROB_THRESHOLD ? real(a[8]) : 0.f;
    need(PyList_Check(a[9]) || PyTuple_Check(a[9]));
    const Py_ssize_t n_pay = PySequence_Fast_GET_SIZE(a[9]);
    const bool given = a[10] != Py_None;
    need(n_pay <= PROPD_MAX_PAYLOADS);
    need(!given || ((PyList_Check(a[10]) || PyTuple_Check(a[10])) && PySequence_Fast_GET_SIZE(a[10]) >= n_pay));
    // held here: the lists are not looked at again, other threads may change them
    at::Tensor src[PROPD_MAX_PAYLOADS], dst[PROPD_MAX_PAYLOADS];
    Owned dst_object[PROPD_MAX_PAYLOADS];
    for (Py_ssize_t i = 0; i < n_pay; ++i) {
      src[i] = tensor(PySequence_Fast_GET_ITEM(a[9], i));
      need(src[i].is_cuda() && src[i].is_contiguous() && (src[i].dim() == 3 || src[i].dim() == 4));
      need(src[i].size(0) == B && src[i].size(-2) == T);
      if (!given) continue;
      PyObject *const o = PySequence_Fast_GET_ITEM(a[10], i);
      dst[i] = tensor(o);
      need(dst[i].sizes() == src[i].sizes() && dst[i].scalar_type() == src[i].scalar_type() && dst[i].is_contiguous());
      dst_object[i] = object(o);
    }
    // per-node and per-sequence outputs in one allocation each, every one of them on a multiple of 16 bytes
    const bool rank = top_k && extra;
    std::vector<at::Tensor> nodes, counts;
    at::Tensor keep, cu, anc, more;
    {
      const Unlocked u;
      const auto i32 = hid.options().dtype(at::kInt), i64 = hid.options().dtype(at::kLong);
      nodes = at::empty_strided({rank ? 6 : 5, B, T}, {(B * T + 3) / 4 * 4, T, 1}, i32).unbind(0);
      counts = at::empty_strided({2, B}, {(B + 3) / 4 * 4, 1}, i32).unbind(0);
      keep = at::empty({B, 2}, i64);
      cu = at::empty({B + 1}, i32);
      anc = at::empty({B, T, 2}, i64);
      if (rank) more = nodes[5];
      if (!top_k && extra) more = at::empty({B, T}, hid.options().dtype(at::kFloat));
      for (Py_ssize_t i = 0; i < n_pay && !given; ++i) dst[i] = at::empty_like(src[i]);
    }
    propd_payload pay[PROPD_MAX_PAYLOADS];
    for (Py_ssize_t i = 0; i < n_pay; ++i) {
      const int64_t outer = src[i].dim() == 3 ? 1 : src[i].size(1), row = src[i].size(-1) * src[i].element_size();
      pay[i] = propd_payload{src[i].data_ptr(), dst[i].data_ptr(), (size_t)row, outer, outer * T * row, T * row, row};
      if (!given) dst_object[i] = object(dst[i]);
    }
    int32_t *node[5];
    for (int i = 0; i < 5; ++i) node[i] = (int32_t *)nodes[i].data_ptr();
    propd_tree_out out;
    out.n_nodes = (int32_t *)counts[1].data_ptr();
    out.parent = node[2];
    out.token = node[3];
    out.depth = node[4];
    out.anc = (uint64_t *)anc.data_ptr();
    const Workspace w = workspace(a[12], entries.workspace_bytes(PROPD_WS_EARLY_PRUNE, tree.B, tree.T_max, 0, 0, 0, size32(hidden),
                                                                 size32(vocab)), hid);
    uint64_t *keep_p = (uint64_t *)keep.data_ptr();
    int32_t *kept_p = (int32_t *)counts[0].data_ptr(), *cu_p = (int32_t *)cu.data_ptr();
    Owned moved = owned(PyList_New(n_pay));
    for (Py_ssize_t i = 0; i < n_pay; ++i) PyList_SET_ITEM(moved.get(), i, dst_object[i].release());
    Owned result = tuple_of(object(keep), object(nodes[0]), object(nodes[1]), object(counts[0]), object(cu), object(counts[1]),
                            object(nodes[2]), object(nodes[3]), object(nodes[4]), object(anc), object(more), std::move(moved));
    void *st = stream_of(a[13]);
    if (top_k)
      call(entries.early_prune, &tree, dt, size32(hidden), size32(vocab), count, hid.data_ptr(), head.data_ptr(), keep_p, node[0], node[1],
           kept_p, cu_p, &out, rank ? (int32_t *)more.data_ptr() : nullptr, (int32_t)n_pay, pay, w.ptr, w.bytes, st);
    else
      call(entries.early_prune_prob, &tree, dt, size32(hidden), size32(vocab), (propd_prob_mode)mode, threshold, count, hid.data_ptr(),
           head.data_ptr(), keep_p, node[0], node[1], kept_p, cu_p, &out, more.defined() ? (float *)more.data_ptr() : nullptr,
           (int32_t)n_pay, pay, w.ptr, w.bytes, st);
    return result;
  });
}

// accept_path(*tree, logits, path_stride or None, workspace, stream) -> (accept_len, path, next_token)
PyObject *py_accept_path(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded([&]() -> Owned {
    need(n == 9);
    const propd_tree tree = tree_of(a);
    const at::Tensor &logits = tensor(a[5]);
    const propd_dtype dt = type_of(logits);
    need(logits.dim() == 3 && logits.is_cuda() && logits.is_contiguous() && tree.B == logits.size(0) && tree.T_max == logits.size(1));
    const int32_t vocab = size32(logits.size(2)), stride = a[6] == Py_None ? tree.T_max : whole32(a[6]);
    need(stride >= 0);
    at::Tensor len, path, next;
    {
      const Unlocked u;
      const auto i32 = logits.options().dtype(at::kInt);
      len = at::empty({tree.B}, i32);
      path = at::empty({tree.B, stride}, i32);
      next = at::empty({tree.B}, i32);
    }
    const Workspace w = workspace(a[7], entries.workspace_bytes(PROPD_WS_ACCEPT_PATH, tree.B, tree.T_max, 0, 0, 0, 0, vocab), logits);
    Owned result = tuple_of(object(len), object(path), object(next));
    call(entries.accept_path, &tree, dt, vocab, logits.data_ptr(), (int32_t *)len.data_ptr(), (int32_t *)path.data_ptr(), stride,
         (int32_t *)next.data_ptr(), w.ptr, w.bytes, stream_of(a[8]));
    return result;
  });
}

// commit_path(*tree, accept_len, path, next_token, k_tree, v_tree, k_cache, v_cache, seq_lens, out_stride or None, stream) -> tokens
PyObject *py_commit_path(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded([&]() -> Owned {
    need(n == 15);
    const propd_tree tree = tree_of(a);
    const at::Tensor &len = dev(a[5], at::kInt), &path = dev(a[6], at::kInt), &next = dev(a[7], at::kInt), &seq = dev(a[12], at::kInt);
    const at::Tensor &kt = tensor(a[8]);
    const propd_dtype dt = type_of(kt);
    need(kt.dim() == 4 && kt.is_cuda() && kt.is_contiguous() && path.dim() >= 2);
    const at::Tensor &vt = dev(a[9], kt.scalar_type()), &kc = dev(a[10], kt.scalar_type()), &vc = dev(a[11], kt.scalar_type());
    const int64_t B = kt.size(0), H = kt.size(1), T = kt.size(2), d = kt.size(3);
    need(kc.dim() == 4);
    const int64_t L = kc.size(2);
    need(vt.sizes() == kt.sizes() && kc.sizes() == at::IntArrayRef({B, H, L, d}) && vc.sizes() == kc.sizes() && tree.B == B && tree.T_max == T);
    const int32_t stride = size32(path.size(1)), out_stride = a[13] == Py_None ? stride : whole32(a[13]);
    need(out_stride >= 0);
    const at::Tensor out = unlocked([&] { return at::empty({B, out_stride}, kt.options().dtype(at::kInt)); });
    Owned result = object(out);
    call(entries.commit_path, &tree, dt, size32(H), size32(d), (const int32_t *)len.data_ptr(), (const int32_t *)path.data_ptr(), stride,
         (const int32_t *)next.data_ptr(), kt.data_ptr(), vt.data_ptr(), kc.data_ptr(), vc.data_ptr(), size32(L),
         (int32_t *)seq.data_ptr(), (int32_t *)out.data_ptr(), out_stride, stream_of(a[14]));
    return result;
  });
}

#define METHOD(name) {#name, (PyCFunction)(void (*)(void))py_##name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(init),        METHOD(tree_mask),   METHOD(tree_attention), METHOD(early_prune),
                         METHOD(accept_path), METHOD(commit_path), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject *PyInit__marshal() { return PyModule_Create(&module); }
