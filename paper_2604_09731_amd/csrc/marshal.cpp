// The binding's calls in native code: output allocation, argument marshalling and the library call of the device entry
// points, for binding.py.  A small call waits for the host, not for the GPU (a draft layer's kernel takes 4.8 us, the call took
// 7.5 us of host time, of which the launch is 3.3): each output tensor made and each address passed from Python costs 0.1 ..
// 1.4 us there.  No arithmetic and no checks beyond those the Python side made; the entry points come as addresses, so that
// this module works with whichever build of the library the binding loaded.
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/autograd/python_variable.h>

#include <vector>

#include "smart_tree.h"

namespace {

// In the order of binding.py's _NATIVE_ENTRIES.
struct Entries {
  decltype(&smart_select_begin_device) begin;
  decltype(&smart_select_layer_device) layer;
  decltype(&tree_compact_pack_fill) compact;
  decltype(&tree_upload_pack) upload_pack;
  decltype(&tree_rope) rope;
  decltype(&kv_cache_write) cache_write;
  decltype(&kv_cache_write_fp8) cache_write_fp8;
  decltype(&tree_verify_attention) attention;
  decltype(&tree_verify_attention_static) attention_static;
  decltype(&tree_accept) accept;
  decltype(&tree_accept_sample) sample;
  decltype(&tree_commit) commit;
  decltype(&tree_commit_fp8) commit_fp8;
} lib;
PyObject *check_call, *get_device, *raw_stream;

struct Failed {};  // a Python exception is set

PyObject* must(PyObject* x) {
  if (!x) throw Failed();
  return x;
}
const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_TypeError, "expected a tensor, got %s", Py_TYPE(o)->tp_name);
    throw Failed();
  }
  return THPVariable_Unpack(o);
}
template <typename T = void>
T* address(const at::Tensor& t) {
  return (T*)t.data_ptr();
}
template <typename T = void>
T* address(PyObject* o) {  // None: NULL
  return o == Py_None ? nullptr : (T*)tensor(o).data_ptr();
}
uint64_t low_bits(PyObject* n) {  // of an int, whose reference it takes
  const unsigned long long v = PyLong_AsUnsignedLongLongMask(must(n));
  Py_DECREF(n);
  if (v == (unsigned long long)-1 && PyErr_Occurred()) throw Failed();
  return v;
}
uint64_t bits64(PyObject* o) { return low_bits(PyNumber_Long(o)); }  // what int(o) gives, modulo 2^64
// An integer; anything else, a float of a whole value among them, is refused as ctypes refuses it.
int64_t integer(PyObject* o) { return (int64_t)low_bits(PyNumber_Index(o)); }
bool truth(PyObject* o) {
  const int v = PyObject_IsTrue(o);
  if (v < 0) throw Failed();
  return v != 0;
}
double real(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw Failed();
  return v;
}
template <typename T>
T* pointer(PyObject* o) {
  return (T*)(uintptr_t)integer(o);
}
void at_least(const at::Tensor& t, int64_t dims) {
  if (t.dim() >= dims) return;
  PyErr_SetString(PyExc_IndexError, "tensor has too few dimensions");
  throw Failed();
}
int64_t extent(const at::Tensor& t, int64_t dim) {
  at_least(t, dim + 1);
  return t.size(dim);
}
void three_dims(const at::Tensor& t) {
  if (t.dim() != 3) {
    PyErr_Format(PyExc_ValueError, "expected 3 dimensions, got %d", (int)t.dim());
    throw Failed();
  }
}
int32_t element_type(const at::Tensor& t) {
  if (t.scalar_type() == at::kFloat) return SMART_F32;
  if (t.scalar_type() == at::kBFloat16) return SMART_BF16;
  PyErr_Format(PyExc_TypeError, "unsupported element type %s", toString(t.scalar_type()));
  throw Failed();
}
void* stream() {
  PyObject* device = must(PyObject_CallNoArgs(get_device));
  PyObject* s = PyObject_CallOneArg(raw_stream, device);
  Py_DECREF(device);
  must(s);
  void* p = PyLong_AsVoidPtr(s);
  Py_DECREF(s);
  if (!p && PyErr_Occurred()) throw Failed();
  return p;
}

constexpr int64_t kRow = 128;  // int32 elements: where an allocation of its own would begin (multiples of 512 bytes)
int64_t whole_rows(int64_t n) { return (n + kRow - 1) / kRow * kRow; }
at::Tensor fresh(const at::Tensor& like, at::ScalarType type, at::IntArrayRef shape) {
  return at::empty(shape, at::TensorOptions().dtype(type).device(like.device()));
}
std::vector<at::Tensor> i32_rows(int64_t rows, int64_t n, const at::Tensor& like) {
  return at::empty_strided({rows, n}, {whole_rows(n), 1}, at::TensorOptions().dtype(at::kInt).device(like.device())).unbind(0);
}

// Runs the library call without the interpreter lock, then binding.py's check of its result.
template <typename F>
void call(const char* what, F f) {
  int32_t rc;
  {
    struct Unlocked {
      PyThreadState* state = PyEval_SaveThread();
      ~Unlocked() { PyEval_RestoreThread(state); }
    } unlocked;
    rc = f();
  }
  if (rc == SMART_OK) return;
  PyObject* r = PyObject_CallFunction(check_call, "is", (int)rc, what);
  Py_XDECREF(r);
  throw Failed();  // (check_call raises)
}

PyObject* wrap(const at::Tensor& t) { return must(THPVariable_Wrap(t)); }
PyObject* none_or(const at::Tensor& t) {
  if (t.defined()) return wrap(t);
  Py_RETURN_NONE;
}
template <typename... Ts>
PyObject* tuple_of(const Ts&... ts) {
  PyObject* items[] = {none_or(ts)...};
  PyObject* r = must(PyTuple_New(sizeof...(ts)));
  for (size_t i = 0; i < sizeof...(ts); ++i) PyTuple_SET_ITEM(r, i, items[i]);
  return r;
}

// The C++ side of a Python call: argument count, and exceptions of either kind turned into Python's.
template <int kArgs, PyObject* (*kBody)(PyObject* const*)>
PyObject* entry(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != kArgs) {
    PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", kArgs, n);
    return nullptr;
  }
  try {
    return kBody(a);
  } catch (const Failed&) {
    return nullptr;
  } catch (const c10::OutOfMemoryError& e) {
    PyObject* torch = PyImport_ImportModule("torch");
    PyObject* type = torch ? PyObject_GetAttrString(torch, "OutOfMemoryError") : nullptr;
    PyErr_SetString(type ? type : PyExc_MemoryError, e.what_without_backtrace());
    Py_XDECREF(type);
    Py_XDECREF(torch);
    return nullptr;
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

PyObject* setup(PyObject* const* a) {  // addresses, check, current device, raw stream
  void** at = (void**)&lib;
  constexpr Py_ssize_t kEntries = sizeof(lib) / sizeof(void*);
  if (!PyTuple_Check(a[0]) || PyTuple_GET_SIZE(a[0]) != kEntries) {
    PyErr_SetString(PyExc_TypeError, "setup: a tuple of all entry points");
    throw Failed();
  }
  for (Py_ssize_t i = 0; i < kEntries; ++i) at[i] = pointer<void>(PyTuple_GET_ITEM(a[0], i));
  PyObject** keep[] = {&check_call, &get_device, &raw_stream};
  for (int i = 0; i < 3; ++i) {
    Py_INCREF(a[1 + i]);
    Py_XDECREF(*keep[i]);
    *keep[i] = a[1 + i];
  }
  Py_RETURN_NONE;
}

PyObject* select_begin(PyObject* const* a) {  // ctx, state, root tokens, cost
  auto ctx = pointer<smart_ctx>(a[0]);
  auto state = pointer<const smart_layer_state>(a[1]);
  auto root = address<int32_t>(a[2]);
  auto cost = address<double>(a[3]);
  void* s = stream();
  call("smart_select_begin_device", [&] { return lib.begin(ctx, s, state, root, cost); });
  Py_RETURN_NONE;
}

// ctx, state, batch, cand_cu, cand_parent_node, cand_prob, cand_token, cost, dcost, alpha, dilution, out_node, status
PyObject* select_layer(PyObject* const* a) {
  auto ctx = pointer<smart_ctx>(a[0]);
  auto state = pointer<const smart_layer_state>(a[1]);
  const int64_t batch = integer(a[2]);
  const at::Tensor& cu = tensor(a[3]);
  const int64_t cap = extent(tensor(a[4]), 0);
  const double alpha = real(a[9]);
  const int32_t dilution = (int32_t)bits64(a[10]);
  at::Tensor out = a[11] == Py_None ? fresh(cu, at::kInt, {std::max<int64_t>(1, cap)}) : tensor(a[11]);
  at::Tensor status = a[12] == Py_None ? fresh(cu, at::kInt, {std::max<int64_t>(1, batch)}) : tensor(a[12]);
  auto parent = address<int32_t>(a[4]);
  auto prob = address<double>(a[5]);
  auto token = address<int32_t>(a[6]);
  auto cost = address<double>(a[7]);
  auto dcost = address<double>(a[8]);
  void* s = stream();
  call("smart_select_layer_device", [&] {
    return lib.layer(ctx, s, state, address<int32_t>(cu), parent, prob, token, cap, cost, dcost, alpha, dilution,
                     address<int32_t>(out), address<int32_t>(status));
  });
  if (extent(out, 0) != cap) out = out.slice(0, 0, cap);
  if (extent(status, 0) != batch) status = status.slice(0, 0, batch);
  return tuple_of(out, status);
}

PyObject* compact(PyObject* const* a) {  // ctx, state, batch, rows, prefix_len
  auto ctx = pointer<smart_ctx>(a[0]);
  auto state = pointer<const smart_layer_state>(a[1]);
  const int64_t batch = integer(a[2]), rows = (int64_t)bits64(a[3]);
  const at::Tensor& prefix = tensor(a[4]);
  // one allocation for everything: the masks (16 bytes a node), the rows of node values, the offsets, the statuses, each in
  // whole rows; the launch writes all of it
  const int64_t n1 = std::max<int64_t>(1, rows), b1 = std::max<int64_t>(1, batch), p = whole_rows(n1), at = whole_rows(4 * n1);
  const int64_t words = at + 5 * p + whole_rows(batch + 1) + b1;
  at::Tensor buf = fresh(prefix, at::kInt, {words});
  at::Tensor mask = buf.slice(0, 0, 4 * n1).view(at::kLong).view({n1, 2});
  at::Tensor row[5];
  for (int i = 0; i < 5; ++i) row[i] = buf.as_strided({n1}, {1}, at + i * p);
  at::Tensor cu = buf.as_strided({batch + 1}, {1}, at + 5 * p);
  at::Tensor status = buf.as_strided({b1}, {1}, at + 5 * p + whole_rows(batch + 1));
  void* s = stream();
  call("tree_compact_pack", [&] {  // (named as the binding's call)
    return lib.compact(ctx, s, state, (int32_t)rows, address<int32_t>(prefix), address<int32_t>(cu), address<int32_t>(row[0]),
                       address<int32_t>(row[1]), address<int32_t>(row[2]), address<int32_t>(row[3]), address<int32_t>(row[4]),
                       address<uint64_t>(mask), address<int32_t>(status));
  });
  if (rows == 0 || batch == 0) {
    for (at::Tensor& r : row) r = r.slice(0, 0, rows);
    mask = mask.slice(0, 0, rows);
    status = status.slice(0, 0, batch);
  }
  return tuple_of(cu, row[0], row[1], row[2], row[3], row[4], mask, status);
}

PyObject* upload_pack(PyObject* const* a) {  // ctx, pinned offsets, parents, tokens (or None), prefix_len
  auto ctx = pointer<smart_ctx>(a[0]);
  const at::Tensor& h_cu = tensor(a[1]);
  const at::Tensor& prefix = tensor(a[4]);
  const int64_t batch = extent(h_cu, 0) - 1;
  const bool plain = h_cu.is_cpu() && h_cu.scalar_type() == at::kInt && h_cu.dim() == 1 && h_cu.is_contiguous() && batch >= 0;
  const int64_t nodes = plain ? address<int32_t>(h_cu)[batch] : h_cu.select(0, batch).item<int64_t>();
  auto h_parent = address<int32_t>(a[2]), h_token = address<int32_t>(a[3]);
  auto rows = i32_rows(a[3] == Py_None ? 4 : 5, nodes, prefix);
  at::Tensor token = rows.size() > 4 ? rows[4] : at::Tensor();
  at::Tensor cu = fresh(prefix, at::kInt, {batch + 1}), status = fresh(prefix, at::kInt, {batch});
  at::Tensor mask = fresh(prefix, at::kLong, {nodes, 2});
  void* s = stream();
  call("tree_upload_pack", [&] {
    return lib.upload_pack(ctx, s, (int32_t)batch, (int32_t)nodes, address<int32_t>(h_cu), h_parent, h_token,
                           address<int32_t>(cu), address<int32_t>(rows[0]), token.defined() ? address<int32_t>(token) : nullptr,
                           address<int32_t>(prefix), address<int32_t>(rows[1]), address<int32_t>(rows[2]),
                           address<int32_t>(rows[3]), address<uint64_t>(mask), address<int32_t>(status));
  });
  return tuple_of(cu, rows[0], token, rows[1], rows[2], rows[3], mask, status);
}

PyObject* rope(PyObject* const* a) {  // ctx, position, q, k_tree, base, rotary_dim (or None), pairing
  auto ctx = pointer<smart_ctx>(a[0]);
  auto position = address<int32_t>(a[1]);
  const at::Tensor &q = tensor(a[2]), &k = tensor(a[3]);
  three_dims(q);
  const int32_t nodes = (int32_t)q.size(0), Hq = (int32_t)q.size(1), D = (int32_t)q.size(2), Hkv = (int32_t)extent(k, 1);
  const double base = real(a[4]);
  const int32_t type = element_type(q), rotary = a[5] == Py_None ? D : (int32_t)bits64(a[5]), pairing = (int32_t)bits64(a[6]);
  void* s = stream();
  call("tree_rope", [&] {
    return lib.rope(ctx, s, type, nodes, Hq, Hkv, D, rotary, pairing, base, position, address(q), address(k));
  });
  Py_RETURN_NONE;
}

// ctx, k_src, v_src, slots, k_cache, v_cache, layout, block_size, num_blocks, three strides, fp8, k_scale, v_scale
PyObject* cache_write(PyObject* const* a) {
  auto ctx = pointer<smart_ctx>(a[0]);
  const at::Tensor& k = tensor(a[1]);
  three_dims(k);
  const int32_t n = (int32_t)k.size(0), Hkv = (int32_t)k.size(1), D = (int32_t)k.size(2), type = element_type(k);
  auto v = address(a[2]), kc = address(a[4]), vc = address(a[5]);
  auto slots = address<int64_t>(a[3]);
  const int32_t layout = (int32_t)integer(a[6]), bs = (int32_t)integer(a[7]), nb = (int32_t)integer(a[8]);
  const int64_t block = integer(a[9]), head = integer(a[10]), token = integer(a[11]);
  void* s = stream();
  if (truth(a[12])) {
    const float ks = (float)real(a[13]), vs = (float)real(a[14]);
    call("kv_cache_write_fp8", [&] {
      return lib.cache_write_fp8(ctx, s, type, layout, n, Hkv, D, bs, nb, address(k), v, slots, kc, vc, block, head, token, ks, vs);
    });
  } else {
    call("kv_cache_write", [&] {
      return lib.cache_write(ctx, s, type, layout, n, Hkv, D, bs, nb, address(k), v, slots, kc, vc, block, head, token);
    });
  }
  Py_RETURN_NONE;
}

// ctx, q, k_tree, v_tree, k_cache, v_cache, block_table, prefix_len, cu_nodes, anc_mask, scale, layout, block_size, out, lse,
// want_lse, address of the host's offsets, k_scale, v_scale, static, status
PyObject* attention(PyObject* const* a) {
  auto ctx = pointer<smart_ctx>(a[0]);
  const at::Tensor &q = tensor(a[1]), &kt = tensor(a[2]), &vt = tensor(a[3]), &cu = tensor(a[8]);
  three_dims(q);
  at::Tensor out = a[13] == Py_None ? at::empty_like(q) : tensor(a[13]), lse;
  const bool want_lse = truth(a[15]);
  tva_params p = {};
  p.dtype = element_type(q);
  p.kv_layout = (int32_t)integer(a[11]);
  p.batch = (int32_t)(extent(cu, 0) - 1);
  p.total_nodes = (int32_t)q.size(0);
  p.num_q_heads = (int32_t)q.size(1);
  p.num_kv_heads = (int32_t)extent(kt, 1);
  p.head_dim = (int32_t)q.size(2);
  p.block_size = (int32_t)integer(a[12]);
  p.max_blocks_per_seq = a[6] == Py_None ? 0 : (int32_t)extent(tensor(a[6]), 1);
  p.softmax_scale = (float)real(a[10]);
  p.d_q = address(q);
  p.d_k_tree = address(kt);
  p.d_v_tree = address(vt);
  if (a[4] != Py_None) {
    const at::Tensor &kc = tensor(a[4]), &vc = tensor(a[5]);
    at_least(kc, 2);
    at_least(vc, 2);
    if (kc.stride(0) != vc.stride(0) || kc.stride(1) != vc.stride(1)) {
      PyErr_SetString(PyExc_AssertionError, "the two caches have different strides");
      throw Failed();
    }
    p.num_blocks = (int32_t)kc.size(0);
    p.d_k_cache = address(kc);
    p.d_v_cache = address(vc);
    p.cache_block_stride = kc.stride(0);
    p.cache_head_stride = kc.stride(1);
    p.cache_token_stride = p.head_dim;
    if (p.kv_layout == SMART_KV_PLAIN) {
      at_least(kc, 3);
      p.cache_token_stride = kc.stride(2);
    }
    p.d_block_table = address<int32_t>(tensor(a[6]));
    if (kc.scalar_type() == at::kByte) {  // an fp8 (E4M3) cache
      p.kv_cache_dtype = SMART_FP8_E4M3;
      p.k_scale = (float)real(a[17]);
      p.v_scale = (float)real(a[18]);
    }
  } else {
    p.cache_block_stride = p.cache_head_stride = (int64_t)p.block_size * p.head_dim;
    p.cache_token_stride = p.head_dim;
  }
  if (a[14] != Py_None) lse = tensor(a[14]);
  else if (want_lse) lse = fresh(q, at::kFloat, {q.size(0), q.size(1)});
  p.d_prefix_len = address<int32_t>(tensor(a[7]));
  p.d_cu_nodes = address<int32_t>(cu);
  p.d_anc_mask = address<uint64_t>(tensor(a[9]));
  p.d_out = address(out);
  p.d_lse = lse.defined() ? address<float>(lse) : nullptr;
  p.d_status = address<int32_t>(a[20]);
  p.h_cu_nodes = pointer<const int32_t>(a[16]);
  void* s = stream();
  if (truth(a[19])) call("tree_verify_attention_static", [&] { return lib.attention_static(ctx, s, &p); });
  else call("tree_verify_attention", [&] { return lib.attention(ctx, s, &p); });
  return lse.defined() ? tuple_of(out, lse) : wrap(out);
}

PyObject* accept(PyObject* const* a) {  // ctx, cu_nodes, parent, token, target_next, max_depth
  auto ctx = pointer<smart_ctx>(a[0]);
  const at::Tensor& cu = tensor(a[1]);
  const int64_t batch = extent(cu, 0) - 1, depth = integer(a[5]);
  auto parent = address<int32_t>(a[2]), token = address<int32_t>(a[3]), target = address<int32_t>(a[4]);
  auto rows = i32_rows(2, batch, cu);
  at::Tensor path = fresh(cu, at::kInt, {batch, depth + 1});
  void* s = stream();
  call("tree_accept", [&] {
    return lib.accept(ctx, s, (int32_t)batch, (int32_t)depth, address<int32_t>(cu), parent, token, target,
                      address<int32_t>(rows[0]), address<int32_t>(path), address<int32_t>(rows[1]));
  });
  return tuple_of(rows[0], path, rows[1]);
}

PyObject* sample(PyObject* const* a) {  // ctx, cu_nodes, parent, token, target_prob, max_depth, seed, step
  auto ctx = pointer<smart_ctx>(a[0]);
  const at::Tensor &cu = tensor(a[1]), &prob = tensor(a[4]);
  if (prob.dim() != 2 || prob.scalar_type() != at::kFloat || prob.stride(1) != 1) {
    PyErr_SetString(PyExc_AssertionError, "target_prob: [nodes, vocabulary] float32, rows of contiguous elements");
    throw Failed();
  }
  const int64_t batch = extent(cu, 0) - 1, depth = integer(a[5]);
  auto parent = address<int32_t>(a[2]), token = address<int32_t>(a[3]);
  const uint64_t seed = bits64(a[6]), step = bits64(a[7]);
  auto rows = i32_rows(2, batch, cu);
  at::Tensor path = fresh(cu, at::kInt, {batch, depth + 1});
  void* s = stream();
  call("tree_accept_sample", [&] {
    return lib.sample(ctx, s, (int32_t)batch, (int32_t)prob.size(0), (int32_t)depth, (int32_t)prob.size(1), address<int32_t>(cu),
                      parent, token, address<float>(prob), prob.stride(0), seed, step, address<int32_t>(rows[0]),
                      address<int32_t>(path), address<int32_t>(rows[1]));
  });
  return tuple_of(rows[0], path, rows[1]);
}

// ctx, cu_nodes, accept_len, accept_path, k_tree, v_tree, k_cache, v_cache, block_table, prefix_len, layout, block_size,
// num_blocks, three strides, k_scale, v_scale
PyObject* commit(PyObject* const* a) {
  auto ctx = pointer<smart_ctx>(a[0]);
  const at::Tensor &cu = tensor(a[1]), &path = tensor(a[3]), &kt = tensor(a[4]), &kc = tensor(a[6]), &table = tensor(a[8]);
  three_dims(kt);
  const int32_t batch = (int32_t)(extent(cu, 0) - 1), depth = (int32_t)(extent(path, 1) - 1), Hkv = (int32_t)kt.size(1),
                D = (int32_t)kt.size(2), type = element_type(kt), blocks = (int32_t)extent(table, 1);
  auto length = address<int32_t>(a[2]), prefix = address<int32_t>(a[9]);
  auto vt = address(a[5]), vc = address(a[7]);
  const int32_t layout = (int32_t)integer(a[10]), bs = (int32_t)integer(a[11]), nb = (int32_t)integer(a[12]);
  const int64_t block = integer(a[13]), head = integer(a[14]), token = integer(a[15]);
  auto rows = i32_rows(2, batch, cu);
  void* s = stream();
  if (kc.scalar_type() == at::kByte) {  // an fp8 (E4M3) cache
    const float ks = (float)real(a[16]), vs = (float)real(a[17]);
    call("tree_commit", [&] {
      return lib.commit_fp8(ctx, s, type, layout, batch, depth, Hkv, D, bs, blocks, nb, address<int32_t>(cu), length,
                            address<int32_t>(path), address(kt), vt, address<int32_t>(table), prefix, address(kc), vc, block,
                            head, token, address<int32_t>(rows[0]), address<int32_t>(rows[1]), ks, vs);
    });
  } else {
    call("tree_commit", [&] {
      return lib.commit(ctx, s, type, layout, batch, depth, Hkv, D, bs, blocks, nb, address<int32_t>(cu), length,
                        address<int32_t>(path), address(kt), vt, address<int32_t>(table), prefix, address(kc), vc, block, head,
                        token, address<int32_t>(rows[0]), address<int32_t>(rows[1]));
    });
  }
  return tuple_of(rows[0], rows[1]);
}

#define SMART_METHOD(NAME, ARGS) {#NAME, (PyCFunction)(void (*)())entry<ARGS, NAME>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {SMART_METHOD(setup, 4),       SMART_METHOD(select_begin, 4),      SMART_METHOD(select_layer, 13),
                         SMART_METHOD(compact, 5),     SMART_METHOD(upload_pack, 5),
                         SMART_METHOD(rope, 7),        SMART_METHOD(cache_write, 15), SMART_METHOD(attention, 21),
                         SMART_METHOD(accept, 6),      SMART_METHOD(sample, 8),     SMART_METHOD(commit, 18),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef marshal_module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&marshal_module); }
