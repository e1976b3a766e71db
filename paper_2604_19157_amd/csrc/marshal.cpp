// Argument marshalling of the binding's hot calls: torch tensors and cache objects -> the C ABI of include/saw.h.
//
// The checks and conversions are those of binding.py, one Python-level attribute or method at a time there (13-17 us a
// decode call, 2.4 us per layer of a store for many layers: 77 us for 32 layers, whose kernel takes 5.6).  Here a call reads
// the cache object's attributes, looks at the tensors directly and launches (32 layers 8.4 us in all, a small store 10.6 -> 4.5, a
// fused step of four 256-token sequences 12.3 -> 10.8); nothing is kept between calls, because a caller may
// replace a cache's tensors at any time.  Functions return the C call's code; a failed check raises AssertionError.
// The C call itself runs without the interpreter lock, as a ctypes call does: a launch can wait - for room in the stream's queue, for
// its code object - and what it waits for can need another Python thread.  Everything Python is read before, and what the call's
// pointers belong to is held until it is back.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>
#include <vector>

#include "saw.h"

namespace {

struct Raised {};                                            // a Python exception is set

// interned attribute names
PyObject *s_k_codes, *s_v_codes, *s_k_meta, *s_v_meta, *s_num_pages, *s_n_kv_heads, *s_page_size, *s_head_dim, *s_had_block,
    *s_rotate_mask, *s_sign_bits, *s_dense_rot, *s_k_pages, *s_v_pages, *s_dtype;

struct Ref {                                                 // an owned reference
  PyObject* o;
  explicit Ref(PyObject* p) : o(p) { if (!o) throw Raised(); }
  ~Ref() { Py_DECREF(o); }
  Ref(const Ref&) = delete;
  Ref& operator=(const Ref&) = delete;
};

class Held {                                                 // references kept until the C call is back
  std::vector<PyObject*> v_;
 public:
  Held() { v_.reserve(8); }
  void room(size_t n) { v_.reserve(n); }
  ~Held() { for (PyObject* o : v_) Py_DECREF(o); }
  Held(const Held&) = delete;
  Held& operator=(const Held&) = delete;
  PyObject* owned(PyObject* o) {
    if (!o) throw Raised();
    v_.push_back(o);
    return o;
  }
};

class Unlocked {                                             // the interpreter lock is another thread's meanwhile
  PyThreadState* s_;
 public:
  Unlocked() : s_(PyEval_SaveThread()) {}
  ~Unlocked() { PyEval_RestoreThread(s_); }
  Unlocked(const Unlocked&) = delete;
  Unlocked& operator=(const Unlocked&) = delete;
};

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_TypeError, "expected a tensor, got %.100s", Py_TYPE(o)->tp_name);
    throw Raised();
  }
  return THPVariable_Unpack(o);
}
void check(bool ok, const char* what) {
  if (!ok) {
    PyErr_SetString(PyExc_AssertionError, what);
    throw Raised();
  }
}
int32_t as_int(PyObject* o) {
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw Raised();
  return (int32_t)v;
}
float as_float(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw Raised();
  return (float)v;
}
int code_of(at::ScalarType t) {
  if (t == at::kHalf) return SAW_F16;
  if (t == at::kBFloat16) return SAW_BF16;
  if (t == at::kFloat) return SAW_F32;
  PyErr_SetString(PyExc_KeyError, c10::toString(t));
  throw Raised();
}
void* stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

void* data_attr(PyObject* cache, PyObject* name, Held& held) {
  PyObject* const o = held.owned(PyObject_GetAttr(cache, name));
  return o == Py_None ? nullptr : tensor(o).data_ptr();
}
int32_t int_attr(PyObject* cache, PyObject* name) {
  Ref r(PyObject_GetAttr(cache, name));
  return as_int(r.o);
}
void shape_of(PyObject* cache, saw_cache_t& c) {
  c.num_pages = int_attr(cache, s_num_pages);
  c.n_kv_heads = int_attr(cache, s_n_kv_heads);
  c.page_size = int_attr(cache, s_page_size);
  c.head_dim = int_attr(cache, s_head_dim);
}
void cache_of(PyObject* cache, saw_cache_t& c, Held& held) {
  c.k_codes = (uint8_t*)data_attr(cache, s_k_codes, held);
  c.v_codes = (uint8_t*)data_attr(cache, s_v_codes, held);
  c.k_meta = (float*)data_attr(cache, s_k_meta, held);
  c.v_meta = (float*)data_attr(cache, s_v_meta, held);
  shape_of(cache, c);
  c.had_block = int_attr(cache, s_had_block);
  c.rotate_mask = int_attr(cache, s_rotate_mask);
  Ref bits(PyObject_GetAttr(cache, s_sign_bits));
  Ref seq(PySequence_Fast(bits.o, "sign_bits is a sequence"));
  const Py_ssize_t n = PySequence_Fast_GET_SIZE(seq.o);
  check(n <= 4, "sign_bits has at most four words");
  for (int i = 0; i < 4; ++i) {
    c.sign_bits[i] = 0;
    if (i < n) {
      c.sign_bits[i] = (uint32_t)PyLong_AsUnsignedLongMask(PySequence_Fast_GET_ITEM(seq.o, i));
      if (PyErr_Occurred()) throw Raised();
    }
  }
  c.dense_rot = data_attr(cache, s_dense_rot, held);
}
bool is_i32(const at::Tensor& t) { return t.scalar_type() == at::kInt; }

// the C call, its arguments worked out before the lock is given away
template <typename F, typename... A>
int run(F f, A... args) {
  Unlocked unlocked;
  return f(args...);
}

template <typename F>
PyObject* call(Py_ssize_t got, Py_ssize_t want, F&& f) {
  if (got != want) {
    PyErr_Format(PyExc_TypeError, "%zd arguments, %zd expected", got, want);
    return nullptr;
  }
  try {
    Held held;
    return PyLong_FromLong(f(held));
  } catch (const Raised&) {
    return nullptr;
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

// (cache, K, V, page_table, slots)
PyObject* store(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return call(n, 5, [&](Held& held) {
    saw_cache_t c;
    cache_of(a[0], c, held);
    const at::Tensor &K = tensor(a[1]), &V = tensor(a[2]), &pt = tensor(a[3]), &slots = tensor(a[4]);
    check(K.dim() == 3 && K.scalar_type() == V.scalar_type() && K.sizes() == V.sizes() && K.stride(2) == 1 && K.stride(1) == c.head_dim,
          "K and V are [T][n_kv_heads][head_dim] of one type, heads dense");
    const int64_t T = K.size(0);
    check(V.strides() == K.strides() && is_i32(pt) && is_i32(slots), "V is laid out as K; page_table and slots are int32");
    check(pt.dim() == 2 && pt.is_contiguous() && slots.is_contiguous() && slots.dim() == 2 && slots.size(0) == T && slots.size(1) == 2,
          "page_table [n_seqs][max_pages] and slots [T][2] are contiguous");
    const int type = code_of(K.scalar_type());
    return run(saw_rotate_quant_store, &c, K.data_ptr(), V.data_ptr(), type, T,
               T > 1 ? K.stride(0) : (int64_t)c.n_kv_heads * c.head_dim, (const int32_t*)pt.data_ptr(), (int32_t)pt.size(0),
               (int32_t)pt.size(1), (const int32_t*)slots.data_ptr(), stream());
  });
}

// (caches, Ks, Vs, page_table, slots)
PyObject* store_layers(PyObject*, PyObject* const* a, Py_ssize_t n_args) {
  return call(n_args, 5, [&](Held& held) {
    // (tuples of their own: another thread may change the caller's lists while the lock is away)
    Ref cs(PySequence_Tuple(a[0])), ks(PySequence_Tuple(a[1])), vs(PySequence_Tuple(a[2]));
    const Py_ssize_t n = PyTuple_GET_SIZE(cs.o);
    if (n < 1) { PyErr_SetString(PyExc_IndexError, "no caches"); throw Raised(); }
    check(PyTuple_GET_SIZE(ks.o) == n && PyTuple_GET_SIZE(vs.o) == n, "one K and one V per cache");
    const at::Tensor &pt = tensor(a[3]), &slots = tensor(a[4]);
    held.room(5 * (size_t)n);
    std::vector<saw_cache_t> c(n);
    std::vector<const void*> K(n), V(n);
    const at::Tensor& K0 = tensor(PyTuple_GET_ITEM(ks.o, 0));
    check(K0.dim() == 3, "K is [T][n_kv_heads][head_dim]");
    const int64_t T = K0.size(0);
    for (Py_ssize_t l = 0; l < n; ++l) {
      cache_of(PyTuple_GET_ITEM(cs.o, l), c[l], held);
      const at::Tensor &k = tensor(PyTuple_GET_ITEM(ks.o, l)), &v = tensor(PyTuple_GET_ITEM(vs.o, l));
      check(k.scalar_type() == K0.scalar_type() && k.sizes() == K0.sizes() && v.sizes() == K0.sizes() && k.stride(2) == 1 && k.stride(1) == c[0].head_dim,
            "every layer's K and V are [T][n_kv_heads][head_dim] of one type, heads dense");
      check(v.strides() == k.strides() && (T <= 1 || k.stride(0) == K0.stride(0)), "every layer's K and V are laid out alike");
      K[l] = k.data_ptr();
      V[l] = v.data_ptr();
    }
    check(pt.dim() == 2 && pt.is_contiguous() && slots.is_contiguous() && slots.dim() == 2 && slots.size(0) == T && slots.size(1) == 2,
          "page_table [n_seqs][max_pages] and slots [T][2] are contiguous");
    const int type = code_of(K0.scalar_type());
    return run(saw_rotate_quant_store_layers, c.data(), K.data(), V.data(), (int32_t)n, type, T,
               T > 1 ? K0.stride(0) : (int64_t)c[0].n_kv_heads * c[0].head_dim, (const int32_t*)pt.data_ptr(),
               (int32_t)pt.size(0), (int32_t)pt.size(1), (const int32_t*)slots.data_ptr(), stream());
  });
}

const int32_t* order_of(PyObject* o, int64_t B) {
  if (o == Py_None) return nullptr;
  const at::Tensor& t = tensor(o);
  check(is_i32(t) && t.numel() == B && t.is_contiguous(), "order is a contiguous int32 tensor of the batch's length");
  return (const int32_t*)t.data_ptr();
}

// (cache, q, page_table, seq_lens, max_seq_len, sm_scale, out, workspace, num_splits, order or None)
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return call(n, 10, [&](Held& held) {
    saw_cache_t c;
    cache_of(a[0], c, held);
    const at::Tensor &q = tensor(a[1]), &pt = tensor(a[2]), &lens = tensor(a[3]), &out = tensor(a[6]), &ws = tensor(a[7]);
    check(q.dim() == 3 && pt.dim() == 2 && q.is_contiguous() && pt.is_contiguous() && is_i32(lens),
          "q [B][n_q_heads][head_dim] and page_table are contiguous, seq_lens is int32");
    const saw_decode_hints_t hints = {order_of(a[9], q.size(0))};
    const int q_type = code_of(q.scalar_type()), out_type = code_of(out.scalar_type());
    const int32_t bound = as_int(a[4]), splits = as_int(a[8]);
    const float scale = as_float(a[5]);
    return run(saw_paged_decode_attn_hinted, &c, q.data_ptr(), q_type, (int32_t)q.size(0), (int32_t)q.size(1),
               (const int32_t*)pt.data_ptr(), (int32_t)pt.size(1), (const int32_t*)lens.data_ptr(), bound, scale,
               out.data_ptr(), out_type, ws.data_ptr(), (size_t)ws.numel(), splits, &hints, stream());
  });
}

// (cache, K_new, V_new, q, page_table, seq_lens, max_seq_len, sm_scale, out, workspace, order or None)
PyObject* append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return call(n, 11, [&](Held& held) {
    saw_cache_t c;
    cache_of(a[0], c, held);
    const at::Tensor &K = tensor(a[1]), &V = tensor(a[2]), &q = tensor(a[3]), &pt = tensor(a[4]), &lens = tensor(a[5]), &out = tensor(a[8]), &ws = tensor(a[9]);
    check(q.dim() == 3 && q.is_contiguous() && K.is_contiguous() && V.is_contiguous() && K.scalar_type() == V.scalar_type(),
          "q, K_new and V_new are contiguous, K_new and V_new of one type");
    check(pt.dim() == 2 && pt.is_contiguous() && is_i32(lens), "page_table is contiguous, seq_lens is int32");
    const saw_decode_hints_t hints = {order_of(a[10], q.size(0))};
    const int type = code_of(K.scalar_type()), q_type = code_of(q.scalar_type()), out_type = code_of(out.scalar_type());
    const int32_t bound = as_int(a[6]);
    const float scale = as_float(a[7]);
    return run(saw_append_decode_attn_hinted, &c, K.data_ptr(), V.data_ptr(), type, q.data_ptr(), q_type, (int32_t)q.size(0),
               (int32_t)q.size(1), (const int32_t*)pt.data_ptr(), (int32_t)pt.size(1), (const int32_t*)lens.data_ptr(), bound,
               scale, out.data_ptr(), out_type, ws.data_ptr(), (size_t)ws.numel(), &hints, stream());
  });
}

// (cache, page_table, seq, pos_begin, pos_end, unrotate, k_out or None, v_out or None), one of the outputs given
PyObject* flatten(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return call(n, 8, [&](Held& held) {
    saw_cache_t c;
    cache_of(a[0], c, held);
    const at::Tensor& pt = tensor(a[1]);
    check(pt.dim() == 2, "page_table is [n_seqs][max_pages]");
    const int32_t begin = as_int(a[3]), end = as_int(a[4]);
    const at::Tensor& ref = tensor(a[6] != Py_None ? a[6] : a[7]);
    void* const k = a[6] != Py_None ? tensor(a[6]).data_ptr() : nullptr;
    void* const v = a[7] != Py_None ? tensor(a[7]).data_ptr() : nullptr;
    const int unrotate = PyObject_IsTrue(a[5]);
    if (unrotate < 0) throw Raised();
    const int type = code_of(ref.scalar_type());
    const int32_t seq = as_int(a[2]);
    return run(saw_flatten_dequant, &c, (const int32_t*)pt.data_ptr(), (int32_t)pt.size(1), seq, begin, end, unrotate, type, k,
               v, end > begin ? ref.stride(0) : (int64_t)c.n_kv_heads * c.head_dim, stream());
  });
}

// (16-bit cache, q, page_table, seq_lens, max_seq_len, sm_scale, out, workspace, num_splits)
PyObject* kv16_decode(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return call(n, 9, [&](Held& held) {
    saw_cache_t c = {};
    shape_of(a[0], c);
    c.had_block = 1;
    void *const k = data_attr(a[0], s_k_pages, held), *const v = data_attr(a[0], s_v_pages, held);
    Ref type(PyObject_GetAttr(a[0], s_dtype));
    check(THPDtype_Check(type.o), "dtype is a torch dtype");
    const at::Tensor &q = tensor(a[1]), &pt = tensor(a[2]), &lens = tensor(a[3]), &out = tensor(a[6]), &ws = tensor(a[7]);
    check(q.dim() == 3 && pt.dim() == 2, "q is [B][n_q_heads][head_dim], page_table [B][max_pages]");
    const int kv_type = code_of(((THPDtype*)type.o)->scalar_type), q_type = code_of(q.scalar_type()), out_type = code_of(out.scalar_type());
    const int32_t bound = as_int(a[4]), splits = as_int(a[8]);
    const float scale = as_float(a[5]);
    return run(saw_kv16_paged_decode_attn, &c, k, v, kv_type, q.data_ptr(), q_type, (int32_t)q.size(0), (int32_t)q.size(1),
               (const int32_t*)pt.data_ptr(), (int32_t)pt.size(1), (const int32_t*)lens.data_ptr(), bound, scale,
               out.data_ptr(), out_type, ws.data_ptr(), (size_t)ws.numel(), splits, stream());
  });
}

#define FAST(f) {#f, (PyCFunction)(void*)f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(store), FAST(store_layers), FAST(decode), FAST(append), FAST(flatten), FAST(kv16_decode),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
#define NAME(n) if (!(s_##n = PyUnicode_InternFromString(#n))) return nullptr;
  NAME(k_codes) NAME(v_codes) NAME(k_meta) NAME(v_meta) NAME(num_pages) NAME(n_kv_heads) NAME(page_size) NAME(head_dim)
  NAME(had_block) NAME(rotate_mask) NAME(sign_bits) NAME(dense_rot) NAME(k_pages) NAME(v_pages) NAME(dtype)
  return PyModule_Create(&module);
}
