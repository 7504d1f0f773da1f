// Argument marshalling of the Python binding, in native code: every call checks
// its tensors (device, type, contiguity, size) and passes their pointers to the
// C ABI.  In Python the checks of a call cost 5 to 15 us, those of a block call
// about 80, more than the launches they guard.  Nothing is kept between calls;
// the interpreter lock is released around the C call.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <string>

#include "lancet_moe.h"

namespace {

struct Abi {   // addresses in the loaded library, given by init()
  decltype(&moe_workspace_bytes) workspace_bytes;
  decltype(&moe_block_workspace_bytes) block_workspace_bytes;
  decltype(&moe_gate_topk) gate_topk;
  decltype(&moe_dispatch) dispatch;
  decltype(&moe_dispatch_noalloc) dispatch_noalloc;
  decltype(&moe_dispatch_bpr) dispatch_bpr;
  decltype(&moe_pack_weights) pack_weights;
  decltype(&moe_expert_ffn_fwd) expert_ffn_fwd;
  decltype(&moe_combine) combine;
  decltype(&moe_bwd_dx) bwd_dx;
  decltype(&moe_bwd_dw) bwd_dw;
  decltype(&moe_block_chunked) block_chunked;
} g_abi;
PyObject* g_stream;      // the module's function from a stream argument to a raw stream
PyObject* g_cfg_type;    // the ctypes structures
PyObject* g_block_type;

struct Error {};   // a Python exception is set

constexpr auto kBf16 = at::kBFloat16;
constexpr auto kF32 = at::kFloat;
constexpr auto kI32 = at::kInt;

// Element counts before the C ABI has checked the sizes they come from: a product
// of four 31-bit factors, or of 63 and 31 bits, is exact.
using Num = __int128;
std::string str(Num v) {
  std::string s;
  const bool neg = v < 0;
  for (unsigned __int128 u = neg ? -(unsigned __int128)v : v; u || s.empty(); u /= 10) s.insert(s.begin(), '0' + (int)(u % 10));
  return neg ? "-" + s : s;
}

const char* type_name(at::ScalarType t) {
  switch (t) {
    case at::kBFloat16: return "torch.bfloat16";
    case at::kFloat: return "torch.float32";
    case at::kInt: return "torch.int32";
    case at::kByte: return "torch.uint8";
    default: return nullptr;
  }
}

// The pointer of tensor o (NULL for an absent or empty one), checked.
void* ptr(PyObject* o, const char* name, at::ScalarType type, Num numel, bool nullable = false) {
  if (o == Py_None) {
    if (nullable) return nullptr;
    PyErr_Format(PyExc_ValueError, "%s is required", name);
    throw Error();
  }
  if (!THPVariable_Check(o)) {
    PyErr_Format(PyExc_ValueError, "%s must be a device tensor", name);
    throw Error();
  }
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda()) {
    PyErr_Format(PyExc_ValueError, "%s must be a device tensor", name);
    throw Error();
  }
  if (t.scalar_type() != type) {
    PyObject* got = PyObject_GetAttrString(o, "dtype");
    PyErr_Format(PyExc_ValueError, "%s must be %s, got %S", name, type_name(type), got ? got : Py_None);
    Py_XDECREF(got);
    throw Error();
  }
  if (!t.is_contiguous()) {
    PyErr_Format(PyExc_ValueError, "%s must be contiguous", name);
    throw Error();
  }
  if (t.numel() < numel) {
    PyErr_Format(PyExc_ValueError, "%s has %lld elements, the call touches %s", name, (long long)t.numel(),
                 str(numel).c_str());
    throw Error();
  }
  return t.numel() ? t.data_ptr() : nullptr;
}
int64_t numel_or_0(PyObject* o) { return o == Py_None ? 0 : THPVariable_Unpack(o).numel(); }

// A ctypes structure's bytes.
template <typename T>
struct Struct {
  Py_buffer buf;
  explicit Struct(PyObject* o) {
    PyObject* type = std::is_same<T, moe_cfg>::value ? g_cfg_type : g_block_type;
    const int is = PyObject_IsInstance(o, type);
    if (is == 0) PyErr_Format(PyExc_TypeError, "cfg must be a %s", ((PyTypeObject*)type)->tp_name);
    if (is != 1 || PyObject_GetBuffer(o, &buf, PyBUF_SIMPLE) != 0) throw Error();
    if (buf.len < (Py_ssize_t)sizeof(T)) {
      PyBuffer_Release(&buf);
      PyErr_SetString(PyExc_TypeError, "cfg is too small");
      throw Error();
    }
  }
  Struct(const Struct&) = delete;
  ~Struct() { PyBuffer_Release(&buf); }
  const T* operator->() const { return (const T*)buf.buf; }
  operator const T*() const { return (const T*)buf.buf; }
};

at::ScalarType dtype_of(const moe_cfg* c) { return c->dtype == MOE_BF16 ? kBf16 : kF32; }
// Elements of an [E][C][X] expert buffer.
Num expert_numel(const moe_cfg* c, Num X) {
  const Num rows = c->dtype == MOE_BF16 ? ((Num)c->C + 15) / 16 * 16 : c->C;
  return c->E * rows * X;
}

// An integer argument, its magnitude bounded to 64 bits.
Num big(PyObject* o) {
  PyObject* i = PyNumber_Index(o);
  if (!i) throw Error();
  int over = 0;
  const long long v = PyLong_AsLongLongAndOverflow(i, &over);
  Py_DECREF(i);
  return over ? (Num)over << 64 : (Num)v;
}

void* stream_arg(PyObject* o) {
  PyObject* raw = PyObject_CallOneArg(g_stream, o);
  if (!raw) throw Error();
  void* s = PyLong_AsVoidPtr(raw);
  Py_DECREF(raw);
  if (!s && PyErr_Occurred()) throw Error();
  return s;
}

// The C call without the interpreter lock, which is held again however it ends.
template <typename F>
PyObject* status(F&& call) {
  struct Unlocked {
    PyThreadState* state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
  };
  moe_status st;
  {
    Unlocked u;
    st = call();
  }
  return PyLong_FromLong(st);
}

// An entry point: N positional arguments, the body's errors as Python exceptions.
template <typename F>
PyObject* entry(Py_ssize_t n, Py_ssize_t want, F&& body) {
  if (n != want) {
    PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
    return nullptr;
  }
  try {
    return body();
  } catch (const Error&) {
    return nullptr;
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}
#define ENTRY(NAME) PyObject* NAME(PyObject*, PyObject* const* a, Py_ssize_t n)

ENTRY(gate_topk) {   // cfg, x, Wg, bias, logits, idx, w, stream
  return entry(n, 8, [&] {
    Struct<moe_cfg> c(a[0]);
    const auto dt = dtype_of(c);
    const Num T = c->T, d = c->d_model, E = c->E, k = c->k;
    const void* x = ptr(a[1], "x", dt, T * d);
    const void* Wg = ptr(a[2], "Wg", dt, E * d);
    const float* bias = (const float*)ptr(a[3], "bias", kF32, E, true);
    float* logits = (float*)ptr(a[4], "logits", kF32, T * E);
    int32_t* idx = (int32_t*)ptr(a[5], "idx", kI32, T * k);
    float* w = (float*)ptr(a[6], "w", kF32, T * k);
    void* s = stream_arg(a[7]);
    return status([&] { return g_abi.gate_topk(c, x, Wg, bias, logits, idx, w, s); });
  });
}

// cfg, x, idx, carry, fill, slot, send_buf, [ws,] stream
PyObject* dispatch_any(PyObject* const* a, bool ws_arg) {
  Struct<moe_cfg> c(a[0]);
  const auto dt = dtype_of(c);
  const Num T = c->T, d = c->d_model, E = c->E, k = c->k;
  const size_t need = ws_arg ? g_abi.workspace_bytes(c, MOE_CALL_DISPATCH) : 0;
  const void* x = ptr(a[1], "x", dt, T * d);
  const int32_t* idx = (const int32_t*)ptr(a[2], "idx", kI32, T * k);
  const int32_t* carry = (const int32_t*)ptr(a[3], "carry", kI32, E, true);
  int32_t* fill = (int32_t*)ptr(a[4], "fill", kI32, E);
  int32_t* slot = (int32_t*)ptr(a[5], "slot", kI32, T * k);
  void* send = ptr(a[6], "send_buf", dt, expert_numel(c, d));
  if (!ws_arg) {
    void* s = stream_arg(a[7]);
    return status([&] { return g_abi.dispatch_noalloc(c, x, idx, carry, fill, slot, send, s); });
  }
  void* ws = ptr(a[7], "ws", at::kByte, need, need == 0);
  const size_t wsn = numel_or_0(a[7]);
  void* s = stream_arg(a[8]);
  return status([&] { return g_abi.dispatch(c, x, idx, carry, fill, slot, send, ws, wsn, s); });
}
ENTRY(dispatch) { return entry(n, 9, [&] { return dispatch_any(a, true); }); }
ENTRY(dispatch_noalloc) { return entry(n, 8, [&] { return dispatch_any(a, false); }); }

ENTRY(dispatch_bpr) {   // cfg, x, logits, idx, fill, slot, send_buf, order, ws, stream
  return entry(n, 10, [&] {
    Struct<moe_cfg> c(a[0]);
    const auto dt = dtype_of(c);
    const Num T = c->T, d = c->d_model, E = c->E, k = c->k;
    const size_t need = g_abi.workspace_bytes(c, MOE_CALL_DISPATCH_BPR);
    const void* x = ptr(a[1], "x", dt, T * d);
    const float* logits = (const float*)ptr(a[2], "logits", kF32, T * E);
    const int32_t* idx = (const int32_t*)ptr(a[3], "idx", kI32, T * k);
    int32_t* fill = (int32_t*)ptr(a[4], "fill", kI32, E);
    int32_t* slot = (int32_t*)ptr(a[5], "slot", kI32, T * k);
    void* send = ptr(a[6], "send_buf", dt, expert_numel(c, d));
    int32_t* order = (int32_t*)ptr(a[7], "order", kI32, T, true);
    void* ws = ptr(a[8], "ws", at::kByte, need, need == 0);
    const size_t wsn = numel_or_0(a[8]);
    void* s = stream_arg(a[9]);
    return status([&] { return g_abi.dispatch_bpr(c, x, logits, idx, fill, slot, send, order, ws, wsn, s); });
  });
}

ENTRY(pack_weights) {   // cfg, W1, W2, W1p, W2p, stream
  return entry(n, 6, [&] {
    Struct<moe_cfg> c(a[0]);
    const auto dt = dtype_of(c);
    const Num m = (Num)c->E * c->d_ff * c->d_model;
    const void* W1 = ptr(a[1], "W1", dt, m);
    const void* W2 = ptr(a[2], "W2", dt, m);
    void* W1p = ptr(a[3], "W1p", dt, m);
    void* W2p = ptr(a[4], "W2p", dt, m);
    void* s = stream_arg(a[5]);
    return status([&] { return g_abi.pack_weights(c, W1, W2, W1p, W2p, s); });
  });
}

ENTRY(expert_ffn_fwd) {   // cfg, send_buf, row_begin, row_end, W1p, W2p, H, A, expert_out, ws, stream
  return entry(n, 11, [&] {
    Struct<moe_cfg> c(a[0]);
    const auto dt = dtype_of(c);
    const Num d = c->d_model, f = c->d_ff, E = c->E;
    const size_t need = g_abi.workspace_bytes(c, MOE_CALL_FFN_FWD);
    const void* send = ptr(a[1], "send_buf", dt, expert_numel(c, d));
    const int32_t* rb = (const int32_t*)ptr(a[2], "row_begin", kI32, E, true);
    const int32_t* re = (const int32_t*)ptr(a[3], "row_end", kI32, E);
    const void* W1p = ptr(a[4], "W1p", dt, E * f * d);
    const void* W2p = ptr(a[5], "W2p", dt, E * d * f);
    void* H = ptr(a[6], "H", dt, expert_numel(c, f));
    void* A = ptr(a[7], "A", dt, expert_numel(c, f));
    void* O = ptr(a[8], "expert_out", dt, expert_numel(c, d));
    void* ws = ptr(a[9], "ws", at::kByte, need, need == 0);
    const size_t wsn = numel_or_0(a[9]);
    void* s = stream_arg(a[10]);
    return status([&] { return g_abi.expert_ffn_fwd(c, send, rb, re, W1p, W2p, H, A, O, ws, wsn, s); });
  });
}

ENTRY(combine) {   // cfg, expert_out, idx, slot, w, y, stream
  return entry(n, 7, [&] {
    Struct<moe_cfg> c(a[0]);
    const auto dt = dtype_of(c);
    const Num T = c->T, d = c->d_model, k = c->k;
    const void* O = ptr(a[1], "expert_out", dt, expert_numel(c, d));
    const int32_t* idx = (const int32_t*)ptr(a[2], "idx", kI32, T * k);
    const int32_t* slot = (const int32_t*)ptr(a[3], "slot", kI32, T * k);
    const float* w = (const float*)ptr(a[4], "w", kF32, T * k);
    void* y = ptr(a[5], "y", dt, T * d);
    void* s = stream_arg(a[6]);
    return status([&] { return g_abi.combine(c, O, idx, slot, w, y, s); });
  });
}

// cfg, Wg, logits, idx, w, slot, row_begin, row_end, H, expert_out, W1p, W2p, dy, dO, dH, dXe, dlogits, dx, ws, stream
ENTRY(bwd_dx) {
  return entry(n, 20, [&] {
    Struct<moe_cfg> c(a[0]);
    const auto dt = dtype_of(c);
    const Num T = c->T, d = c->d_model, f = c->d_ff, E = c->E, k = c->k;
    const Num nd = expert_numel(c, d), nf = expert_numel(c, f);
    const size_t need = g_abi.workspace_bytes(c, MOE_CALL_BWD_DX);
    const void* Wg = ptr(a[1], "Wg", dt, E * d);
    const float* logits = (const float*)ptr(a[2], "logits", kF32, T * E);
    const int32_t* idx = (const int32_t*)ptr(a[3], "idx", kI32, T * k);
    const float* w = (const float*)ptr(a[4], "w", kF32, T * k);
    const int32_t* slot = (const int32_t*)ptr(a[5], "slot", kI32, T * k);
    const int32_t* rb = (const int32_t*)ptr(a[6], "row_begin", kI32, E, true);
    const int32_t* re = (const int32_t*)ptr(a[7], "row_end", kI32, E);
    const void* H = ptr(a[8], "H", dt, nf);
    const void* O = ptr(a[9], "expert_out", dt, nd);
    const void* W1p = ptr(a[10], "W1p", dt, E * f * d);
    const void* W2p = ptr(a[11], "W2p", dt, E * d * f);
    const void* dy = ptr(a[12], "dy", dt, T * d);
    void* dO = ptr(a[13], "dO", dt, nd);
    void* dH = ptr(a[14], "dH", dt, nf);
    void* dXe = ptr(a[15], "dXe", dt, nd);
    float* dl = (float*)ptr(a[16], "dlogits", kF32, T * E);
    void* dx = ptr(a[17], "dx", dt, T * d);
    void* ws = ptr(a[18], "ws", at::kByte, need, need == 0);
    const size_t wsn = numel_or_0(a[18]);
    void* s = stream_arg(a[19]);
    return status([&] {
      return g_abi.bwd_dx(c, Wg, logits, idx, w, slot, rb, re, H, O, W1p, W2p, dy, dO, dH, dXe, dl, dx, ws, wsn, s);
    });
  });
}

// cfg, x, dlogits, row_begin, row_end, send_buf, A, dO, dH, dW1, dW2, dWg, ws, stream
ENTRY(bwd_dw) {
  return entry(n, 14, [&] {
    Struct<moe_cfg> c(a[0]);
    const auto dt = dtype_of(c);
    const Num T = c->T, d = c->d_model, f = c->d_ff, E = c->E;
    const Num nd = expert_numel(c, d), nf = expert_numel(c, f);
    const size_t need = g_abi.workspace_bytes(c, MOE_CALL_BWD_DW);
    const void* x = ptr(a[1], "x", dt, T * d, T == 0);
    const float* dl = (const float*)ptr(a[2], "dlogits", kF32, T * E);
    const int32_t* rb = (const int32_t*)ptr(a[3], "row_begin", kI32, E, true);
    const int32_t* re = (const int32_t*)ptr(a[4], "row_end", kI32, E);
    const void* send = ptr(a[5], "send_buf", dt, nd);
    const void* A = ptr(a[6], "A", dt, nf);
    const void* dO = ptr(a[7], "dO", dt, nd);
    const void* dH = ptr(a[8], "dH", dt, nf);
    void* dW1 = ptr(a[9], "dW1", dt, E * f * d);
    void* dW2 = ptr(a[10], "dW2", dt, E * d * f);
    float* dWg = (float*)ptr(a[11], "dWg", kF32, E * d);
    void* ws = ptr(a[12], "ws", at::kByte, need, need == 0);
    const size_t wsn = numel_or_0(a[12]);
    void* s = stream_arg(a[13]);
    return status([&] { return g_abi.bwd_dw(c, x, dl, rb, re, send, A, dO, dH, dW1, dW2, dWg, ws, wsn, s); });
  });
}

// d[name] (KeyError if missing; any mapping).  The caller owns the reference.
struct Item {
  PyObject* o;
  Item(PyObject* d, const char* name) {
    PyObject* key = PyUnicode_InternFromString(name);
    o = key ? PyObject_GetItem(d, key) : nullptr;
    Py_XDECREF(key);
    if (!o) throw Error();
  }
  ~Item() { Py_DECREF(o); }
};
// The pointer of d[name], checked.  The mapping keeps the tensor alive.
template <typename T>
void item(T*& out, PyObject* d, const char* name, at::ScalarType type, Num numel) {
  Item it(d, name);
  out = (T*)ptr(it.o, name, type, numel);
}

// cfg, weights, grads, x, out, dy, dx, acts, passes, n_chunks, (stream, stream, stream), ws
ENTRY(block_chunked) {
  return entry(n, 12, [&] {
    Struct<moe_block_cfg> c(a[0]);
    const moe_cfg* m = &c->moe;
    // The C ABI takes the low 32 bits; the size of `fill` is checked for the number as given.
    const int passes = (int)PyLong_AsUnsignedLongMask(a[8]), chunks = (int)PyLong_AsUnsignedLongMask(a[9]);
    if (PyErr_Occurred()) throw Error();
    const Num given = big(a[9]);
    const bool fwd = passes & MOE_BLOCK_FWD, bwd = passes & MOE_BLOCK_BWD;
    const Num T = m->T, d = m->d_model, f = m->d_ff, E = m->E, k = m->k;
    const Num nd = expert_numel(m, d), nf = expert_numel(m, f), nw = E * f * d;
    const Num st = (Num)c->B * c->heads * (((Num)c->S + 63) / 64 * 64);
    moe_block_weights W;
    PyObject* w = a[1];
    item(W.ln1_g, w, "ln1_g", kBf16, d);
    item(W.ln1_b, w, "ln1_b", kBf16, d);
    item(W.Wqkv, w, "Wqkv", kBf16, 3 * d * d);
    item(W.Wo, w, "Wo", kBf16, d * d);
    item(W.ln2_g, w, "ln2_g", kBf16, d);
    item(W.ln2_b, w, "ln2_b", kBf16, d);
    item(W.Wg, w, "Wg", kBf16, E * d);
    item(W.W1, w, "W1", kBf16, nw);
    item(W.W2, w, "W2", kBf16, nw);
    moe_block_grads G = {};
    if (bwd) {
      PyObject* g = a[2];
      item(G.dln1_g, g, "dln1_g", kF32, d);
      item(G.dln1_b, g, "dln1_b", kF32, d);
      item(G.dWqkv, g, "dWqkv", kBf16, 3 * d * d);
      item(G.dWo, g, "dWo", kBf16, d * d);
      item(G.dln2_g, g, "dln2_g", kF32, d);
      item(G.dln2_b, g, "dln2_b", kF32, d);
      item(G.dWg, g, "dWg", kF32, E * d);
      item(G.dW1, g, "dW1", kBf16, nw);
      item(G.dW2, g, "dW2", kBf16, nw);
    }
    moe_block_acts A = {};
    PyObject* q = a[7];
    item(A.a, q, "a", kBf16, T * d);
    item(A.ln1_mean, q, "ln1_mean", kF32, T);
    item(A.ln1_rstd, q, "ln1_rstd", kF32, T);
    item(A.qkv, q, "qkv", kBf16, T * 3 * d);
    item(A.attn, q, "attn", kBf16, T * d);
    item(A.lse, q, "lse", kF32, st);
    item(A.h, q, "h", kBf16, T * d);
    item(A.ln2_mean, q, "ln2_mean", kF32, T);
    item(A.ln2_rstd, q, "ln2_rstd", kF32, T);
    item(A.m, q, "m", kBf16, T * d);
    item(A.logits, q, "logits", kF32, T * E);
    item(A.idx, q, "idx", kI32, T * k);
    item(A.w, q, "w", kF32, T * k);
    item(A.slot, q, "slot", kI32, T * k);
    item(A.fill, q, "fill", kI32, given * E);
    item(A.send_buf, q, "send_buf", kBf16, nd);
    item(A.H, q, "H", kBf16, nf);
    item(A.A, q, "A", kBf16, nf);
    item(A.expert_out, q, "expert_out", kBf16, nd);
    item(A.W1p, q, "W1p", kBf16, nw);
    item(A.W2p, q, "W2p", kBf16, nw);
    if (bwd) {
      item(A.dO, q, "dO", kBf16, nd);
      item(A.dH, q, "dH", kBf16, nf);
      item(A.dXe, q, "dXe", kBf16, nd);
      item(A.dlogits, q, "dlogits", kF32, T * E);
      item(A.dm, q, "dm", kBf16, T * d);
      item(A.dh, q, "dh", kBf16, T * d);
      item(A.dattn, q, "dattn", kBf16, T * d);
      item(A.delta, q, "delta", kF32, st);
      item(A.dqkv, q, "dqkv", kBf16, T * 3 * d);
      item(A.da, q, "da", kBf16, T * d);
    }
    const size_t need = g_abi.block_workspace_bytes(c, chunks);
    moe_stream_t s[3] = {nullptr, nullptr, nullptr};
    PyObject* list = PySequence_List(a[10]);
    if (!list) throw Error();
    struct Ref {
      PyObject* o;
      ~Ref() { Py_DECREF(o); }
    } hold{list};
    if (PyList_GET_SIZE(list) > 3) {
      PyErr_SetString(PyExc_IndexError, "streams: three at most");
      throw Error();
    }
    for (Py_ssize_t i = 0; i < PyList_GET_SIZE(list); ++i) s[i] = stream_arg(PyList_GET_ITEM(list, i));
    const void* x = ptr(a[3], "x", kBf16, T * d);
    void* out = fwd ? ptr(a[4], "out", kBf16, T * d) : nullptr;
    const void* dy = bwd ? ptr(a[5], "dy", kBf16, T * d) : nullptr;
    void* dx = bwd ? ptr(a[6], "dx", kBf16, T * d) : nullptr;
    void* ws = ptr(a[11], "ws", at::kByte, need);
    const size_t wsn = numel_or_0(a[11]);
    return status([&] {
      return g_abi.block_chunked(c, &W, bwd ? &G : nullptr, x, out, dy, dx, &A, passes, chunks, s, ws, wsn);
    });
  });
}

// init({C ABI name: address}, stream function, moe_cfg type, moe_block_cfg type)
ENTRY(init) {
  if (n != 4) return PyErr_Format(PyExc_TypeError, "init takes 4 arguments");
  PyObject* d = a[0];
  auto set = [&](auto& fn, const char* name) {
    Item it(d, name);
    void* p = PyLong_AsVoidPtr(it.o);
    if (!p) {
      if (!PyErr_Occurred()) PyErr_Format(PyExc_ValueError, "%s has no address", name);
      throw Error();
    }
    fn = (std::remove_reference_t<decltype(fn)>)p;
  };
  try {
    set(g_abi.workspace_bytes, "moe_workspace_bytes");
    set(g_abi.block_workspace_bytes, "moe_block_workspace_bytes");
    set(g_abi.gate_topk, "moe_gate_topk");
    set(g_abi.dispatch, "moe_dispatch");
    set(g_abi.dispatch_noalloc, "moe_dispatch_noalloc");
    set(g_abi.dispatch_bpr, "moe_dispatch_bpr");
    set(g_abi.pack_weights, "moe_pack_weights");
    set(g_abi.expert_ffn_fwd, "moe_expert_ffn_fwd");
    set(g_abi.combine, "moe_combine");
    set(g_abi.bwd_dx, "moe_bwd_dx");
    set(g_abi.bwd_dw, "moe_bwd_dw");
    set(g_abi.block_chunked, "moe_block_chunked");
  } catch (const Error&) {
    return nullptr;
  }
  PyObject** slots[] = {&g_stream, &g_cfg_type, &g_block_type};
  for (int i = 0; i < 3; ++i) {
    Py_INCREF(a[i + 1]);
    Py_XSETREF(*slots[i], a[i + 1]);
  }
  Py_RETURN_NONE;
}

#define METHOD(NAME) {#NAME, (PyCFunction)(void (*)(void))NAME, METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {METHOD(init),
                          METHOD(gate_topk),
                          METHOD(dispatch),
                          METHOD(dispatch_noalloc),
                          METHOD(dispatch_bpr),
                          METHOD(pack_weights),
                          METHOD(expert_ffn_fwd),
                          METHOD(combine),
                          METHOD(bwd_dx),
                          METHOD(bwd_dw),
                          METHOD(block_chunked),
                          {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_bind", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__bind(void) { return PyModule_Create(&kModule); }
