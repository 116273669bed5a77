// Host side of the Python binding: takes tensors, allocates outputs, calls the C ABI (include/lstm_abi.h).  No device code.
//
// What bounds a small call (a decoder step for one sentence, a short sentence's encoding) is not the device but the time
// the host needs to hand the work over: in Python, with ctypes, a call cost 16 - 21 us before the first kernel was enqueued
// (a dozen tensors checked and their addresses taken, the descriptor built, four outputs allocated, fifteen arguments
// converted).  The same work here takes 7 - 11 us.  The functions are positional and private to binding.py, which keeps the public
// names, keyword arguments and results.
//
// The library's entry points are handed over as addresses (`bind`), so that binding.py alone decides which library is
// loaded.  Every function returns the library's status first; binding.py turns it into an exception.
#include <Python.h>
#include <ATen/ATen.h>
#include <torch/csrc/autograd/python_variable.h>

#include <vector>

#include "../../include/lstm_abi.h"

namespace {

struct Abi {
  decltype(&lstm_query) query;
  decltype(&lstm_fwd) fwd;
  decltype(&blstm_fwd) bfwd;
  decltype(&lstm_bwd) bwd;
  decltype(&blstm_bwd) bbwd;
  decltype(&lstm_gemm) gemm;
  decltype(&lstm_attention_query) att_query;
  decltype(&lstm_attention_step) att_step;
  decltype(&lstm_readout_query) ro_query;
  decltype(&lstm_readout) ro;
  decltype(&lstm_beam_query) beam_query;
  decltype(&lstm_beam_step) beam;
  decltype(&lstm_beam_gather_many) gather_many;
  decltype(&lstm_embed) embed;
  decltype(&lstm_time_pool_fwd) pool_fwd;
  decltype(&lstm_time_pool_bwd) pool_bwd;
} abi;

struct Failed {};                                   // a Python exception is set

[[noreturn]] void fail(PyObject* type, const char* what) {
  PyErr_SetString(type, what);
  throw Failed();
}
void require(bool ok, const char* what) {
  if (!ok) fail(PyExc_AssertionError, what);
}
const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) fail(PyExc_TypeError, "expected a torch.Tensor");
  return THPVariable_Unpack(o);
}
// address of an optional tensor that crosses the ABI whole (an address given as a number passes through)
void* ptr(PyObject* o) {
  if (o == Py_None) return nullptr;
  if (PyLong_Check(o)) {
    void* p = PyLong_AsVoidPtr(o);
    if (PyErr_Occurred()) throw Failed();
    return p;
  }
  const at::Tensor& t = tensor(o);
  require(t.is_contiguous(), "tensors crossing the ABI must be contiguous");
  return t.data_ptr();
}
long integer(PyObject* o) {
  const long v = PyLong_AsLong(o);
  if (v == -1 && PyErr_Occurred()) throw Failed();
  return v;
}
bool truth(PyObject* o) {
  const int v = PyObject_IsTrue(o);
  if (v < 0) throw Failed();
  return v != 0;
}
void* stream_of(PyObject* o) {
  void* p = PyLong_AsVoidPtr(o);
  if (!p && PyErr_Occurred()) throw Failed();
  return p;
}
// calls an entry point without the interpreter lock (enqueueing may have to wait for room in the stream's queue)
struct Unlocked {
  PyThreadState* state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};
template <typename F, typename... A>
int call(F f, A... args) {
  Unlocked u;
  return f(args...);
}
PyObject* wrapped(const at::Tensor& t) {
  if (!t.defined()) Py_RETURN_NONE;
  return THPVariable_Wrap(t);
}
int storage(const at::Tensor& x) { return x.scalar_type() == at::kBFloat16 ? LSTM_BF16_F32STATE : LSTM_F32; }
at::Tensor bytes_like(const at::Tensor& x, int64_t n) { return at::empty({n}, x.options().dtype(at::kByte)); }
// `o` if it is a tensor of at least `need` elements, otherwise a new byte tensor
at::Tensor workspace_of(PyObject* o, const at::Tensor& like, uint64_t need) {
  if (o != Py_None) {
    const at::Tensor& t = tensor(o);
    if ((uint64_t)t.numel() >= need) {
      require(t.is_contiguous(), "tensors crossing the ABI must be contiguous");
      return t;
    }
  }
  return bytes_like(like, (int64_t)need);
}

template <int N, typename F>
PyObject* guarded(Py_ssize_t nargs, F&& body) {
  try {
    if (nargs != N) fail(PyExc_TypeError, "wrong number of arguments");
    return body();
  } catch (const Failed&) {
    return nullptr;
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}
#define FAST(name) PyObject* name(PyObject*, PyObject* const* a, Py_ssize_t nargs)

// x W_x W_h b h0 c0 lens | bidirectional direction flags workspace want_c want_state poison stream
//   -> (status, y, c, hT, cT, reserve, workspace, reserve bytes)
FAST(forward) {
  return guarded<15>(nargs, [&]() -> PyObject* {
    const at::Tensor &x = tensor(a[0]), &W_h = tensor(a[2]);
    require(x.dim() == 3 && W_h.dim() >= 2, "x is [T, B, n_in]");
    const int64_t T = x.size(0), B = x.size(1), n_in = x.size(2), n = W_h.size(-2);
    const bool both = truth(a[7]), want_c = truth(a[11]), want_state = truth(a[12]), poison = truth(a[13]);
    const int flags = (int)integer(a[9]);
    const bool infer = flags & LSTM_FLAG_INFERENCE;
    lstm_desc d = {(int32_t)T, (int32_t)B, (int32_t)n_in, (int32_t)n, (int32_t)integer(a[8]), storage(x), flags, 0, 0, 0};
    size_t rb = 0, wb = 0;
    int rc = abi.query(&d, both, &rb, &wb);
    if (rc) return Py_BuildValue("(i)", rc);
    at::Tensor reserve = infer ? at::Tensor() : bytes_like(x, (int64_t)rb), ws = workspace_of(a[10], x, wb);
    if (poison) {                                    // tests: every byte the library has not written reads as NaN
      ws.fill_(0xFF);
      if (!infer) reserve.fill_(0xFF);
    }
    d.reserve_bytes = infer ? 0 : rb;
    d.workspace_bytes = (uint64_t)ws.numel();
    const auto f32 = x.options().dtype(at::kFloat);
    const at::Tensor y = at::empty({T, B, both ? 2 * n : n}, x.options());
    at::Tensor c, hT, cT;
    if (want_c || !infer) c = both ? at::empty({2, T, B, n}, f32) : at::empty({T, B, n}, f32);
    if (want_state) {
      hT = both ? at::empty({2, B, n}, f32) : at::empty({B, n}, f32);
      cT = both ? at::empty({2, B, n}, f32) : at::empty({B, n}, f32);
    }
    const auto p = [](const at::Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; };
    rc = call(both ? abi.bfwd : abi.fwd, &d, ptr(a[0]), ptr(a[1]), ptr(a[2]), ptr(a[3]), ptr(a[4]), ptr(a[5]), (const int32_t*)ptr(a[6]), p(y),
                                     p(c), p(hT), p(cT), p(reserve), p(ws), stream_of(a[14]));
    return Py_BuildValue("(iNNNNNNK)", rc, wrapped(y), wrapped(c), wrapped(hT), wrapped(cT), wrapped(reserve), wrapped(ws),
                         (unsigned long long)(infer ? 0 : rb));
  });
}

// desc (address) bidirectional | x W_x W_h h0 c0 lens y c reserve dy dhT dcT | dW_x dW_h db (or None) | want_dx want_dstate workspace stream
//   -> (status, dx, dW_x, dW_h, db, dh0, dc0)
FAST(backward) {
  return guarded<21>(nargs, [&]() -> PyObject* {
    const lstm_desc* d = (const lstm_desc*)PyLong_AsVoidPtr(a[0]);
    if (!d) fail(PyExc_TypeError, "no descriptor");
    const bool both = truth(a[1]);
    const at::Tensor &x = tensor(a[2]), &W_x = tensor(a[3]), &W_h = tensor(a[4]);
    require(x.dim() == 3 && W_h.dim() >= 2 && W_x.dim() >= 2, "x is [T, B, n_in]");
    const int64_t B = x.size(1), n = W_h.size(-2);
    const auto f32 = x.options().dtype(at::kFloat);
    at::Tensor dW_x, dW_h, db, dx, dh0, dc0;
    if (a[14] != Py_None) {
      dW_x = tensor(a[14]); dW_h = tensor(a[15]); db = tensor(a[16]);
    } else {
      dW_x = at::empty(W_x.sizes(), f32);
      dW_h = at::empty(W_h.sizes(), f32);
      auto shape = W_x.sizes().vec();
      shape.pop_back();
      shape.back() = 4 * n;
      db = at::empty(shape, f32);
    }
    if (truth(a[17])) dx = at::empty_like(x);
    if (truth(a[18])) {
      dh0 = both ? at::empty({2, B, n}, f32) : at::empty({B, n}, f32);
      dc0 = both ? at::empty({2, B, n}, f32) : at::empty({B, n}, f32);
    }
    const auto p = [](const at::Tensor& t) {
      if (!t.defined()) return (void*)nullptr;
      require(t.is_contiguous(), "tensors crossing the ABI must be contiguous");
      return t.data_ptr();
    };
    const int rc = call(both ? abi.bbwd : abi.bwd, d, ptr(a[2]), ptr(a[3]), ptr(a[4]), ptr(a[5]), ptr(a[6]), (const int32_t*)ptr(a[7]), ptr(a[8]),
                                               ptr(a[9]), ptr(a[10]), ptr(a[11]), ptr(a[12]), ptr(a[13]), p(dx), p(dW_x), p(dW_h), p(db),
                                               p(dh0), p(dc0), ptr(a[19]), stream_of(a[20]));
    return Py_BuildValue("(iNNNNNN)", rc, wrapped(dx), wrapped(dW_x), wrapped(dW_h), wrapped(db), wrapped(dh0), wrapped(dc0));
  });
}

// A B C bias lens | a_kcontig b_kcontig M N K accumulate Bt T out_bf16 stream  -> (status, C)
FAST(gemm) {
  return guarded<15>(nargs, [&]() -> PyObject* {
    const at::Tensor &A = tensor(a[0]), &B = tensor(a[1]);
    const bool in_bf16 = A.scalar_type() == at::kBFloat16;
    const long M = integer(a[7]), N = integer(a[8]), K = integer(a[9]);
    at::Tensor C = a[2] != Py_None ? tensor(a[2]) : at::empty({M, N}, A.options().dtype(truth(a[13]) ? at::kBFloat16 : at::kFloat));
    require(A.is_contiguous() && B.is_contiguous() && C.is_contiguous(), "tensors crossing the ABI must be contiguous");
    const int rc = call(abi.gemm, in_bf16, C.scalar_type() == at::kBFloat16, truth(a[5]), truth(a[6]), (int)M, (int)N, (int)K, A.data_ptr(), A.stride(0),
                            B.data_ptr(), B.stride(0), C.data_ptr(), C.stride(0), (const float*)ptr(a[3]), truth(a[10]), (const int32_t*)ptr(a[4]),
                            (int)integer(a[11]), (int)integer(a[12]), stream_of(a[14]));
    return Py_BuildValue("(iN)", rc, wrapped(C));
  });
}

// enc enc_ctx src_lens beam s W_s b_s w_fb b_fb v b_e accum | att workspace want_a stream  -> (status, a, accum, att, workspace)
FAST(attention_step) {
  return guarded<16>(nargs, [&]() -> PyObject* {
    const at::Tensor &enc = tensor(a[0]), &ctx = tensor(a[1]), &s = tensor(a[4]), &accum = tensor(a[11]);
    require(enc.dim() == 3 && ctx.dim() == 3 && s.dim() == 2, "enc is [S, Q, E], enc_ctx [S, Q, A], s [B, n]");
    const int64_t S = enc.size(0), Q = enc.size(1), E = enc.size(2), A = ctx.size(2), B = s.size(0), n = s.size(1);
    lstm_att_desc d = {(int32_t)S, (int32_t)Q, (int32_t)integer(a[3]), (int32_t)A, (int32_t)E, (int32_t)n, 0};
    uint64_t need = 0;
    int rc = abi.att_query(&d, &need);
    if (rc) return Py_BuildValue("(i)", rc);
    const at::Tensor ws = workspace_of(a[13], enc, need);
    d.workspace_bytes = (uint64_t)ws.numel();
    const auto f32 = enc.options().dtype(at::kFloat);
    at::Tensor att = a[12] != Py_None ? tensor(a[12]) : at::empty({B, E}, enc.options().dtype(at::kBFloat16)), w;
    if (truth(a[14])) w = at::empty({B, S}, f32);
    const at::Tensor out = at::empty({B, S}, f32);
    require(enc.is_contiguous() && ctx.is_contiguous() && accum.is_contiguous() && s.stride(1) == 1 && att.stride(1) == 1,
            "enc, enc_ctx and accum are contiguous, s and att have contiguous rows");
    const double b_e = PyFloat_AsDouble(a[10]);
    if (b_e == -1.0 && PyErr_Occurred()) throw Failed();
    rc = call(abi.att_step, &d, enc.data_ptr(), ctx.data_ptr(), (const int32_t*)ptr(a[2]), s.data_ptr(), s.stride(0), ptr(a[5]), (const float*)ptr(a[6]),
                      (const float*)ptr(a[7]), (const float*)ptr(a[8]), (const float*)ptr(a[9]), (float)b_e, (const float*)accum.data_ptr(),
                      (float*)out.data_ptr(), w.defined() ? (float*)w.data_ptr() : nullptr, att.data_ptr(), att.stride(0), ws.data_ptr(),
                      stream_of(a[15]));
    return Py_BuildValue("(iNNNN)", rc, wrapped(w), wrapped(out), wrapped(att), wrapped(ws));
  });
}

// s trg att W_r b_r | out workspace flags stream  -> (status, out)
FAST(readout) {
  return guarded<9>(nargs, [&]() -> PyObject* {
    const at::Tensor &s = tensor(a[0]), &trg = tensor(a[1]), &att = tensor(a[2]), &W = tensor(a[3]);
    require(s.dim() == 2 && trg.dim() == 2 && att.dim() == 2 && W.dim() == 2, "s, trg, att and W_r are matrices");
    const int64_t B = s.size(0), n = s.size(1), nt = trg.size(1), E = att.size(1), R = W.size(0);
    uint64_t need = 0;
    int rc = abi.ro_query((int)B, (int)R, (int)n, (int)nt, (int)E, &need);
    if (rc) return Py_BuildValue("(i)", rc);
    const at::Tensor ws = workspace_of(a[6], s, need);
    const at::Tensor out = a[5] != Py_None ? tensor(a[5]) : at::empty({B, R}, s.options().dtype(at::kBFloat16));
    require(s.stride(1) == 1 && trg.stride(1) == 1 && att.stride(1) == 1 && W.is_contiguous() && out.stride(1) == 1,
            "W_r is contiguous, the others have contiguous rows");
    rc = call(abi.ro, (int)integer(a[7]), (int)B, (int)R, s.data_ptr(), s.stride(0), (int)n, trg.data_ptr(), trg.stride(0), (int)nt, att.data_ptr(),
                att.stride(0), (int)E, W.data_ptr(), (const float*)ptr(a[4]), out.data_ptr(), out.stride(0), ws.data_ptr(), (uint64_t)ws.numel(),
                stream_of(a[8]));
    return Py_BuildValue("(iN)", rc, wrapped(out));
  });
}

// logits score | workspace stream  -> (status, score, src, label, workspace)
FAST(beam_step) {
  return guarded<4>(nargs, [&]() -> PyObject* {
    const at::Tensor &logits = tensor(a[0]), &score = tensor(a[1]);
    require(logits.dim() == 2 && score.dim() == 2, "logits and score are matrices");
    const int64_t Q = score.size(0), beam = score.size(1), V = logits.size(1);
    uint64_t need = 0;
    int rc = abi.beam_query((int)Q, (int)beam, (int)V, &need);
    if (rc) return Py_BuildValue("(i)", rc);
    const at::Tensor ws = workspace_of(a[2], logits, need);
    const auto i32 = logits.options().dtype(at::kInt);
    const at::Tensor out = at::empty({Q, beam}, logits.options().dtype(at::kFloat)), src = at::empty({Q, beam}, i32), label = at::empty({Q, beam}, i32);
    require(logits.stride(1) == 1 && logits.scalar_type() == at::kFloat && score.scalar_type() == at::kFloat, "logits and score are float");
    rc = call(abi.beam, (int)Q, (int)beam, (int)V, (const float*)logits.data_ptr(), logits.stride(0), (const float*)ptr(a[1]), (float*)out.data_ptr(),
                  (int32_t*)src.data_ptr(), (int32_t*)label.data_ptr(), ws.data_ptr(), (uint64_t)ws.numel(), stream_of(a[3]));
    return Py_BuildValue("(iNNNN)", rc, wrapped(out), wrapped(src), wrapped(label), wrapped(ws));
  });
}

// states outs (sequences of the same length) src stream  -> status
FAST(gather_many) {
  return guarded<4>(nargs, [&]() -> PyObject* {
    const Py_ssize_t count = PySequence_Size(a[0]);
    if (count < 0) throw Failed();
    std::vector<lstm_gather_item> item(count);
    std::vector<at::Tensor> held;                    // (a sequence may make its items on access)
    held.reserve(2 * count);
    const auto item_of = [&](PyObject* seq, Py_ssize_t i) -> const at::Tensor& {
      struct Ref { PyObject* o; ~Ref() { Py_XDECREF(o); } } ref{PySequence_GetItem(seq, i)};
      if (!ref.o) throw Failed();
      held.push_back(tensor(ref.o));
      return held.back();
    };
    const at::Tensor& src = tensor(a[2]);
    require(src.dim() == 2 && PySequence_Size(a[1]) == count, "src is [Q, beam], one output per state");
    for (Py_ssize_t i = 0; i < count; ++i) {
      const at::Tensor &in = item_of(a[0], i), &out = item_of(a[1], i);
      require(in.dim() == 2 && in.stride(1) == 1 && out.dim() == 2 && out.stride(1) == 1 && in.scalar_type() == out.scalar_type() &&
                  in.sizes() == out.sizes(), "states are matrices with contiguous rows, outputs like them");
      item[i] = {(int32_t)in.element_size(), (int32_t)in.size(1), in.data_ptr(), in.stride(0), out.data_ptr(), out.stride(0)};
    }
    return PyLong_FromLong(call(abi.gather_many, (int)src.size(0), (int)src.size(1), (int)count, item.data(), (const int32_t*)ptr(a[2]), stream_of(a[3])));
  });
}

// label W_trg b_trg out stream  -> (status, out)
FAST(embed) {
  return guarded<5>(nargs, [&]() -> PyObject* {
    const at::Tensor &label = tensor(a[0]), &W = tensor(a[1]);
    require(W.dim() == 2, "W_trg is [V, n]");
    const int64_t B = label.numel(), n = W.size(1);
    const at::Tensor out = a[3] != Py_None ? tensor(a[3]) : at::empty({B, n}, W.options().dtype(at::kBFloat16));
    const int rc = call(abi.embed, (int)B, (int)n, (int)W.size(0), (const int32_t*)ptr(a[0]), ptr(a[1]), (const float*)ptr(a[2]), out.data_ptr(), out.stride(0),
                             stream_of(a[4]));
    return Py_BuildValue("(iN)", rc, wrapped(out));
  });
}

// y lens pool want_arg stream  -> (status, out, lens, arg)
FAST(time_pool_fwd) {
  return guarded<5>(nargs, [&]() -> PyObject* {
    const at::Tensor& y = tensor(a[0]);
    require(y.dim() == 3, "y is [T, B, F]");
    const int64_t T = y.size(0), B = y.size(1), F = y.size(2), pool = integer(a[2]);
    if (pool == 0) fail(PyExc_ZeroDivisionError, "pool is 0");
    require(y.stride(2) == 1 && y.stride(0) == B * y.stride(1), "frames of y follow each other with contiguous rows");
    const int64_t Tp = pool > 0 ? (T + pool - 1) / pool : 0;
    const at::Tensor out = at::empty({Tp, B, F}, y.options()), lens = at::empty({B}, y.options().dtype(at::kInt));
    at::Tensor arg;
    if (truth(a[3])) arg = at::empty({Tp, B, F}, y.options().dtype(at::kByte));
    const int rc = call(abi.pool_fwd, storage(y), (int)T, (int)B, (int)F, (int)pool, y.data_ptr(), y.stride(1), (const int32_t*)ptr(a[1]), out.data_ptr(), F,
                                arg.defined() ? (uint8_t*)arg.data_ptr() : nullptr, (int32_t*)lens.data_ptr(), stream_of(a[4]));
    return Py_BuildValue("(iNNN)", rc, wrapped(out), wrapped(lens), wrapped(arg));
  });
}

// dout arg lens pool T stream  -> (status, dy)
FAST(time_pool_bwd) {
  return guarded<6>(nargs, [&]() -> PyObject* {
    const at::Tensor& dout = tensor(a[0]);
    require(dout.dim() == 3 && dout.is_contiguous(), "dout is [T', B, F], contiguous");
    const int64_t B = dout.size(1), F = dout.size(2), T = integer(a[4]);
    const at::Tensor dy = at::empty({T, B, F}, dout.options());
    const int rc = call(abi.pool_bwd, storage(dout), (int)T, (int)B, (int)F, (int)integer(a[3]), dout.data_ptr(), F, (const uint8_t*)ptr(a[1]),
                                (const int32_t*)ptr(a[2]), dy.data_ptr(), F, stream_of(a[5]));
    return Py_BuildValue("(iN)", rc, wrapped(dy));
  });
}

// dict: entry point name -> address
PyObject* bind(PyObject*, PyObject* table) {
  const auto at_name = [&](const char* name) -> void* {
    PyObject* v = PyDict_Check(table) ? PyDict_GetItemString(table, name) : nullptr;
    return v ? PyLong_AsVoidPtr(v) : nullptr;
  };
  struct { void** slot; const char* name; } want[] = {
      {(void**)&abi.query, "lstm_query"}, {(void**)&abi.fwd, "lstm_fwd"}, {(void**)&abi.bfwd, "blstm_fwd"}, {(void**)&abi.bwd, "lstm_bwd"},
      {(void**)&abi.bbwd, "blstm_bwd"}, {(void**)&abi.gemm, "lstm_gemm"}, {(void**)&abi.att_query, "lstm_attention_query"},
      {(void**)&abi.att_step, "lstm_attention_step"}, {(void**)&abi.ro_query, "lstm_readout_query"}, {(void**)&abi.ro, "lstm_readout"},
      {(void**)&abi.beam_query, "lstm_beam_query"}, {(void**)&abi.beam, "lstm_beam_step"}, {(void**)&abi.gather_many, "lstm_beam_gather_many"},
      {(void**)&abi.embed, "lstm_embed"}, {(void**)&abi.pool_fwd, "lstm_time_pool_fwd"}, {(void**)&abi.pool_bwd, "lstm_time_pool_bwd"}};
  for (auto& w : want) {
    *w.slot = at_name(w.name);
    if (!*w.slot) {
      PyErr_Format(PyExc_ImportError, "the library has no entry point %s", w.name);
      return nullptr;
    }
  }
  Py_RETURN_NONE;
}

#define ENTRY(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"bind", bind, METH_O, nullptr}, ENTRY(forward), ENTRY(backward), ENTRY(gemm), ENTRY(attention_step), ENTRY(readout),
                         ENTRY(beam_step), ENTRY(gather_many), ENTRY(embed), ENTRY(time_pool_fwd), ENTRY(time_pool_bwd), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
