// Native marshalling of the Python binding's calls (spot.py): checks the
// tensors and passes raw pointers, sizes and the stream to libspot's C entry
// points.
//
// A call from Python cost 13-17 us of host time, more than the kernels of a
// short decode step or a front end take: per tensor five attribute look-ups
// (0.4 us), the current stream object (3 us) and ctypes' conversions.  Here a
// tensor costs tens of nanoseconds; a fused step of 24 arguments is issued
// in about a quarter of the time.
//
// Every function mirrors the Python function of the same name, argument by
// argument, and accepts only what that function would pass on: exact
// torch.Tensor objects on the device, contiguous, 16-byte aligned, of an
// allowed type and large enough, and plain ints and floats in range.  For
// anything else -- also where a check raises -- it returns None and nothing
// has been enqueued; the caller then takes the checked Python path, which
// accepts or raises as it always did.  Otherwise it returns the status.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "spot.h"

namespace {

// Read from the file before it is imported (build.py, binding_fits).
__attribute__((used)) const char kBuiltFor[] = "spot binding for torch " SPOT_TORCH;

// Entry points of the loaded libspot, in the order spot.py passes them.
enum Fn {
  kScore, kScoreQ, kScoreTokensBlk, kProject, kProjectPooled, kPool, kSelect, kSparseBlk, kDense,
  kPrefill, kStep, kStepQ, kStepStatic, kFns
};
void* g_fn[kFns];
PyObject* g_stream_type;    // torch.cuda.Stream
PyObject* g_stream_attr;    // "cuda_stream"

template <typename F>
F fn(Fn i, F) { return reinterpret_cast<F>(g_fn[i]); }

enum : unsigned { BF16 = 1, I16 = 2, I32 = 4, F32 = 8, U8 = 16, I8 = 32, F16 = 64, ANY = ~0u };
constexpr unsigned kBf = BF16 | I16;

unsigned dtype_bit(at::ScalarType t) {
  switch (t) {
    case at::kBFloat16: return BF16;
    case at::kShort: return I16;
    case at::kInt: return I32;
    case at::kFloat: return F32;
    case at::kByte: return U8;
    case at::kChar: return I8;
    case at::kHalf: return F16;
    default: return 0;
  }
}

// Element counts: products of up to four int sizes, which 64 bits cannot hold.
typedef __int128 big;

// The arguments of one call, taken in order; `ok` turns false at the first
// one that needs the Python path.
struct Args {
  PyObject* const* a;
  Py_ssize_t n, i = 0;
  bool ok = true;

  PyObject* next() {
    if (i >= n) ok = false;
    return ok ? a[i++] : nullptr;
  }
  int32_t integer() {
    PyObject* o = next();
    if (!o || !PyLong_Check(o)) return ok = false, 0;
    int over = 0;
    const long v = PyLong_AsLongAndOverflow(o, &over);
    if (over || v < INT32_MIN || v > INT32_MAX) return ok = false, 0;
    return (int32_t)v;
  }
  float real() {
    PyObject* o = next();
    if (!o) return 0.f;
    if (PyFloat_Check(o)) return (float)PyFloat_AS_DOUBLE(o);
    if (!PyLong_Check(o)) return ok = false, 0.f;
    const double v = PyLong_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) PyErr_Clear(), ok = false;
    return (float)v;
  }
  int format() {
    PyObject* o = next();
    if (!o) return 0;
    if (PyUnicode_Check(o)) {
      static const char* const names[] = {"bf16", "int4", "mxfp4", "int8", "mxfp8"};
      for (int f = 0; f < 5; ++f)
        if (PyUnicode_CompareWithASCIIString(o, names[f]) == 0) return f;
      return ok = false, 0;
    }
    --i;
    return integer();
  }
  void* stream() {
    PyObject* o = next();
    if (!o) return nullptr;
    if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
    if ((PyObject*)Py_TYPE(o) != g_stream_type) return ok = false, nullptr;
    PyObject* v = PyObject_GetAttr(o, g_stream_attr);
    void* p = v ? PyLong_AsVoidPtr(v) : nullptr;
    Py_XDECREF(v);
    if (PyErr_Occurred()) PyErr_Clear(), ok = false;
    return p;
  }
};

// A tensor argument; its checks come once the sizes are known.
struct Dev {
  PyObject* o;
  explicit Dev(Args& a) : o(a.next()) {}
  bool none() const { return o == Py_None; }
  // The device pointer, `numel` elements of one of `types` checked.
  void* ptr(Args& a, unsigned types, big numel) const {
    if (!a.ok || !THPVariable_CheckExact(o)) return a.ok = false, nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous() ||
        (types != ANY && !(dtype_bit(t.scalar_type()) & types)) || t.numel() < numel)
      return a.ok = false, nullptr;
    void* p = t.data_ptr();
    if (reinterpret_cast<uintptr_t>(p) & 15u) a.ok = false;
    return p;
  }
  void* opt(Args& a, unsigned types, big numel) const {
    return none() ? nullptr : ptr(a, types, numel);
  }
  size_t bytes() const { return THPVariable_Unpack(o).nbytes(); }
};

// Selector keys or queries: n of h_s x d_s elements in format f, with scales.
struct Keys {
  Dev k, s;
  void *kp = nullptr, *sp = nullptr;
  Keys(const Dev& k_, const Dev& s_) : k(k_), s(s_) {}
  void take(Args& a, int f, big n, big hs, big ds) {
    if (f == 0) {
      kp = k.ptr(a, kBf, n * hs * ds);
      if (!s.none()) sp = s.ptr(a, ANY, 0);
      return;
    }
    kp = k.ptr(a, U8 | I8, n * (f == 3 || f == 4 ? hs * ds : hs * ds / 2));
    sp = s.ptr(a, f == 1 || f == 3 ? F16 | I16 : U8, n * hs * ds / 32);
  }
};

PyObject* python_path() { Py_RETURN_NONE; }

// Runs `call` without the GIL unless an argument needs the Python path.
template <typename Call>
PyObject* finish(const Args& a, const Call& call) {
  if (!a.ok || a.i != a.n) return python_path();
  spot_status st;
  Py_BEGIN_ALLOW_THREADS
  st = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

const int32_t* ip(void* p) { return static_cast<const int32_t*>(p); }
const float* fp(void* p) { return static_cast<const float*>(p); }

// q_sel, w, k_sel, k_scale, kfmt, n_seq, rows_per_seq, nblk, h_s, d_s, n_valid, scores, stream
PyObject* selector_score(Args a) {
  Dev q(a), w(a), k(a), ks(a);
  const int f = a.format(), ns = a.integer(), rps = a.integer(), nb = a.integer(),
            hs = a.integer(), ds = a.integer();
  Dev nv(a), out(a);
  void* st = a.stream();
  const big rows = (big)ns * rps;
  Keys key(k, ks);
  void* qp = q.ptr(a, kBf, rows * hs * ds);
  void* wp = w.ptr(a, F32, rows * hs);
  if (a.ok) key.take(a, f, (big)ns * nb, hs, ds);
  void* nvp = nv.opt(a, I32, rows);
  void* op = out.ptr(a, F32, rows * nb);
  return finish(a, [&] {
    return fn(kScore, &spot_selector_score)(qp, fp(wp), key.kp, key.sp, f, ns, rps, nb, hs, ds,
                                            ip(nvp), static_cast<float*>(op), st);
  });
}

// q_sel, q_scale, qfmt, w, k_sel, k_scale, kfmt, n_seq, rows_per_seq, nblk, h_s, d_s, n_valid,
// scores, stream
PyObject* selector_score_q(Args a) {
  Dev q(a), qs(a);
  const int qf = a.format();
  Dev w(a), k(a), ks(a);
  const int f = a.format(), ns = a.integer(), rps = a.integer(), nb = a.integer(),
            hs = a.integer(), ds = a.integer();
  Dev nv(a), out(a);
  void* st = a.stream();
  const big rows = (big)ns * rps;
  Keys qk(q, qs), key(k, ks);
  if (a.ok) qk.take(a, qf, rows, hs, ds);
  void* wp = w.ptr(a, F32, rows * hs);
  if (a.ok) key.take(a, f, (big)ns * nb, hs, ds);
  void* nvp = nv.opt(a, I32, rows);
  void* op = out.ptr(a, F32, rows * nb);
  return finish(a, [&] {
    return fn(kScoreQ, &spot_selector_score_q)(qk.kp, qk.sp, qf, fp(wp), key.kp, key.sp, f, ns,
                                               rps, nb, hs, ds, ip(nvp), static_cast<float*>(op),
                                               st);
  });
}

// q_sel, w, k_tok, k_scale, kfmt, n_seq, rows_per_seq, l_cap, blk, h_s, d_s, seq_len, scores,
// stream
PyObject* selector_score_tokens_blk(Args a) {
  Dev q(a), w(a), k(a), ks(a);
  const int f = a.format(), ns = a.integer(), rps = a.integer(), lc = a.integer(),
            blk = a.integer(), hs = a.integer(), ds = a.integer();
  Dev sl(a), out(a);
  void* st = a.stream();
  const big rows = (big)ns * rps;
  Keys key(k, ks);
  if (blk < 1 || lc < 0) a.ok = false;
  void* qp = q.ptr(a, kBf, rows * hs * ds);
  void* wp = w.ptr(a, F32, rows * hs);
  if (a.ok) key.take(a, f, (big)ns * lc, hs, ds);
  void* slp = sl.opt(a, I32, rows);
  void* op = a.ok ? out.ptr(a, F32, rows * (lc / blk)) : nullptr;
  return finish(a, [&] {
    return fn(kScoreTokensBlk, &spot_selector_score_tokens_blk)(
        qp, fp(wp), key.kp, key.sp, f, ns, rps, lc, blk, hs, ds, ip(slp),
        static_cast<float*>(op), st);
  });
}

// h, w_q, w_k, w_w, pos, rows, d_model, h_s, d_s, rope_dim, rope_base, q_out, w_out, k_cache,
// rows_per_seq, l_cap, stream
PyObject* selector_project(Args a) {
  Dev h(a), wq(a), wk(a), ww(a), pos(a);
  const int rows = a.integer(), dm = a.integer(), hs = a.integer(), ds = a.integer(),
            rope = a.integer();
  const float base = a.real();
  Dev qo(a), wo(a), kc(a);
  const int rps = a.integer(), lc = a.integer();
  void* st = a.stream();
  if (rows < 0) a.ok = false;
  const big n = (big)hs * ds;
  void *hp = h.ptr(a, kBf, (big)rows * dm), *wqp = wq.ptr(a, kBf, n * dm),
       *wkp = wk.ptr(a, kBf, n * dm), *wwp = ww.ptr(a, kBf, (big)hs * dm),
       *pp = pos.ptr(a, I32, rows), *qop = qo.ptr(a, kBf, (big)rows * n),
       *wop = wo.ptr(a, F32, (big)rows * hs),
       *kcp = kc.ptr(a, kBf, (big)(rows / (rps > 1 ? rps : 1)) * lc * n);
  return finish(a, [&] {
    return fn(kProject, &spot_selector_project)(hp, wqp, wkp, wwp, ip(pp), rows, dm, hs, ds, rope,
                                                base, qop, static_cast<float*>(wop), kcp, rps, lc,
                                                st);
  });
}

// h, w_q, w_k, w_w, pos, seq_len, n_seq, d_model, h_s, d_s, rope_dim, rope_base, q_out, w_out,
// k_cache, k_pool, l_cap, stream
PyObject* selector_project_pooled(Args a) {
  Dev h(a), wq(a), wk(a), ww(a), pos(a), sl(a);
  const int ns = a.integer(), dm = a.integer(), hs = a.integer(), ds = a.integer(),
            rope = a.integer();
  const float base = a.real();
  Dev qo(a), wo(a), kc(a), kp(a);
  const int lc = a.integer();
  void* st = a.stream();
  if (lc < 0) a.ok = false;
  const big n = (big)hs * ds;
  void *hp = h.ptr(a, kBf, (big)ns * dm), *wqp = wq.ptr(a, kBf, n * dm),
       *wkp = wk.ptr(a, kBf, n * dm), *wwp = ww.ptr(a, kBf, (big)hs * dm),
       *pp = pos.ptr(a, I32, ns), *slp = sl.opt(a, I32, ns), *qop = qo.ptr(a, kBf, (big)ns * n),
       *wop = wo.ptr(a, F32, (big)ns * hs), *kcp = kc.ptr(a, kBf, (big)ns * lc * n),
       *kpp = kp.ptr(a, kBf, (big)ns * (lc / 64) * n);
  return finish(a, [&] {
    return fn(kProjectPooled, &spot_selector_project_pooled)(
        hp, wqp, wkp, wwp, ip(pp), ip(slp), ns, dm, hs, ds, rope, base, qop,
        static_cast<float*>(wop), kcp, kpp, lc, st);
  });
}

// k_tok, k_pool, n_seq, l_cap, h_s, d_s, seq_len, first_block, max_blocks, stream
PyObject* selector_pool(Args a) {
  Dev kt(a), kp(a);
  const int ns = a.integer(), lc = a.integer(), hs = a.integer(), ds = a.integer();
  Dev sl(a), fb(a);
  PyObject* mb = a.next();
  int max_blocks = 0;
  if (mb == Py_None)
    max_blocks = lc / 64;
  else if (mb)
    --a.i, max_blocks = a.integer();
  void* st = a.stream();
  if (lc < 0) a.ok = false;
  const big n = (big)hs * ds;
  void *ktp = kt.ptr(a, kBf, (big)ns * lc * n), *kpp = kp.ptr(a, kBf, (big)ns * (lc / 64) * n),
       *slp = sl.opt(a, I32, ns), *fbp = fb.opt(a, I32, ns);
  return finish(a, [&] {
    return fn(kPool, &spot_selector_pool)(ktp, kpp, ns, lc, hs, ds, ip(slp), ip(fbp), max_blocks,
                                          st);
  });
}

// scores, rows, nblk, n_valid, top_p, k_max, k_min, n_sink, n_recent, idx, count, nuc_mass, stream
PyObject* select_blocks(Args a) {
  Dev sc(a);
  const int rows = a.integer(), nb = a.integer();
  Dev nv(a);
  const float p = a.real();
  const int kmax = a.integer(), kmin = a.integer(), sink = a.integer(), rec = a.integer();
  Dev idx(a), cnt(a), mass(a);
  void* st = a.stream();
  void *scp = sc.ptr(a, F32, (big)rows * nb), *nvp = nv.opt(a, I32, rows),
       *ixp = idx.ptr(a, I32, (big)rows * kmax), *cp = cnt.ptr(a, I32, rows),
       *mp = mass.opt(a, F32, rows);
  return finish(a, [&] {
    return fn(kSelect, &spot_select_blocks)(fp(scp), rows, nb, ip(nvp), p, kmax, kmin, sink, rec,
                                            static_cast<int32_t*>(ixp), static_cast<int32_t*>(cp),
                                            static_cast<float*>(mp), st);
  });
}

// q, k, v, seq_len, idx, count, k_max, blk, batch, h_q, h_kv, d, l_cap, sm_scale, out, lse, ws,
// stream
PyObject* sparse_decode_blk(Args a) {
  Dev q(a), k(a), v(a), sl(a), idx(a), cnt(a);
  const int kmax = a.integer(), blk = a.integer(), b = a.integer(), hq = a.integer(),
            hkv = a.integer(), d = a.integer(), lc = a.integer();
  const float scale = a.real();
  Dev out(a), lse(a), ws(a);
  void* st = a.stream();
  const big kv = (big)b * hkv * lc * d, qn = (big)b * hq * d;
  void *qp = q.ptr(a, kBf, qn), *kp = k.ptr(a, kBf, kv), *vp = v.ptr(a, kBf, kv),
       *slp = sl.ptr(a, I32, b), *ixp = idx.ptr(a, I32, (big)b * kmax), *cp = cnt.ptr(a, I32, b),
       *op = out.ptr(a, kBf, qn), *lp = lse.opt(a, F32, (big)b * hq), *wp = ws.ptr(a, ANY, 0);
  const size_t wb = a.ok ? ws.bytes() : 0;
  return finish(a, [&] {
    return fn(kSparseBlk, &spot_sparse_decode_blk)(qp, kp, vp, ip(slp), ip(ixp), ip(cp), kmax, blk,
                                                   b, hq, hkv, d, lc, scale, op,
                                                   static_cast<float*>(lp), wp, wb, st);
  });
}

// q, k, v, seq_len, batch, h_q, h_kv, d, l_cap, sm_scale, out, lse, ws, stream
PyObject* dense_decode(Args a) {
  Dev q(a), k(a), v(a), sl(a);
  const int b = a.integer(), hq = a.integer(), hkv = a.integer(), d = a.integer(),
            lc = a.integer();
  const float scale = a.real();
  Dev out(a), lse(a), ws(a);
  void* st = a.stream();
  const big kv = (big)b * hkv * lc * d, qn = (big)b * hq * d;
  void *qp = q.ptr(a, kBf, qn), *kp = k.ptr(a, kBf, kv), *vp = v.ptr(a, kBf, kv),
       *slp = sl.ptr(a, I32, b), *op = out.ptr(a, kBf, qn),
       *lp = lse.opt(a, F32, (big)b * hq), *wp = ws.ptr(a, ANY, 0);
  const size_t wb = a.ok ? ws.bytes() : 0;
  return finish(a, [&] {
    return fn(kDense, &spot_dense_decode)(qp, kp, vp, ip(slp), b, hq, hkv, d, lc, scale, op,
                                          static_cast<float*>(lp), wp, wb, st);
  });
}

// q, k, v, L, idx, count, k_max, batch, h_q, h_kv, d, sm_scale, out, lse, stream
PyObject* sparse_prefill(Args a) {
  Dev q(a), k(a), v(a);
  const int L = a.integer();
  Dev idx(a), cnt(a);
  const int kmax = a.integer(), b = a.integer(), hq = a.integer(), hkv = a.integer(),
            d = a.integer();
  const float scale = a.real();
  Dev out(a), lse(a);
  void* st = a.stream();
  if (L < 0) a.ok = false;
  const big rows = (big)b * (L / 64), kv = (big)b * hkv * L * d, qn = (big)b * hq * L * d;
  void *qp = q.ptr(a, kBf, qn), *kp = k.ptr(a, kBf, kv), *vp = v.ptr(a, kBf, kv),
       *ixp = idx.ptr(a, I32, rows * kmax), *cp = cnt.ptr(a, I32, rows),
       *op = out.ptr(a, kBf, qn), *lp = lse.opt(a, F32, (big)b * hq * L);
  return finish(a, [&] {
    return fn(kPrefill, &spot_sparse_prefill)(qp, kp, vp, L, ip(ixp), ip(cp), kmax, b, hq, hkv, d,
                                              scale, op, static_cast<float*>(lp), st);
  });
}

// The arguments spot_decode_step, _q and _static share, in spot.py's order:
// q_sel, w, k_sel, k_scale, kfmt, h_s, d_s, n_valid, top_p, k_max, k_min, n_sink, n_recent, q, k,
// v, seq_len, batch, h_q, h_kv, d, l_cap, sm_scale, scores, idx, count, nuc_mass, out, lse
struct Step {
  Dev q_sel, w, k_sel, k_scale;
  int f, hs, ds;
  Dev nv;
  float p;
  int kmax, kmin, sink, rec;
  Dev q, k, v, sl;
  int b, hq, hkv, d, lc;
  float scale;
  Dev scores, idx, cnt, mass, out, lse;
  void *wp, *nvp, *qp, *kp, *vp, *slp, *scp, *ixp, *cp, *mp, *op, *lp;

  explicit Step(Args& a)
      : q_sel(a), w(a), k_sel(a), k_scale(a), f(a.format()), hs(a.integer()), ds(a.integer()),
        nv(a), p(a.real()), kmax(a.integer()), kmin(a.integer()), sink(a.integer()),
        rec(a.integer()), q(a), k(a), v(a), sl(a), b(a.integer()), hq(a.integer()),
        hkv(a.integer()), d(a.integer()), lc(a.integer()), scale(a.real()), scores(a), idx(a),
        cnt(a), mass(a), out(a), lse(a) {}
  void take(Args& a) {
    if (lc < 0) a.ok = false;
    const big kv = (big)b * hkv * lc * d, qn = (big)b * hq * d, nb = lc / 64;
    wp = w.ptr(a, F32, (big)b * hs);
    nvp = nv.opt(a, I32, b);
    qp = q.ptr(a, kBf, qn);
    kp = k.ptr(a, kBf, kv);
    vp = v.ptr(a, kBf, kv);
    slp = sl.ptr(a, I32, b);
    scp = scores.ptr(a, F32, nb * b);
    ixp = idx.ptr(a, I32, (big)b * kmax);
    cp = cnt.ptr(a, I32, b);
    mp = mass.opt(a, F32, b);
    op = out.ptr(a, kBf, qn);
    lp = lse.opt(a, F32, (big)b * hq);
  }
};

// the shared arguments, ws, stream, q_scale, qfmt
PyObject* decode_step(Args a) {
  Step s(a);
  Dev ws(a);
  void* st = a.stream();
  Dev q_scale(a);
  const int qf = a.format();
  if (a.ok) s.take(a);
  Keys qk(s.q_sel, q_scale), key(s.k_sel, s.k_scale);
  if (a.ok) qk.take(a, qf, s.b, s.hs, s.ds);
  if (a.ok) key.take(a, s.f, (big)s.b * (s.lc / 64), s.hs, s.ds);
  void* wsp = a.ok ? ws.ptr(a, ANY, 0) : nullptr;
  const size_t wb = a.ok ? ws.bytes() : 0;
  return finish(a, [&] {
    if (qf == 0)
      return fn(kStep, &spot_decode_step)(
          qk.kp, fp(s.wp), key.kp, key.sp, s.f, s.hs, s.ds, ip(s.nvp), s.p, s.kmax, s.kmin, s.sink,
          s.rec, s.qp, s.kp, s.vp, ip(s.slp), s.b, s.hq, s.hkv, s.d, s.lc, s.scale,
          static_cast<float*>(s.scp), static_cast<int32_t*>(s.ixp), static_cast<int32_t*>(s.cp),
          static_cast<float*>(s.mp), s.op, static_cast<float*>(s.lp), wsp, wb, st);
    return fn(kStepQ, &spot_decode_step_q)(
        qk.kp, qk.sp, qf, fp(s.wp), key.kp, key.sp, s.f, s.hs, s.ds, ip(s.nvp), s.p, s.kmax,
        s.kmin, s.sink, s.rec, s.qp, s.kp, s.vp, ip(s.slp), s.b, s.hq, s.hkv, s.d, s.lc, s.scale,
        static_cast<float*>(s.scp), static_cast<int32_t*>(s.ixp), static_cast<int32_t*>(s.cp),
        static_cast<float*>(s.mp), s.op, static_cast<float*>(s.lp), wsp, wb, st);
  });
}

// the shared arguments, stream
PyObject* decode_step_static(Args a) {
  Step s(a);
  void* st = a.stream();
  if (a.ok) s.take(a);
  Keys key(s.k_sel, s.k_scale);
  if (a.ok) key.take(a, s.f, (big)s.b * (s.lc / 64), s.hs, s.ds);
  void* qp = a.ok ? s.q_sel.ptr(a, kBf, (big)s.b * s.hs * s.ds) : nullptr;
  return finish(a, [&] {
    return fn(kStepStatic, &spot_decode_step_static)(
        qp, fp(s.wp), key.kp, key.sp, s.f, s.hs, s.ds, ip(s.nvp), s.p, s.kmax, s.kmin, s.sink,
        s.rec, s.qp, s.kp, s.vp, ip(s.slp), s.b, s.hq, s.hkv, s.d, s.lc, s.scale,
        static_cast<float*>(s.scp), static_cast<int32_t*>(s.ixp), static_cast<int32_t*>(s.cp),
        static_cast<float*>(s.mp), s.op, static_cast<float*>(s.lp), st);
  });
}

// A tensor without storage or of a wrapped kind throws from its accessors:
// the Python path then raises as it always did.
template <PyObject* (*F)(Args)>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (!g_fn[0]) return python_path();
  try {
    return F(Args{args, n});
  } catch (...) {
    PyErr_Clear();
    return python_path();
  }
}

// init(addresses of the entry points in Fn's order, torch.cuda.Stream)
PyObject* init(PyObject*, PyObject* args) {
  PyObject *fns, *type;
  if (!PyArg_ParseTuple(args, "O!O", &PyTuple_Type, &fns, &type)) return nullptr;
  if (PyTuple_GET_SIZE(fns) != kFns) {
    PyErr_SetString(PyExc_ValueError, "init: wrong number of entry points");
    return nullptr;
  }
  void* p[kFns];
  for (int i = 0; i < kFns; ++i) {
    p[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(fns, i));
    if (PyErr_Occurred()) return nullptr;
  }
  Py_INCREF(type);
  g_stream_type = type;
  if (!g_stream_attr) g_stream_attr = PyUnicode_InternFromString("cuda_stream");
  for (int i = 0; i < kFns; ++i) g_fn[i] = p[i];
  Py_RETURN_NONE;
}

#define SPOT_ENTRY(f) {#f, (PyCFunction)(void (*)(void))entry<f>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"init", init, METH_VARARGS, nullptr},
                         SPOT_ENTRY(selector_score),
                         SPOT_ENTRY(selector_score_q),
                         SPOT_ENTRY(selector_score_tokens_blk),
                         SPOT_ENTRY(selector_project),
                         SPOT_ENTRY(selector_project_pooled),
                         SPOT_ENTRY(selector_pool),
                         SPOT_ENTRY(select_blocks),
                         SPOT_ENTRY(sparse_decode_blk),
                         SPOT_ENTRY(dense_decode),
                         SPOT_ENTRY(sparse_prefill),
                         SPOT_ENTRY(decode_step),
                         SPOT_ENTRY(decode_step_static),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
