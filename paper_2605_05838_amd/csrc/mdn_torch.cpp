// The entry points of binding.py, natively: argument checks, output allocation, stream and pointer marshalling for the
// C ABI of include/mdn.h.  A small call (a decode step: two loads and two stores of 1 MB) is 3.2 us of GPU time; with the
// same work done in Python over ctypes it took 12.9 us from call to call, here 4.4.
// Functions take every argument positionally (binding.py gives them their names and defaults) and raise
// binding.MdnError.  Nothing of the path runs here, and there is no CPU path: PyTorch supplies memory and the stream.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cmath>
#include <initializer_list>
#include <string>
#include <vector>

#include "../../include/mdn.h"

namespace {

PyObject *g_error = nullptr, *g_oom = nullptr; // binding.MdnError, torch.OutOfMemoryError

struct Fail {}; // the Python error is set

[[noreturn]] void fail(const std::string &what) {
    PyErr_SetString(g_error ? g_error : PyExc_RuntimeError, what.c_str());
    throw Fail{};
}

struct Ref { // an owned reference
    PyObject *p;
    explicit Ref(PyObject *o = nullptr) : p(o) {}
    Ref(const Ref &) = delete;
    Ref(Ref &&o) noexcept : p(o.p) { o.p = nullptr; }
    ~Ref() { Py_XDECREF(p); }
};

typedef const at::Tensor *Opt; // a tensor argument, or null for None

Opt opt(PyObject *o, const char *name) {
    if (!o || o == Py_None) return nullptr;
    if (!THPVariable_Check(o)) fail(std::string(name) + " must be a tensor");
    return &THPVariable_Unpack(o);
}
const at::Tensor &need(PyObject *o, const char *name) {
    Opt t = opt(o, name);
    if (!t) fail(std::string(name) + " is required");
    return *t;
}

std::string str(at::IntArrayRef s) {
    std::string r = "(";
    for (size_t i = 0; i < s.size(); ++i) r += (i ? ", " : "") + std::to_string(s[i]);
    return r + (s.size() == 1 ? ",)" : ")");
}
const char *dtype_name(at::ScalarType t) {
    switch (t) {
    case at::kFloat: return "torch.float32";
    case at::kBFloat16: return "torch.bfloat16";
    case at::kHalf: return "torch.float16";
    case at::kDouble: return "torch.float64";
    default: return c10::toString(t);
    }
}

// Shape, dtype, device and layout of one tensor against what the call's first tensor implies.  The C ABI takes raw
// pointers and trusts them: a tensor of the wrong size would be read or written out of bounds on the device, so every
// tensor is checked, before anything is launched.
void expect(const char *name, Opt t, std::initializer_list<int64_t> shape, at::ScalarType dtype, const at::Tensor &like) {
    if (!t) return;
    const at::IntArrayRef want(shape.begin(), shape.size());
    if (t->sizes() != want) fail(std::string(name) + ": expected shape " + str(want) + ", got " + str(t->sizes()));
    if (t->scalar_type() != dtype)
        fail(std::string(name) + ": expected dtype " + dtype_name(dtype) + ", got " + dtype_name(t->scalar_type()));
    if (t->device() != like.device())
        fail(std::string(name) + " is on " + t->device().str() + ", q on " + like.device().str() + ": all tensors of a call share one device");
    if (!t->is_contiguous()) fail(std::string(name) + " must be contiguous");
}
// An opaque buffer (workspace, kept states / operands): at least nbytes
void expect_bytes(const char *name, Opt t, size_t nbytes, const at::Tensor &like) {
    if (!t) return;
    const size_t have = (size_t)t->numel() * t->element_size();
    if (have < nbytes) fail(std::string(name) + ": " + std::to_string(have) + " bytes, the call needs " + std::to_string(nbytes));
    if (t->device() != like.device())
        fail(std::string(name) + " is on " + t->device().str() + ", q on " + like.device().str() + ": all tensors of a call share one device");
    if (!t->is_contiguous()) fail(std::string(name) + " must be contiguous");
}
// after the checks above one tensor stands for all of a call's
void on_gpu(const at::Tensor &t) {
    if (!t.is_cuda()) fail("MDN tensors must live on the GPU (no CPU path exists)");
}

int dtype_code(const at::Tensor &t) {
    if (t.scalar_type() == at::kBFloat16) return MDN_DTYPE_BF16;
    if (t.scalar_type() == at::kFloat) return MDN_DTYPE_F32;
    fail("q/k/v must be bfloat16 or float32");
}

// without the interpreter lock from here to the end of the scope, however it is left
struct Unlocked {
    PyThreadState *t = PyEval_SaveThread();
    Unlocked() = default;
    Unlocked(const Unlocked &) = delete;
    ~Unlocked() { PyEval_RestoreThread(t); }
};
void check(int rc, const char *what) {
    if (rc) fail(std::string(what) + ": " + mdn_strerror(rc) + " (code " + std::to_string(rc) + ")");
}
// The library call itself, without the interpreter lock (a launch may wait for room in the stream's queue).  The arguments
// are values by then: taking a pointer can raise (a tensor that has no storage), which needs the lock.
template <typename... P, typename... A> void call(const char *what, int (*f)(P...), A... args) {
    int rc;
    {
        const Unlocked u;
        rc = f(args...);
    }
    check(rc, what);
}

double number(PyObject *o) { // float(o)
    if (PyFloat_CheckExact(o)) return PyFloat_AS_DOUBLE(o);
    const Ref v(PyNumber_Float(o));
    if (!v.p) throw Fail{};
    return PyFloat_AS_DOUBLE(v.p);
}
long integer(PyObject *o) {
    const long v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) throw Fail{};
    return v;
}
bool truth(PyObject *o) {
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw Fail{};
    return v != 0;
}

void *stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

template <typename T = void> T *ptr(const at::Tensor &t) { return static_cast<T *>(t.data_ptr()); }
template <typename T = void> T *ptr(Opt t) { return t ? static_cast<T *>(t->data_ptr()) : nullptr; }
template <typename T = void> T *ptr(const c10::optional<at::Tensor> &t) { return t ? static_cast<T *>(t->data_ptr()) : nullptr; }

at::Tensor empty(at::IntArrayRef shape, at::ScalarType dt, const at::Tensor &like) {
    return at::empty(shape, at::TensorOptions().dtype(dt).device(like.device()));
}
at::Tensor bytes(size_t n, const at::Tensor &like) { return empty({(int64_t)n}, at::kByte, like); }

// the result dict, filled key by key; `out`: the caller's tensors of an earlier call, or nothing
struct Dict {
    PyObject *d;
    Dict() : d(PyDict_New()) {
        if (!d) throw Fail{};
    }
    ~Dict() { Py_XDECREF(d); }
    void set(const char *key, const at::Tensor &t) {
        Ref v(THPVariable_Wrap(t));
        if (!v.p || PyDict_SetItemString(d, key, v.p) < 0) throw Fail{};
    }
    void set(const char *key, Opt t) { t ? set(key, *t) : none(key); }
    void set(const char *key, const c10::optional<at::Tensor> &t) { t ? set(key, *t) : none(key); }
    void none(const char *key) {
        if (PyDict_SetItemString(d, key, Py_None) < 0) throw Fail{};
    }
    PyObject *release() {
        PyObject *r = d;
        d = nullptr;
        return r;
    }
};
// out.get(key) of a dict (or of anything with a get method); None and absence alike give null
Ref out_get(PyObject *out, const char *key) {
    if (!out || out == Py_None) return Ref();
    PyObject *v;
    if (PyDict_Check(out)) {
        v = PyDict_GetItemString(out, key);
        Py_XINCREF(v);
    } else {
        v = PyObject_CallMethod(out, "get", "s", key);
        if (!v) throw Fail{};
    }
    if (v == Py_None) {
        Py_DECREF(v);
        v = nullptr;
    }
    return Ref(v);
}
// a caller's output tensor, checked, or a new one
at::Tensor output(PyObject *out, const char *key, std::initializer_list<int64_t> shape, at::ScalarType dt, const at::Tensor &like) {
    Ref r = out_get(out, key);
    if (!r.p) return empty(at::IntArrayRef(shape.begin(), shape.size()), dt, like);
    const std::string name = std::string("out['") + key + "']";
    const at::Tensor &t = need(r.p, name.c_str());
    expect(name.c_str(), &t, shape, dt, like);
    return t;
}
at::Tensor output_bytes(PyObject *out, const char *key, size_t n, const at::Tensor &like) {
    Ref r = out_get(out, key);
    if (!r.p) return bytes(n, like);
    const std::string name = std::string("out['") + key + "']";
    const at::Tensor &t = need(r.p, name.c_str());
    expect_bytes(name.c_str(), &t, n, like);
    return t;
}

// the inputs that every chunkwise / recurrent call takes, checked against q
struct Inputs {
    const at::Tensor &q, &k, &v, &beta, &alpha, &mu;
    Opt eta, S0, M0;
    mdn_shape s;
    at::ScalarType dt;
    int64_t B, T, H, dk, dv;
    // states_batch < 0: B
    Inputs(PyObject *const *x, PyObject *eta_, PyObject *S0_, PyObject *M0_, PyObject *scale, long C, int64_t states_batch = -1)
        : q(need(x[0], "q")), k(need(x[1], "k")), v(need(x[2], "v")), beta(need(x[3], "beta")), alpha(need(x[4], "alpha")),
          mu(need(x[5], "mu")), eta(opt(eta_, "eta")), S0(opt(S0_, "S0")), M0(opt(M0_, "M0")) {
        if (q.dim() != 4 || v.dim() != 4) fail("q, v must be [B, T, H, d]; got " + str(q.sizes()) + ", " + str(v.sizes()));
        s.dtype = dtype_code(q);
        dt = q.scalar_type();
        B = q.size(0); T = q.size(1); H = q.size(2); dk = q.size(3); dv = v.size(3);
        expect("k", &k, {B, T, H, dk}, dt, q);
        expect("v", &v, {B, T, H, dv}, dt, q);
        expect("beta", &beta, {B, T, H}, at::kFloat, q);
        expect("alpha", &alpha, {B, T, H}, at::kFloat, q);
        expect("mu", &mu, {B, T, H}, at::kFloat, q);
        expect("eta", eta, {B, T, H}, at::kFloat, q);
        const int64_t nb = states_batch < 0 ? B : states_batch;
        expect("S0", S0, {nb, H, dk, dv}, at::kFloat, q);
        expect("M0", M0, {nb, H, dk, dv}, at::kFloat, q);
        if (!q.is_contiguous()) fail("q must be contiguous");
        s.B = (int32_t)B; s.T = (int32_t)T; s.H = (int32_t)H; s.dk = (int32_t)dk; s.dv = (int32_t)dv; s.C = (int32_t)C;
        s.scale = (float)(scale && scale != Py_None ? number(scale) : std::pow((double)dk, -0.5));
    }
};

size_t workspace_bytes(const mdn_shape &s, int which) {
    size_t n = 0;
    check(mdn_workspace_bytes(&s, which, &n), "mdn_workspace_bytes");
    return n;
}
size_t states_bytes(const mdn_shape &s) {
    size_t n = 0;
    check(mdn_saved_states_bytes(&s, &n), "mdn_saved_states_bytes");
    return n;
}
size_t operands_bytes(const mdn_shape &s) {
    size_t n = 0;
    check(mdn_saved_operands_bytes(&s, &n), "mdn_saved_operands_bytes");
    return n;
}
at::Tensor workspace(PyObject *o, size_t n, const at::Tensor &like) {
    Opt w = opt(o, "workspace");
    expect_bytes("workspace", w, n, like);
    return w ? *w : bytes(n, like);
}
size_t size_of(const at::Tensor &t) { return (size_t)t.numel() * t.element_size(); }

// the host array of sequence offsets of a packed batch
std::vector<int32_t> offsets(PyObject *o, int64_t T) {
    const Ref seq(PySequence_Tuple(o)); // (a tuple of its own: int(item) may run code that changes a list)
    if (!seq.p) throw Fail{};
    const Py_ssize_t n = PyTuple_GET_SIZE(seq.p);
    std::vector<int32_t> cu((size_t)n);
    std::string seen;
    bool good = n >= 2;
    for (Py_ssize_t i = 0; i < n; ++i) {
        const Ref item(PyNumber_Long(PyTuple_GET_ITEM(seq.p, i)));
        if (!item.p) throw Fail{};
        int overflow;
        const long v = PyLong_AsLongAndOverflow(item.p, &overflow);
        good = good && !overflow && v >= 0 && v <= 0x7fffffffL && (i == 0 ? v == 0 : v > cu[i - 1]);
        cu[i] = (int32_t)v;
        if (i < 8) seen += (i ? ", " : "") + (overflow ? std::string("out of range") : std::to_string(v));
    }
    if (!good || cu[n - 1] != T)
        fail("cu_seqlens must rise from 0 to T = " + std::to_string(T) + " without empty sequences; got [" + seen + "]" + (n > 8 ? "..." : ""));
    return cu;
}

// ---- the entry points.  x: the positional arguments, in the order of the signatures in binding.py

// q k v beta alpha mu | eta S0 M0 scale save_vt save_states save_operands output_final_state workspace out chunk_size
PyObject *chunk_fwd(PyObject *const *x) {
    const Inputs in(x, x[6], x[7], x[8], x[9], integer(x[16]));
    PyObject *out = x[15];
    at::Tensor o = output(out, "o", {in.B, in.T, in.H, in.dv}, in.dt, in.q);
    c10::optional<at::Tensor> S, M, vt, states, operands;
    if (truth(x[13])) {
        S = output(out, "S", {in.B, in.H, in.dk, in.dv}, at::kFloat, in.q);
        M = output(out, "M", {in.B, in.H, in.dk, in.dv}, at::kFloat, in.q);
    }
    if (truth(x[10])) vt = output(out, "vt", {in.B, in.T, in.H, in.dv}, in.dt, in.q);
    if (truth(x[11])) states = output_bytes(out, "states", states_bytes(in.s), in.q);
    if (truth(x[12])) operands = output_bytes(out, "operands", operands_bytes(in.s), in.q);
    at::Tensor ws = workspace(x[14], workspace_bytes(in.s, MDN_WS_FWD), in.q);
    on_gpu(in.q);
    void *st = stream();
    call("mdn_chunk_fwd", mdn_chunk_fwd, &in.s, ptr(in.q), ptr(in.k), ptr(in.v), ptr<float>(in.beta), ptr<float>(in.alpha),
         ptr<float>(in.mu), ptr<float>(in.eta), ptr<float>(in.S0), ptr<float>(in.M0), ptr(o), ptr<float>(S), ptr<float>(M),
         ptr(vt), ptr(states), ptr(operands), ptr(ws), size_of(ws), st);
    Dict r;
    r.set("o", o);
    r.set("S", S);
    r.set("M", M);
    r.set("vt", vt);
    r.set("states", states);
    r.set("operands", operands);
    r.set("workspace", ws);
    return r.release();
}

// q k v beta alpha mu out | eta S0 M0 scale chunk_size
PyObject *chunk_fwd_noalloc(PyObject *const *x) {
    const Inputs in(x, x[7], x[8], x[9], x[10], integer(x[11]));
    Ref ro = out_get(x[6], "o"), rS = out_get(x[6], "S"), rM = out_get(x[6], "M"), rvt = out_get(x[6], "vt");
    Opt o = &need(ro.p, "out['o']"), S = opt(rS.p, "out['S']"), M = opt(rM.p, "out['M']"), vt = opt(rvt.p, "out['vt']");
    expect("out['o']", o, {in.B, in.T, in.H, in.dv}, in.dt, in.q);
    expect("out['S']", S, {in.B, in.H, in.dk, in.dv}, at::kFloat, in.q);
    expect("out['M']", M, {in.B, in.H, in.dk, in.dv}, at::kFloat, in.q);
    expect("out['vt']", vt, {in.B, in.T, in.H, in.dv}, in.dt, in.q);
    on_gpu(in.q);
    void *st = stream();
    call("mdn_chunk_fwd_noalloc", mdn_chunk_fwd_noalloc, &in.s, ptr(in.q), ptr(in.k), ptr(in.v), ptr<float>(in.beta),
         ptr<float>(in.alpha), ptr<float>(in.mu), ptr<float>(in.eta), ptr<float>(in.S0), ptr<float>(in.M0), ptr(o),
         ptr<float>(S), ptr<float>(M), ptr(vt), st);
    Py_INCREF(x[6]);
    return x[6];
}

// the gradients of a backward call: the caller's tensors (out) or new ones
struct Grads {
    at::Tensor dq, dk, dv, dbeta, dalpha, dmu;
    c10::optional<at::Tensor> deta, dS0, dM0;
    Grads(PyObject *out, const Inputs &in, bool want_deta, bool want_states, int64_t states_batch)
        : dq(output(out, "dq", {in.B, in.T, in.H, in.dk}, in.dt, in.q)), dk(output(out, "dk", {in.B, in.T, in.H, in.dk}, in.dt, in.q)),
          dv(output(out, "dv", {in.B, in.T, in.H, in.dv}, in.dt, in.q)),
          dbeta(output(out, "dbeta", {in.B, in.T, in.H}, at::kFloat, in.q)),
          dalpha(output(out, "dalpha", {in.B, in.T, in.H}, at::kFloat, in.q)),
          dmu(output(out, "dmu", {in.B, in.T, in.H}, at::kFloat, in.q)) {
        if (want_deta) deta = output(out, "deta", {in.B, in.T, in.H}, at::kFloat, in.q);
        if (want_states) {
            dS0 = output(out, "dS0", {states_batch, in.H, in.dk, in.dv}, at::kFloat, in.q);
            dM0 = output(out, "dM0", {states_batch, in.H, in.dk, in.dv}, at::kFloat, in.q);
        }
    }
    void into(Dict &r) const {
        r.set("dq", dq);
        r.set("dk", dk);
        r.set("dv", dv);
        r.set("dbeta", dbeta);
        r.set("dalpha", dalpha);
        r.set("dmu", dmu);
        r.set("deta", deta);
        r.set("dS0", dS0);
        r.set("dM0", dM0);
    }
};

// q k v beta alpha mu vt dO | eta S0 M0 states operands dS_final dM_final scale want_deta want_dstates workspace out chunk_size
PyObject *chunk_bwd(PyObject *const *x) {
    const Inputs in(x, x[8], x[9], x[10], x[15], integer(x[20]));
    const at::Tensor &vt = need(x[6], "vt"), &dO = need(x[7], "dO");
    Opt states = opt(x[11], "states"), operands = opt(x[12], "operands"), dS = opt(x[13], "dS_final"), dM = opt(x[14], "dM_final");
    expect("vt", &vt, {in.B, in.T, in.H, in.dv}, in.dt, in.q);
    expect("dO", &dO, {in.B, in.T, in.H, in.dv}, in.dt, in.q);
    expect("dS_final", dS, {in.B, in.H, in.dk, in.dv}, at::kFloat, in.q);
    expect("dM_final", dM, {in.B, in.H, in.dk, in.dv}, at::kFloat, in.q);
    if (states) expect_bytes("states", states, states_bytes(in.s), in.q);
    if (operands) expect_bytes("operands", operands, operands_bytes(in.s), in.q);
    const Grads g(x[19], in, truth(x[16]), truth(x[17]), in.B);
    at::Tensor ws = workspace(x[18], workspace_bytes(in.s, dS || dM ? MDN_WS_BWD_STATE_ADJOINTS : MDN_WS_BWD), in.q);
    on_gpu(in.q);
    void *st = stream();
    call("mdn_chunk_bwd", mdn_chunk_bwd, &in.s, ptr(in.q), ptr(in.k), ptr(in.v), ptr<float>(in.beta), ptr<float>(in.alpha),
         ptr<float>(in.mu), ptr<float>(in.eta), ptr<float>(in.S0), ptr<float>(in.M0), ptr(vt), ptr(states), ptr(operands),
         ptr(dO), ptr<float>(dS), ptr<float>(dM), ptr(g.dq), ptr(g.dk), ptr(g.dv), ptr<float>(g.dbeta), ptr<float>(g.dalpha),
         ptr<float>(g.dmu), ptr<float>(g.deta), ptr<float>(g.dS0), ptr<float>(g.dM0), ptr(ws), size_of(ws), st);
    Dict r;
    g.into(r);
    r.set("workspace", ws);
    return r.release();
}

// q k v beta alpha mu S M | eta scale out
PyObject *recurrent_step(PyObject *const *x) {
    const Inputs in(x, x[8], x[6], x[7], x[9], 64);
    if (!in.S0 || !in.M0) fail("S and M are required (they are advanced in place)");
    Opt given = opt(x[10], "out");
    expect("out", given, {in.B, in.T, in.H, in.dv}, in.dt, in.q);
    at::Tensor o = given ? *given : empty({in.B, in.T, in.H, in.dv}, in.dt, in.q);
    on_gpu(in.q);
    void *st = stream();
    call("mdn_recurrent_step", mdn_recurrent_step, &in.s, ptr(in.q), ptr(in.k), ptr(in.v), ptr<float>(in.beta),
         ptr<float>(in.alpha), ptr<float>(in.mu), ptr<float>(in.eta), ptr<float>(in.S0), ptr<float>(in.M0), ptr(o), st);
    if (given) {
        Py_INCREF(x[10]);
        return x[10];
    }
    return THPVariable_Wrap(o);
}

// q k v beta alpha mu cu_seqlens | eta S0 M0 scale save_vt want_states
PyObject *chunk_fwd_varlen(PyObject *const *x) {
    const at::Tensor &q = need(x[0], "q");
    if (q.dim() != 4 || q.size(0) != 1) fail("packed batches are [1, T, H, d]; got q " + str(q.sizes()));
    const std::vector<int32_t> cu = offsets(x[6], q.size(1));
    const int64_t n = (int64_t)cu.size() - 1;
    const Inputs in(x, x[7], x[8], x[9], x[10], 64, n);
    at::Tensor o = empty({1, in.T, in.H, in.dv}, in.dt, q);
    c10::optional<at::Tensor> S, M, vt;
    if (truth(x[12])) {
        S = empty({n, in.H, in.dk, in.dv}, at::kFloat, q);
        M = empty({n, in.H, in.dk, in.dv}, at::kFloat, q);
    }
    if (truth(x[11])) vt = empty({1, in.T, in.H, in.dv}, in.dt, q);
    size_t nb = 0;
    const int which = in.S0 || in.M0 || S ? MDN_WS_FWD : MDN_WS_FWD_NO_STATES;
    check(mdn_workspace_bytes_varlen(&in.s, cu.data(), (int32_t)n, which, &nb), "mdn_workspace_bytes_varlen");
    at::Tensor ws = bytes(nb, q);
    on_gpu(q);
    void *st = stream();
    call("mdn_chunk_fwd_varlen", mdn_chunk_fwd_varlen, &in.s, cu.data(), (int32_t)n, ptr(q), ptr(in.k), ptr(in.v),
         ptr<float>(in.beta), ptr<float>(in.alpha), ptr<float>(in.mu), ptr<float>(in.eta), ptr<float>(in.S0), ptr<float>(in.M0),
         ptr(o), ptr<float>(S), ptr<float>(M), ptr(vt), ptr(ws), nb, st);
    Dict r;
    r.set("o", o);
    r.set("S", S);
    r.set("M", M);
    r.set("vt", vt);
    return r.release();
}

// q k v beta alpha mu vt dO cu_seqlens | eta S0 M0 dS_final dM_final scale want_deta want_state_grads
PyObject *chunk_bwd_varlen(PyObject *const *x) {
    const at::Tensor &q = need(x[0], "q");
    if (q.dim() != 4 || q.size(0) != 1) fail("packed batches are [1, T, H, d]; got q " + str(q.sizes()));
    const std::vector<int32_t> cu = offsets(x[8], q.size(1));
    const int64_t n = (int64_t)cu.size() - 1;
    const Inputs in(x, x[9], x[10], x[11], x[14], 64, n);
    const at::Tensor &vt = need(x[6], "vt"), &dO = need(x[7], "dO");
    Opt dS = opt(x[12], "dS_final"), dM = opt(x[13], "dM_final");
    expect("vt", &vt, {1, in.T, in.H, in.dv}, in.dt, q);
    expect("dO", &dO, {1, in.T, in.H, in.dv}, in.dt, q);
    expect("dS_final", dS, {n, in.H, in.dk, in.dv}, at::kFloat, q);
    expect("dM_final", dM, {n, in.H, in.dk, in.dv}, at::kFloat, q);
    const Grads g(nullptr, in, truth(x[15]), truth(x[16]), n);
    size_t nb = 0;
    const int which = dS || dM ? MDN_WS_BWD : in.S0 || in.M0 || g.dS0 ? MDN_WS_BWD_NO_STATE_ADJOINTS : MDN_WS_BWD_NO_STATES;
    check(mdn_workspace_bytes_varlen(&in.s, cu.data(), (int32_t)n, which, &nb), "mdn_workspace_bytes_varlen");
    at::Tensor ws = bytes(nb, q);
    on_gpu(q);
    void *st = stream();
    call("mdn_chunk_bwd_varlen", mdn_chunk_bwd_varlen, &in.s, cu.data(), (int32_t)n, ptr(q), ptr(in.k), ptr(in.v),
         ptr<float>(in.beta), ptr<float>(in.alpha), ptr<float>(in.mu), ptr<float>(in.eta), ptr<float>(in.S0), ptr<float>(in.M0),
         ptr(vt), ptr(dO), ptr<float>(dS), ptr<float>(dM), ptr(g.dq), ptr(g.dk), ptr(g.dv), ptr<float>(g.dbeta),
         ptr<float>(g.dalpha), ptr<float>(g.dmu), ptr<float>(g.deta), ptr<float>(g.dS0), ptr<float>(g.dM0), ptr(ws), nb, st);
    Dict r;
    g.into(r);
    return r.release();
}

// the four projections x_alpha x_mu x_beta x_eta, the four per-head vectors, and the scalars
struct GateInputs {
    const at::Tensor &xa, &xm, &xb, &xe;
    mdn_gate_params p;
    GateInputs(PyObject *const *x, PyObject *s, PyObject *tau, PyObject *mu_log_min)
        : xa(need(x[0], "x_alpha")), xm(need(x[1], "x_mu")), xb(need(x[2], "x_beta")), xe(need(x[3], "x_eta")) {
        same("x_alpha", xa);
        same("x_mu", xm);
        same("x_beta", xb);
        same("x_eta", xe);
        if (xa.dim() != 3) fail("gate projections must be [B, T, H]; got " + str(xa.sizes()));
        static const char *const names[4] = {"a_alpha", "b_alpha", "a_mu", "b_mu"};
        const float *v[4];
        for (int i = 0; i < 4; ++i) {
            const at::Tensor &t = need(x[4 + i], names[i]);
            expect(names[i], &t, {xa.size(2)}, at::kFloat, xa);
            v[i] = ptr<const float>(t);
        }
        p.B = (int32_t)xa.size(0); p.T = (int32_t)xa.size(1); p.H = (int32_t)xa.size(2);
        p.a_alpha = v[0]; p.b_alpha = v[1]; p.a_mu = v[2]; p.b_mu = v[3];
        p.s = (float)number(s); p.tau = (float)number(tau); p.mu_log_min = (float)number(mu_log_min);
    }
    // a [B, T, H] fp32 tensor like x_alpha
    void same(const char *name, const at::Tensor &t) const {
        if (t.sizes() != xa.sizes()) fail(std::string(name) + ": expected shape " + str(xa.sizes()) + ", got " + str(t.sizes()));
        if (t.scalar_type() != at::kFloat)
            fail(std::string(name) + ": expected dtype torch.float32, got " + dtype_name(t.scalar_type()));
        if (t.device() != xa.device())
            fail(std::string(name) + " is on " + t.device().str() + ", x_alpha on " + xa.device().str() + ": all tensors of a call share one device");
        if (!t.is_contiguous()) fail(std::string(name) + " must be contiguous");
    }
};

// x_alpha x_mu x_beta x_eta a_alpha b_alpha a_mu b_mu s tau mu_log_min
PyObject *gates_fwd(PyObject *const *x) {
    const GateInputs in(x, x[8], x[9], x[10]);
    on_gpu(in.xa);
    at::Tensor alpha = empty(in.xa.sizes(), at::kFloat, in.xa), beta = empty(in.xa.sizes(), at::kFloat, in.xa),
               mu = empty(in.xa.sizes(), at::kFloat, in.xa), eta = empty(in.xa.sizes(), at::kFloat, in.xa);
    void *st = stream();
    call("mdn_gates_fwd", mdn_gates_fwd, &in.p, ptr<float>(in.xa), ptr<float>(in.xm), ptr<float>(in.xb), ptr<float>(in.xe),
         ptr<float>(alpha), ptr<float>(beta), ptr<float>(mu), ptr<float>(eta), st);
    Dict r;
    r.set("alpha", alpha);
    r.set("beta", beta);
    r.set("mu", mu);
    r.set("eta", eta);
    return r.release();
}

// x_alpha x_mu x_beta x_eta a_alpha b_alpha a_mu b_mu s tau dalpha dbeta dmu deta mu_log_min want_dparams
PyObject *gates_bwd(PyObject *const *x) {
    const GateInputs in(x, x[8], x[9], x[14]);
    const at::Tensor &da = need(x[10], "dalpha"), &db = need(x[11], "dbeta"), &dm = need(x[12], "dmu"), &de = need(x[13], "deta");
    in.same("dalpha", da);
    in.same("dbeta", db);
    in.same("dmu", dm);
    in.same("deta", de);
    on_gpu(in.xa);
    at::Tensor xa = empty(in.xa.sizes(), at::kFloat, in.xa), xm = empty(in.xa.sizes(), at::kFloat, in.xa),
               xb = empty(in.xa.sizes(), at::kFloat, in.xa), xe = empty(in.xa.sizes(), at::kFloat, in.xa);
    c10::optional<at::Tensor> par;
    if (truth(x[15])) par = empty({4, in.xa.size(2)}, at::kFloat, in.xa);
    void *st = stream();
    call("mdn_gates_bwd", mdn_gates_bwd, &in.p, ptr<float>(in.xa), ptr<float>(in.xm), ptr<float>(in.xb), ptr<float>(in.xe),
         ptr<float>(da), ptr<float>(db), ptr<float>(dm), ptr<float>(de), ptr<float>(xa), ptr<float>(xm), ptr<float>(xb),
         ptr<float>(xe), ptr<float>(par), st);
    Dict r;
    r.set("dx_alpha", xa);
    r.set("dx_mu", xm);
    r.set("dx_beta", xb);
    r.set("dx_eta", xe);
    r.set("dparams", par);
    return r.release();
}

// x_q, x_k, x_v, d of the front end
struct FrontInputs {
    const at::Tensor &q, &k, &v, &d;
    at::ScalarType dt;
    mdn_shape s;
    explicit FrontInputs(PyObject *const *x) : q(need(x[0], "x_q")), k(need(x[1], "x_k")), v(need(x[2], "x_v")), d(need(x[3], "d")) {
        if (q.dim() != 4 || v.dim() != 4) fail("x_q, x_v must be [B, T, H, d]; got " + str(q.sizes()) + ", " + str(v.sizes()));
        s = mdn_shape{(int32_t)q.size(0), (int32_t)q.size(1), (int32_t)q.size(2), (int32_t)q.size(3), (int32_t)v.size(3), 64, dtype_code(q), 1.f};
        dt = q.scalar_type();
        expect("x_q", &q, {q.size(0), q.size(1), q.size(2), q.size(3)}, dt, q);
        expect("x_k", &k, {q.size(0), q.size(1), q.size(2), q.size(3)}, dt, q);
        expect("x_v", &v, {q.size(0), q.size(1), q.size(2), v.size(3)}, dt, q);
        expect("d", &d, {q.size(2)}, at::kFloat, q);
    }
};

// x_q x_k x_v d eps
PyObject *frontend_fwd(PyObject *const *x) {
    const FrontInputs in(x);
    const double eps = number(x[4]);
    on_gpu(in.q);
    at::Tensor q = empty(in.q.sizes(), in.dt, in.q), k = empty(in.k.sizes(), in.dt, in.q), v = empty(in.v.sizes(), in.dt, in.q);
    void *st = stream();
    call("mdn_frontend_fwd", mdn_frontend_fwd, &in.s, ptr(in.q), ptr(in.k), ptr(in.v), ptr<float>(in.d), (float)eps, ptr(q),
         ptr(k), ptr(v), st);
    Dict r;
    r.set("q", q);
    r.set("k", k);
    r.set("v", v);
    return r.release();
}

// x_q x_k x_v d dq dk dv eps want_dd
PyObject *frontend_bwd(PyObject *const *x) {
    const FrontInputs in(x);
    const at::Tensor &dq = need(x[4], "dq"), &dk = need(x[5], "dk"), &dv = need(x[6], "dv");
    const int64_t B = in.s.B, T = in.s.T, H = in.s.H;
    expect("dq", &dq, {B, T, H, in.s.dk}, in.dt, in.q);
    expect("dk", &dk, {B, T, H, in.s.dk}, in.dt, in.q);
    expect("dv", &dv, {B, T, H, in.s.dv}, in.dt, in.q);
    const double eps = number(x[7]);
    on_gpu(in.q);
    at::Tensor q = empty(in.q.sizes(), in.dt, in.q), k = empty(in.k.sizes(), in.dt, in.q), v = empty(in.v.sizes(), in.dt, in.q);
    c10::optional<at::Tensor> dd;
    if (truth(x[8])) dd = empty(in.d.sizes(), at::kFloat, in.q);
    void *st = stream();
    call("mdn_frontend_bwd", mdn_frontend_bwd, &in.s, ptr(in.q), ptr(in.k), ptr(in.v), ptr<float>(in.d), (float)eps, ptr(dq),
         ptr(dk), ptr(dv), ptr(q), ptr(k), ptr(v), ptr<float>(dd), st);
    Dict r;
    r.set("dx_q", q);
    r.set("dx_k", k);
    r.set("dx_v", v);
    r.set("dd", dd);
    return r.release();
}

// o, g, w of the back end
struct BackInputs {
    const at::Tensor &o, &g, &w;
    at::ScalarType dt;
    mdn_shape s;
    explicit BackInputs(PyObject *const *x) : o(need(x[0], "o")), g(need(x[1], "g")), w(need(x[2], "w")) {
        if (o.dim() != 4) fail("o must be [B, T, H, dv]; got " + str(o.sizes()));
        s = mdn_shape{(int32_t)o.size(0), (int32_t)o.size(1), (int32_t)o.size(2), (int32_t)o.size(3), (int32_t)o.size(3), 64, dtype_code(o), 1.f};
        dt = o.scalar_type();
        expect("o", &o, {o.size(0), o.size(1), o.size(2), o.size(3)}, dt, o);
        expect("g", &g, {o.size(0), o.size(1), o.size(2), o.size(3)}, dt, o);
        expect("w", &w, {o.size(3)}, at::kFloat, o);
    }
};

// o g w eps
PyObject *epilogue_fwd(PyObject *const *x) {
    const BackInputs in(x);
    const double eps = number(x[3]);
    on_gpu(in.o);
    at::Tensor y = empty(in.o.sizes(), in.dt, in.o);
    void *st = stream();
    call("mdn_epilogue_fwd", mdn_epilogue_fwd, &in.s, ptr(in.o), ptr(in.g), ptr<float>(in.w), (float)eps, ptr(y), st);
    return THPVariable_Wrap(y);
}

// o g w dy eps want_dw
PyObject *epilogue_bwd(PyObject *const *x) {
    const BackInputs in(x);
    const at::Tensor &dy = need(x[3], "dy");
    expect("dy", &dy, {in.s.B, in.s.T, in.s.H, in.s.dv}, in.dt, in.o);
    const double eps = number(x[4]);
    on_gpu(in.o);
    at::Tensor d_o = empty(in.o.sizes(), in.dt, in.o), dg = empty(in.o.sizes(), in.dt, in.o);
    c10::optional<at::Tensor> dw;
    if (truth(x[5])) dw = empty(in.w.sizes(), at::kFloat, in.o);
    void *st = stream();
    call("mdn_epilogue_bwd", mdn_epilogue_bwd, &in.s, ptr(in.o), ptr(in.g), ptr<float>(in.w), (float)eps, ptr(dy), ptr(d_o),
         ptr(dg), ptr<float>(dw), st);
    Dict r;
    r.set("do", d_o);
    r.set("dg", dg);
    r.set("dw", dw);
    return r.release();
}

template <PyObject *(*F)(PyObject *const *), int N> PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", N, n);
        return nullptr;
    }
    try {
        return F(args);
    } catch (const Fail &) {
        return nullptr;
    } catch (const c10::OutOfMemoryError &e) {
        PyErr_SetString(g_oom ? g_oom : PyExc_RuntimeError, e.what_without_backtrace());
        return nullptr;
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

PyObject *set_error_types(PyObject *, PyObject *types) { // (MdnError, torch.OutOfMemoryError)
    PyObject *e, *oom;
    if (!PyArg_ParseTuple(types, "OO", &e, &oom)) return nullptr;
    Py_INCREF(e);
    Py_INCREF(oom);
    Py_XSETREF(g_error, e);
    Py_XSETREF(g_oom, oom);
    Py_RETURN_NONE;
}

#define MDN_ENTRY(name, n) \
    {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<name, n>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {MDN_ENTRY(chunk_fwd, 17), MDN_ENTRY(chunk_fwd_noalloc, 12), MDN_ENTRY(chunk_bwd, 21),
                         MDN_ENTRY(recurrent_step, 11), MDN_ENTRY(chunk_fwd_varlen, 13), MDN_ENTRY(chunk_bwd_varlen, 17),
                         MDN_ENTRY(gates_fwd, 11), MDN_ENTRY(gates_bwd, 16), MDN_ENTRY(frontend_fwd, 5),
                         MDN_ENTRY(frontend_bwd, 9), MDN_ENTRY(epilogue_fwd, 4), MDN_ENTRY(epilogue_bwd, 6),
                         {"set_error_types", set_error_types, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_mdn_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__mdn_torch(void) { return PyModule_Create(&module); }
