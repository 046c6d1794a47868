// swr_binding.cpp -- the Python binding's fast path: tensors to pointers and
// strides, outputs allocated, one call of the C ABI, in native code.
//
// Host time binds small calls: checking, allocating and marshalling one call
// in Python and ctypes took about 17 us, twice what its kernel takes on a
// problem of a few MB.  Each function here takes one entry point's arguments in
// a fixed order and handles the ordinary call: plain strided GPU tensors that
// pass every check.  It returns None for anything else, and the caller then
// runs the Python path, which raises what there is to raise and which serves
// every call where this module cannot be built or loaded; a status of the C
// ABI comes back as an int.  Nothing is kept between calls: the C ABI's entry
// points are the only state, bound when the library is loaded.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/swr.h"

// What this module was built from and for; the build looks for it in the file.
extern "C" __attribute__((used)) const char swr_binding_key[] = "swr-binding-key:" SWR_BINDING_KEY;

namespace {

// The C ABI's entry points (the addresses that the loaded library has).
struct Abi {
    decltype(&swr_forward) forward;
    decltype(&swr_backward) backward;
    decltype(&swr_exact_workspace_bytes) exact_workspace_bytes;
    decltype(&swr_exact_forward) exact_forward;
    decltype(&swr_exact_backward) exact_backward;
    decltype(&swr_step) step;
    decltype(&swr_exact_step) exact_step;
    decltype(&swr_decode_state) decode_state;
    decltype(&swr_uniform_forward) uniform_forward;
    decltype(&swr_uniform_backward) uniform_backward;
    decltype(&swr_forward_shared_gates) forward_shared_gates;
    decltype(&swr_backward_shared_gates) backward_shared_gates;
    decltype(&swr_shared_gates_workspace_bytes) shared_gates_workspace_bytes;
};
constexpr int kEntries = sizeof(Abi) / sizeof(void*);
union {
    Abi fn;
    void* address[kEntries];
} abi;

// Arguments of one call, taken in order; ok turns false at the first that is
// not what the fast path handles.
struct Args {
    PyObject* const* v;
    bool ok = true;

    const at::Tensor& tensor() {   // a plain torch.Tensor or Parameter
        static const at::Tensor undefined;
        PyObject* o = *v++;
        if (!THPVariable_CheckExact(o)) { ok = false; return undefined; }
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.defined() || t.layout() != c10::kStrided) ok = false;
        return t;
    }
    at::Tensor optional() {        // None or a tensor
        if (*v == Py_None) { ++v; return {}; }
        return tensor();
    }
    int64_t integer() {
        PyObject* o = *v++;
        if (!PyLong_Check(o)) { ok = false; return 0; }
        const int64_t r = PyLong_AsLongLong(o);
        if (r == -1 && PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        return r;
    }
    bool truth() { return *v++ == Py_True; }
};

bool same_layout(const at::Tensor& x, const at::Tensor& t) {
    return t.scalar_type() == x.scalar_type() && t.device() == x.device() && t.sizes() == x.sizes() &&
           t.strides() == x.strides();
}

bool float_state(const at::Tensor& t, const at::Tensor& x, at::IntArrayRef shape) {
    return t.scalar_type() == at::kFloat && t.device() == x.device() && t.sizes() == shape && t.is_contiguous();
}

// The problem of x, a and the scalars, with every check of the Python path.
bool problem(const at::Tensor& x, const at::Tensor& a, int64_t block, int64_t flags, int64_t run_len,
             swr_problem_t* p) {
    if (x.dim() != 4 || !x.is_cuda() || a.device() != x.device() || a.scalar_type() != x.scalar_type()) return false;
    const bool pc = a.dim() == 4;
    if (pc ? a.sizes() != x.sizes() || a.strides() != x.strides()
           : a.dim() != 3 || a.sizes() != x.sizes().slice(0, 3))
        return false;
    if (x.stride(3) != 1 && x.size(3) > 1) return false;
    if (x.scalar_type() != at::kBFloat16 && x.scalar_type() != at::kFloat) return false;
    if (block <= 0) return false;
    *p = swr_problem_t{};
    p->abi_version = SWR_ABI_VERSION;
    p->dtype = x.scalar_type() == at::kBFloat16 ? SWR_DTYPE_BF16 : SWR_DTYPE_F32;
    p->B = x.size(0); p->T = x.size(1); p->H = x.size(2); p->D = x.size(3);
    p->block = block;
    p->flags = (uint32_t)flags | (pc ? SWR_FLAG_PER_CHANNEL_DECAY : 0);
    p->sx_b = x.stride(0); p->sx_t = x.stride(1); p->sx_h = x.stride(2);
    p->sa_b = a.stride(0); p->sa_t = a.stride(1); p->sa_h = a.stride(2);
    p->run_len = run_len;
    return true;
}

// Allocating and launching run without the interpreter's lock, so that other
// Python threads go on where one waits for the allocator or a full queue.
struct Unlocked {
    PyThreadState* state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};

template <typename F, typename... A>
int call(F entry, A... args) {
    const Unlocked unlocked;
    return entry(args...);
}

void* ptr(const at::Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }
float* fptr(const at::Tensor& t) { return (float*)ptr(t); }

at::Tensor like(const at::Tensor& x) {
    const Unlocked unlocked;
    return at::empty_strided(x.sizes(), x.strides(), x.options().requires_grad(false));
}
at::Tensor floats(const at::Tensor& x, at::IntArrayRef shape) {
    const Unlocked unlocked;
    return at::empty(shape, x.options().dtype(at::kFloat).requires_grad(false));
}
at::Tensor decay_gradient(const at::Tensor& a) {
    const Unlocked unlocked;
    return at::empty_strided(a.sizes(), a.strides(), a.options().dtype(at::kFloat).requires_grad(false));
}

std::array<int64_t, 4> carrier_shape(const swr_problem_t& p) {
    return {p.B, p.H, (p.T + p.block - 1) / p.block, p.D};
}

// The stream argument (an address, or None: x's device's current stream).
void* stream_of(PyObject* o, const at::Tensor& x, bool* ok) {
    if (o == Py_None) return (void*)c10::hip::getCurrentHIPStream(x.device().index()).stream();
    if (!PyLong_Check(o)) { *ok = false; return nullptr; }
    return PyLong_AsVoidPtr(o);
}

// n floats that only one call's kernels use, on its stream (o, st: the stream
// argument and its address).  The tensor is let go when the call returns, so
// it is taken from that stream's memory: whoever gets it next is ordered
// behind those kernels there, and it has no other stream's work pending.
at::Tensor workspace(const at::Tensor& x, int64_t n, PyObject* o, void* st) {
    if (o == Py_None) return floats(x, {n});
    struct On {
        const c10::hip::HIPStream before;
        On(c10::DeviceIndex d, void* s) : before(c10::hip::getCurrentHIPStream(d)) {
            c10::hip::setCurrentHIPStream(s ? c10::hip::getStreamFromExternal((hipStream_t)s, d)
                                            : c10::hip::getDefaultHIPStream(d));
        }
        ~On() { c10::hip::setCurrentHIPStream(before); }
    } on(x.device().index(), st);
    return floats(x, {n});
}

PyObject* none() { Py_RETURN_NONE; }

PyObject* results(int rc, std::initializer_list<at::Tensor> ts) {
    if (rc != 0) return PyLong_FromLong(rc);
    if (ts.size() == 1) return THPVariable_Wrap(*ts.begin());
    PyObject* r = PyTuple_New((Py_ssize_t)ts.size());
    if (!r) return nullptr;
    Py_ssize_t i = 0;
    for (const at::Tensor& t : ts) {
        PyObject* o = nullptr;
        if (t.defined()) o = THPVariable_Wrap(t);
        else { o = Py_None; Py_INCREF(o); }
        if (!o) { Py_DECREF(r); return nullptr; }
        PyTuple_SET_ITEM(r, i++, o);
    }
    return r;
}

// x, a, b, c of the calls whose b and c have x's layout.
struct Inputs {
    const at::Tensor &x, &a, &b, &c;
    explicit Inputs(Args& g) : x(g.tensor()), a(g.tensor()), b(g.tensor()), c(g.tensor()) {}
    bool check(const Args& g, int64_t block, int64_t flags, int64_t run_len, swr_problem_t* p) const {
        return g.ok && problem(x, a, block, flags, run_len, p) && same_layout(x, b) && same_layout(x, c);
    }
};

// forward(x, a, b, c, block, flags, run_len, y, carriers, want_carriers, stream) -> (y, carriers)
PyObject* forward(PyObject*, PyObject* const* v, Py_ssize_t) {
    HANDLE_TH_ERRORS
    Args g{v};
    const Inputs in(g);
    const int64_t block = g.integer(), flags = g.integer(), run_len = g.integer();
    at::Tensor y = g.optional(), s = g.optional();
    const bool want = g.truth();
    swr_problem_t p;
    if (!in.check(g, block, flags, run_len, &p)) return none();
    void* st = stream_of(*g.v, in.x, &g.ok);
    const auto vs = carrier_shape(p);
    if (!g.ok || (y.defined() && !same_layout(in.x, y)) || (s.defined() && !float_state(s, in.x, vs))) return none();
    if (!y.defined()) y = like(in.x);
    if (want && !s.defined()) s = floats(in.x, vs);
    return results(call(abi.fn.forward, &p, ptr(in.x), ptr(in.a), ptr(in.b), ptr(in.c), ptr(y), fptr(s), st), {y, s});
    END_HANDLE_TH_ERRORS
}

// backward(x, a, b, c, dy, carriers, block, flags, run_len, stream) -> (dx, da, db, dc)
PyObject* backward(PyObject*, PyObject* const* v, Py_ssize_t) {
    HANDLE_TH_ERRORS
    Args g{v};
    const Inputs in(g);
    const at::Tensor& dy = g.tensor();
    const at::Tensor s = g.optional();
    const int64_t block = g.integer(), flags = g.integer(), run_len = g.integer();
    swr_problem_t p;
    if (!in.check(g, block, flags, run_len, &p) || !same_layout(in.x, dy)) return none();
    void* st = stream_of(*g.v, in.x, &g.ok);
    if (!g.ok || (s.defined() && !float_state(s, in.x, carrier_shape(p)))) return none();
    const at::Tensor dx = like(in.x), db = like(in.x), dc = like(in.x), da = decay_gradient(in.a);
    return results(call(abi.fn.backward, &p, ptr(in.x), ptr(in.a), ptr(in.b), ptr(in.c), ptr(dy), fptr(s), ptr(dx),
                          fptr(da),
                                   ptr(db), ptr(dc), st), {dx, da, db, dc});
    END_HANDLE_TH_ERRORS
}

// exact_forward(x, a, b, c, block, flags, run_len, h0, want_carriers, want_h_last, stream)
//     -> (y, carriers, h_last)
PyObject* exact_forward(PyObject*, PyObject* const* v, Py_ssize_t) {
    HANDLE_TH_ERRORS
    Args g{v};
    const Inputs in(g);
    const int64_t block = g.integer(), flags = g.integer(), run_len = g.integer();
    const at::Tensor h0 = g.optional();
    const bool want_v = g.truth(), want_h = g.truth();
    swr_problem_t p;
    if (!in.check(g, block, flags, run_len, &p)) return none();
    void* st = stream_of(*g.v, in.x, &g.ok);
    const std::array<int64_t, 3> hs{p.B, p.H, p.D};
    if (!g.ok || (h0.defined() && !float_state(h0, in.x, hs))) return none();
    const int64_t ws = abi.fn.exact_workspace_bytes(&p);
    if (ws < 0) return none();
    const at::Tensor y = like(in.x);
    at::Tensor s, hl;
    if (want_v) s = floats(in.x, carrier_shape(p));
    if (want_h) hl = floats(in.x, hs);
    const at::Tensor work = workspace(in.x, std::max<int64_t>(ws / 4, 1), *g.v, st);
    return results(call(abi.fn.exact_forward, &p, ptr(in.x), ptr(in.a), ptr(in.b), ptr(in.c), fptr(h0), ptr(y), fptr(s),
                                        fptr(hl), ptr(work), st), {y, s, hl});
    END_HANDLE_TH_ERRORS
}

// exact_backward(x, a, b, c, dy, carriers, block, flags, run_len, h0, dh_last, want_dh0, stream)
//     -> (dx, da, db, dc, dh0)
PyObject* exact_backward(PyObject*, PyObject* const* v, Py_ssize_t) {
    HANDLE_TH_ERRORS
    Args g{v};
    const Inputs in(g);
    const at::Tensor &dy = g.tensor(), &s = g.tensor();
    const int64_t block = g.integer(), flags = g.integer(), run_len = g.integer();
    const at::Tensor h0 = g.optional(), dhl = g.optional();
    const bool want = g.truth();
    swr_problem_t p;
    if (!in.check(g, block, flags, run_len, &p) || !same_layout(in.x, dy)) return none();
    void* st = stream_of(*g.v, in.x, &g.ok);
    const std::array<int64_t, 3> hs{p.B, p.H, p.D};
    if (!g.ok || !float_state(s, in.x, carrier_shape(p)) || (h0.defined() && !float_state(h0, in.x, hs)) ||
        (dhl.defined() && !float_state(dhl, in.x, hs)))
        return none();
    const int64_t ws = abi.fn.exact_workspace_bytes(&p);
    if (ws < 0) return none();
    const at::Tensor dx = like(in.x), db = like(in.x), dc = like(in.x), da = decay_gradient(in.a);
    at::Tensor dh0;
    if (want) dh0 = floats(in.x, hs);
    const at::Tensor work = workspace(in.x, std::max<int64_t>(ws / 4, 1), *g.v, st);
    return results(call(abi.fn.exact_backward, &p, ptr(in.x), ptr(in.a), ptr(in.b), ptr(in.c), ptr(dy), fptr(h0),
                          fptr(s),
                                         fptr(dhl), ptr(dx), fptr(da), ptr(db), ptr(dc), fptr(dh0), ptr(work), st),
                   {dx, da, db, dc, dh0});
    END_HANDLE_TH_ERRORS
}

// step(x, a, b, c, block, flags, t0, state, y, stream) -> y; t0 < 0: the exact recurrence
PyObject* step(PyObject*, PyObject* const* v, Py_ssize_t) {
    HANDLE_TH_ERRORS
    Args g{v};
    const Inputs in(g);
    const int64_t block = g.integer(), flags = g.integer(), t0 = g.integer();
    const at::Tensor& state = g.tensor();
    at::Tensor y = g.optional();
    swr_problem_t p;
    if (!in.check(g, block, flags, 0, &p)) return none();
    void* st = stream_of(*g.v, in.x, &g.ok);
    const std::array<int64_t, 4> js{p.B, p.H, 2, p.D};
    const std::array<int64_t, 3> hs{p.B, p.H, p.D};
    if (!g.ok || !float_state(state, in.x, t0 < 0 ? at::IntArrayRef(hs) : at::IntArrayRef(js)) ||
        (y.defined() && !same_layout(in.x, y)))
        return none();
    if (!y.defined()) y = like(in.x);
    const int rc = t0 < 0 ? call(abi.fn.exact_step, &p, ptr(in.x), ptr(in.a), ptr(in.b), ptr(in.c), ptr(y),
          fptr(state), st)
                          : call(abi.fn.step, &p, t0, ptr(in.x), ptr(in.a), ptr(in.b), ptr(in.c), ptr(y), fptr(state),
                                st);
    return results(rc, {y});
    END_HANDLE_TH_ERRORS
}

// decode_state(x, a, carriers, block, flags, stream) -> state
PyObject* decode_state(PyObject*, PyObject* const* v, Py_ssize_t) {
    HANDLE_TH_ERRORS
    Args g{v};
    const at::Tensor &x = g.tensor(), &a = g.tensor(), &s = g.tensor();
    const int64_t block = g.integer(), flags = g.integer();
    swr_problem_t p;
    if (!g.ok || !problem(x, a, block, flags, 0, &p)) return none();
    void* st = stream_of(*g.v, x, &g.ok);
    if (!g.ok || !float_state(s, x, carrier_shape(p))) return none();
    const at::Tensor state = floats(x, {p.B, p.H, 2, p.D});
    return results(call(abi.fn.decode_state, &p, ptr(a), fptr(s), fptr(state), st), {state});
    END_HANDLE_TH_ERRORS
}

// uniform_forward(x, a, b, c, window, flags, run_len, stream) -> y
PyObject* uniform_forward(PyObject*, PyObject* const* v, Py_ssize_t) {
    HANDLE_TH_ERRORS
    Args g{v};
    const Inputs in(g);
    const int64_t block = g.integer(), flags = g.integer(), run_len = g.integer();
    swr_problem_t p;
    if (!in.check(g, block, flags, run_len, &p)) return none();
    void* st = stream_of(*g.v, in.x, &g.ok);
    if (!g.ok) return none();
    const at::Tensor y = like(in.x);
    return results(call(abi.fn.uniform_forward, &p, ptr(in.x), ptr(in.a), ptr(in.b), ptr(in.c), ptr(y), st), {y});
    END_HANDLE_TH_ERRORS
}

// uniform_backward(x, a, b, c, dy, window, flags, run_len, stream) -> (dx, da, db, dc)
PyObject* uniform_backward(PyObject*, PyObject* const* v, Py_ssize_t) {
    HANDLE_TH_ERRORS
    Args g{v};
    const Inputs in(g);
    const at::Tensor& dy = g.tensor();
    const int64_t block = g.integer(), flags = g.integer(), run_len = g.integer();
    swr_problem_t p;
    if (!in.check(g, block, flags, run_len, &p) || !same_layout(in.x, dy)) return none();
    void* st = stream_of(*g.v, in.x, &g.ok);
    if (!g.ok) return none();
    const at::Tensor dx = like(in.x), db = like(in.x), dc = like(in.x), da = decay_gradient(in.a);
    return results(call(abi.fn.uniform_backward, &p, ptr(in.x), ptr(in.a), ptr(in.b), ptr(in.c), ptr(dy), ptr(dx),
                          fptr(da),
                                           ptr(db), ptr(dc), st), {dx, da, db, dc});
    END_HANDLE_TH_ERRORS
}

// The gates' checks: [B, T, H / group, D] with contiguous channels, b and c alike.
bool gates(const Args& g, const at::Tensor& x, const at::Tensor& a, const at::Tensor& b, const at::Tensor& c,
           int64_t group, int64_t block, int64_t flags, int64_t run_len, swr_problem_t* p) {
    if (!g.ok || !problem(x, a, block, flags, run_len, p) || group < 1 || p->H % group != 0) return false;
    const std::array<int64_t, 4> gs{p->B, p->T, p->H / group, p->D};
    return b.sizes() == at::IntArrayRef(gs) && b.scalar_type() == x.scalar_type() && b.device() == x.device() &&
           (b.stride(3) == 1 || p->D <= 1) && same_layout(b, c);
}

// forward_shared_gates(x, a, b, c, block, flags, run_len, group, want_carriers, stream) -> (y, carriers)
PyObject* forward_shared_gates(PyObject*, PyObject* const* v, Py_ssize_t) {
    HANDLE_TH_ERRORS
    Args g{v};
    const Inputs in(g);
    const int64_t block = g.integer(), flags = g.integer(), run_len = g.integer(), group = g.integer();
    const bool want = g.truth();
    swr_problem_t p;
    if (!gates(g, in.x, in.a, in.b, in.c, group, block, flags, run_len, &p)) return none();
    void* st = stream_of(*g.v, in.x, &g.ok);
    if (!g.ok) return none();
    const at::Tensor y = like(in.x);
    at::Tensor s;
    if (want) s = floats(in.x, carrier_shape(p));
    return results(call(abi.fn.forward_shared_gates, &p, group, in.b.strides().data(), ptr(in.x), ptr(in.a), ptr(in.b),
                                               ptr(in.c), ptr(y), fptr(s), st), {y, s});
    END_HANDLE_TH_ERRORS
}

// backward_shared_gates(x, a, b, c, dy, carriers, block, flags, run_len, group, stream) -> (dx, da, db, dc)
PyObject* backward_shared_gates(PyObject*, PyObject* const* v, Py_ssize_t) {
    HANDLE_TH_ERRORS
    Args g{v};
    const Inputs in(g);
    const at::Tensor &dy = g.tensor(), &s = g.tensor();
    const int64_t block = g.integer(), flags = g.integer(), run_len = g.integer(), group = g.integer();
    swr_problem_t p;
    if (!gates(g, in.x, in.a, in.b, in.c, group, block, flags, run_len, &p) || !same_layout(in.x, dy)) return none();
    void* st = stream_of(*g.v, in.x, &g.ok);
    if (!g.ok || !float_state(s, in.x, carrier_shape(p))) return none();
    const int64_t ws = abi.fn.shared_gates_workspace_bytes(&p, group);
    if (ws < 0) return none();
    const at::Tensor dx = like(in.x), db = like(in.b), dc = like(in.b), da = decay_gradient(in.a);
    at::Tensor work;
    if (ws > 0) work = workspace(in.x, ws / 4, *g.v, st);
    return results(call(abi.fn.backward_shared_gates, &p, group, in.b.strides().data(), ptr(in.x), ptr(in.a), ptr(in.b),
                                                ptr(in.c), ptr(dy), fptr(s), ptr(dx), fptr(da), ptr(db), ptr(dc),
                                                ptr(work), st), {dx, da, db, dc});
    END_HANDLE_TH_ERRORS
}

// bind(address, ...): the C ABI's entry points, in Abi's order
PyObject* bind(PyObject*, PyObject* const* v, Py_ssize_t n) {
    if (n != kEntries) {
        PyErr_SetString(PyExc_TypeError, "bind: wrong number of entry points");
        return nullptr;
    }
    for (int i = 0; i < kEntries; ++i) abi.address[i] = PyLong_AsVoidPtr(v[i]);
    if (PyErr_Occurred()) return nullptr;
    Py_RETURN_NONE;
}

#define ENTRY(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ENTRY(bind), ENTRY(forward), ENTRY(backward), ENTRY(exact_forward), ENTRY(exact_backward),
                         ENTRY(step), ENTRY(decode_state), ENTRY(uniform_forward), ENTRY(uniform_backward),
                         ENTRY(forward_shared_gates), ENTRY(backward_shared_gates), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
