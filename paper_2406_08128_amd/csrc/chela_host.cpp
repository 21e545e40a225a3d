// The host path of the decode step and of whole sequences without the interpreter: checks, the outputs' allocation, the current
// stream and the call into libchela.so for plain device tensors.  A step is over in 4.5 us on the GPU; through the binding's own lines, a dozen attribute
// look-ups, torch.empty() and ctypes, the host needed 8.9 us for it, of which the launch is 3.4.
//
// step(function, q, k, v, g or None, S, eps, y or None, stream or None) -> y, a status of the library (int, not 0), or None:
// "not the plain case", and nothing has been done.  The binding then takes its own path, which says what is wrong or serves the
// case (other devices, subclasses, modes).  function: address of chela_linattn_step (g is None) or chela_linattn_step_gated.
//
// Likewise, with the functions' addresses first and the stream last:
//   forward(f, f32, Q, K, V, S_in, S_out, chunk, stream) -> O; with f32 = None (chela_linattn_fwd_state: bf16 only) -> (O, S_out)
//   backward(f, f32, Q, K, V, dO, chunk, stream) -> (dQ, dK, dV); f32 = None: chela_linattn_noncausal_bwd, bf16 only, chunk not looked at
//   gated(f, saved_bytes, Q or Z, K or affine, V, G, eps, want_O, want_saved, stream) -> (Y, O or None, saved or None);
//       saved_bytes = None: chela_linattn_noncausal_fwd_gated
//   gate_norm_bwd(f, O, G, dY, eps, stream) -> (dO, dG)
//   zbwd_saved(f, Z, affine, V, dO, saved, stream) -> (dZ, d_affine, dV)
//   spectrum(f, bytes, k_long, stream) -> spectrum
//   conv_fwd(f, f32, X, w_short, spectrum, stream) -> Z;  conv_bwd(f, f32, X, w_short, spectrum, dZ, stream) -> (dX, d_w_short, d_k_long)
// Host side of a call, us, the binding's own lines and these: forward, one launch, 8.5 and 4.4, two launches 9.7 and 6.2; with the
// state 9.9 and 4.8, 12.1 and 7.2; backward, two launches, 11.4 and 7.5; the three calls of a gated layer's step, six launches, 39.6 and 23;
// spectrum, forward and gradient of a convolution, 22.5 and 15.
#include <Python.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

typedef int (*step_fn)(const void*, const void*, const void*, float*, void*, int, int, int, int, void*);
typedef int (*step_gated_fn)(const void*, const void*, const void*, const void*, float*, void*, float, int, int, int, int, void*);

// a dense device tensor of exactly the class torch.Tensor
bool plain(PyObject* o, at::ScalarType type, c10::DeviceIndex dev)
{
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor& t = THPVariable_Unpack(o);
    return t.defined() && t.is_cuda() && t.layout() == at::kStrided && t.has_storage() && t.scalar_type() == type &&
           t.get_device() == dev && t.is_contiguous() && !t.key_set().has_any(c10::DispatchKeySet({c10::DispatchKey::FuncTorchBatched,
               c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize, c10::DispatchKey::Python}));
}

// (before there is a current device to ask for: a machine may have none)
bool on_gpu(PyObject* o) { return THPVariable_CheckExact(o) && THPVariable_Unpack(o).defined() && THPVariable_Unpack(o).is_cuda(); }

// something that wants to see, or to change, what is done with tensors
bool modes() { return at::impl::PythonTorchFunctionTLS::stack_len() > 0 || c10::impl::TorchDispatchModeTLS::any_modes_set(); }

struct without_interpreter_lock {
    PyThreadState* const state = PyEval_SaveThread();
    ~without_interpreter_lock() { PyEval_RestoreThread(state); }
};

PyObject* step(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 9) { PyErr_SetString(PyExc_TypeError, "step takes nine arguments"); return nullptr; }
    if (modes()) Py_RETURN_NONE;
    PyObject *oq = a[1], *ok = a[2], *ov = a[3], *og = a[4], *oS = a[5], *oy = a[7], *ostream = a[8];
    if (!THPVariable_CheckExact(oq) || (ostream != Py_None) || !PyFloat_CheckExact(a[6])) Py_RETURN_NONE;
    const at::Tensor& q = THPVariable_Unpack(oq);
    if (!q.defined() || !q.is_cuda()) Py_RETURN_NONE;
    const c10::DeviceIndex dev = c10::hip::current_device();
    if (!plain(oq, at::kBFloat16, dev) || !plain(ok, at::kBFloat16, dev) || !plain(ov, at::kBFloat16, dev) ||
        !plain(oS, at::kFloat, dev) || (og != Py_None && !plain(og, at::kBFloat16, dev)) ||
        (oy != Py_None && !plain(oy, at::kBFloat16, dev)))
        Py_RETURN_NONE;
    const at::Tensor &k = THPVariable_Unpack(ok), &v = THPVariable_Unpack(ov), &S = THPVariable_Unpack(oS);
    if (q.dim() != 3 || k.sizes() != q.sizes() || v.dim() != 3) Py_RETURN_NONE;
    const int64_t B = q.size(0), H = q.size(1), dk = q.size(2), dv = v.size(2);
    const int64_t lim = 0x7fffffff;
    if (v.size(0) != B || v.size(1) != H || B > lim || H > lim || dk > lim || dv > lim) Py_RETURN_NONE;
    if (S.dim() != 4 || S.size(0) != B || S.size(1) != H || S.size(2) != dk || S.size(3) != dv) Py_RETURN_NONE;
    if (og != Py_None && THPVariable_Unpack(og).sizes() != v.sizes()) Py_RETURN_NONE;
    if (oy != Py_None && THPVariable_Unpack(oy).sizes() != v.sizes()) Py_RETURN_NONE;
    const unsigned long long fn = PyLong_AsUnsignedLongLong(a[0]);
    if (PyErr_Occurred()) return nullptr;
    const void *pq = q.data_ptr(), *pk = k.data_ptr(), *pv = v.data_ptr();
    const void* pg = og != Py_None ? THPVariable_Unpack(og).data_ptr() : nullptr;
    float *pS = (float*)S.data_ptr(), eps = (float)PyFloat_AS_DOUBLE(a[6]);
    const at::TensorOptions like = q.options().requires_grad(false);
    at::Tensor y;
    if (oy != Py_None) y = THPVariable_Unpack(oy);
    int rc;
    {
        // (both may wait for the GPU, the launch for room in a queue: other threads go on, as they do through ctypes)
        const without_interpreter_lock free;
        if (oy == Py_None) y = at::empty({B, H, dv}, like);
        void *py = y.data_ptr(), *st = (void*)c10::hip::getCurrentHIPStream(dev).stream();
        rc = og == Py_None
                 ? reinterpret_cast<step_fn>(fn)(pq, pk, pv, pS, py, (int)B, (int)H, (int)dk, (int)dv, st)
                 : reinterpret_cast<step_gated_fn>(fn)(pq, pk, pv, pg, pS, py, eps, (int)B, (int)H, (int)dk, (int)dv, st);
    }
    if (rc != 0) return PyLong_FromLong(rc);
    if (oy != Py_None) { Py_INCREF(oy); return oy; }
    return THPVariable_Wrap(std::move(y));
    END_HANDLE_TH_ERRORS
}

typedef int (*fwd_fn)(const void*, const void*, const void*, void*, int, int, int, int, int, int, void*);
typedef int (*fwd_state_fn)(const void*, const void*, const void*, const float*, void*, float*, int, int, int, int, int, int, void*);
typedef int (*bwd_fn)(const void*, const void*, const void*, const void*, void*, void*, void*, int, int, int, int, int, int, void*);
typedef int (*noncausal_bwd_fn)(const void*, const void*, const void*, const void*, void*, void*, void*, int, int, int, int, int, void*);
typedef int (*gated_fn)(const void*, const void*, const void*, const void*, void*, void*, void*, float, int, int, int, int, int, int, void*);
typedef int (*noncausal_gated_fn)(const void*, const void*, const void*, const void*, void*, void*, float, int, int, int, int, int, void*);
typedef size_t (*saved_bytes_fn)(int, int, int, int, int, int);
typedef int (*gate_norm_bwd_fn)(const void*, const void*, const void*, void*, void*, float, long long, int, void*);
typedef int (*zbwd_saved_fn)(const void*, const float*, const void*, const void*, const void*, void*, float*, void*, int, int, int, int, int,
                             int, void*);
typedef size_t (*spectrum_bytes_fn)(int, int);
typedef int (*spectrum_fn)(const float*, void*, int, int, void*);
typedef int (*conv_fwd_fn)(const void*, const float*, int, const void*, void*, int, int, int, void*);
typedef int (*conv_bwd_fn)(const void*, const float*, int, const void*, const void*, void*, float*, float*, int, int, int, void*);

// Q, K [B,H,N,dk] and V [B,H,N,dv], plain and of one type that there is a function for.
struct Sequences {
    int B, H, N, dk, dv, chunk;
    c10::DeviceIndex dev;
    at::ScalarType type;
    bool read(PyObject* const* qkv, bool f32_too, PyObject* ochunk, PyObject* ostream)
    {
        if (modes() || ostream != Py_None || !on_gpu(qkv[0])) return false;
        const int64_t lim = 0x7fffffff;
        int overflow = 0;
        long c = 64;
        if (ochunk != nullptr) {
            if (!PyLong_CheckExact(ochunk)) return false;
            c = PyLong_AsLongAndOverflow(ochunk, &overflow);
            if (overflow || c < 0 || c > lim) return false;
        }
        const at::Tensor& q = THPVariable_Unpack(qkv[0]);
        type = q.scalar_type();
        dev = c10::hip::current_device();
        if (type != at::kBFloat16 && !(f32_too && type == at::kFloat)) return false;
        for (int i = 0; i < 3; ++i) if (!plain(qkv[i], type, dev)) return false;
        const at::Tensor &k = THPVariable_Unpack(qkv[1]), &v = THPVariable_Unpack(qkv[2]);
        if (q.dim() != 4 || k.sizes() != q.sizes() || v.dim() != 4) return false;
        for (int i = 0; i < 4; ++i) if (q.size(i) > lim || v.size(i) > lim || (i < 3 && v.size(i) != q.size(i))) return false;
        B = (int)q.size(0); H = (int)q.size(1); N = (int)q.size(2); dk = (int)q.size(3); dv = (int)v.size(3);
        chunk = (int)c;
        return true;
    }
    bool is_affine(PyObject* o) const
    {
        if (!plain(o, at::kFloat, dev)) return false;
        const at::Tensor& t = THPVariable_Unpack(o);
        return t.dim() == 3 && t.size(0) == 4 && t.size(1) == H && t.size(2) == dk;
    }
    bool is_state(PyObject* o) const
    {
        if (!plain(o, at::kFloat, dev)) return false;
        const at::Tensor& t = THPVariable_Unpack(o);
        return t.dim() == 4 && t.size(0) == B && t.size(1) == H && t.size(2) == dk && t.size(3) == dv;
    }
};

PyObject* none() { Py_INCREF(Py_None); return Py_None; }

// The tensors as a tuple, None for those that are not there.
template <size_t N>
PyObject* wrap(at::Tensor (&t)[N])
{
    PyObject* all = PyTuple_New(N);
    for (size_t i = 0; all != nullptr && i < N; ++i) {
        PyObject* o = t[i].defined() ? THPVariable_Wrap(std::move(t[i])) : none();
        if (o == nullptr) { Py_DECREF(all); return nullptr; }
        PyTuple_SET_ITEM(all, i, o);
    }
    return all;
}

template <typename F>
F address(PyObject* o) { return reinterpret_cast<F>(PyLong_AsUnsignedLongLong(o)); }
void* stream_of(c10::DeviceIndex dev) { return (void*)c10::hip::getCurrentHIPStream(dev).stream(); }
at::TensorOptions like(const at::Tensor& t) { return t.options().requires_grad(false); }

PyObject* forward(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 9) { PyErr_SetString(PyExc_TypeError, "forward takes nine arguments"); return nullptr; }
    const bool with_state = a[1] == Py_None;
    Sequences x;
    if (!x.read(a + 2, !with_state, a[7], a[8])) Py_RETURN_NONE;
    PyObject *oin = a[5], *oout = a[6];
    if ((oin != Py_None && !(with_state && x.is_state(oin))) || (oout != Py_None && !(with_state && x.is_state(oout)))) Py_RETURN_NONE;
    PyObject* const of = a[x.type == at::kFloat ? 1 : 0];
    const auto f = address<fwd_fn>(of);
    const auto f_state = address<fwd_state_fn>(of);
    if (PyErr_Occurred()) return nullptr;
    const at::Tensor& q = THPVariable_Unpack(a[2]);
    const void *pq = q.data_ptr(), *pk = THPVariable_Unpack(a[3]).data_ptr(), *pv = THPVariable_Unpack(a[4]).data_ptr();
    const float* pin = oin != Py_None ? (const float*)THPVariable_Unpack(oin).data_ptr() : nullptr;
    at::Tensor out[2];
    if (oout != Py_None) out[1] = THPVariable_Unpack(oout);
    int rc;
    {
        const without_interpreter_lock free;
        out[0] = at::empty({x.B, x.H, x.N, x.dv}, like(q));
        if (with_state && oout == Py_None) out[1] = at::empty({x.B, x.H, x.dk, x.dv}, like(q).dtype(at::kFloat));
        void *po = out[0].data_ptr(), *st = stream_of(x.dev);
        rc = with_state ? f_state(pq, pk, pv, pin, po, (float*)out[1].data_ptr(), x.B, x.H, x.N, x.dk, x.dv, x.chunk, st)
                        : f(pq, pk, pv, po, x.B, x.H, x.N, x.dk, x.dv, x.chunk, st);
    }
    if (rc != 0) return PyLong_FromLong(rc);
    return with_state ? wrap(out) : THPVariable_Wrap(std::move(out[0]));       // (S_out as it came: a tensor has one Python object)
    END_HANDLE_TH_ERRORS
}

PyObject* backward(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 8) { PyErr_SetString(PyExc_TypeError, "backward takes eight arguments"); return nullptr; }
    const bool causal = a[1] != Py_None;
    Sequences x;
    if (!x.read(a + 2, causal, causal ? a[6] : nullptr, a[7]) || !plain(a[5], x.type, x.dev)) Py_RETURN_NONE;
    const at::Tensor &q = THPVariable_Unpack(a[2]), &v = THPVariable_Unpack(a[4]), &d = THPVariable_Unpack(a[5]);
    if (d.sizes() != v.sizes()) Py_RETURN_NONE;
    PyObject* const of = a[x.type == at::kFloat ? 1 : 0];
    const auto f = address<bwd_fn>(of);
    const auto f_noncausal = address<noncausal_bwd_fn>(of);
    if (PyErr_Occurred()) return nullptr;
    const void *pq = q.data_ptr(), *pk = THPVariable_Unpack(a[3]).data_ptr(), *pv = v.data_ptr(), *pd = d.data_ptr();
    at::Tensor g[3];
    int rc;
    {
        const without_interpreter_lock free;
        for (int i = 0; i < 3; ++i) g[i] = at::empty({x.B, x.H, x.N, i < 2 ? x.dk : x.dv}, like(q));
        void *p0 = g[0].data_ptr(), *p1 = g[1].data_ptr(), *p2 = g[2].data_ptr(), *st = stream_of(x.dev);
        rc = causal ? f(pq, pk, pv, pd, p0, p1, p2, x.B, x.H, x.N, x.dk, x.dv, x.chunk, st)
                    : f_noncausal(pq, pk, pv, pd, p0, p1, p2, x.B, x.H, x.N, x.dk, x.dv, st);
    }
    return rc != 0 ? PyLong_FromLong(rc) : wrap(g);
    END_HANDLE_TH_ERRORS
}

PyObject* gated(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 10) { PyErr_SetString(PyExc_TypeError, "gated takes ten arguments"); return nullptr; }
    const bool causal = a[1] != Py_None;
    Sequences x;
    // (the second operand: keys of the first one's shape, or the affine parameters [4,H,dk])
    PyObject* const first[3] = {a[2], a[2], a[4]};
    if (!x.read(first, false, nullptr, a[9]) || !PyFloat_CheckExact(a[6])) Py_RETURN_NONE;
    const at::Tensor &q = THPVariable_Unpack(a[2]), &v = THPVariable_Unpack(a[4]);
    if (plain(a[3], at::kBFloat16, x.dev) ? THPVariable_Unpack(a[3]).sizes() != q.sizes() : !(causal && x.is_affine(a[3]))) Py_RETURN_NONE;
    if (!plain(a[5], at::kBFloat16, x.dev) || THPVariable_Unpack(a[5]).sizes() != v.sizes()) Py_RETURN_NONE;
    const int want_O = PyObject_IsTrue(a[7]), want_saved = PyObject_IsTrue(a[8]);
    if (want_O < 0 || want_saved < 0) return nullptr;
    const auto f = address<gated_fn>(a[0]);
    const auto f_noncausal = address<noncausal_gated_fn>(a[0]);
    const auto bytes = causal ? address<saved_bytes_fn>(a[1]) : nullptr;
    if (PyErr_Occurred()) return nullptr;
    const void *pq = q.data_ptr(), *pk = THPVariable_Unpack(a[3]).data_ptr(), *pv = v.data_ptr(), *pg = THPVariable_Unpack(a[5]).data_ptr();
    const float eps = (float)PyFloat_AS_DOUBLE(a[6]);
    at::Tensor out[3];      // Y, O, saved
    int rc;
    {
        const without_interpreter_lock free;
        for (int i = 0; i < (want_O ? 2 : 1); ++i) out[i] = at::empty({x.B, x.H, x.N, x.dv}, like(q));
        if (causal && want_saved) {
            const size_t need = bytes(x.B, x.H, x.N, x.dk, x.dv, 64);
            out[2] = at::empty({(int64_t)(need < 16 ? 16 : need) / 4}, like(q).dtype(at::kFloat));
        }
        void *pY = out[0].data_ptr(), *pO = want_O ? out[1].data_ptr() : nullptr, *ps = out[2].defined() ? out[2].data_ptr() : nullptr;
        rc = causal ? f(pq, pk, pv, pg, pO, pY, ps, eps, x.B, x.H, x.N, x.dk, x.dv, 64, stream_of(x.dev))
                    : f_noncausal(pq, pk, pv, pg, pO, pY, eps, x.B, x.H, x.N, x.dk, x.dv, stream_of(x.dev));
    }
    return rc != 0 ? PyLong_FromLong(rc) : wrap(out);
    END_HANDLE_TH_ERRORS
}

PyObject* gate_norm_bwd(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 6) { PyErr_SetString(PyExc_TypeError, "gate_norm_bwd takes six arguments"); return nullptr; }
    if (modes() || a[5] != Py_None || !PyFloat_CheckExact(a[4]) || !on_gpu(a[1])) Py_RETURN_NONE;
    const c10::DeviceIndex dev = c10::hip::current_device();
    for (int i = 1; i < 4; ++i) if (!plain(a[i], at::kBFloat16, dev)) Py_RETURN_NONE;
    const at::Tensor &o = THPVariable_Unpack(a[1]), &g = THPVariable_Unpack(a[2]), &d = THPVariable_Unpack(a[3]);
    if (o.dim() < 1 || g.sizes() != o.sizes() || d.sizes() != o.sizes() || o.size(-1) < 1 || o.size(-1) > 0x7fffffff) Py_RETURN_NONE;
    const auto f = address<gate_norm_bwd_fn>(a[0]);
    if (PyErr_Occurred()) return nullptr;
    const void *po = o.data_ptr(), *pg = g.data_ptr(), *pd = d.data_ptr();
    const float eps = (float)PyFloat_AS_DOUBLE(a[4]);
    at::Tensor out[2];
    int rc;
    {
        const without_interpreter_lock free;
        for (at::Tensor& t : out) t = at::empty(o.sizes(), like(o));
        rc = f(po, pg, pd, out[0].data_ptr(), out[1].data_ptr(), eps, (long long)(o.numel() / o.size(-1)), (int)o.size(-1), stream_of(dev));
    }
    return rc != 0 ? PyLong_FromLong(rc) : wrap(out);
    END_HANDLE_TH_ERRORS
}

PyObject* zbwd_saved(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 7) { PyErr_SetString(PyExc_TypeError, "zbwd_saved takes seven arguments"); return nullptr; }
    Sequences x;
    PyObject* const zv[3] = {a[1], a[1], a[3]};
    if (!x.read(zv, false, nullptr, a[6]) || !x.is_affine(a[2]) || !plain(a[4], at::kBFloat16, x.dev) || !plain(a[5], at::kFloat, x.dev))
        Py_RETURN_NONE;
    const at::Tensor &z = THPVariable_Unpack(a[1]), &v = THPVariable_Unpack(a[3]), &d = THPVariable_Unpack(a[4]);
    if (d.sizes() != v.sizes()) Py_RETURN_NONE;
    const auto f = address<zbwd_saved_fn>(a[0]);
    if (PyErr_Occurred()) return nullptr;
    const void *pz = z.data_ptr(), *pv = v.data_ptr(), *pd = d.data_ptr(), *ps = THPVariable_Unpack(a[5]).data_ptr();
    const float* pa = (const float*)THPVariable_Unpack(a[2]).data_ptr();
    at::Tensor g[3];
    int rc;
    {
        const without_interpreter_lock free;
        g[0] = at::empty({x.B, x.H, x.N, x.dk}, like(z));
        g[1] = at::empty({4, x.H, x.dk}, like(z).dtype(at::kFloat));
        g[2] = at::empty({x.B, x.H, x.N, x.dv}, like(z));
        rc = f(pz, pa, pv, pd, ps, g[0].data_ptr(), (float*)g[1].data_ptr(), g[2].data_ptr(), x.B, x.H, x.N, x.dk, x.dv, 64, stream_of(x.dev));
    }
    return rc != 0 ? PyLong_FromLong(rc) : wrap(g);
    END_HANDLE_TH_ERRORS
}

// A plain tensor of the type with as many dimensions, none beyond an int.
bool plain_sizes(PyObject* o, at::ScalarType type, c10::DeviceIndex dev, int64_t dims)
{
    if (!plain(o, type, dev)) return false;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (t.dim() != dims) return false;
    for (int64_t i = 0; i < dims; ++i) if (t.size(i) > 0x7fffffff) return false;
    return true;
}

PyObject* spectrum(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 4) { PyErr_SetString(PyExc_TypeError, "spectrum takes four arguments"); return nullptr; }
    if (modes() || a[3] != Py_None || !on_gpu(a[2])) Py_RETURN_NONE;
    const c10::DeviceIndex dev = c10::hip::current_device();
    if (!plain_sizes(a[2], at::kFloat, dev, 2)) Py_RETURN_NONE;
    const at::Tensor& k = THPVariable_Unpack(a[2]);
    const int d = (int)k.size(0), L = (int)k.size(1);
    const auto f = address<spectrum_fn>(a[0]);
    const auto bytes = address<spectrum_bytes_fn>(a[1]);
    if (PyErr_Occurred()) return nullptr;
    const size_t need = bytes(d, L);
    if (need == 0) Py_RETURN_NONE;
    const float* pk = (const float*)k.data_ptr();
    at::Tensor s;
    int rc;
    {
        const without_interpreter_lock free;
        s = at::empty({(int64_t)(need < 16 ? 16 : need) / 4}, like(k));
        rc = f(pk, s.data_ptr(), d, L, stream_of(dev));
    }
    return rc != 0 ? PyLong_FromLong(rc) : THPVariable_Wrap(std::move(s));
    END_HANDLE_TH_ERRORS
}

// X [B,d,L], w_short [d,m] or None, the spectrum (whatever its size: that is the caller's business, as in the binding).
struct Conv {
    int B, d, L, m;
    c10::DeviceIndex dev;
    at::ScalarType type;
    const float* w;
    bool read(PyObject* ox, PyObject* ow, PyObject* os, PyObject* ostream)
    {
        if (modes() || ostream != Py_None || !on_gpu(ox)) return false;
        const at::Tensor& x = THPVariable_Unpack(ox);
        type = x.scalar_type();
        dev = c10::hip::current_device();
        if ((type != at::kBFloat16 && type != at::kFloat) || !plain_sizes(ox, type, dev, 3) || !plain(os, at::kFloat, dev)) return false;
        B = (int)x.size(0); d = (int)x.size(1); L = (int)x.size(2); m = 0; w = nullptr;
        if (ow == Py_None) return true;
        if (!plain_sizes(ow, at::kFloat, dev, 2) || THPVariable_Unpack(ow).size(0) != d) return false;
        m = (int)THPVariable_Unpack(ow).size(1);
        w = (const float*)THPVariable_Unpack(ow).data_ptr();
        return true;
    }
};

PyObject* conv_fwd(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 6) { PyErr_SetString(PyExc_TypeError, "conv_fwd takes six arguments"); return nullptr; }
    Conv c;
    if (!c.read(a[2], a[3], a[4], a[5])) Py_RETURN_NONE;
    const auto f = address<conv_fwd_fn>(a[c.type == at::kFloat ? 1 : 0]);
    if (PyErr_Occurred()) return nullptr;
    const at::Tensor& x = THPVariable_Unpack(a[2]);
    const void *px = x.data_ptr(), *ps = THPVariable_Unpack(a[4]).data_ptr();
    at::Tensor z;
    int rc;
    {
        const without_interpreter_lock free;
        z = at::empty({c.B, c.d, c.L}, like(x));
        rc = f(px, c.w, c.m, ps, z.data_ptr(), c.B, c.d, c.L, stream_of(c.dev));
    }
    return rc != 0 ? PyLong_FromLong(rc) : THPVariable_Wrap(std::move(z));
    END_HANDLE_TH_ERRORS
}

PyObject* conv_bwd(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 7) { PyErr_SetString(PyExc_TypeError, "conv_bwd takes seven arguments"); return nullptr; }
    Conv c;
    if (!c.read(a[2], a[3], a[4], a[6]) || !plain(a[5], c.type, c.dev)) Py_RETURN_NONE;
    const at::Tensor &x = THPVariable_Unpack(a[2]), &dz = THPVariable_Unpack(a[5]);
    if (dz.sizes() != x.sizes()) Py_RETURN_NONE;
    const auto f = address<conv_bwd_fn>(a[c.type == at::kFloat ? 1 : 0]);
    if (PyErr_Occurred()) return nullptr;
    const void *px = x.data_ptr(), *ps = THPVariable_Unpack(a[4]).data_ptr(), *pd = dz.data_ptr();
    at::Tensor g[3];        // dX, d_w_short, d_k_long
    int rc;
    {
        const without_interpreter_lock free;
        g[0] = at::empty({c.B, c.d, c.L}, like(x));
        if (c.w != nullptr || a[3] != Py_None) g[1] = at::empty({c.d, c.m}, like(x).dtype(at::kFloat));
        g[2] = at::empty({c.d, c.L}, like(x).dtype(at::kFloat));
        rc = f(px, c.w, c.m, ps, pd, g[0].data_ptr(), g[1].defined() ? (float*)g[1].data_ptr() : nullptr, (float*)g[2].data_ptr(), c.B, c.d,
               c.L, stream_of(c.dev));
    }
    return rc != 0 ? PyLong_FromLong(rc) : wrap(g);
    END_HANDLE_TH_ERRORS
}

#define CHELA_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {CHELA_METHOD(step), CHELA_METHOD(forward), CHELA_METHOD(backward), CHELA_METHOD(gated),
                         CHELA_METHOD(gate_norm_bwd), CHELA_METHOD(zbwd_saved), CHELA_METHOD(spectrum), CHELA_METHOD(conv_fwd),
                         CHELA_METHOD(conv_bwd), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_chela_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__chela_host() { return PyModule_Create(&module); }
