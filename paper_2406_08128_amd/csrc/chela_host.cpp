// The decode step's host path without the interpreter: checks, the output's allocation, the current stream and the call into
// libchela.so for plain device tensors.  A step is over in 4.5 us on the GPU; through the binding's own lines, a dozen attribute
// look-ups, torch.empty() and ctypes, the host needed 8.9 us for it, of which the launch is 3.4.
//
// step(function, q, k, v, g or None, S, eps, y or None, stream or None) -> y, a status of the library (int, not 0), or None:
// "not the plain case", and nothing has been done.  The binding then takes its own path, which says what is wrong or serves the
// case (other devices, subclasses, modes).  function: address of chela_linattn_step (g is None) or chela_linattn_step_gated.
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

struct without_interpreter_lock {
    PyThreadState* const state = PyEval_SaveThread();
    ~without_interpreter_lock() { PyEval_RestoreThread(state); }
};

PyObject* step(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 9) { PyErr_SetString(PyExc_TypeError, "step takes nine arguments"); return nullptr; }
    if (at::impl::PythonTorchFunctionTLS::stack_len() > 0 || c10::impl::TorchDispatchModeTLS::any_modes_set()) Py_RETURN_NONE;
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

PyMethodDef methods[] = {{"step", (PyCFunction)(void (*)(void))step, METH_FASTCALL, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_chela_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__chela_host() { return PyModule_Create(&module); }
