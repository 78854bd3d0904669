// attention() of the package as one native call: checks, O and LSE allocated by torch, the C entry on torch's current stream.
//
// Host code only.  In Python the same steps took longer than a small launch: 9.0 us a call (1.2 and 1.8 for the two allocations, 1.0 for the
// checks, 0.9 for the arguments, 3.7 for the C entry through ctypes), and the kernel of one sequence of 512 keys, 4 heads, 7.1.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/DeviceGuard.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <cmath>

namespace {

using Entry = int (*)(const void *, const void *, const void *, void *, float *, int, int, int, int, int, int, int, float, void *);
Entry entry = nullptr;

PyObject *refuse(const char *why)
{
    PyErr_SetString(PyExc_ValueError, why);
    return nullptr;
}

// call(q, k, v, causal, scale): (O, LSE); a status code of the C entry if it is not 0; None if this is not its business (a tensor of another
// type than torch.Tensor itself, a torch function mode, sizes beyond an int, a scale that is no number, a C++ exception of torch's): the
// caller has a general form.
PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    if (nargs != 5) return refuse("call(q, k, v, causal, scale)");
    if (entry == nullptr || at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
    for (int i = 0; i < 3; ++i)
        if (!THPVariable_CheckExact(args[i])) Py_RETURN_NONE;
    try {
        const at::Tensor &q = THPVariable_Unpack(args[0]), &k = THPVariable_Unpack(args[1]), &v = THPVariable_Unpack(args[2]);
        const at::Tensor *all[3] = {&q, &k, &v};
        for (const at::Tensor *t : all)
            if (!t->is_cuda()) return refuse("attention() needs device tensors; there is no CPU path");
        for (const at::Tensor *t : all)
            if (t->scalar_type() != at::kBFloat16 || !t->is_contiguous() || t->dim() != 4)
                return refuse("q, k, v must be contiguous 4-d BF16 tensors [B, S, H, D]");
        const int64_t B = q.size(0), Sq = q.size(1), Hq = q.size(2), D = q.size(3), Skv = k.size(1), Hkv = k.size(2);
        if (k.size(0) != B || k.size(3) != D || k.sizes() != v.sizes()) return refuse("inconsistent q/k/v shapes");
        for (int64_t n : {B, Sq, Hq, D, Skv, Hkv})
            if (n > INT_MAX) Py_RETURN_NONE;
        float scale;
        if (args[4] == Py_None) {
            if (D == 0) Py_RETURN_NONE;
            scale = (float)std::pow((double)D, -0.5);
        } else {
            const double s = PyFloat_AsDouble(args[4]);
            if (s == -1.0 && PyErr_Occurred()) {
                PyErr_Clear();
                Py_RETURN_NONE;
            }
            scale = (float)s;
        }
        const int causal = PyObject_IsTrue(args[3]);
        if (causal < 0) return nullptr;
        const at::Tensor o = at::empty_like(q), lse = at::empty({B, Hq, Sq}, q.options().dtype(at::kFloat));
        const auto index = q.get_device();
        void *stream = (void *)c10::hip::getCurrentHIPStream(index).stream();
        const void *pq = q.data_ptr(), *pk = k.data_ptr(), *pv = v.data_ptr();
        void *po = o.data_ptr();
        float *pl = (float *)lse.data_ptr();
        int rc;
        auto launch = [&]() {
            Py_BEGIN_ALLOW_THREADS
            rc = entry(pq, pk, pv, po, pl, (int)B, (int)Hq, (int)Hkv, (int)Sq, (int)Skv, (int)D, causal, scale, stream);
            Py_END_ALLOW_THREADS
        };
        if (index == c10::hip::current_device()) {
            launch();
        } else {
            const c10::DeviceGuard guard(q.device());
            launch();
        }
        if (rc != 0) return PyLong_FromLong(rc);
        PyObject *po_ = THPVariable_Wrap(o), *pl_ = po_ ? THPVariable_Wrap(lse) : nullptr;
        PyObject *both = pl_ ? PyTuple_Pack(2, po_, pl_) : nullptr;
        Py_XDECREF(po_);
        Py_XDECREF(pl_);
        return both;
    } catch (python_error &e) {     // of a dispatch mode, for instance: the exception itself, whether the interpreter still holds it or `e` does
        e.restore();
    } catch (const std::exception &) {
    }
    if (PyErr_Occurred()) return nullptr;
    Py_RETURN_NONE;         // (the general form meets it again, and torch raises its own exception)
}

// bind(address of attn_fwd)
PyObject *bind(PyObject *, PyObject *address)
{
    void *p = PyLong_AsVoidPtr(address);
    if (p == nullptr && PyErr_Occurred()) return nullptr;
    entry = (Entry)p;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL, "attention() on tensors"},
                         {"bind", bind, METH_O, "sets the C entry"},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_attn_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__attn_call() { return PyModule_Create(&module); }
