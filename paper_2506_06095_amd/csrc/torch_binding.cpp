// Plan.forward for ordinary calls, as one native call: checks of shapes and types, the output's allocation, the current
// stream and smha_forward.  A call with a short kernel lasts as long as its host side: 8 us in Python through ctypes, 4.7 so, of which
// the launch is 3.5 and the output's allocation 0.6 (window 1 x 2 x 128 x 64 8.0 -> 4.9 us a call; a launch of torch's own 4 to 5).
//
// It answers for plain dense tensors only, and leaves every other call, those that are errors among them, to
// binding.smha_forward (by returning None): subclasses, named, functorch-wrapped, tracked by a mode, other layouts, a shape or type
// that does not fit.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "smha.h"

namespace {

using Forward = decltype(&smha_forward);

bool plain(PyObject *obj) {
    if (!THPVariable_CheckExact(obj)) return false;
    const at::Tensor &t = THPVariable_Unpack(obj);
    constexpr c10::DispatchKeySet ordinary({c10::DispatchKey::CUDA, c10::DispatchKey::AutogradCUDA, c10::DispatchKey::ADInplaceOrView,
                                            c10::DispatchKey::AutocastCUDA});
    return t.defined() && (t.key_set() | ordinary) == ordinary && t.is_cuda() && t.dim() == 4 && !t.has_names() &&
           !t.unsafeGetTensorImpl()->has_symbolic_sizes_strides();
}

int code_of(at::ScalarType type) {
    return type == at::kHalf ? SMHA_F16 : type == at::kBFloat16 ? SMHA_BF16 : type == at::kFloat ? SMHA_F32 : -1;
}

// the three leading strides, or null where the tensor is packed; ok is cleared where a head's elements do not follow each other
const int64_t *strides_of(const at::Tensor &t, bool &ok) {
    if (t.is_contiguous()) return nullptr;
    ok = ok && t.strides()[3] == 1;
    return t.strides().data();
}

// forward(address of smha_forward, plan handle, S, Sk, Q, K, V, out or None, out_dtype or None, scale, kernel) -> the output, a status that is
// not SMHA_OK, or None
PyObject *forward(PyObject *, PyObject *const *args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 11 || at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set()) Py_RETURN_NONE;
    if (!plain(args[4]) || !plain(args[5]) || !plain(args[6])) Py_RETURN_NONE;
    if (!PyLong_CheckExact(args[1]) || !PyFloat_CheckExact(args[9]) || !PyLong_CheckExact(args[10])) Py_RETURN_NONE;
    const auto entry = reinterpret_cast<Forward>(PyLong_AsVoidPtr(args[0]));
    const auto *plan = static_cast<const smha_plan_t *>(PyLong_AsVoidPtr(args[1]));
    const int64_t S = PyLong_AsLongLong(args[2]), Sk = PyLong_AsLongLong(args[3]);
    const double scale = PyFloat_AS_DOUBLE(args[9]);
    const long kernel = PyLong_AsLong(args[10]);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    const at::Tensor &q = THPVariable_Unpack(args[4]), &k = THPVariable_Unpack(args[5]), &v = THPVariable_Unpack(args[6]);
    const at::ScalarType type = q.scalar_type();
    const int in = code_of(type);
    if (in < 0 || in == SMHA_F32 || k.scalar_type() != type || v.scalar_type() != type) Py_RETURN_NONE;
    const at::IntArrayRef qn = q.sizes(), kn = k.sizes();
    if (kn != v.sizes() || qn[0] != kn[0] || qn[1] != kn[1] || qn[3] != kn[3] || qn[2] != S || kn[2] != Sk) Py_RETURN_NONE;
    if (qn[0] > INT32_MAX || qn[1] > INT32_MAX || qn[3] > INT32_MAX) Py_RETURN_NONE;
    at::Tensor o;
    if (args[7] == Py_None) {
        at::ScalarType out_type = type;
        if (args[8] != Py_None) {
            if (!THPDtype_Check(args[8])) Py_RETURN_NONE;
            out_type = reinterpret_cast<THPDtype *>(args[8])->scalar_type;
        }
        if (code_of(out_type) < 0) Py_RETURN_NONE;
        o = at::empty(qn, q.options().dtype(out_type), at::MemoryFormat::Contiguous);
    } else {
        if (!plain(args[7])) Py_RETURN_NONE;
        o = THPVariable_Unpack(args[7]);
        if (o.sizes() != qn) Py_RETURN_NONE;
    }
    const int out = code_of(o.scalar_type());
    bool ok = out >= 0;
    const int64_t *qs = strides_of(q, ok), *ks = strides_of(k, ok), *vs = strides_of(v, ok), *os = strides_of(o, ok);
    if (!ok) Py_RETURN_NONE;
    void *const stream = c10::hip::getCurrentHIPStream(q.device().index()).stream();
    const void *const qp = q.data_ptr(), *const kp = k.data_ptr(), *const vp = v.data_ptr();
    void *const op = o.data_ptr();
    smha_status_t status;
    Py_BEGIN_ALLOW_THREADS
    status = entry(plan, qp, kp, vp, op, (int)qn[0], (int)qn[1], (int)qn[3], (smha_dtype_t)in, (smha_dtype_t)out, qs, ks, vs, os, (float)scale,
                   (smha_kernel_t)kernel, stream);
    Py_END_ALLOW_THREADS
    if (status != SMHA_OK) return PyLong_FromLong((long)status);
    if (args[7] != Py_None) {
        Py_INCREF(args[7]);
        return args[7];
    }
    return THPVariable_Wrap(std::move(o));
    END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {{"forward", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(forward)), METH_FASTCALL, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_smha_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__smha_torch() {
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "stamp", SMHA_STAMP) < 0) Py_CLEAR(m);  // what it was built from: build.py looks for it in the file
    return m;
}
