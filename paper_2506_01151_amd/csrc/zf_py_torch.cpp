// Extension module _native_torch: what the binding has to know of a torch tensor, read from the tensor itself instead of through a
// dozen Python attribute look-ups (2 us a call).
#define PY_SSIZE_T_CLEAN
#include <torch/csrc/autograd/python_variable.h>
#include <c10/hip/HIPStream.h>
#include "zf_py.h"

namespace {

// What cannot be looked at -- a tensor whose size, strides or address torch refuses to give (nested tensors, the wrappers of vmap and
// grad, all of which pass for plain ones) -- is not an ordinary case: its exception must not leave a C function, and the twin raises its own.
bool look(void *o, zfpy::TensorInfo *out) noexcept {
    PyObject *obj = (PyObject *)o;
    if (!THPVariable_CheckExact(obj)) return false;
    try {
        const at::Tensor &t = THPVariable_Unpack(obj);
        if (t.layout() != at::kStrided || t.is_nested() || t.dim() > 2 || t.unsafeGetTensorImpl()->has_symbolic_sizes_strides() || t.is_neg() || t.is_conj()) return false;
        out->dim = (int32_t)t.dim();
        for (int k = 0; k < out->dim; k++) { out->size[k] = t.size(k); out->stride[k] = t.stride(k); }
        out->device = t.is_cuda() ? (int32_t)t.get_device() : -1;
        const auto st = t.scalar_type();
        out->dtype = st == at::kFloat ? 0 : st == at::kBFloat16 ? 1 : st == at::kInt ? 2 : -1;
        out->contiguous = t.is_contiguous();
        out->data = out->device >= 0 ? t.data_ptr() : nullptr;
    } catch (...) { return false; }
    return true;
}

bool stream(int32_t device, void **out) noexcept {
    try { *out = (void *)c10::hip::getCurrentHIPStream((c10::DeviceIndex)device).stream(); } catch (...) { return false; }
    return true;
}

zfpy::TensorCalls calls = {look, stream};

PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_native_torch", "Access to torch tensors for the _native module.", -1, nullptr, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native_torch(void) {
    PyObject *m = PyModule_Create(&module_def);
    if (!m) return nullptr;
    PyObject *c = PyCapsule_New(&calls, zfpy::TENSOR_CALLS_NAME, nullptr);
    if (!c || PyModule_AddObject(m, "calls", c) < 0) { Py_XDECREF(c); Py_DECREF(m); return nullptr; }
    return m;
}
