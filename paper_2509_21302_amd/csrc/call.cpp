// What DsfqLinear does on the host between two launches, in native code: the checks of a call's tensors, the output's allocation, the current
// stream, the call of the C entry point with the interpreter's lock released.  The same as the Python functions of binding.py do one by one
// (a call of two launches, 64 x 128 -> 128 in f32 when it was one: 11.5 us with them, 8.9 this way, of which 7.2 are the launches).
//
// linear(kind, X, signs, inv_smooth, gelu_table, W, w_scale, bias, out, workspace, N, bits)
//   -> the output, or the entry point's status where it is not 0, or NotImplemented, before anything is launched, where a call is not an ordinary
//      one: an argument that is no plain contiguous GPU tensor (a subclass, a wrapper, a view that is not contiguous), an X that is not
//      two-dimensional bf16 or f32, an output that cannot be allocated.  The caller's Python path takes it then, with its errors.  As there, types
//      of the other operands and which GPU holds what are the caller's to get right.
// bind(kind, address): the C entry point of a kind.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>

#include <cstdint>

namespace {

enum Kind { kPacked, kE2m3, kGelu, kInt8, kInt8Blocks, kKinds };
void *entry[kKinds];

using PackedFn = int (*)(const void *, int, int, int, int, const void *, const void *, const void *, const void *, const void *, void *, void *, size_t, void *);
using GeluFn = int (*)(const void *, int, int, int, int, const void *, const void *, const void *, const void *, const void *, const void *, void *, void *, size_t, void *);
using Int8Fn = int (*)(const void *, int, int, int, int, const void *, const void *, int, const void *, const void *, const void *, void *, void *, size_t, void *);

// the tensor behind an argument, if it is an ordinary one on the GPU, contiguous and with memory of its own kind; nullptr otherwise
const at::Tensor *ordinary(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || t.layout() != at::kStrided || !t.has_storage() || !t.is_cuda() || !t.is_contiguous() || t.is_conj() || t.is_neg()) return nullptr;
    return &t;
}

// device address of a tensor, or nullptr for None; false if the argument is neither
bool address(PyObject *o, const void **p)
{
    *p = nullptr;
    if (o == Py_None) return true;
    const at::Tensor *t = ordinary(o);
    if (t == nullptr) return false;
    *p = t->const_data_ptr();
    return true;
}

PyObject *linear(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 12) {
        PyErr_SetString(PyExc_TypeError, "linear takes 12 arguments");
        return nullptr;
    }
    bool launched = false;
    try {
        const long kind = PyLong_AsLong(args[0]), N_layer = PyLong_AsLong(args[10]), bits = PyLong_AsLong(args[11]);
        if (PyErr_Occurred()) return nullptr;
        if (kind < 0 || kind >= kKinds || entry[kind] == nullptr) Py_RETURN_NOTIMPLEMENTED;
        const at::Tensor *X = ordinary(args[1]), *ws = ordinary(args[9]);
        if (X == nullptr || ws == nullptr || X->dim() != 2 || X->size(0) > INT32_MAX || X->size(1) > INT32_MAX) Py_RETURN_NOTIMPLEMENTED;
        const at::ScalarType type = X->scalar_type();
        if (type != at::kBFloat16 && type != at::kFloat) Py_RETURN_NOTIMPLEMENTED;
        const void *signs, *inv, *table, *W, *w_scale, *bias;
        if (!address(args[2], &signs) || !address(args[3], &inv) || !address(args[4], &table) || !address(args[5], &W) || !address(args[6], &w_scale) ||
            !address(args[7], &bias))
            Py_RETURN_NOTIMPLEMENTED;
        const int M = (int)X->size(0), K = (int)X->size(1);
        at::Tensor made;
        const at::Tensor *Y = nullptr;
        if (args[8] == Py_None) {
            made = at::empty({M, N_layer}, X->options().dtype(at::kBFloat16));
            Y = &made;
        } else {
            Y = ordinary(args[8]);
            if (Y == nullptr || Y->dim() != 2 || Y->size(1) > INT32_MAX) Py_RETURN_NOTIMPLEMENTED;
        }
        const int N = (int)Y->size(1);
        const void *x = X->const_data_ptr();
        void *y = Y->data_ptr(), *w = ws->data_ptr();
        const size_t w_bytes = (size_t)ws->numel() * ws->element_size();
        const int dtype = type == at::kFloat;                       // QVGGT_BF16 = 0, QVGGT_F32 = 1
        void *stream = reinterpret_cast<void *>(c10::hip::getCurrentHIPStream(c10::hip::current_device()).stream());
        int status;
        launched = true;
        Py_BEGIN_ALLOW_THREADS
        switch (kind) {
            case kGelu: status = reinterpret_cast<GeluFn>(entry[kind])(x, dtype, M, N, K, signs, inv, table, W, w_scale, bias, y, w, w_bytes, stream); break;
            case kInt8:
            case kInt8Blocks: status = reinterpret_cast<Int8Fn>(entry[kind])(x, dtype, M, N, K, signs, inv, (int)bits, W, w_scale, bias, y, w, w_bytes, stream); break;
            default: status = reinterpret_cast<PackedFn>(entry[kind])(x, dtype, M, N, K, signs, inv, W, w_scale, bias, y, w, w_bytes, stream); break;
        }
        Py_END_ALLOW_THREADS
        if (status != 0) return PyLong_FromLong(status);
        if (args[8] == Py_None) return THPVariable_Wrap(std::move(made));
        Py_INCREF(args[8]);
        return args[8];
    } catch (python_error &e) {                                     // raised in Python: a dispatch mode that sees the allocation
        e.restore();
        return nullptr;
    } catch (const std::exception &e) {
        if (!launched) Py_RETURN_NOTIMPLEMENTED;                    // torch's own errors, the allocator's among them: torch.empty raises them as Python knows them
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

PyObject *bind(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 2) {
        PyErr_SetString(PyExc_TypeError, "bind takes 2 arguments");
        return nullptr;
    }
    const long kind = PyLong_AsLong(args[0]);
    void *const address = PyLong_AsVoidPtr(args[1]);
    if (PyErr_Occurred()) return nullptr;
    if (kind < 0 || kind >= kKinds) {
        PyErr_SetString(PyExc_ValueError, "no such kind");
        return nullptr;
    }
    entry[kind] = address;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"linear", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(linear)), METH_FASTCALL, nullptr},
                         {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(bind)), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call()
{
    PyObject *const m = PyModule_Create(&module);
    if (m != nullptr && PyModule_AddStringConstant(m, "torch_version", QVGGT_TORCH_VERSION) != 0) {       // binding.py compares it
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
