// Single-tensor calls of the Python binding: the checks of srs.py on the tensors and the call into libsrs.so in one step.  The
// functions return what the library returned, or None where any argument is not what the checks ask for (or is anything but
// a plain tensor or integer): srs.py then goes its general way, which raises the errors.  What bounds a call on a small
// tensor is the host: extract and apply of 4096 elements took 11.7 us from Python and ctypes; it takes
// 7.8 us this way (8.1 against 12.1 us per pair in a loop of their own).
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/TensorSubclassLikeUtils.h>

#include <cstdint>

namespace {

// A plain contiguous tensor on the GPU of `width` bytes per element; null otherwise.
const at::Tensor *on_gpu(PyObject *o, size_t width) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || at::isTensorSubclassLike(t) || !t.is_cuda() || t.layout() != at::kStrided) return nullptr;
    if ((size_t)t.element_size() != width || !t.is_contiguous()) return nullptr;
    return &t;
}

bool number(PyObject *o, uint64_t &v) {
    if (!PyLong_CheckExact(o)) return false;
    v = PyLong_AsUnsignedLongLong(o);
    if (v == (uint64_t)-1 && PyErr_Occurred()) { PyErr_Clear(); return false; }
    return true;
}

struct Payload { void *I, *V, *counts; };

bool payload(PyObject *const *args, uint64_t n, uint64_t be, uint64_t cap, size_t width, Payload &p) {
    if (be == 0 || cap == 0 || be > 0x7fffffffull || cap > 0x7fffffffull) return false;
    const at::Tensor *I = on_gpu(args[0], 4), *V = on_gpu(args[1], width), *c = on_gpu(args[2], 4);
    if (!I || !V || !c || I->scalar_type() != at::kInt) return false;
    const uint64_t nb = (n + be - 1) / be;
    if ((uint64_t)I->numel() < nb * cap || (uint64_t)V->numel() < nb * cap || (uint64_t)c->numel() < nb) return false;
    p = Payload{I->data_ptr(), V->data_ptr(), c->data_ptr()};
    return true;
}

typedef int (*ExtractFn)(void *, void *, const void *, uint64_t, uint64_t, void *, void *, void *, uint64_t, void *);
typedef int (*ApplyFn)(void *, void *, uint64_t, uint64_t, const void *, const void *, const void *, uint64_t, void *);

// Nothing that torch throws leaves a function: the general way meets the same tensor and reports it.
// extract(function, context, old, new, bucket_elems, I, V, counts, cap, stream, width, new_width)
PyObject *extract(PyObject *, PyObject *const *args, Py_ssize_t n_args) {
    uint64_t fn, ctx, be, cap, stream, width, new_width;
    if (n_args != 12 || !number(args[0], fn) || !number(args[1], ctx) || !number(args[4], be) || !number(args[8], cap) ||
        !number(args[9], stream) || !number(args[10], width) || !number(args[11], new_width))
        Py_RETURN_NONE;
    uint64_t n;
    Payload p;
    void *old_p, *new_p;
    try {
        const at::Tensor *o = on_gpu(args[2], width), *w = on_gpu(args[3], new_width);
        if (!o || !w || o->numel() != w->numel() || (new_width != width && w->scalar_type() != at::kFloat)) Py_RETURN_NONE;
        n = (uint64_t)o->numel();
        if (n > 0x7fffffffull || !payload(args + 5, n, be, cap, width, p)) Py_RETURN_NONE;
        old_p = o->data_ptr(), new_p = w->data_ptr();
    } catch (...) {
        Py_RETURN_NONE;
    }
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = ((ExtractFn)fn)((void *)ctx, old_p, new_p, n, be, p.I, p.V, p.counts, cap, (void *)stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// apply(function, context, weights, bucket_elems, I, V, counts, cap, stream, width)
PyObject *apply(PyObject *, PyObject *const *args, Py_ssize_t n_args) {
    uint64_t fn, ctx, be, cap, stream, width;
    if (n_args != 10 || !number(args[0], fn) || !number(args[1], ctx) || !number(args[3], be) || !number(args[7], cap) ||
        !number(args[8], stream) || !number(args[9], width))
        Py_RETURN_NONE;
    uint64_t n;
    Payload p;
    void *weights;
    try {
        const at::Tensor *w = on_gpu(args[2], width);
        if (!w) Py_RETURN_NONE;
        n = (uint64_t)w->numel();
        if (n > 0x7fffffffull || !payload(args + 4, n, be, cap, width, p)) Py_RETURN_NONE;
        weights = w->data_ptr();
    } catch (...) {
        Py_RETURN_NONE;
    }
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = ((ApplyFn)fn)((void *)ctx, weights, n, be, p.I, p.V, p.counts, cap, (void *)stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

PyMethodDef methods[] = {{"extract", (PyCFunction)(void (*)(void))extract, METH_FASTCALL, nullptr},
                         {"apply", (PyCFunction)(void (*)(void))apply, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// The version of the torch whose headers this was built against: srs.py takes the module only where it is the running one's.
PyMODINIT_FUNC PyInit__call(void) {
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", SRS_TORCH_VERSION) < 0) { Py_DECREF(m); return nullptr; }
    return m;
}
