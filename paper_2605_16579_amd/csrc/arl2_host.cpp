// The host side of a small call: checks a call's tensors, fills the descriptor and calls the C ABI, without the per-tensor Python work.
//
//   call(function address, kinds, sm_scale, l2_eps, stream, workspace or None, tensors...) -> status, or None
//
// None means that something is not as a plain call has it (another type than torch.Tensor, not in device memory, not
// contiguous, another shape or type): nothing has been called, and the Python binding goes through its own checks, which
// raise what is to be raised.  One character of `kinds` per tensor says what it must be; None stands for NULL except for k:
//   q  [B][Lq][H][D], the inputs' type (the first tensor, which names the sizes and the type)      k  [B][Lkv][H][D], likewise
//   S  [B][H][D][D] fp32    W  [H][D][D], the inputs' type    r  [Lq][D/2] fp32    a  [B][H] fp32    t  [B][Lq][H] fp32
//   g  [B][Lq][H], [B][Lq] or [B][Lq][H][D], fp32 or bf16: sets the descriptor's gate mode and type
// Measured: a call of the smallest size took 7 us to issue through ctypes, of them 3.5 in the library and the runtime.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/arl2.h"

namespace {

constexpr int kMaxTensors = 10;

struct Checked {
    arl2_desc d{};
    const void *p[kMaxTensors] = {};
    bool sized = false;
};

int type_code(const at::Tensor &t)
{
    return t.scalar_type() == at::kFloat ? ARL2_F32 : t.scalar_type() == at::kBFloat16 ? ARL2_BF16 : -1;
}

bool is_shape(const at::Tensor &t, std::initializer_list<int64_t> want) { return t.sizes().equals(at::IntArrayRef(want)); }

// A plain tensor in device memory, contiguous; nullptr otherwise.
const at::Tensor *plain(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.defined() && t.is_cuda() && t.is_contiguous() ? &t : nullptr;
}

bool check(Checked &c, char kind, PyObject *o, int i)
{
    arl2_desc &d = c.d;
    if (o == Py_None && i > 0) return kind != 'k';      // (keys name a size: the binding's checks refuse None)
    const at::Tensor *t = plain(o);
    if (t == nullptr) return false;
    const int type = type_code(*t);
    if (type < 0) return false;
    if (i == 0) {
        if (kind != 'q' || t->dim() != 4) return false;
        for (int64_t n : t->sizes())
            if (n > INT32_MAX) return false;
        d.B = (int32_t)t->size(0); d.Lq = d.Lkv = (int32_t)t->size(1); d.H = (int32_t)t->size(2); d.D = (int32_t)t->size(3);
        d.io_dtype = type;
    }
    const int64_t B = d.B, H = d.H, Lq = d.Lq, D = d.D;
    bool ok = false;
    switch (kind) {
    case 'q': ok = type == d.io_dtype && is_shape(*t, {B, Lq, H, D}); break;
    case 'k':
        if (!c.sized) {                       // the first of them names Lkv
            if (t->dim() != 4 || t->size(1) > INT32_MAX) return false;
            d.Lkv = (int32_t)t->size(1);
            c.sized = true;
        }
        ok = type == d.io_dtype && is_shape(*t, {B, d.Lkv, H, D});
        break;
    case 'W': ok = type == d.io_dtype && is_shape(*t, {H, D, D}); break;
    case 'S': ok = type == ARL2_F32 && is_shape(*t, {B, H, D, D}); break;
    case 'r': ok = type == ARL2_F32 && is_shape(*t, {Lq, D / 2}); break;
    case 'a': ok = type == ARL2_F32 && is_shape(*t, {B, H}); break;
    case 't': ok = type == ARL2_F32 && is_shape(*t, {B, Lq, H}); break;
    case 'g':
        d.g_dtype = type;
        d.g_mode = t->dim() == 4 ? ARL2_GATE_PER_ELEMENT : t->dim() == 2 ? ARL2_GATE_PER_TOKEN : ARL2_GATE_PER_HEAD;
        ok = t->dim() == 4 ? is_shape(*t, {B, Lq, H, D}) : t->dim() == 2 ? is_shape(*t, {B, Lq}) : is_shape(*t, {B, Lq, H});
        break;
    }
    if (ok) c.p[i] = t->data_ptr();
    return ok;
}

int invoke(void *f, const arl2_desc *d, const void *const *p, int n)
{
    typedef const void *P;
    switch (n) {
    case 3: return ((int (*)(const arl2_desc *, P, P, P))f)(d, p[0], p[1], p[2]);
    case 4: return ((int (*)(const arl2_desc *, P, P, P, P))f)(d, p[0], p[1], p[2], p[3]);
    case 5: return ((int (*)(const arl2_desc *, P, P, P, P, P))f)(d, p[0], p[1], p[2], p[3], p[4]);
    case 6: return ((int (*)(const arl2_desc *, P, P, P, P, P, P))f)(d, p[0], p[1], p[2], p[3], p[4], p[5]);
    case 7: return ((int (*)(const arl2_desc *, P, P, P, P, P, P, P))f)(d, p[0], p[1], p[2], p[3], p[4], p[5], p[6]);
    case 8: return ((int (*)(const arl2_desc *, P, P, P, P, P, P, P, P))f)(d, p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7]);
    case 10:
        return ((int (*)(const arl2_desc *, P, P, P, P, P, P, P, P, P, P))f)(d, p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7], p[8], p[9]);
    }
    return -1;
}

PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    constexpr Py_ssize_t kFixed = 6;
    if (nargs <= kFixed || !PyBytes_CheckExact(args[1]) || PyBytes_GET_SIZE(args[1]) != nargs - kFixed || nargs - kFixed > kMaxTensors) Py_RETURN_NONE;
    const int n = (int)(nargs - kFixed);
    const char *kinds = PyBytes_AS_STRING(args[1]);
    void *f = PyLong_AsVoidPtr(args[0]);
    const double sm_scale = PyFloat_AsDouble(args[2]), l2_eps = PyFloat_AsDouble(args[3]);
    void *stream = PyLong_Check(args[4]) ? PyLong_AsVoidPtr(args[4]) : nullptr;
    if (PyErr_Occurred() || f == nullptr || !PyLong_Check(args[4])) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    Checked c;
    try {
        for (int i = 0; i < n; ++i)
            if (!check(c, kinds[i], args[kFixed + i], i)) Py_RETURN_NONE;
        if (args[5] != Py_None) {
            const at::Tensor *w = plain(args[5]);
            if (w == nullptr) Py_RETURN_NONE;
            c.d.workspace = w->data_ptr();
            c.d.workspace_bytes = w->nbytes();
        }
    } catch (...) {                           // a tensor without storage, or of a layout that has no such notion
        Py_RETURN_NONE;
    }
    c.d.sm_scale = (float)sm_scale;
    c.d.l2_eps = (float)l2_eps;
    c.d.stream = stream;
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = invoke(f, &c.d, c.p, n);
    Py_END_ALLOW_THREADS
    if (st < 0) Py_RETURN_NONE;
    return PyLong_FromLong(st);
}

PyMethodDef methods[] = {{"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL, "Checks a call's tensors and calls the C ABI."},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_arl2_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__arl2_host(void)
{
    PyObject *m = PyModule_Create(&module);
    if (m != nullptr && PyModule_AddStringConstant(m, "built_for", ARL2_HOST_FOR) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
