// Argument marshalling of binding.py's three calls in native code: a CPython module, one function per C entry point.
//
// A step of a small problem takes the GPU 50 us and a layer call 10, and the same checks written in Python (five attribute
// look-ups per tensor, a dictionary per layer, ctypes arrays) took 25-80 us of host time per call.  Every
// function here handles the ordinary call only: GPU tensors that are contiguous, of the right element size and long
// enough, passed as the entry point wants them.  Anything else (a raw address, a short tensor, a tuple as workspace,
// taps) makes it return None, and binding.py then takes its own path, which raises what there is to raise.  That path also
// does the work alone where this module is missing.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <vector>

#include "../../include/phantom.h"

namespace {

typedef ph_status (*FwdFn)(const ph_problem *, const void *, const void *, const void *, const void *, const void *, const void *,
                           void *, void *, void *, void *, size_t, void *);
typedef ph_status (*BwdFn)(const ph_problem *, const void *, const void *, const void *, const void *, const void *, const void *,
                           const void *, void *, void *, float *, float *, float *, float *, void *, void *, size_t, void *);
typedef ph_status (*StepFn)(const ph_problem *, const ph_step_args *, void *, size_t, void *);
typedef ph_status (*StaticFn)(const ph_problem *, const ph_step_args *, void *);
FwdFn g_fwd;
BwdFn g_bwd;
StepFn g_step;
StaticFn g_static;

// what binding.py's _check_layer_tensors knows of a layer
struct Counts {
    int64_t in, out, L, C, D, b, g, send, gathered;
    int64_t esz;
};

bool problem_of(PyObject *obj, const ph_problem **prob, Py_buffer *view)
{
    if (PyObject_GetBuffer(obj, view, PyBUF_SIMPLE) != 0) { PyErr_Clear(); return false; }
    if (view->len < (Py_ssize_t)sizeof(ph_problem)) { PyBuffer_Release(view); return false; }
    *prob = (const ph_problem *)view->buf;
    return true;
}

bool counts_of(const ph_problem *pr, int layer, Counts &c)
{
    if (pr->p < 1 || pr->batch < 1 || layer >= pr->layers) return false;
    const int64_t q = pr->p - 1, B = pr->batch, groups = pr->rank < 0 ? pr->p : 1;
    const int64_t si = (pr->widths ? pr->widths[layer] : pr->n) / pr->p, so = (pr->widths ? pr->widths[layer + 1] : pr->n) / pr->p;
    const int64_t k = q > 0 ? (pr->widths && pr->ks ? pr->ks[layer] : pr->k) : 0;
    c.in = groups * B * si; c.out = groups * B * so; c.L = groups * so * si; c.C = groups * k * si; c.D = groups * q * so * k;
    c.b = groups * so; c.g = groups * B * k; c.send = groups * q * B * k; c.gathered = (pr->rank < 0 ? pr->p : q) * B * k;
    c.esz = pr->dtype == PH_BF16 ? 2 : 4;
    return true;
}

// None -> NULL, a fitting GPU tensor -> its address; anything else: false
bool address(PyObject *obj, int64_t elems, int64_t elem_bytes, void **out)
{
    *out = nullptr;
    if (obj == Py_None) return true;
    if (!THPVariable_Check(obj)) return false;
    const at::Tensor &t = THPVariable_Unpack(obj);
    if (elems > 0 && (!t.is_cuda() || !t.is_contiguous() || (int64_t)t.element_size() != elem_bytes || t.numel() < elems)) return false;
    if (!t.is_cuda()) return false;
    *out = t.data_ptr();
    return true;
}

bool workspace_of(PyObject *obj, void **ws, size_t *bytes)
{
    *ws = nullptr;
    *bytes = 0;
    if (obj == Py_None) return true;
    if (!THPVariable_Check(obj)) return false;
    const at::Tensor &t = THPVariable_Unpack(obj);
    *ws = t.data_ptr();
    *bytes = t.numel() * t.element_size();
    return true;
}

bool stream_of(PyObject *obj, void **stream)
{
    if (obj == Py_None) {
        *stream = (void *)c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    if (!PyLong_Check(obj)) return false;
    *stream = PyLong_AsVoidPtr(obj);
    if (PyErr_Occurred()) { PyErr_Clear(); return false; }
    return true;
}

struct Released {             // the problem's buffer, given back on every way out
    Py_buffer view{};
    bool held = false;
    ~Released() { if (held) PyBuffer_Release(&view); }
};

struct WithoutGil {           // taken back on every way out
    PyThreadState *state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

PyObject *none() { Py_RETURN_NONE; }

// Tensor and stream queries throw (a sparse tensor has no address, a host without a GPU no stream) and CPython is C: an
// exception must not leave here.  None sends the call down binding.py's path, where torch raises its own error.
template <PyObject *(*Body)(PyObject *const *, Py_ssize_t)>
PyObject *guarded(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    try {
        return Body(a, n);
    } catch (...) {
        PyErr_Clear();
        return none();
    }
}

// (prob, X, Lw, Cw, Dw, bias, G, Y, g_own, A_save, workspace, stream)
PyObject *layer_fwd(PyObject *const *a, Py_ssize_t n)
{
    Released r;
    const ph_problem *pr;
    Counts c;
    if (n != 12 || !(r.held = problem_of(a[0], &pr, &r.view)) || !counts_of(pr, 0, c)) return none();
    const int64_t elems[9] = {c.in, c.L, c.C, c.D, c.b, pr->rank < 0 ? 0 : c.gathered, c.out, c.g, c.out};
    void *p[9], *ws, *stream;
    size_t bytes;
    for (int i = 0; i < 9; ++i)
        if (!address(a[1 + i], elems[i], c.esz, &p[i])) return none();
    if (!workspace_of(a[10], &ws, &bytes) || !stream_of(a[11], &stream)) return none();
    int st;
    {
        WithoutGil released;
        st = g_fwd(pr, p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7], p[8], ws, bytes, stream);
    }
    return PyLong_FromLong(st);
}

// (prob, dY, X, A_or_Y, Lw, Cw, Dw, G, dg_own, dX, dLw, dCw, dDw, dbias, dG_send, workspace, stream)
PyObject *layer_bwd(PyObject *const *a, Py_ssize_t n)
{
    Released r;
    const ph_problem *pr;
    Counts c;
    if (n != 17 || !(r.held = problem_of(a[0], &pr, &r.view)) || !counts_of(pr, 0, c)) return none();
    const int64_t elems[14] = {c.out, c.in, c.out, c.L, c.C, c.D, c.gathered, c.g, c.in, c.L, c.C, c.D, c.b, c.send};
    void *p[14], *ws, *stream;
    size_t bytes;
    for (int i = 0; i < 14; ++i)
        if (!address(a[1 + i], elems[i], i >= 9 && i <= 12 ? 4 : c.esz, &p[i])) return none();
    if (!workspace_of(a[15], &ws, &bytes) || !stream_of(a[16], &stream)) return none();
    int st;
    {
        WithoutGil released;
        st = g_bwd(pr, p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7], p[8], (float *)p[9], (float *)p[10], (float *)p[11], (float *)p[12],
                   p[13], ws, bytes, stream);
    }
    return PyLong_FromLong(st);
}

// (prob, X0, T, Y_out, loss, lr, mode, static, workspace, stream, and the 14 per-layer sequences
//  Lw Cw Dw bias, their masters, G dg_own, dLw dCw dDw dbias)
PyObject *ffn_step(PyObject *const *a, Py_ssize_t n)
{
    Released r;
    const ph_problem *pr;
    if (n != 24 || !(r.held = problem_of(a[0], &pr, &r.view)) || pr->layers < 1) return none();
    const int L = pr->layers;
    std::vector<void *> ptrs((size_t)L * 14);
    void **arrays[14];
    std::vector<Counts> counts((size_t)L);
    for (int l = 0; l < L; ++l)
        if (!counts_of(pr, l, counts[(size_t)l])) return none();
    for (int i = 0; i < 14; ++i) {
        PyObject *seq = a[10 + i];
        arrays[i] = nullptr;
        if (seq == Py_None) continue;
        if (!PyList_Check(seq) && !PyTuple_Check(seq)) return none();
        if (PySequence_Fast_GET_SIZE(seq) != L) return none();
        arrays[i] = ptrs.data() + (size_t)i * L;
        for (int l = 0; l < L; ++l) {
            const Counts &c = counts[(size_t)l];
            const int64_t elems[14] = {c.L, c.C, c.D, c.b, c.L, c.C, c.D, c.b, pr->rank < 0 ? 0 : c.gathered, pr->rank < 0 ? 0 : c.g,
                                       c.L, c.C, c.D, c.b};
            const bool as_float = (i >= 4 && i <= 7) || i >= 10;
            if (!address(PySequence_Fast_GET_ITEM(seq, l), elems[i], as_float ? 4 : c.esz, &arrays[i][l])) return none();
        }
    }
    ph_step_args args{};
    void *x0, *t, *y, *loss, *ws, *stream;
    size_t bytes;
    const Counts &first = counts.front(), &last = counts.back();
    if (!address(a[1], first.in, first.esz, &x0) || !address(a[2], last.out, last.esz, &t) || !address(a[3], last.out, last.esz, &y) ||
        !address(a[4], 1, 4, &loss) || !workspace_of(a[8], &ws, &bytes) || !stream_of(a[9], &stream))
        return none();
    args.lr = (float)PyFloat_AsDouble(a[5]);
    args.mode = (int32_t)PyLong_AsLong(a[6]);
    const bool own = PyObject_IsTrue(a[7]) == 1;
    if (PyErr_Occurred()) { PyErr_Clear(); return none(); }
    args.X0 = x0; args.T = t; args.Y_out = y; args.loss = (float *)loss;
    args.Lw = arrays[0]; args.Cw = arrays[1]; args.Dw = arrays[2]; args.bias = arrays[3];
    args.Lw_master = (float *const *)arrays[4]; args.Cw_master = (float *const *)arrays[5];
    args.Dw_master = (float *const *)arrays[6]; args.bias_master = (float *const *)arrays[7];
    args.G = (const void *const *)arrays[8]; args.dg_own = (const void *const *)arrays[9];
    args.dLw = (float *const *)arrays[10]; args.dCw = (float *const *)arrays[11];
    args.dDw = (float *const *)arrays[12]; args.dbias = (float *const *)arrays[13];
    int st;
    {
        WithoutGil released;
        st = own ? g_static(pr, &args, stream) : g_step(pr, &args, ws, bytes, stream);
    }
    return PyLong_FromLong(st);
}

// addresses of phantom_layer_fwd, phantom_layer_bwd, phantom_ffn_step, phantom_ffn_step_static
PyObject *bind(PyObject *, PyObject *args)
{
    unsigned long long f, b, s, t;
    if (!PyArg_ParseTuple(args, "KKKK", &f, &b, &s, &t)) return nullptr;
    g_fwd = (FwdFn)(uintptr_t)f; g_bwd = (BwdFn)(uintptr_t)b; g_step = (StepFn)(uintptr_t)s; g_static = (StaticFn)(uintptr_t)t;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    {"layer_fwd", (PyCFunction)(void (*)(void))guarded<layer_fwd>, METH_FASTCALL, nullptr},
    {"layer_bwd", (PyCFunction)(void (*)(void))guarded<layer_bwd>, METH_FASTCALL, nullptr},
    {"ffn_step", (PyCFunction)(void (*)(void))guarded<ffn_step>, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
// (build.py looks for the stamp in the file: it names the sources, the Python and the torch that this module was built for)
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", PHANTOM_MARSHAL_STAMP, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
