// pk_torch.cpp -- the tensor calls of binding.py (gemm, conv2d_fwd,
// conv2d_winograd) marshalled natively: torch tensors in, one C-ABI call on the
// current stream, the output tensor out.
//
// Why: a 64 x 64 x 64 product takes the GPU 4 us, the C-ABI call 0.8 us and
// its launch 2.9 us, but marshalled in Python (attribute reads, two ctypes
// calls, the allocations) a call took 12.5 us of host time, and that was the
// rate at which a program could issue small calls; marshalled here it takes
// 4.1 or 5.0 us (one or the other for the life of a process).
//
// Each function answers None whenever a call is anything but the plain case
// (a tensor subclass, an active torch mode, another type, device, layout or
// argument form, a shape that does not match, a C-ABI status that refuses the
// call): binding.py then runs its own checks and the same C-ABI call, so errors
// and unusual forms behave as they always did.  A failed launch is raised here:
// what went before it on the stream must not run twice.  Nothing is kept
// between calls.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>

#include "../../include/pk.h"

namespace {

// the C-ABI of the library binding.py loaded (set once by bind())
decltype(&pk_sgemm_ws) f_sgemm_ws;
decltype(&pk_sgemm_workspace_bytes_for) f_sgemm_workspace_bytes;
decltype(&pk_conv2d_fwd) f_conv2d_fwd;
decltype(&pk_conv2d_workspace_bytes_for) f_conv2d_workspace_bytes;
decltype(&pk_conv2d_out_dims) f_out_dims;
decltype(&pk_conv2d_same_pads) f_same_pads;
decltype(&pk_conv2d_winograd_tile_fwd) f_winograd;
decltype(&pk_conv2d_winograd_tile_workspace_bytes) f_winograd_workspace_bytes;
PyObject *f_check;  // binding._check(status, entry point): raises

// The answer to a status other than PK_OK.
PyObject *refused(int st, const char *entry)
{
    if (st != PK_ERR_LAUNCH) Py_RETURN_NONE;
    return PyObject_CallFunction(f_check, "is", st, entry);
}

// A plain fp32 tensor on a GPU, or NULL.
const at::Tensor *plain(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.scalar_type() == at::kFloat && t.is_cuda() && t.layout() == at::kStrided ? &t : nullptr;
}

bool modes_active()
{
    return at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set();
}

// Leading dimension of a row-major 2-D view whose rows do not overlap, or -1.
int64_t ld_2d(const at::Tensor &t)
{
    if (t.dim() != 2 || (t.size(1) > 1 && t.stride(1) != 1)) return -1;
    if (t.size(0) > 1 && t.stride(0) < t.size(1)) return -1;
    return std::max<int64_t>(std::max(t.stride(0), t.size(1)), 1);
}

bool as_int(PyObject *o, int64_t *v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    *v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return !overflow;
}

bool as_float(PyObject *o, float *v)
{
    if (PyFloat_CheckExact(o)) {
        const double d = PyFloat_AS_DOUBLE(o);
        *v = (float)d;
        return *v != 0.f || d == 0.0;  // a beta that underflows isn't "no beta"
    }
    int64_t i;
    if (!as_int(o, &i) || i < -(1 << 24) || i > (1 << 24)) return false;
    *v = (float)i;
    return true;
}

// A workspace of at least `need` bytes, or the caller's: false when it is not
// a plain tensor.  `own` keeps an allocated one until the call has returned
// (the allocator reuses it in stream order).
bool workspace_for(PyObject *given, size_t need, const at::Tensor &like, at::Tensor *own, void **ptr, size_t *bytes)
{
    *ptr = nullptr;
    *bytes = 0;
    if (given != Py_None) {
        const at::Tensor *w = plain(given);
        if (!w) return false;
        *ptr = w->data_ptr();
        *bytes = (size_t)w->numel() * 4;
    } else if (need) {
        *own = at::empty({(int64_t)((need + 3) / 4)}, like.options());
        *ptr = own->data_ptr();
        *bytes = (size_t)own->numel() * 4;
    }
    return true;
}

void *stream_of(const at::Tensor &t) { return (void *)c10::hip::getCurrentHIPStream(t.device().index()).stream(); }

// gemm(a, b, c, alpha, beta, trans_a, trans_b, workspace)
PyObject *py_gemm(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    HANDLE_TH_ERRORS
    float alpha, beta;
    if (nargs != 8 || !PyBool_Check(args[5]) || !PyBool_Check(args[6]) || !as_float(args[3], &alpha) ||
        !as_float(args[4], &beta) || modes_active())
        Py_RETURN_NONE;
    const at::Tensor *a = plain(args[0]), *b = plain(args[1]);
    if (!a || !b) Py_RETURN_NONE;
    const bool ta = args[5] == Py_True, tb = args[6] == Py_True;
    const int64_t lda = ld_2d(*a), ldb = ld_2d(*b);
    if (lda < 0 || ldb < 0) Py_RETURN_NONE;
    const int64_t M = a->size(ta ? 1 : 0), K = a->size(ta ? 0 : 1), N = b->size(tb ? 0 : 1);
    if (b->size(tb ? 1 : 0) != K) Py_RETURN_NONE;
    at::Tensor c;
    const bool fresh = args[2] == Py_None;
    if (fresh) {
        if (beta != 0.f) Py_RETURN_NONE;
        c = at::empty({M, N}, a->options());
    } else {
        const at::Tensor *p = plain(args[2]);
        if (!p || p->dim() != 2 || p->size(0) != M || p->size(1) != N) Py_RETURN_NONE;
        c = *p;
    }
    const int64_t ldc = ld_2d(c);
    if (ldc < 0) Py_RETURN_NONE;
    const char fa = ta ? 'T' : 'N', fb = tb ? 'T' : 'N';
    const float *pa = (const float *)a->data_ptr(), *pb = (const float *)b->data_ptr();
    at::Tensor own;
    void *ws;
    size_t ws_bytes;
    const size_t need = args[7] == Py_None ? f_sgemm_workspace_bytes(fa, fb, M, N, K, pa, lda, pb, ldb, ldc) : 0;
    if (!workspace_for(args[7], need, *a, &own, &ws, &ws_bytes)) Py_RETURN_NONE;
    float *pc = (float *)c.data_ptr();
    void *stream = stream_of(c);
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = f_sgemm_ws(fa, fb, M, N, K, alpha, pa, lda, pb, ldb, beta, pc, ldc, ws, ws_bytes, stream);
    Py_END_ALLOW_THREADS
    if (st != PK_OK) return refused(st, "pk_sgemm_ws");
    if (fresh) return THPVariable_Wrap(std::move(c));
    Py_INCREF(args[2]);
    return args[2];
    END_HANDLE_TH_ERRORS
}

// The geometry both convolutions share, from x (N, H, W, Cin), w (KH, KW,
// Cin, Cout), a stride and a padding argument; false: not the plain case.
struct Geometry {
    const at::Tensor *x, *w;
    int64_t N, H, W, Cin, KH, KW, Cout, sh, sw, p[4], Ho, Wo;
};

bool geometry(PyObject *x, PyObject *w, PyObject *stride, PyObject *padding, Geometry *g)
{
    g->x = plain(x);
    g->w = plain(w);
    if (!g->x || !g->w || g->x->dim() != 4 || g->w->dim() != 4 || !g->x->is_contiguous() || !g->w->is_contiguous())
        return false;
    g->N = g->x->size(0);
    g->H = g->x->size(1);
    g->W = g->x->size(2);
    g->Cin = g->x->size(3);
    g->KH = g->w->size(0);
    g->KW = g->w->size(1);
    g->Cout = g->w->size(3);
    if (g->w->size(2) != g->Cin) return false;
    if (stride == Py_None) {
        g->sh = g->sw = 1;
    } else if (PyLong_CheckExact(stride)) {
        if (!as_int(stride, &g->sh)) return false;
        g->sw = g->sh;
    } else if (!PyTuple_CheckExact(stride) || PyTuple_GET_SIZE(stride) != 2 ||
               !as_int(PyTuple_GET_ITEM(stride, 0), &g->sh) || !as_int(PyTuple_GET_ITEM(stride, 1), &g->sw)) {
        return false;
    }
    if (PyUnicode_CheckExact(padding)) {
        if (PyUnicode_CompareWithASCIIString(padding, "SAME") == 0) {
            if (f_same_pads(g->H, g->W, g->KH, g->KW, g->sh, g->sw, g->p) != PK_OK) return false;
        } else if (PyUnicode_CompareWithASCIIString(padding, "VALID") == 0) {
            memset(g->p, 0, sizeof(g->p));
        } else {
            return false;
        }
    } else {
        if (!PyTuple_CheckExact(padding) || PyTuple_GET_SIZE(padding) != 4) return false;
        for (int i = 0; i < 4; ++i)
            if (!as_int(PyTuple_GET_ITEM(padding, i), &g->p[i])) return false;
    }
    return f_out_dims(g->H, g->W, g->KH, g->KW, g->sh, g->sw, g->p[0], g->p[1], g->p[2], g->p[3], &g->Ho, &g->Wo) ==
           PK_OK;
}

// The output tensor: the caller's (plain, contiguous, of this shape) or a new one.
bool output_for(PyObject *given, const Geometry &g, at::Tensor *y)
{
    if (given == Py_None) {
        *y = at::empty({g.N, g.Ho, g.Wo, g.Cout}, g.x->options());
        return true;
    }
    const at::Tensor *p = plain(given);
    if (!p || p->dim() != 4 || p->size(0) != g.N || p->size(1) != g.Ho || p->size(2) != g.Wo || p->size(3) != g.Cout ||
        !p->is_contiguous())
        return false;
    *y = *p;
    return true;
}

PyObject *answer(PyObject *given, at::Tensor &&y)
{
    if (given == Py_None) return THPVariable_Wrap(std::move(y));
    Py_INCREF(given);
    return given;
}

// conv2d_fwd(x, w, stride, padding, out, workspace)
PyObject *py_conv2d_fwd(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    HANDLE_TH_ERRORS
    Geometry g;
    at::Tensor y, own;
    if (nargs != 6 || args[2] == Py_None || modes_active() || !geometry(args[0], args[1], args[2], args[3], &g) ||
        !output_for(args[4], g, &y))
        Py_RETURN_NONE;
    const float *px = (const float *)g.x->data_ptr(), *pw = (const float *)g.w->data_ptr();
    const size_t need = args[5] == Py_None
                            ? f_conv2d_workspace_bytes(px, g.N, g.H, g.W, g.Cin, pw, g.KH, g.KW, g.Cout, g.sh, g.sw,
                                                       g.p[0], g.p[1], g.p[2], g.p[3])
                            : 0;
    void *ws;
    size_t ws_bytes;
    if (!workspace_for(args[5], need, *g.x, &own, &ws, &ws_bytes)) Py_RETURN_NONE;
    float *py = (float *)y.data_ptr();
    void *stream = stream_of(y);
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = f_conv2d_fwd(px, g.N, g.H, g.W, g.Cin, pw, g.KH, g.KW, g.Cout, g.sh, g.sw, g.p[0], g.p[1], g.p[2], g.p[3],
                      py, g.Ho, g.Wo, ws, ws_bytes, stream);
    Py_END_ALLOW_THREADS
    if (st != PK_OK) return refused(st, "pk_conv2d_fwd");
    return answer(args[4], std::move(y));
    END_HANDLE_TH_ERRORS
}

// conv2d_winograd(x, w, padding, out, workspace, tile)
PyObject *py_conv2d_winograd(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    HANDLE_TH_ERRORS
    Geometry g;
    at::Tensor y, own;
    int64_t m;
    if (nargs != 6 || !as_int(args[5], &m) || modes_active() ||
        !geometry(args[0], args[1], Py_None, args[2], &g) || !output_for(args[3], g, &y))
        Py_RETURN_NONE;
    size_t need = 0;
    if (args[4] == Py_None) {
        need = f_winograd_workspace_bytes(m, g.N, g.H, g.W, g.Cin, g.Cout, g.p[0], g.p[1], g.p[2], g.p[3]);
        if (need < 4) need = 4;
    }
    void *ws;
    size_t ws_bytes;
    if (!workspace_for(args[4], need, *g.x, &own, &ws, &ws_bytes)) Py_RETURN_NONE;
    const float *px = (const float *)g.x->data_ptr(), *pw = (const float *)g.w->data_ptr();
    float *py = (float *)y.data_ptr();
    void *stream = stream_of(y);
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = f_winograd(px, g.N, g.H, g.W, g.Cin, pw, g.KH, g.KW, g.Cout, 1, 1, g.p[0], g.p[1], g.p[2], g.p[3], py, g.Ho,
                    g.Wo, m, ws, ws_bytes, stream);
    Py_END_ALLOW_THREADS
    if (st != PK_OK) return refused(st, "pk_conv2d_winograd_tile_fwd");
    return answer(args[3], std::move(y));
    END_HANDLE_TH_ERRORS
}

// bind(addresses, check): the eight entry points above, in their order, and the
// function that raises for a status.
PyObject *py_bind(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    if (nargs != 9) {
        PyErr_SetString(PyExc_TypeError, "bind takes the addresses of eight entry points and a function");
        return nullptr;
    }
    void *p[8];
    for (int i = 0; i < 8; ++i) {
        p[i] = PyLong_AsVoidPtr(args[i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null entry point");
            return nullptr;
        }
    }
    f_sgemm_ws = (decltype(f_sgemm_ws))p[0];
    f_sgemm_workspace_bytes = (decltype(f_sgemm_workspace_bytes))p[1];
    f_conv2d_fwd = (decltype(f_conv2d_fwd))p[2];
    f_conv2d_workspace_bytes = (decltype(f_conv2d_workspace_bytes))p[3];
    f_out_dims = (decltype(f_out_dims))p[4];
    f_same_pads = (decltype(f_same_pads))p[5];
    f_winograd = (decltype(f_winograd))p[6];
    f_winograd_workspace_bytes = (decltype(f_winograd_workspace_bytes))p[7];
    Py_INCREF(args[8]);
    Py_XSETREF(f_check, args[8]);
    Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"bind", (PyCFunction)(void (*)(void))py_bind, METH_FASTCALL, nullptr},
    {"gemm", (PyCFunction)(void (*)(void))py_gemm, METH_FASTCALL, nullptr},
    {"conv2d_fwd", (PyCFunction)(void (*)(void))py_conv2d_fwd, METH_FASTCALL, nullptr},
    {"conv2d_winograd", (PyCFunction)(void (*)(void))py_conv2d_winograd, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_pk_torch", "Native marshalling of the tensor calls.", -1, kMethods,
                       nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pk_torch(void)
{
    PyObject *m = PyModule_Create(&kModule);
    // the torch this was built for: binding.py takes no other
    if (m && PyModule_AddStringConstant(m, "torch_version", PK_TORCH_VERSION) < 0) Py_CLEAR(m);
    return m;
}
