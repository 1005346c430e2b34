// Host side of the calls a program makes every step: checks, output allocation and the C ABI call in
// one native function each.  The same work in Python (nine tensors through is_cuda / is_contiguous / dtype /
// shape / data_ptr, ctypes conversions, the stream query) took 18 us per decode step and 25 us per
// forward on the host, more than the kernels of a small call take on the GPU.
// CPython + libtorch; no kernels in here, and nothing is kept between calls.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>

#include "swimba.h"
#include "unlocked.hpp"

namespace {

using swimba::unlocked;

PyObject *g_mixer_out = nullptr, *g_step_out = nullptr, *g_error = nullptr;   // classes of the Python module

struct Raised {};   // a Python exception is set

[[noreturn]] void raise(PyObject *type, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    PyErr_FormatV(type, fmt, ap);
    va_end(ap);
    throw Raised{};
}

// size tuple as Python prints it: "(2, 3)", "(2,)"
std::string show(c10::IntArrayRef s)
{
    std::string r = "(";
    for (size_t i = 0; i < s.size(); ++i) r += (i ? ", " : "") + std::to_string(s[i]);
    return r + (s.size() == 1 ? ",)" : ")");
}

const at::Tensor &tensor(PyObject *o, const char *name)
{
    if (!THPVariable_Check(o)) raise(PyExc_TypeError, "%s must be a tensor", name);
    return THPVariable_Unpack(o);
}

// the tensor, with as many dimensions as the caller reads sizes from
const at::Tensor &tensor_of_rank(PyObject *o, const char *name, int64_t rank)
{
    const at::Tensor &t = tensor(o, name);
    if (t.dim() != rank) raise(PyExc_ValueError, "%s must have %d dimensions, got %d", name, (int)rank, (int)t.dim());
    return t;
}

int32_t io_code(const at::Tensor &t)
{
    if (t.scalar_type() == at::kFloat) return SWIMBA_F32;
    if (t.scalar_type() == at::kBFloat16) return SWIMBA_BF16;
    raise(PyExc_TypeError, "io tensors must be float32 or bfloat16, got %s", c10::toString(t.scalar_type()));
}

// Device pointer of an argument (NULL for None) that has to be a contiguous GPU tensor of this type and shape.
void *ptr(PyObject *o, const char *name, at::ScalarType dtype, c10::IntArrayRef shape)
{
    if (o == Py_None) return nullptr;
    const at::Tensor &t = tensor(o, name);
    if (!t.is_cuda()) raise(PyExc_ValueError, "%s must be a GPU tensor (this library has no CPU path)", name);
    if (!t.is_contiguous()) raise(PyExc_ValueError, "%s must be contiguous", name);
    if (t.scalar_type() != dtype)
        raise(PyExc_TypeError, "%s must have dtype %s, got %s", name, c10::toString(dtype),
              c10::toString(t.scalar_type()));
    if (t.sizes() != shape)
        raise(PyExc_ValueError, "%s must have shape %s, got %s", name, show(shape).c_str(), show(t.sizes()).c_str());
    return t.data_ptr();
}

int32_t integer(PyObject *o)
{
    const long v = PyLong_AsLong(o);
    if (v == -1 && PyErr_Occurred()) throw Raised{};
    return (int32_t)v;
}

bool truth(PyObject *o)
{
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw Raised{};
    return v != 0;
}

// A new reference to `given`, or to a new tensor where it is None and wanted; its device pointer in *data.
struct Out {
    PyObject *obj = nullptr;
    void *data = nullptr;
    ~Out() { Py_XDECREF(obj); }
    void take(PyObject *given, bool wanted, const char *name, at::ScalarType dtype, c10::IntArrayRef shape,
              at::Device dev)
    {
        if (given != Py_None || !wanted) {
            data = ptr(given, name, dtype, shape);
            obj = Py_NewRef(given);
            return;
        }
        at::TensorBase t = at::detail::empty_cuda(shape, dtype, dev, std::nullopt);
        data = t.data_ptr();
        obj = THPVariable_Wrap(std::move(t));
        if (!obj) throw Raised{};
    }
    PyObject *release() { PyObject *o = obj; obj = nullptr; return o; }
};

void check(swimba_status st, const char *where)
{
    if (st == SWIMBA_OK) return;
    PyObject *e = PyObject_CallFunction(g_error, "is", (int)st, where);
    if (e) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    throw Raised{};
}

// The caller's workspace, or one of `want` bytes for this call.  Sizes that the library refuses (want == 0): those of a
// forward raise their status here, before an output is allocated for them; a decode call refuses them by itself.
struct Workspace {
    at::TensorBase own;
    void *data = nullptr;
    size_t bytes = 0;
    Workspace(PyObject *given, size_t want, at::Device dev, const swimba_dims *forward = nullptr,
              const char *query = nullptr)
    {
        if (given == Py_None) {
            if (want == 0) {
                if (!forward) return;
                swimba_ws_layout lo;
                const swimba_status st = swimba_mixer_workspace_layout(forward, &lo);
                check(st != SWIMBA_OK ? st : SWIMBA_ERR_SHAPE, query);
            }
            own = at::detail::empty_cuda({(int64_t)want}, at::kByte, dev, std::nullopt);
            data = own.data_ptr();
            bytes = want;
            return;
        }
        const at::Tensor &t = tensor(given, "workspace");
        data = ptr(given, "workspace", at::kByte, t.sizes());
        bytes = (size_t)t.numel();
    }
};

at::Device gpu_of(const at::Tensor &t, const char *name)
{
    if (!t.is_cuda()) raise(PyExc_ValueError, "%s must be a GPU tensor (this library has no CPU path)", name);
    return t.device();
}

// asked for while the lock is held: the query can throw
void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

// MixerOut / StepOut: named tuples, made without their Python-level constructor
PyObject *named(PyObject *cls, std::initializer_list<Out *> outs)
{
    PyObject *t = PyTuple_New((Py_ssize_t)outs.size());
    if (!t) throw Raised{};
    Py_ssize_t i = 0;
    for (Out *o : outs) PyTuple_SET_ITEM(t, i++, o->release());
    PyObject *arg = PyTuple_Pack(1, t);
    Py_DECREF(t);
    if (!arg) throw Raised{};
    PyObject *r = PyTuple_Type.tp_new((PyTypeObject *)cls, arg, nullptr);
    Py_DECREF(arg);
    if (!r) throw Raised{};
    return r;
}

swimba_dims dims_of(int64_t B, int64_t L, int64_t H, int64_t P, int64_t N, int64_t G, int64_t E, int32_t k, int32_t Q,
                    int32_t io)
{
    return swimba_dims{(int32_t)B, (int32_t)L, (int32_t)H, (int32_t)P, (int32_t)N, (int32_t)G, (int32_t)E, k, Q, io};
}

// x dt A D B_experts C_experts router_logits top_k chunk h0 y h_final topk_idx topk_w workspace want_h_final want_topk
PyObject *mixer_fwd(PyObject *const *a)
{
    const at::Tensor &x = tensor_of_rank(a[0], "x", 4), &Be = tensor_of_rank(a[4], "B_experts", 5);
    const int64_t B = x.size(0), L = x.size(1), H = x.size(2), P = x.size(3);
    const int64_t E = Be.size(2), G = Be.size(3), N = Be.size(4);
    const int32_t k = integer(a[7]);
    const swimba_dims d = dims_of(B, L, H, P, N, G, E, k, integer(a[8]), io_code(x));
    const at::ScalarType io = x.scalar_type(), f32 = at::kFloat;
    const at::Device dev = gpu_of(x, "x");
    const bool topk = truth(a[16]);
    void *px = ptr(a[0], "x", io, {B, L, H, P}), *pdt = ptr(a[1], "dt", io, {B, L, H});
    void *pA = ptr(a[2], "A", f32, {H}), *pD = ptr(a[3], "D", f32, {H});
    void *pB = ptr(a[4], "B_experts", io, {B, L, E, G, N}), *pC = ptr(a[5], "C_experts", io, {B, L, E, G, N});
    void *pg = ptr(a[6], "router_logits", io, {B, L, E}), *ph = ptr(a[9], "h0", f32, {B, H, P, N});
    const Workspace ws(a[14], a[14] == Py_None ? swimba_mixer_workspace_bytes(&d) : 0, dev, &d,
                       "swimba_mixer_workspace_bytes");
    Out y, hf, idx, w;
    y.take(a[10], true, "y", io, {B, L, H, P}, dev);
    hf.take(a[11], truth(a[15]), "h_final", f32, {B, H, P, N}, dev);
    idx.take(a[12], topk, "topk_idx", at::kInt, {B, L, k}, dev);
    w.take(a[13], topk, "topk_w", f32, {B, L, k}, dev);
    void *const hs = stream();
    check(unlocked([&] {
              return swimba_mixer_fwd(&d, px, pdt, (float *)pA, (float *)pD, pB, pC, pg, (float *)ph, y.data,
                                      (float *)hf.data, (int32_t *)idx.data, (float *)w.data, ws.data, ws.bytes, hs);
          }), "swimba_mixer_fwd");
    return named(g_mixer_out, {&y, &hf, &idx, &w});
}

// u W_g router_logits
PyObject *router_linear(PyObject *const *a)
{
    const at::Tensor &u = tensor(a[0], "u"), &W = tensor_of_rank(a[1], "W_g", 2);
    if (u.dim() < 1) raise(PyExc_ValueError, "u must have at least one dimension");
    const int64_t Dm = u.size(-1), E = W.size(0);
    const at::ScalarType io = u.scalar_type();
    const int32_t code = io_code(u);
    c10::SmallVector<int64_t, 6> shape(u.sizes().begin(), u.sizes().end());
    void *pu = ptr(a[0], "u", io, u.sizes()), *pW = ptr(a[1], "W_g", io, {E, Dm});
    shape.back() = E;
    Out g;
    g.take(a[2], true, "router_logits", io, shape, gpu_of(u, "u"));
    const int64_t tokens = Dm ? u.numel() / Dm : 0;
    void *const hs = stream();
    check(unlocked([&] {
              return swimba_router_linear(tokens, (int32_t)Dm, (int32_t)E, code, pu, pW, g.data, hs);
          }), "swimba_router_linear");
    return g.release();
}

// x dt A D B_sel C_sel topk_w chunk h0 y h_final workspace want_h_final
PyObject *mixer_fwd_selected(PyObject *const *a)
{
    const at::Tensor &x = tensor_of_rank(a[0], "x", 4), &Bs = tensor_of_rank(a[4], "B_sel", 5);
    const int64_t B = x.size(0), L = x.size(1), H = x.size(2), P = x.size(3);
    const int64_t K = Bs.size(2), G = Bs.size(3), N = Bs.size(4);
    const swimba_dims d = dims_of(B, L, H, P, N, G, K, (int32_t)K, integer(a[7]), io_code(x));
    const at::ScalarType io = x.scalar_type(), f32 = at::kFloat;
    const at::Device dev = gpu_of(x, "x");
    void *px = ptr(a[0], "x", io, {B, L, H, P}), *pdt = ptr(a[1], "dt", io, {B, L, H});
    void *pA = ptr(a[2], "A", f32, {H}), *pD = ptr(a[3], "D", f32, {H});
    void *pB = ptr(a[4], "B_sel", io, {B, L, K, G, N}), *pC = ptr(a[5], "C_sel", io, {B, L, K, G, N});
    void *pw = ptr(a[6], "topk_w", f32, {B, L, K}), *ph = ptr(a[8], "h0", f32, {B, H, P, N});
    const Workspace ws(a[11], a[11] == Py_None ? swimba_mixer_workspace_bytes(&d) : 0, dev, &d,
                       "swimba_mixer_workspace_bytes");
    Out y, hf, none1, none2;
    y.take(a[9], true, "y", io, {B, L, H, P}, dev);
    hf.take(a[10], truth(a[12]), "h_final", f32, {B, H, P, N}, dev);
    none1.obj = Py_NewRef(Py_None);
    none2.obj = Py_NewRef(Py_None);
    void *const hs = stream();
    check(unlocked([&] {
              return swimba_mixer_fwd_selected(&d, px, pdt, (float *)pA, (float *)pD, pB, pC, (float *)pw, (float *)ph,
                                               y.data, (float *)hf.data, ws.data, ws.bytes, hs);
          }), "swimba_mixer_fwd_selected");
    return named(g_mixer_out, {&y, &hf, &none1, &none2});
}

// u W_B W_C x dt A D router_logits top_k chunk h0 y h_final workspace want_h_final want_topk
PyObject *mixer_fwd_proj(PyObject *const *a)
{
    const at::Tensor &x = tensor_of_rank(a[3], "x", 4), &WB = tensor_of_rank(a[1], "W_B", 4);
    const int64_t B = x.size(0), L = x.size(1), H = x.size(2), P = x.size(3);
    const int64_t E = WB.size(0), G = WB.size(1), N = WB.size(2), Dm = WB.size(3);
    const int32_t k = integer(a[8]);
    const swimba_dims d = dims_of(B, L, H, P, N, G, E, k, integer(a[9]), io_code(x));
    const at::ScalarType io = x.scalar_type(), f32 = at::kFloat;
    const at::Device dev = gpu_of(x, "x");
    const bool topk = truth(a[15]);
    void *pu = ptr(a[0], "u", io, {B, L, Dm}), *pWB = ptr(a[1], "W_B", io, {E, G, N, Dm});
    void *pWC = ptr(a[2], "W_C", io, {E, G, N, Dm}), *px = ptr(a[3], "x", io, {B, L, H, P});
    void *pdt = ptr(a[4], "dt", io, {B, L, H}), *pA = ptr(a[5], "A", f32, {H}), *pD = ptr(a[6], "D", f32, {H});
    void *pg = ptr(a[7], "router_logits", io, {B, L, E}), *ph = ptr(a[10], "h0", f32, {B, H, P, N});
    const Workspace ws(a[13], a[13] == Py_None ? swimba_mixer_proj_workspace_bytes(&d, (int32_t)Dm) : 0, dev, &d,
                       "swimba_mixer_proj_workspace_bytes");
    Out y, hf, idx, w;
    y.take(a[11], true, "y", io, {B, L, H, P}, dev);
    hf.take(a[12], truth(a[14]), "h_final", f32, {B, H, P, N}, dev);
    idx.take(Py_None, topk, "topk_idx", at::kInt, {B, L, k}, dev);
    w.take(Py_None, topk, "topk_w", f32, {B, L, k}, dev);
    void *const hs = stream();
    check(unlocked([&] {
              return swimba_mixer_fwd_proj(&d, (int32_t)Dm, pu, pWB, pWC, px, pdt, (float *)pA, (float *)pD, pg,
                                           (float *)ph, y.data, (float *)hf.data, (int32_t *)idx.data, (float *)w.data,
                                           ws.data, ws.bytes, hs);
          }), "swimba_mixer_fwd_proj");
    return named(g_mixer_out, {&y, &hf, &idx, &w});
}

// u W_B W_C W_X dt A D router_logits top_k chunk h0 y h_final workspace want_h_final want_topk
PyObject *mixer_fwd_xe_proj(PyObject *const *a)
{
    const at::Tensor &u = tensor_of_rank(a[0], "u", 3), &WB = tensor_of_rank(a[1], "W_B", 4);
    const at::Tensor &WX = tensor_of_rank(a[3], "W_X", 4);
    const int64_t B = u.size(0), L = u.size(1), Dm = u.size(2);
    const int64_t E = WB.size(0), G = WB.size(1), N = WB.size(2), H = WX.size(1), P = WX.size(2);
    const int32_t k = integer(a[8]);
    const swimba_dims d = dims_of(B, L, H, P, N, G, E, k, integer(a[9]), io_code(u));
    const at::ScalarType io = u.scalar_type(), f32 = at::kFloat;
    const at::Device dev = gpu_of(u, "u");
    const bool topk = truth(a[15]);
    void *pu = ptr(a[0], "u", io, {B, L, Dm}), *pWB = ptr(a[1], "W_B", io, {E, G, N, Dm});
    void *pWC = ptr(a[2], "W_C", io, {E, G, N, Dm}), *pWX = ptr(a[3], "W_X", io, {E, H, P, Dm});
    void *pdt = ptr(a[4], "dt", io, {B, L, H}), *pA = ptr(a[5], "A", f32, {H}), *pD = ptr(a[6], "D", f32, {H});
    void *pg = ptr(a[7], "router_logits", io, {B, L, E}), *ph = ptr(a[10], "h0", f32, {B, H, P, N});
    const Workspace ws(a[13], a[13] == Py_None ? swimba_mixer_xe_proj_workspace_bytes(&d, (int32_t)Dm) : 0, dev, &d,
                       "swimba_mixer_xe_proj_workspace_bytes");
    Out y, hf, idx, w;
    y.take(a[11], true, "y", io, {B, L, H, P}, dev);
    hf.take(a[12], truth(a[14]), "h_final", f32, {B, H, P, N}, dev);
    idx.take(Py_None, topk, "topk_idx", at::kInt, {B, L, k}, dev);
    w.take(Py_None, topk, "topk_w", f32, {B, L, k}, dev);
    void *const hs = stream();
    check(unlocked([&] {
              return swimba_mixer_fwd_xe_proj(&d, (int32_t)Dm, pu, pWB, pWC, pWX, pdt, (float *)pA, (float *)pD, pg,
                                              (float *)ph, y.data, (float *)hf.data, (int32_t *)idx.data,
                                              (float *)w.data, ws.data, ws.bytes, hs);
          }), "swimba_mixer_fwd_xe_proj");
    return named(g_mixer_out, {&y, &hf, &idx, &w});
}

// state x dt A D B_experts C_experts router_logits top_k state_out y topk_idx workspace want_topk
// MULTI: x (B,L,H,P) and so on, otherwise one token per sequence without the L axis
template <bool MULTI>
PyObject *step(PyObject *const *a)
{
    const at::Tensor &x = tensor_of_rank(a[1], "x", MULTI ? 4 : 3);
    const at::Tensor &Be = tensor_of_rank(a[5], "B_experts", MULTI ? 5 : 4);
    const int64_t B = x.size(0), L = MULTI ? x.size(1) : 1, H = x.size(-2), P = x.size(-1);
    const int64_t E = Be.size(-3), G = Be.size(-2), N = Be.size(-1);
    const int32_t k = integer(a[8]);
    const swimba_dims d = dims_of(B, L, H, P, N, G, E, k, 0, io_code(x));
    const at::ScalarType io = x.scalar_type(), f32 = at::kFloat;
    const at::Device dev = gpu_of(x, "x");
    using Sizes = c10::SmallVector<int64_t, 6>;
    auto lead = [&](std::initializer_list<int64_t> rest) {   // (B[, L]) + rest
        Sizes s{B};
        if (MULTI) s.push_back(L);
        s.append(rest.begin(), rest.end());
        return s;
    };
    void *ps = ptr(a[0], "state", f32, {B, H, P, N});
    PyObject *so = a[9] == Py_None ? a[0] : a[9];
    void *pso = a[9] == Py_None ? ps : ptr(a[9], "state_out", f32, {B, H, P, N});
    void *px = ptr(a[1], "x", io, lead({H, P})), *pdt = ptr(a[2], "dt", io, lead({H}));
    void *pA = ptr(a[3], "A", f32, {H}), *pD = ptr(a[4], "D", f32, {H});
    void *pB = ptr(a[5], "B_experts", io, lead({E, G, N})), *pC = ptr(a[6], "C_experts", io, lead({E, G, N}));
    void *pg = ptr(a[7], "router_logits", io, lead({E}));
    const Workspace ws(a[12], a[12] != Py_None ? 0 : MULTI ? swimba_step_multi_workspace_bytes(&d)
                                                           : swimba_step_workspace_bytes(&d), dev);
    Out y, idx, state;
    y.take(a[10], true, "y", io, lead({H, P}), dev);
    idx.take(a[11], truth(a[13]), "topk_idx", at::kInt, lead({k}), dev);
    state.obj = Py_NewRef(so);
    void *const hs = stream();
    check(unlocked([&] {
              return (MULTI ? swimba_step_multi : swimba_step)(&d, (float *)ps, (float *)pso, px, pdt, (float *)pA,
                                                               (float *)pD, pB, pC, pg, y.data, (int32_t *)idx.data,
                                                               ws.data, ws.bytes, hs);
          }), MULTI ? "swimba_step_multi" : "swimba_step");
    return named(g_step_out, {&y, &state, &idx});
}

template <PyObject *(*F)(PyObject *const *), Py_ssize_t NARGS>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != NARGS) {
        PyErr_Format(PyExc_TypeError, "%zd arguments expected, got %zd", NARGS, n);
        return nullptr;
    }
    try {
        return F(args);
    } catch (const Raised &) {
    } catch (...) {
        torch::translate_exception_to_python(std::current_exception());   // torch.OutOfMemoryError and its like
    }
    return nullptr;
}

// classes(MixerOut, StepOut, SwimbaError): what the calls return and raise
PyObject *classes(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 3) {
        PyErr_SetString(PyExc_TypeError, "three classes expected");
        return nullptr;
    }
    g_mixer_out = Py_NewRef(args[0]);
    g_step_out = Py_NewRef(args[1]);
    g_error = Py_NewRef(args[2]);
    Py_RETURN_NONE;
}

#define ENTRY(name, f, n) {name, (PyCFunction)(void (*)(void))entry<f, n>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"classes", (PyCFunction)(void (*)(void))classes, METH_FASTCALL, nullptr},
    ENTRY("mixer_fwd", mixer_fwd, 17),
    ENTRY("router_linear", router_linear, 3),
    ENTRY("mixer_fwd_selected", mixer_fwd_selected, 13),
    ENTRY("mixer_fwd_proj", mixer_fwd_proj, 16),
    ENTRY("mixer_fwd_xe_proj", mixer_fwd_xe_proj, 16),
    ENTRY("step", step<false>, 14),
    ENTRY("step_multi", step<true>, 14),
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&module); }
