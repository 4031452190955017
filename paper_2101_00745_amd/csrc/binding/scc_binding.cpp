// The plain calls of the Python binding in native code: checks, allocation of the outputs and of the workspace, launch.
//
// One image through a small layer, or a network of small blocks, is bound by the host.  us per call on the host, through ctypes -> here:
// scc_forward 7.7 -> 4.5 (its launch: 3.6), scc_backward 10.5 -> 5.9, scc_dw_backward 21 -> 11; a training step of the 13-block stack at
// batch 128 925 -> 709 (then bound by its kernels), its forward at batch 16 145 -> 114, one 8x8 image forward and backward 18.6 -> 11.6.
// Each function here serves the call that a program makes all day (dense,
// contiguous tensors of the right shapes on the current device, no `out`, no workspace, no modes) and returns None for
// everything else, errors included: scc.py then goes its general way, which raises what there is to raise.  Nothing is kept
// from one call to the next.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>

#include "scc.h"

namespace {

// A dense contiguous tensor on the current device in one of the library's types (and, for the second overload, those of x).
bool plain(const at::Tensor& t)
{
    return t.defined() && t.is_cuda() && t.layout() == at::kStrided && t.has_storage() && t.is_contiguous() &&
           (t.scalar_type() == at::kFloat || t.scalar_type() == at::kBFloat16) &&
           t.get_device() == c10::hip::current_device();
}

bool plain(const at::Tensor& t, const at::Tensor& x) { return plain(t) && t.scalar_type() == x.scalar_type(); }

bool fits(const at::Tensor& t)
{
    for (const int64_t s : t.sizes())
        if (s < 1 || s > INT_MAX) return false;
    return true;
}

// Arguments of a call: `tensors` tensors that are no subclass (Parameter aside), cg, co and, with `strided`, the stage's stride.
struct Args {
    const at::Tensor* t[4];
    int cg, stride;
    double co;
};

bool integer(PyObject* o, int* v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long l = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || l < 1 || l > INT_MAX) return false;
    *v = (int)l;
    return true;
}

bool parse(PyObject* const* a, Py_ssize_t n, int tensors, bool strided, Args* out)
{
    if (n != tensors + 2 + (strided ? 1 : 0)) return false;
    if (c10::impl::TorchDispatchModeTLS::any_modes_set() || at::impl::PythonTorchFunctionTLS::stack_len() > 0) return false;
    for (int i = 0; i < tensors; ++i) {
        if (!THPVariable_CheckExact(a[i])) return false;
        out->t[i] = &THPVariable_Unpack(a[i]);
    }
    out->stride = 1;
    if (!integer(a[tensors], &out->cg) || (strided && !integer(a[tensors + 2], &out->stride))) return false;
    if (!PyFloat_CheckExact(a[tensors + 1])) return false;
    out->co = PyFloat_AS_DOUBLE(a[tensors + 1]);
    return true;
}

// x [N,Cin,H,W] and w [Cout,Cin/cg] as a layer; the map behind a depthwise stage of the given stride is Ho x Wo.
struct Layer {
    int N, Cin, Cout, H, W, Ho, Wo;
    scc_dtype dtype;
};

bool layer(const Args& a, const at::Tensor& x, const at::Tensor& w, Layer* l)
{
    if (!plain(x) || !plain(w, x) || x.dim() != 4 || w.dim() != 2 || !fits(x) || !fits(w)) return false;
    l->N = (int)x.size(0);
    l->Cin = (int)x.size(1);
    l->Cout = (int)w.size(0);
    l->H = (int)x.size(2);
    l->W = (int)x.size(3);
    l->Ho = (l->H - 1) / a.stride + 1;
    l->Wo = (l->W - 1) / a.stride + 1;
    l->dtype = x.scalar_type() == at::kFloat ? SCC_F32 : SCC_BF16;
    return l->Cin % a.cg == 0 && w.size(1) == l->Cin / a.cg;
}

bool taps(const at::Tensor& k, const at::Tensor& x, const Layer& l)
{
    return plain(k, x) && k.dim() == 3 && k.size(0) == l.Cin && k.size(1) == 3 && k.size(2) == 3;
}

bool outputs(const at::Tensor& g, const at::Tensor& x, const Layer& l)
{
    return plain(g, x) && g.dim() == 4 && g.size(0) == l.N && g.size(1) == l.Cout && g.size(2) == l.Ho && g.size(3) == l.Wo;
}

at::Tensor scratch(size_t need, const at::Tensor& x)
{
    return need ? at::empty({(int64_t)need}, x.options().dtype(at::kByte)) : at::Tensor();
}

void* address(const at::Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }

// f(stream) without the interpreter's lock, as a call through ctypes runs
struct Unlocked {
    PyThreadState* save = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(save); }
};

void* stream_of(const at::Tensor& x) { return (void*)c10::hip::getCurrentHIPStream(x.get_device()).stream(); }

template <typename F>
int launch(const at::Tensor& x, F&& f)
{
    void* stream = stream_of(x);
    Unlocked unlocked;
    return f(stream);
}

PyObject* tuple_of(std::initializer_list<at::Tensor> ts)
{
    PyObject* r = PyTuple_New((Py_ssize_t)ts.size());
    Py_ssize_t i = 0;
    if (r)
        for (const at::Tensor& t : ts) PyTuple_SET_ITEM(r, i++, THPVariable_Wrap(t));
    return r;
}

PyObject* forward(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    Args a;
    Layer l;
    if (!parse(args, n, 2, false, &a) || !layer(a, *a.t[0], *a.t[1], &l)) Py_RETURN_NONE;
    const at::Tensor &x = *a.t[0], &w = *a.t[1];
    at::Tensor y = at::empty({l.N, l.Cout, l.H, l.W}, x.options());
    const size_t need = scc_forward_workspace_bytes(l.N, l.Cin, l.Cout, l.H, l.W, a.cg, a.co, l.dtype);
    const at::Tensor ws = scratch(need, x);
    const int rc = launch(x, [&](void* st) {
        return scc_forward_ws(x.data_ptr(), w.data_ptr(), y.data_ptr(), l.N, l.Cin, l.Cout, l.H, l.W, a.cg, a.co, l.dtype,
                              address(ws), need, st);
    });
    if (rc != SCC_OK) Py_RETURN_NONE;
    return THPVariable_Wrap(std::move(y));
    END_HANDLE_TH_ERRORS
}

PyObject* backward(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    Args a;
    Layer l;
    if (!parse(args, n, 3, false, &a) || !layer(a, *a.t[0], *a.t[2], &l)) Py_RETURN_NONE;
    const at::Tensor &x = *a.t[0], &dy = *a.t[1], &w = *a.t[2];
    if (!outputs(dy, x, l)) Py_RETURN_NONE;
    at::Tensor dx = at::empty_like(x), dw = at::empty(w.sizes(), x.options().dtype(at::kFloat));
    const size_t need = scc_backward_workspace_bytes(l.N, l.Cin, l.Cout, l.H, l.W, a.cg, a.co, l.dtype);
    const at::Tensor ws = scratch(need, x);
    const int rc = launch(x, [&](void* st) {
        return scc_backward(x.data_ptr(), dy.data_ptr(), w.data_ptr(), dx.data_ptr(), dw.data_ptr(), l.N, l.Cin, l.Cout, l.H, l.W,
                            a.cg, a.co, l.dtype, address(ws), need, st);
    });
    if (rc != SCC_OK) Py_RETURN_NONE;
    return tuple_of({dx, dw});
    END_HANDLE_TH_ERRORS
}

// y of a block; undefined where the call failed
template <typename F>
at::Tensor block_forward(const at::Tensor& x, const at::Tensor& k, const at::Tensor& w, const Args& a, const Layer& l, F&& run)
{
    at::Tensor y = at::empty({l.N, l.Cout, l.Ho, l.Wo}, x.options());
    const size_t need = scc_dw_forward_workspace_bytes(l.N, l.Cin, l.Cout, l.H, l.W, a.stride, a.cg, a.co, l.dtype);
    const at::Tensor ws = scratch(need, x);
    const int rc = run([&](void* st) {
        return scc_dw_forward_scratch(x.data_ptr(), k.data_ptr(), w.data_ptr(), y.data_ptr(), l.N, l.Cin, l.Cout, l.H, l.W,
                                      a.stride, a.cg, a.co, l.dtype, address(ws), need, st);
    });
    return rc == SCC_OK ? y : at::Tensor();
}

// dx, dkdw, dw of a block; none where the call failed
template <typename F>
std::vector<at::Tensor> block_backward(const at::Tensor& x, const at::Tensor& k, const at::Tensor& w, const at::Tensor& dy,
                                       const Args& a, const Layer& l, scc_dtype grad, F&& run)
{
    const at::TensorOptions of = x.options().dtype(grad == SCC_F32 ? at::kFloat : at::kBFloat16);
    at::Tensor dx = at::empty_like(x), dk = at::empty(k.sizes(), of), dw = at::empty(w.sizes(), of);
    const size_t need = scc_dw_backward_as_workspace_bytes(l.N, l.Cin, l.Cout, l.H, l.W, a.stride, a.cg, a.co, l.dtype, grad);
    const at::Tensor ws = scratch(need, x);
    const int rc = run([&](void* st) {
        return scc_dw_backward_as(x.data_ptr(), k.data_ptr(), w.data_ptr(), dy.data_ptr(), dx.data_ptr(), dk.data_ptr(),
                                  dw.data_ptr(), l.N, l.Cin, l.Cout, l.H, l.W, a.stride, a.cg, a.co, l.dtype, grad, address(ws), need,
                                  st);
    });
    if (rc != SCC_OK) return {};
    return {dx, dk, dw};
}

PyObject* dw_forward(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    Args a;
    Layer l;
    if (!parse(args, n, 3, true, &a) || !layer(a, *a.t[0], *a.t[2], &l)) Py_RETURN_NONE;
    const at::Tensor &x = *a.t[0], &k = *a.t[1], &w = *a.t[2];
    if (!taps(k, x, l)) Py_RETURN_NONE;
    at::Tensor y = block_forward(x, k, w, a, l, [&](auto&& f) { return launch(x, f); });
    if (!y.defined()) Py_RETURN_NONE;
    return THPVariable_Wrap(std::move(y));
    END_HANDLE_TH_ERRORS
}

PyObject* dw_backward(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    Args a;
    Layer l;
    if (n != 8 || !PyBool_Check(args[7]) || !parse(args, 7, 4, true, &a) || !layer(a, *a.t[0], *a.t[2], &l)) Py_RETURN_NONE;
    const at::Tensor &x = *a.t[0], &k = *a.t[1], &w = *a.t[2], &dy = *a.t[3];
    if (!taps(k, x, l) || !outputs(dy, x, l)) Py_RETURN_NONE;
    const std::vector<at::Tensor> g = block_backward(x, k, w, dy, a, l, args[7] == Py_True ? l.dtype : SCC_F32,
                                                     [&](auto&& f) { return launch(x, f); });
    if (g.empty()) Py_RETURN_NONE;
    return tuple_of({g[0], g[1], g[2]});
    END_HANDLE_TH_ERRORS
}

// nn._FirstOrder: gradients under create_graph, which only differentiating them makes an error of
struct FirstOrder : torch::autograd::Function<FirstOrder> {
    static torch::autograd::variable_list forward(torch::autograd::AutogradContext*, const at::Tensor& dx, const at::Tensor& dk,
                                                  const at::Tensor& dw, const at::Tensor&, const at::Tensor&, const at::Tensor&,
                                                  const at::Tensor&)
    {
        return {dx.detach(), dk.detach(), dw.detach()};
    }

    static torch::autograd::variable_list backward(torch::autograd::AutogradContext*, torch::autograd::variable_list)
    {
        TORCH_CHECK(false, "sliding-channel convolution has no second derivative");
    }
};

// A block under autograd: nn.DWSCCFunction for the training step of a plain call, all of whose tensors want gradients.  Through the Python function
// a block costs 40 us of host time more, forward and backward, than its launches take (128 x 128 -> 256 on 32x32, stride 2, bf16, one
// step: 95 us of which the kernels are 62).
struct Block : torch::autograd::Function<Block> {
    struct Refused {};

    // from a call of the interpreter, whose lock is held
    static at::Tensor forward(torch::autograd::AutogradContext* ctx, const at::Tensor& x, const at::Tensor& k, const at::Tensor& w,
                              int64_t cg, double co, int64_t stride)
    {
        const Args a = {{&x, &k, &w, nullptr}, (int)cg, (int)stride, co};
        Layer l;
        at::Tensor y;
        if (layer(a, x, w, &l)) y = block_forward(x, k, w, a, l, [&](auto&& f) { return launch(x, f); });
        if (!y.defined()) throw Refused();
        ctx->save_for_backward({x, k, w});
        ctx->saved_data["cg"] = cg;
        ctx->saved_data["co"] = co;
        ctx->saved_data["stride"] = stride;
        return y;
    }

    // The engine's thread: the interpreter's lock is not held.
    static torch::autograd::variable_list backward(torch::autograd::AutogradContext* ctx, torch::autograd::variable_list grads)
    {
        const torch::autograd::variable_list saved = ctx->get_saved_variables();
        const at::Tensor &x = saved[0], &k = saved[1], &w = saved[2];
        const at::Tensor dy = grads[0].contiguous();
        Args a = {{&x, &k, &w, &dy}, (int)ctx->saved_data["cg"].toInt(), (int)ctx->saved_data["stride"].toInt(),
                  ctx->saved_data["co"].toDouble()};
        Layer l;
        std::vector<at::Tensor> g;
        if (layer(a, x, w, &l) && taps(k, x, l) && outputs(dy, x, l))
            g = block_backward(x, k, w, dy, a, l, l.dtype, [&](auto&& f) { return f(stream_of(x)); });
        if (g.empty()) g = general(a);
        if (at::GradMode::is_enabled()) g = FirstOrder::apply(g[0], g[1], g[2], x, k, w, dy);
        return {g[0], g[1], g[2], at::Tensor(), at::Tensor(), at::Tensor()};
    }

    // what is not plain any more (tensors that saved-tensor hooks brought back, say), and errors: scc._dw_backward
    static std::vector<at::Tensor> general(const Args& a)
    {
        struct Locked {
            PyGILState_STATE s = PyGILState_Ensure();
            ~Locked() { PyGILState_Release(s); }
        } locked;
        std::vector<at::Tensor> g;
        PyObject* m = PyImport_ImportModule("paper_2101_00745_amd.scc");
        PyObject* t[4] = {};
        for (int i = 0; i < 4; ++i) t[i] = THPVariable_Wrap(*a.t[i]);
        PyObject* r = m ? PyObject_CallMethod(m, "_dw_backward", "OOOOidiO", t[0], t[1], t[2], t[3], a.cg, a.co, a.stride, Py_True) : nullptr;
        for (int i = 0; r && i < 3; ++i) g.push_back(THPVariable_Unpack(PyTuple_GetItem(r, i)));
        for (int i = 0; i < 4; ++i) Py_XDECREF(t[i]);
        Py_XDECREF(r);
        Py_XDECREF(m);
        if (!r) {
            python_error e;
            e.persist();
            throw e;
        }
        return g;
    }
};

PyObject* dw_block(PyObject*, PyObject* const* args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    Args a;
    Layer l;
    if (!at::GradMode::is_enabled() || !parse(args, n, 3, true, &a) || !layer(a, *a.t[0], *a.t[2], &l)) Py_RETURN_NONE;
    const at::Tensor &x = *a.t[0], &k = *a.t[1], &w = *a.t[2];
    if (!taps(k, x, l)) Py_RETURN_NONE;
    for (int i = 0; i < 3; ++i)
        if (!a.t[i]->requires_grad() || a.t[i]->is_inference() || a.t[i]->_fw_grad(0).defined()) Py_RETURN_NONE;
    try {
        return THPVariable_Wrap(Block::apply(x, k, w, (int64_t)a.cg, a.co, (int64_t)a.stride));
    } catch (const Block::Refused&) {
        Py_RETURN_NONE;
    }
    END_HANDLE_TH_ERRORS
}

#define METHOD(name, doc) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, doc}
PyMethodDef methods[] = {METHOD(forward, "(x, w, cg, co) -> y or None"), METHOD(backward, "(x, dy, w, cg, co) -> (dx, dw) or None"),
                         METHOD(dw_forward, "(x, kdw, w, cg, co, stride) -> y or None"),
                         METHOD(dw_block, "(x, kdw, w, cg, co, stride) -> y under autograd, or None"),
                         METHOD(dw_backward, "(x, kdw, w, dy, cg, co, stride, stored) -> (dx, dkdw, dw) or None"),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the torch (and interpreter) whose inlined types this code was compiled with; scc.py compares it before the first call
PyMODINIT_FUNC PyInit__binding()
{
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", SCC_BUILT_FOR) < 0) Py_CLEAR(m);
    return m;
}
