// Host path of the Python package in native code: argument checks, allocation of outputs and
// workspace, the call into librmm.so and the autograd node, without a Python frame or a ctypes
// conversion per argument (a forward + backward through RMMLinear took 92 us of host time in Python,
// more than the kernels of a RoBERTa-base attention projection).
//
// Every function takes its arguments by position and returns
//   - its result,
//   - a negative int: the rmm_status_t of the library call, or
//   - NotImplemented: something about the arguments is unusual (wrong type, device, shape, layout);
//     the caller then goes through the checks in binding.py, which say what.
#include <torch/csrc/autograd/function.h>
#include <torch/csrc/autograd/functions/utils.h>
#include <torch/csrc/autograd/python_cpp_function.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/autograd/saved_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <ATen/ATen.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>

#include "../../include/rmm.h"

namespace {

using at::Tensor;
using torch::autograd::Node;
using torch::autograd::SavedVariable;
using torch::autograd::variable_list;
using namespace torch::autograd;  // (for the property and method tables of Python nodes)

int dtype_code(const Tensor &t) {
    return t.scalar_type() == at::kBFloat16 ? RMM_DTYPE_BF16 : t.scalar_type() == at::kFloat ? RMM_DTYPE_F32 : -1;
}

void *current_stream(const Tensor &t) {
    return c10::hip::getCurrentHIPStreamMasqueradingAsCUDA(t.device().index()).stream();
}

// A dense GPU tensor of the given matrix shape (cols < 0: a vector of `rows`), dtype and device.
bool is_matrix(const Tensor &t, int64_t rows, int64_t cols, const Tensor &like) {
    return t.is_cuda() && t.scalar_type() == like.scalar_type() && t.device() == like.device() && t.is_contiguous() &&
           (cols < 0 ? t.dim() == 1 && t.size(0) == rows : t.dim() == 2 && t.size(0) == rows && t.size(1) == cols);
}

Tensor new_matrix(const Tensor &like, int64_t rows, int64_t cols) { return at::empty({rows, cols}, like.options().requires_grad(false)); }

Tensor scratch(const Tensor &like, size_t need) {
    return at::empty({(int64_t)(need > 16 ? need : 16)}, like.options().dtype(at::kByte).requires_grad(false));
}

const void *ptr(const Tensor &t) { return t.defined() ? t.data_ptr() : nullptr; }
void *mut(const Tensor &t) { return t.defined() ? t.data_ptr() : nullptr; }

struct NoGil {
    PyThreadState *state;
    NoGil() : state(PyGILState_Check() ? PyEval_SaveThread() : nullptr) {}
    ~NoGil() {
        if (state != nullptr) PyEval_RestoreThread(state);
    }
};

// ---- the library calls on checked tensors; undefined tensors = absent / to be allocated

int run_forward(const Tensor &X, const Tensor &W, const Tensor &bias, int64_t k, int kind, rmm_rng_state_t st, Tensor &Y,
                Tensor &X_proj, Tensor ws, bool need_xproj) {
    const int64_t n = X.size(0), d_in = X.size(1), d_out = W.size(0);
    const rmm_layer_desc_t desc = {n, d_in, d_out, k, dtype_code(X), kind};
    if (!Y.defined()) Y = new_matrix(X, n, d_out);
    if (!X_proj.defined() && need_xproj) X_proj = new_matrix(X, k, d_in);
    if (!ws.defined() && need_xproj) {
        const size_t need = rmm_workspace_bytes(&desc, RMM_OP_FORWARD);
        if (need > 0) ws = scratch(X, need);
    }
    void *stream = current_stream(X);
    const size_t ws_bytes = ws.defined() ? ws.nbytes() : 0;
    NoGil free_;
    return rmm_forward(&desc, st, ptr(X), ptr(W), ptr(bias), mut(Y), mut(X_proj), mut(ws), ws_bytes, stream);
}

int run_backward(const Tensor &dY, const Tensor &W, const Tensor &X_proj, int kind, rmm_rng_state_t st, bool need_dX,
                 bool need_db, Tensor &dX, Tensor &dW, Tensor &db, Tensor ws, bool accumulate) {
    const int64_t n = dY.size(0), d_out = dY.size(1), k = X_proj.size(0), d_in = X_proj.size(1);
    const rmm_layer_desc_t desc = {n, d_in, d_out, k, dtype_code(dY), kind};
    if (need_dX && !dX.defined()) dX = new_matrix(dY, n, d_in);
    if (!dW.defined()) dW = new_matrix(dY, d_out, d_in);
    if (need_db && !db.defined()) db = at::empty({d_out}, dY.options().requires_grad(false));
    if (!ws.defined()) ws = scratch(dY, rmm_workspace_bytes(&desc, RMM_OP_BACKWARD));
    void *stream = current_stream(dY);
    const size_t ws_bytes = ws.nbytes();
    NoGil free_;
    return (accumulate ? rmm_backward_accumulate : rmm_backward)(&desc, st, ptr(dY), ptr(W), ptr(X_proj), mut(dX), mut(dW),
                                                                mut(db), mut(ws), ws_bytes, stream);
}

// ---- autograd

struct LinearBackward : public Node {
    SavedVariable W_, X_proj_;  // X itself is not kept
    int kind = 0;
    rmm_rng_state_t st{};
    std::vector<int64_t> x_sizes;
    bool has_bias = false;

    std::mutex &mutex_for_python() { return mutex_; }

    std::string name() const override { return "RMMLinearFunctionBackward"; }

    void release_variables() override {
        std::lock_guard<std::mutex> lock(mutex_);
        W_.reset_data();
        X_proj_.reset_data();
    }

    variable_list apply(variable_list &&grads) override {
        std::lock_guard<std::mutex> lock(mutex_);
        variable_list out(has_bias ? 3 : 2);
        if (!grads[0].defined()) return out;
        const Tensor W = W_.unpack(), X_proj = X_proj_.unpack();
        at::NoGradGuard no_grad;
        const Tensor dY = grads[0].reshape({-1, W.size(0)}).contiguous();
        TORCH_CHECK(dY.scalar_type() == W.scalar_type() && dY.is_cuda(), "RMMLinear: the gradient must be a GPU tensor of dtype ",
                    W.scalar_type());
        Tensor dX, dW, db;
        if (task_should_compute_output(0)) dX = at::empty(x_sizes, dY.options());
        const int rc = run_backward(dY, W, X_proj, kind, st, dX.defined(),
                                    has_bias && task_should_compute_output(2), dX, dW, db, Tensor(), false);
        TORCH_CHECK(rc == RMM_OK, "rmm_backward: ", rmm_status_string(rc), " (status ", rc, ")");
        out[0] = dX;
        out[1] = dW;
        if (has_bias) out[2] = db;
        return out;
    }
};

PyObject *saved_tensors(PyObject *self, void *) {
    HANDLE_TH_ERRORS
    auto *node = static_cast<LinearBackward *>(reinterpret_cast<torch::autograd::THPCppFunction *>(self)->cdata.get());
    Tensor W, X_proj;
    {
        std::lock_guard<std::mutex> lock(node->mutex_for_python());
        W = node->W_.unpack(), X_proj = node->X_proj_.unpack();
    }
    PyObject *out = PyTuple_New(2);
    if (out == nullptr) return nullptr;
    PyTuple_SET_ITEM(out, 0, THPVariable_Wrap(W));
    PyTuple_SET_ITEM(out, 1, THPVariable_Wrap(X_proj));
    return out;
    END_HANDLE_TH_ERRORS
}

// ---- Python arguments

struct Unusual {};  // -> NotImplemented

Tensor arg_tensor(PyObject *o, bool optional = false) {
    if (o == Py_None && optional) return Tensor();
    if (!THPVariable_Check(o)) throw Unusual();
    return THPVariable_Unpack(o);
}
int64_t arg_int(PyObject *o) {
    if (!PyLong_CheckExact(o)) throw Unusual();
    const long long v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred() != nullptr) {
        PyErr_Clear();
        throw Unusual();
    }
    return v;
}
uint64_t arg_u64(PyObject *o) {  // modulo 2^64, as ctypes does it
    if (!PyLong_CheckExact(o)) throw Unusual();
    return PyLong_AsUnsignedLongLongMask(o);
}
int arg_kind(PyObject *o) {
    const int64_t v = arg_int(o);
    if (v < INT32_MIN || v > INT32_MAX) throw Unusual();
    return (int)v;
}
bool arg_bool(PyObject *o) {
    if (o == Py_True) return true;
    if (o == Py_False || o == Py_None) return false;
    throw Unusual();
}
void need(bool ok) {
    if (!ok) throw Unusual();
}
void need_scratch(const Tensor &ws, const Tensor &like) { need(!ws.defined() || (ws.is_cuda() && ws.is_contiguous() && ws.device() == like.device())); }
PyObject *wrap(const Tensor &t) {
    if (!t.defined()) Py_RETURN_NONE;
    return THPVariable_Wrap(t);
}
PyObject *unusual() {
    Py_INCREF(Py_NotImplemented);
    return Py_NotImplemented;
}

#define RMM_BEGIN(COUNT)                                                      \
    HANDLE_TH_ERRORS                                                          \
    if (nargs != COUNT) {                                                     \
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");       \
        return nullptr;                                                       \
    }                                                                         \
    try {
#define RMM_END                                                               \
    }                                                                         \
    catch (const Unusual &) {                                                 \
        return unusual();                                                     \
    }                                                                         \
    END_HANDLE_TH_ERRORS

// forward(X, W, bias, k, kind, seed, offset, Y, X_proj, ws, need_xproj) -> (Y, X_proj)
PyObject *py_forward(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
    RMM_BEGIN(11)
    const Tensor X = arg_tensor(a[0]), W = arg_tensor(a[1]), bias = arg_tensor(a[2], true), ws = arg_tensor(a[9], true);
    Tensor Y = arg_tensor(a[7], true), X_proj = arg_tensor(a[8], true);
    const int64_t k = arg_int(a[3]);
    const int kind = arg_kind(a[4]);
    const rmm_rng_state_t st = {arg_u64(a[5]), arg_u64(a[6])};
    const bool need_xproj = arg_bool(a[10]);
    need(X.is_cuda() && X.dim() == 2 && X.is_contiguous() && dtype_code(X) >= 0 && k >= 1 && W.dim() == 2);
    const int64_t n = X.size(0), d_in = X.size(1), d_out = W.size(0);
    need(is_matrix(W, d_out, d_in, X) && (!bias.defined() || is_matrix(bias, d_out, -1, X)) &&
         (!Y.defined() || is_matrix(Y, n, d_out, X)) && (!X_proj.defined() || is_matrix(X_proj, k, d_in, X)));
    need_scratch(ws, X);
    const int rc = run_forward(X, W, bias, k, kind, st, Y, X_proj, ws, need_xproj);
    if (rc != RMM_OK) return PyLong_FromLong(rc);
    PyObject *out = PyTuple_New(2);
    if (out == nullptr) return nullptr;
    PyTuple_SET_ITEM(out, 0, wrap(Y));
    PyTuple_SET_ITEM(out, 1, wrap(X_proj));
    return out;
    RMM_END
}

// backward(dY, W, X_proj, kind, seed, offset, need_dX, need_dbias, dX, dW, dbias, ws, accumulate) -> (dX, dW, dbias)
PyObject *py_backward(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
    RMM_BEGIN(13)
    const Tensor dY = arg_tensor(a[0]), W = arg_tensor(a[1]), X_proj = arg_tensor(a[2]), ws = arg_tensor(a[11], true);
    Tensor dX = arg_tensor(a[8], true), dW = arg_tensor(a[9], true), db = arg_tensor(a[10], true);
    const int kind = arg_kind(a[3]);
    const rmm_rng_state_t st = {arg_u64(a[4]), arg_u64(a[5])};
    const bool need_dX = arg_bool(a[6]), need_db = arg_bool(a[7]), accumulate = arg_bool(a[12]);
    need(dY.is_cuda() && dY.dim() == 2 && dY.is_contiguous() && dtype_code(dY) >= 0 && X_proj.dim() == 2);
    const int64_t n = dY.size(0), d_out = dY.size(1), k = X_proj.size(0), d_in = X_proj.size(1);
    need(is_matrix(W, d_out, d_in, dY) && is_matrix(X_proj, k, d_in, dY) && (!dX.defined() || is_matrix(dX, n, d_in, dY)) &&
         (!dW.defined() || is_matrix(dW, d_out, d_in, dY)) && (!db.defined() || is_matrix(db, d_out, -1, dY)));
    need(!accumulate || (dW.defined() && (db.defined() || !need_db)));
    need_scratch(ws, dY);
    const int rc = run_backward(dY, W, X_proj, kind, st, need_dX, need_db, dX, dW, db, ws, accumulate);
    if (rc != RMM_OK) return PyLong_FromLong(rc);
    PyObject *out = PyTuple_New(3);
    if (out == nullptr) return nullptr;
    PyTuple_SET_ITEM(out, 0, wrap(dX));
    PyTuple_SET_ITEM(out, 1, wrap(dW));
    PyTuple_SET_ITEM(out, 2, wrap(db));
    return out;
    RMM_END
}

// sketch(A, k, kind, seed, offset, out, ws) -> out
PyObject *py_sketch(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
    RMM_BEGIN(7)
    const Tensor A = arg_tensor(a[0]);
    Tensor out = arg_tensor(a[5], true), ws = arg_tensor(a[6], true);
    const int64_t k = arg_int(a[1]);
    const int kind = arg_kind(a[2]);
    const rmm_rng_state_t st = {arg_u64(a[3]), arg_u64(a[4])};
    need(A.is_cuda() && A.dim() == 2 && A.is_contiguous() && dtype_code(A) >= 0 && k >= 1);
    const int64_t n = A.size(0), d = A.size(1);
    need(!out.defined() || is_matrix(out, k, d, A));
    need_scratch(ws, A);
    if (!out.defined()) out = new_matrix(A, k, d);
    if (!ws.defined()) {
        const rmm_layer_desc_t desc = {n, d, d, k, dtype_code(A), kind};
        ws = scratch(A, rmm_workspace_bytes(&desc, RMM_OP_SKETCH));
    }
    void *stream = current_stream(A);
    int rc;
    {
        NoGil free_;
        rc = rmm_sketch(n, d, k, dtype_code(A), kind, st, ptr(A), mut(out), mut(ws), ws.nbytes(), stream);
    }
    return rc != RMM_OK ? PyLong_FromLong(rc) : wrap(out);
    RMM_END
}

// variance_stats(X, dY, k, kind, out, ws) -> out
PyObject *py_variance_stats(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
    RMM_BEGIN(6)
    const Tensor X = arg_tensor(a[0]), dY = arg_tensor(a[1]);
    Tensor out = arg_tensor(a[4], true), ws = arg_tensor(a[5], true);
    const int64_t k = arg_int(a[2]);
    const int kind = arg_kind(a[3]);
    need(X.is_cuda() && X.dim() == 2 && X.is_contiguous() && dtype_code(X) >= 0 && dY.dim() == 2 && k >= 1);
    const int64_t n = X.size(0), d_in = X.size(1), d_out = dY.size(1);
    need(is_matrix(dY, n, d_out, X));
    need(!out.defined() || (out.is_cuda() && out.device() == X.device() && out.scalar_type() == at::kDouble && out.is_contiguous() &&
                            out.dim() == 1 && out.size(0) == 8));
    need_scratch(ws, X);
    const rmm_layer_desc_t desc = {n, d_in, d_out, k, dtype_code(X), kind};
    if (!out.defined()) out = at::empty({8}, X.options().dtype(at::kDouble).requires_grad(false));
    if (!ws.defined()) ws = scratch(X, rmm_workspace_bytes(&desc, RMM_OP_VARIANCE));
    void *stream = current_stream(X);
    int rc;
    {
        NoGil free_;
        rc = rmm_variance_stats(&desc, ptr(X), ptr(dY), (double *)mut(out), mut(ws), ws.nbytes(), stream);
    }
    return rc != RMM_OK ? PyLong_FromLong(rc) : wrap(out);
    RMM_END
}

// The layer calls below make their output without torch operators and hang their own node on it, so whatever
// watches operators or Python autograd functions would see nothing of them: a trace would hold an allocation that
// nobody fills, a forward-mode derivative would be dropped without a word, and a transform's wrapper has no memory.
// Such calls take the Python function, which torch records or refuses as any other.
bool watched(const Tensor &t) {
    return t.defined() && (t._fw_grad(/*level=*/0).defined() || !t.has_storage());
}
void need_unwatched(const Tensor &X, const Tensor &W, const Tensor &bias) {
    need(!torch::jit::tracer::isTracing() && !watched(X) && !watched(W) && !watched(bias) &&
         !c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode));
}

// X as a dense n x d_in matrix
Tensor rows_of(const Tensor &X, const Tensor &W) {
    need(X.is_cuda() && X.dim() >= 1 && dtype_code(X) >= 0 && X.numel() > 0 && W.dim() == 2 && X.size(-1) == W.size(1));
    return X.dim() == 2 && X.is_contiguous() ? X : X.reshape({-1, X.size(-1)}).contiguous();
}
// An uninitialised tensor of X's leading dimensions and `last` columns (only its address goes to the library).
Tensor like_rows(const Tensor &X, int64_t last) {
    c10::SmallVector<int64_t, 4> s(X.sizes().begin(), X.sizes().end());
    s.back() = last;
    return at::empty(s, X.options().requires_grad(false));
}

// linear(X, W, bias, k, kind, seed, offset) -> Y with the autograd history of RMMLinearFunction
PyObject *py_linear(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
    RMM_BEGIN(7)
    const Tensor X = arg_tensor(a[0]), W = arg_tensor(a[1]), bias = arg_tensor(a[2], true);
    const int64_t k = arg_int(a[3]);
    const int kind = arg_kind(a[4]);
    const rmm_rng_state_t st = {arg_u64(a[5]), arg_u64(a[6])};
    need(k >= 1);
    need_unwatched(X, W, bias);
    Tensor Y, X_proj, Wc;
    {
        at::NoGradGuard no_grad;
        const Tensor X2 = rows_of(X, W);
        Wc = W.contiguous();
        need(is_matrix(Wc, W.size(0), W.size(1), X2) && (!bias.defined() || is_matrix(bias, W.size(0), -1, X2)));
        Y = like_rows(X, W.size(0));
        const int rc = run_forward(X2, Wc, bias, k, kind, st, Y, X_proj, Tensor(), true);
        if (rc != RMM_OK) return PyLong_FromLong(rc);
    }
    if (torch::autograd::compute_requires_grad(X, W, bias)) {
        std::shared_ptr<LinearBackward> node(new LinearBackward(), torch::autograd::deleteNode);
        node->set_next_edges(bias.defined() ? torch::autograd::collect_next_edges(X, W, bias)
                                            : torch::autograd::collect_next_edges(X, W));
        node->W_ = SavedVariable(Wc, false);
        node->X_proj_ = SavedVariable(X_proj, false);
        node->kind = kind, node->st = st, node->has_bias = bias.defined();
        node->x_sizes.assign(X.sizes().begin(), X.sizes().end());
        torch::autograd::set_history(Y, node);
    }
    return wrap(Y);
    RMM_END
}

// infer(X, W, bias, kind) -> Y; nothing is kept, no sketch is made
PyObject *py_infer(PyObject *, PyObject *const *a, Py_ssize_t nargs) {
    RMM_BEGIN(4)
    const Tensor X = arg_tensor(a[0]), W = arg_tensor(a[1]), bias = arg_tensor(a[2], true);
    const int kind = arg_kind(a[3]);
    need_unwatched(X, W, bias);
    at::NoGradGuard no_grad;
    const Tensor X2 = rows_of(X, W), Wc = W.contiguous();
    need(is_matrix(Wc, W.size(0), W.size(1), X2) && (!bias.defined() || is_matrix(bias, W.size(0), -1, X2)));
    Tensor Y = like_rows(X, W.size(0)), X_proj;
    const int rc = run_forward(X2, Wc, bias, 1, kind, rmm_rng_state_t{0, 0}, Y, X_proj, Tensor(), false);
    if (rc != RMM_OK) return PyLong_FromLong(rc);
    return wrap(Y);
    RMM_END
}

#define RMM_METHOD(NAME) {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(py_##NAME)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {RMM_METHOD(forward), RMM_METHOD(backward), RMM_METHOD(sketch), RMM_METHOD(variance_stats),
                         RMM_METHOD(linear),  RMM_METHOD(infer),    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_rmm_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

PyTypeObject node_type;
// (torch's own table of these, THP_FUNCTION_DEFAULT_METHODS, names a function that its headers do not declare)
PyMethodDef node_methods[] = {{"_register_hook_dict", THPCppFunction_register_hook_dict, METH_O, nullptr},
                              {"register_hook", THPCppFunction_register_hook, METH_O, nullptr},
                              {"register_prehook", THPCppFunction_register_prehook, METH_O, nullptr},
                              {"name", THPCppFunction_name, METH_NOARGS, nullptr},
                              {"_sequence_nr", THPCppFunction_sequence_nr, METH_NOARGS, nullptr},
                              {nullptr, nullptr, 0, nullptr}};
PyGetSetDef node_properties[] = {THP_FUNCTION_DEFAULT_PROPERTIES,
                                 {(char *)"saved_tensors", saved_tensors, nullptr, nullptr, nullptr},
                                 {nullptr, nullptr, nullptr, nullptr, nullptr}};

}  // namespace

PyMODINIT_FUNC PyInit__rmm_host(void) {
    PyObject *m = PyModule_Create(&module);
    if (m == nullptr) return nullptr;
    torch::autograd::_initFunctionPyTypeObject(node_type, "RMMLinearFunctionBackward", node_properties, node_methods);
    torch::autograd::registerCppFunction(typeid(LinearBackward), &node_type);
    return m;
}
