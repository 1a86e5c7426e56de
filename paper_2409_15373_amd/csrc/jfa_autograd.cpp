// The differentiable functions of autograd.py as native autograd nodes.
//
// What bounds a training step on a small batch is the host: on 256 samples of 64 rows on average the kernels of a step take
// 44 us, and through torch.autograd.Function the step took 105, since the backward of a Python function is entered on the
// engine's thread with the interpreter's lock to be handed over, and everything around the three launches is Python.  Here
// both directions are C++; the entry points of libjfa.so are called by the addresses that the ctypes binding has loaded.
//
// Only plain calls come here (see autograd.py): anything that the checks below do not find in order is answered with None, and
// the Python function, which raises what is to be raised, takes it.
#include <pybind11/functional.h>
#include <torch/extension.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>

namespace {

using at::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

// C ABI of include/jfa.h
using Forward = int (*)(const void *, const void *, const void *, const int64_t *, int64_t, int64_t, int, int, void *, float *, void *);
using Backward = int (*)(const void *, const void *, const void *, const void *, const void *, const float *, const int64_t *, int64_t, int64_t,
                         int, int, void *, void *, void *, float *, void *);
using ForwardCross = int (*)(const void *, const void *, const void *, const int64_t *, const int64_t *, int64_t, int64_t, int64_t, int, int,
                             void *, float *, void *);
using BackwardCross = int (*)(const void *, const void *, const void *, const void *, const void *, const float *, const int64_t *,
                              const int64_t *, int64_t, int64_t, int64_t, int, int, void *, void *, void *, float *, void *);

using ToDense = int (*)(const void *, const int64_t *, int64_t, int64_t, int64_t, uint32_t, void *, void *);
using ToJagged = int (*)(const void *, const int64_t *, int64_t, int64_t, int64_t, void *, void *);
using Product = int (*)(const void *, const void *, const int64_t *, int64_t, int64_t, int, int, void *, void *);
using Softmax = int (*)(const void *, const int64_t *, int64_t, int64_t, int, void *, void *);
using SoftmaxBackward = int (*)(const void *, const void *, const int64_t *, int64_t, int64_t, int, void *, void *);

struct Library {   // [0]: bf16, [1]: fp32
    Forward forward[2], forward_causal[2];
    Backward backward[2], backward_causal[2];
    ForwardCross forward_cross[2];
    BackwardCross backward_cross[2];
    ToDense to_dense;
    ToJagged to_jagged;
    Product dense_bmm, jagged_bmm;
    Softmax softmax;
    SoftmaxBackward softmax_backward;
    PyObject *check = nullptr;   // binding._check: raises JfaError for a status that is not JFA_OK
    PyObject *pointer = nullptr;   // binding._ptr: raises AssertionError for a tensor that is not contiguous or not on the GPU
};
Library lib;

struct Refused {};   // the call is the Python function's

void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

// In a backward, on the engine's thread: the error that a Python function raises for this argument.
void raise_from(PyObject *function, pybind11::object argument) {
    PyObject *r = PyObject_CallFunctionObjArgs(function, argument.ptr(), nullptr);
    Py_XDECREF(r);
    if (r) throw std::runtime_error("jfa backward failed");
    python_error e;
    e.persist();
    throw std::move(e);
}
void check_backward(int status) {
    if (status == 0) return;
    pybind11::gil_scoped_acquire gil;
    raise_from(lib.check, pybind11::int_(status));
}

bool plain(const Tensor &t) { return t.defined() && t.is_cuda() && t.is_contiguous(); }
bool plain_offsets(const Tensor &t) { return plain(t) && t.dim() == 1 && t.scalar_type() == at::kLong; }
int kind(const Tensor &q) {
    if (q.scalar_type() == at::kBFloat16) return 0;
    if (q.scalar_type() == at::kFloat) return 1;
    throw Refused{};
}
// What the graph gives back for a saved tensor is any tensor that a hook has made of it: it has to be what the kernels take it for.
// (The engine has made dout one of the output's size and type; a hook of the node comes after that.)
void check_on_gpu(const Tensor &t) {
    if (plain(t)) return;
    pybind11::gil_scoped_acquire gil;
    raise_from(lib.pointer, pybind11::cast(t));
}
int check_dout(const Tensor &dout) {
    check_on_gpu(dout);
    TORCH_CHECK(dout.dim() == 3 && (dout.scalar_type() == at::kBFloat16 || dout.scalar_type() == at::kFloat),
                "jagged attention, backward: a gradient of ", dout.sizes(), " ", dout.scalar_type());
    return dout.scalar_type() == at::kFloat;
}
void check_saved(const Tensor &t, at::IntArrayRef sizes, at::ScalarType type, const Tensor &dout) {
    check_on_gpu(t);
    TORCH_CHECK(t.sizes() == sizes && t.scalar_type() == type && t.device() == dout.device(), "jagged attention, backward: a tensor of ", sizes, " ",
                type, " on ", dout.device(), " was saved, ", t.sizes(), " ", t.scalar_type(), " on ", t.device(), " came back");
}
float *floats(const Tensor &t) { return static_cast<float *>(t.data_ptr()); }
const int64_t *longs(const Tensor &t) { return static_cast<const int64_t *>(t.data_ptr()); }
Tensor statistics(const Tensor &q, int64_t planes) { return at::empty({planes, q.size(1), q.size(0)}, q.options().dtype(at::kFloat)); }

struct SelfAttention : torch::autograd::Function<SelfAttention> {
    static Tensor forward(AutogradContext *ctx, const Tensor &q, const Tensor &k, const Tensor &v, const Tensor &offsets, int64_t max_len, bool causal) {
        const int f32 = kind(q);
        const Tensor out = at::empty_like(q), lse = at::empty({q.size(1), q.size(0)}, q.options().dtype(at::kFloat));
        const Forward fn = (causal ? lib.forward_causal : lib.forward)[f32];
        int status;
        {
            pybind11::gil_scoped_release nogil;
            status = fn(q.data_ptr(), k.data_ptr(), v.data_ptr(), longs(offsets), offsets.numel() - 1, max_len, (int)q.size(1), (int)q.size(2),
                        out.data_ptr(), floats(lse), stream());
        }
        if (status != 0) throw Refused{};   // the Python function meets the same error and reports it
        ctx->save_for_backward({q, k, v, out, lse, offsets});
        ctx->saved_data["call"] = std::vector<int64_t>{max_len, causal, offsets.numel()};
        return out;
    }
    static variable_list backward(AutogradContext *ctx, variable_list grads) {
        const variable_list saved = ctx->get_saved_variables();
        const Tensor &q = saved[0], &k = saved[1], &v = saved[2], &out = saved[3], &lse = saved[4], &offsets = saved[5];
        const Tensor dout = grads[0].contiguous();
        const std::vector<int64_t> call = ctx->saved_data["call"].toIntVector();   // max_len, causal, offsets' length
        const int f32 = check_dout(dout);
        for (const Tensor *t : {&q, &k, &v, &out}) check_saved(*t, dout.sizes(), dout.scalar_type(), dout);
        check_saved(lse, {dout.size(1), dout.size(0)}, at::kFloat, dout);
        check_saved(offsets, call[2], at::kLong, dout);
        const Tensor dq = at::empty_like(q), dk = at::empty_like(q), dv = at::empty_like(q), stats = statistics(q, f32 ? 1 : 2);
        const Backward fn = (call[1] ? lib.backward_causal : lib.backward)[f32];
        check_backward(fn(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), dout.data_ptr(), floats(lse), longs(offsets), offsets.numel() - 1,
                          call[0], (int)q.size(1), (int)q.size(2), dq.data_ptr(), dk.data_ptr(), dv.data_ptr(),
                          floats(stats), stream()));
        return {dq, dk, dv, Tensor(), Tensor(), Tensor()};
    }
};

struct CrossAttention : torch::autograd::Function<CrossAttention> {
    static Tensor forward(AutogradContext *ctx, const Tensor &q, const Tensor &k, const Tensor &v, const Tensor &offsets_q, const Tensor &offsets_kv,
                          int64_t max_len_q, int64_t max_len_kv) {
        const int f32 = kind(q);
        const Tensor out = at::empty_like(q), lse = at::empty({q.size(1), q.size(0)}, q.options().dtype(at::kFloat));
        int status;
        {
            pybind11::gil_scoped_release nogil;
            status = lib.forward_cross[f32](q.data_ptr(), k.data_ptr(), v.data_ptr(), longs(offsets_q), longs(offsets_kv), offsets_q.numel() - 1,
                                            max_len_q, max_len_kv, (int)q.size(1), (int)q.size(2), out.data_ptr(), floats(lse), stream());
        }
        if (status != 0) throw Refused{};
        ctx->save_for_backward({q, k, v, out, lse, offsets_q, offsets_kv});
        ctx->saved_data["call"] = std::vector<int64_t>{max_len_q, max_len_kv, offsets_q.numel(), k.size(0)};
        return out;
    }
    static variable_list backward(AutogradContext *ctx, variable_list grads) {
        const variable_list saved = ctx->get_saved_variables();
        const Tensor &q = saved[0], &k = saved[1], &v = saved[2], &out = saved[3], &lse = saved[4], &offsets_q = saved[5], &offsets_kv = saved[6];
        const Tensor dout = grads[0].contiguous();
        const std::vector<int64_t> call = ctx->saved_data["call"].toIntVector();   // max_len_q, max_len_kv, offsets' length, rows of k
        const int f32 = check_dout(dout);
        for (const Tensor *t : {&q, &out}) check_saved(*t, dout.sizes(), dout.scalar_type(), dout);
        for (const Tensor *t : {&k, &v}) check_saved(*t, {call[3], dout.size(1), dout.size(2)}, dout.scalar_type(), dout);
        check_saved(lse, {dout.size(1), dout.size(0)}, at::kFloat, dout);
        for (const Tensor *t : {&offsets_q, &offsets_kv}) check_saved(*t, call[2], at::kLong, dout);
        const Tensor dq = at::empty_like(q), dk = at::empty_like(k), dv = at::empty_like(v), stats = statistics(q, f32 ? 1 : 2);
        check_backward(lib.backward_cross[f32](q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), dout.data_ptr(), floats(lse), longs(offsets_q),
                                               longs(offsets_kv), offsets_q.numel() - 1, call[0], call[1], (int)q.size(1), (int)q.size(2), dq.data_ptr(), dk.data_ptr(),
                                               dv.data_ptr(), floats(stats), stream()));
        return {dq, dk, dv, Tensor(), Tensor(), Tensor(), Tensor()};
    }
};

std::optional<Tensor> self_attention(const Tensor &q, const Tensor &k, const Tensor &v, const Tensor &offsets, int64_t max_len, bool causal) {
    if (!plain(q) || !plain(k) || !plain(v) || !plain_offsets(offsets) || q.dim() != 3 || k.sizes() != q.sizes() || v.sizes() != q.sizes() ||
        k.scalar_type() != q.scalar_type() || v.scalar_type() != q.scalar_type())
        return std::nullopt;
    try {
        return SelfAttention::apply(q, k, v, offsets, max_len, causal);
    } catch (const Refused &) {
        return std::nullopt;
    }
}

std::optional<Tensor> cross_attention(const Tensor &q, const Tensor &k, const Tensor &v, const Tensor &offsets_q, const Tensor &offsets_kv,
                                      int64_t max_len_q, int64_t max_len_kv) {
    if (!plain(q) || !plain(k) || !plain(v) || !plain_offsets(offsets_q) || !plain_offsets(offsets_kv) || q.dim() != 3 || k.dim() != 3 ||
        k.sizes() != v.sizes() || k.size(1) != q.size(1) || k.size(2) != q.size(2) || k.scalar_type() != q.scalar_type() ||
        v.scalar_type() != q.scalar_type() || offsets_q.numel() != offsets_kv.numel())
        return std::nullopt;
    try {
        return CrossAttention::apply(q, k, v, offsets_q, offsets_kv, max_len_q, max_len_kv);
    } catch (const Refused &) {
        return std::nullopt;
    }
}

// ---- the binding's calls without gradients, results allocated here ----
// What bounds a call on a small batch is the host again: the ctypes call and the Python around it took 7.5 us, twice a small batch's
// kernel; from here a call takes 4.4 (four bf16 samples of up to 64 rows; fp32, where the kernel takes longer, 5.4).  The functions take the arguments as the interpreter has them; whatever
// is not exactly what they expect, and whatever goes wrong, is answered with None: the Python function takes the call and raises what there is to raise.
const Tensor *exact_tensor(PyObject *o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const Tensor &t = THPVariable_Unpack(o);
    using c10::DispatchKey;
    // tensors that stand for others (function transforms, fake and functional tensors) have one of these keys
    constexpr c10::DispatchKeySet stands_for_others({DispatchKey::Python, DispatchKey::Functionalize, DispatchKey::FuncTorchBatched,
                                                     DispatchKey::FuncTorchGradWrapper, DispatchKey::BatchedNestedTensor, DispatchKey::Conjugate,
                                                     DispatchKey::Negative, DispatchKey::ZeroTensor});
    return t.key_set().has_any(stands_for_others) || !plain(t) ? nullptr : &t;
}
bool as_int64(PyObject *o, int64_t *x) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    *x = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}
bool nobody_listens() {   // no function mode, dispatch mode, function transform or tracer is to see the allocations
    using c10::DispatchKey;
    constexpr c10::DispatchKeySet modes({DispatchKey::Python, DispatchKey::PythonTLSSnapshot, DispatchKey::FuncTorchDynamicLayerFrontMode,
                                         DispatchKey::FuncTorchVmapMode, DispatchKey::Functionalize});
    return !c10::impl::tls_local_dispatch_key_set().included_.has_any(modes) && !torch::jit::tracer::isTracing() && !at::impl::torch_function_mode_enabled();
}
// (q, k, v, offsets, max_len, causal), or with offsets_kv, max_len_q, max_len_kv for cross attention
template <bool kCross> PyObject *forward_call(PyObject *, PyObject *const *args, Py_ssize_t n_args) {
    HANDLE_TH_ERRORS
    int64_t max_len = 0, max_len_kv = 0;
    const Tensor *q, *k, *v, *offsets, *offsets_kv = nullptr;
    if (n_args != (kCross ? 7 : 6) || !nobody_listens() || !(q = exact_tensor(args[0])) || !(k = exact_tensor(args[1])) || !(v = exact_tensor(args[2])) ||
        !(offsets = exact_tensor(args[3])) || (kCross && !(offsets_kv = exact_tensor(args[4]))) || !as_int64(args[kCross ? 5 : 4], &max_len) ||
        (kCross && !as_int64(args[6], &max_len_kv)) || (!kCross && !PyBool_Check(args[5])))
        Py_RETURN_NONE;
    const at::ScalarType type = q->scalar_type();
    const bool shapes = q->dim() == 3 && k->dim() == 3 && k->sizes() == v->sizes() &&
                        (kCross ? k->size(1) == q->size(1) && k->size(2) == q->size(2) && offsets_kv->numel() == offsets->numel() : k->sizes() == q->sizes());
    if (!shapes || (type != at::kBFloat16 && type != at::kFloat) || k->scalar_type() != type || v->scalar_type() != type || !plain_offsets(*offsets) ||
        (kCross && !plain_offsets(*offsets_kv)))
        Py_RETURN_NONE;
    const int f32 = type == at::kFloat;
    Tensor out, lse;
    int status;
    {
        pybind11::gil_scoped_release nogil;
        out = at::empty(q->sizes(), q->options());
        lse = at::empty({q->size(1), q->size(0)}, q->options().dtype(at::kFloat));
        const int64_t B = offsets->numel() - 1;
        const int H = (int)q->size(1), D = (int)q->size(2);
        if constexpr (kCross)
            status = lib.forward_cross[f32](q->data_ptr(), k->data_ptr(), v->data_ptr(), longs(*offsets), longs(*offsets_kv), B, max_len, max_len_kv, H, D,
                                            out.data_ptr(), floats(lse), stream());
        else
            status = (args[5] == Py_True ? lib.forward_causal : lib.forward)[f32](q->data_ptr(), k->data_ptr(), v->data_ptr(), longs(*offsets), B, max_len, H, D,
                                                                                 out.data_ptr(), floats(lse), stream());
    }
    if (status != 0) Py_RETURN_NONE;
    PyObject *pair = PyTuple_New(2);
    if (!pair) return nullptr;
    PyTuple_SET_ITEM(pair, 0, THPVariable_Wrap(std::move(out)));
    PyTuple_SET_ITEM(pair, 1, THPVariable_Wrap(std::move(lse)));
    return pair;
    END_HANDLE_TH_ERRORS
}
// (values, offsets, max_len): rows past a sample's end become zeros
PyObject *to_dense_call(PyObject *, PyObject *const *args, Py_ssize_t n_args) {
    HANDLE_TH_ERRORS
    int64_t max_len = 0;
    const Tensor *values, *offsets;
    if (n_args != 3 || !nobody_listens() || !(values = exact_tensor(args[0])) || !(offsets = exact_tensor(args[1])) || !as_int64(args[2], &max_len) ||
        max_len < 0 || values->dim() < 1 || !plain_offsets(*offsets) || offsets->numel() < 1)
        Py_RETURN_NONE;
    std::vector<int64_t> sizes{offsets->numel() - 1, max_len};
    int64_t row_bytes = (int64_t)values->element_size();
    for (int64_t d = 1; d < values->dim(); ++d) {
        sizes.push_back(values->size(d));
        row_bytes *= values->size(d);
    }
    Tensor dense;
    int status;
    {
        pybind11::gil_scoped_release nogil;
        dense = at::empty(sizes, values->options());
        status = lib.to_dense(values->data_ptr(), longs(*offsets), sizes[0], max_len, row_bytes, 0, dense.data_ptr(), stream());
    }
    if (status != 0) Py_RETURN_NONE;
    return THPVariable_Wrap(std::move(dense));
    END_HANDLE_TH_ERRORS
}
// (dense, offsets, values): values, filled
PyObject *to_jagged_call(PyObject *, PyObject *const *args, Py_ssize_t n_args) {
    HANDLE_TH_ERRORS
    const Tensor *dense, *offsets, *values;
    if (n_args != 3 || !nobody_listens() || !(dense = exact_tensor(args[0])) || !(offsets = exact_tensor(args[1])) || !(values = exact_tensor(args[2])) ||
        dense->dim() < 2 || values->dim() < 1 || !plain_offsets(*offsets) || offsets->numel() - 1 != dense->size(0))
        Py_RETURN_NONE;
    int64_t row_bytes = (int64_t)dense->element_size(), values_row = (int64_t)values->element_size();
    for (int64_t d = 2; d < dense->dim(); ++d) row_bytes *= dense->size(d);
    for (int64_t d = 1; d < values->dim(); ++d) values_row *= values->size(d);
    if (row_bytes != values_row) Py_RETURN_NONE;
    int status;
    {
        pybind11::gil_scoped_release nogil;
        status = lib.to_jagged(dense->data_ptr(), longs(*offsets), dense->size(0), dense->size(1), row_bytes, values->data_ptr(), stream());
    }
    if (status != 0) Py_RETURN_NONE;
    Py_INCREF(args[2]);
    return args[2];
    END_HANDLE_TH_ERRORS
}
// The feature operators on bf16: (x, w or y, offsets, max_len), the softmax (x, offsets, max_len)
enum class Feature { kDenseBmm, kJaggedBmm, kSoftmax, kSoftmaxBackward };
template <Feature kOp> PyObject *feature_call(PyObject *, PyObject *const *args, Py_ssize_t n_args) {
    HANDLE_TH_ERRORS
    constexpr int kTensors = kOp == Feature::kSoftmax ? 1 : 2;
    int64_t max_len = 0;
    const Tensor *a, *b = nullptr, *offsets;
    if (n_args != kTensors + 2 || !nobody_listens() || !(a = exact_tensor(args[0])) || (kTensors == 2 && !(b = exact_tensor(args[1]))) ||
        !(offsets = exact_tensor(args[kTensors])) || !as_int64(args[kTensors + 1], &max_len) || !plain_offsets(*offsets) || offsets->numel() < 1 ||
        a->dim() != 2 || a->scalar_type() != at::kBFloat16 || (b && b->scalar_type() != at::kBFloat16))
        Py_RETURN_NONE;
    const int64_t B = offsets->numel() - 1, n = a->size(0), D = a->size(1);
    if constexpr (kOp == Feature::kDenseBmm)
        if (b->dim() != 3 || b->size(0) != B || b->size(1) != D) Py_RETURN_NONE;
    if constexpr (kOp == Feature::kJaggedBmm)
        if (b->dim() != 2 || b->size(0) != n) Py_RETURN_NONE;
    if constexpr (kOp == Feature::kSoftmaxBackward)
        if (b->sizes() != a->sizes()) Py_RETURN_NONE;
    if (D > 128 || (b && b->size(-1) > 128)) Py_RETURN_NONE;
    Tensor out;
    int status;
    {
        pybind11::gil_scoped_release nogil;
        if constexpr (kOp == Feature::kDenseBmm || kOp == Feature::kJaggedBmm) {
            const int T = (int)b->size(-1);
            constexpr bool kDense = kOp == Feature::kDenseBmm;
            out = kDense ? at::empty({n, T}, a->options()) : at::empty({B, D, T}, a->options());
            status = (kDense ? lib.dense_bmm : lib.jagged_bmm)(a->data_ptr(), b->data_ptr(), longs(*offsets), B, max_len, (int)D, T, out.data_ptr(), stream());
        } else {
            out = at::empty(a->sizes(), a->options());
            if constexpr (kOp == Feature::kSoftmax)
                status = lib.softmax(a->data_ptr(), longs(*offsets), B, max_len, (int)D, out.data_ptr(), stream());
            else
                status = lib.softmax_backward(a->data_ptr(), b->data_ptr(), longs(*offsets), B, max_len, (int)D, out.data_ptr(), stream());
        }
    }
    if (status != 0) Py_RETURN_NONE;
    return THPVariable_Wrap(std::move(out));
    END_HANDLE_TH_ERRORS
}
#define JFA_CALL(name, function) {name, (PyCFunction)(void (*)())function, METH_FASTCALL, nullptr}
PyMethodDef calls[] = {JFA_CALL("forward", forward_call<false>),
                       JFA_CALL("forward_cross", forward_call<true>),
                       JFA_CALL("to_dense", to_dense_call),
                       JFA_CALL("to_jagged", to_jagged_call),
                       JFA_CALL("dense_bmm", feature_call<Feature::kDenseBmm>),
                       JFA_CALL("jagged_bmm", feature_call<Feature::kJaggedBmm>),
                       JFA_CALL("softmax", feature_call<Feature::kSoftmax>),
                       JFA_CALL("softmax_backward", feature_call<Feature::kSoftmaxBackward>),
                       {nullptr, nullptr, 0, nullptr}};
#undef JFA_CALL

// entry: name of an entry point -> its address
void bind_library(const std::function<int64_t(const std::string &)> &entry, pybind11::object check, pybind11::object pointer) {
    const char *suffix[2] = {"", "_f32"};
    auto at = [&](const char *name, int i) { return (uintptr_t)entry(std::string(name) + suffix[i]); };
    for (int i = 0; i < 2; ++i) {
        lib.forward[i] = reinterpret_cast<Forward>(at("jfa_forward", i));
        lib.forward_causal[i] = reinterpret_cast<Forward>(at("jfa_forward_causal", i));
        lib.backward[i] = reinterpret_cast<Backward>(at("jfa_backward", i));
        lib.backward_causal[i] = reinterpret_cast<Backward>(at("jfa_backward_causal", i));
        lib.forward_cross[i] = reinterpret_cast<ForwardCross>(at("jfa_forward_cross", i));
        lib.backward_cross[i] = reinterpret_cast<BackwardCross>(at("jfa_backward_cross", i));
    }
    auto plain_entry = [&](const char *name) { return (uintptr_t)entry(name); };
    lib.to_dense = reinterpret_cast<ToDense>(plain_entry("jfa_jagged_to_dense"));
    lib.to_jagged = reinterpret_cast<ToJagged>(plain_entry("jfa_dense_to_jagged"));
    lib.dense_bmm = reinterpret_cast<Product>(plain_entry("jfa_jagged_dense_bmm"));
    lib.jagged_bmm = reinterpret_cast<Product>(plain_entry("jfa_jagged_jagged_bmm"));
    lib.softmax = reinterpret_cast<Softmax>(plain_entry("jfa_jagged_softmax"));
    lib.softmax_backward = reinterpret_cast<SoftmaxBackward>(plain_entry("jfa_jagged_softmax_backward"));
    lib.check = check.release().ptr();   // kept for the life of the process
    lib.pointer = pointer.release().ptr();
}

}  // namespace

PYBIND11_MODULE(TORCH_EXTENSION_NAME, m) {
    m.def("bind_library", &bind_library);
    m.def("self_attention", &self_attention);
    m.def("cross_attention", &cross_attention);
    if (PyModule_AddFunctions(m.ptr(), calls) != 0) throw pybind11::error_already_set();
}
