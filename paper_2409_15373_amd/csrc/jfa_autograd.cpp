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

struct Library {   // [0]: bf16, [1]: fp32
    Forward forward[2], forward_causal[2];
    Backward backward[2], backward_causal[2];
    ForwardCross forward_cross[2];
    BackwardCross backward_cross[2];
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
    lib.check = check.release().ptr();   // kept for the life of the process
    lib.pointer = pointer.release().ptr();
}

}  // namespace

PYBIND11_MODULE(TORCH_EXTENSION_NAME, m) {
    m.def("bind_library", &bind_library);
    m.def("self_attention", &self_attention);
    m.def("cross_attention", &cross_attention);
}
