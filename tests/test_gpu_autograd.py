"""The autograd wrappers are marshalling only: their outputs and gradients are the entry points' own, bit for bit, and
(on a small case) match the fp64 oracle within the stated gate."""
import numpy as np
import pytest
import torch

from paper_2409_15373_amd.synthetic import make_custom, offsets_from_lengths
from helpers import f64, gate_bf16, to_device

pytestmark = pytest.mark.gpu


def _rand(n, H, D, dtype, gen):
    return torch.randn(n, H, D, device="cuda", generator=gen).to(dtype)


@pytest.mark.parametrize("dtype,causal,L", [(torch.bfloat16, False, [300, 5, 0, 64, 700]), (torch.bfloat16, True, [300, 5, 0, 64, 700]),
                                            (torch.float32, False, [40, 3, 0, 17])])
def test_self_attention_wrapper_equals_the_entry_points(dtype, causal, L):
    from paper_2409_15373_amd import binding
    from paper_2409_15373_amd.autograd import jagged_flash_attention
    H, D = 2, 128 if dtype == torch.bfloat16 else 32
    off = torch.from_numpy(offsets_from_lengths(np.array(L))).cuda()
    n, max_len = int(off[-1]), max(L)
    gen = torch.Generator(device="cuda").manual_seed(1)
    q, k, v, dout = (_rand(n, H, D, dtype, gen) for _ in range(4))
    qa, ka, va = (t.clone().requires_grad_(True) for t in (q, k, v))
    out = jagged_flash_attention(qa, ka, va, off, max_len, causal=causal)
    out.backward(dout)
    r_out, r_lse = binding.jfa_forward(q, k, v, off, max_len, causal=causal)
    r_dq, r_dk, r_dv, _ = binding.jfa_backward(q, k, v, r_out, dout, r_lse, off, max_len, causal=causal)
    torch.cuda.synchronize()
    for name, a, b in (("out", out, r_out), ("dq", qa.grad, r_dq), ("dk", ka.grad, r_dk), ("dv", va.grad, r_dv)):
        assert torch.equal(a.detach().view(torch.int16 if dtype == torch.bfloat16 else torch.int32),
                           b.view(torch.int16 if dtype == torch.bfloat16 else torch.int32)), name


@pytest.mark.parametrize("max_q", [32, 200])
def test_cross_attention_wrapper_equals_the_entry_points(max_q):
    from paper_2409_15373_amd import binding
    from paper_2409_15373_amd.autograd import jagged_flash_cross_attention
    rng = np.random.default_rng(2)
    B, H, D = 12, 2, 128
    Lq, Lk = rng.integers(0, max_q + 1, B), rng.integers(0, 600, B)
    oq, ok = (torch.from_numpy(offsets_from_lengths(x)).cuda() for x in (Lq, Lk))
    nq, nk = int(oq[-1]), int(ok[-1])
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, dout = _rand(nq, H, D, torch.bfloat16, gen), _rand(nq, H, D, torch.bfloat16, gen)
    k, v = _rand(nk, H, D, torch.bfloat16, gen), _rand(nk, H, D, torch.bfloat16, gen)
    qa, ka, va = (t.clone().requires_grad_(True) for t in (q, k, v))
    out = jagged_flash_cross_attention(qa, ka, va, oq, ok, max_q, 599)
    out.backward(dout)
    r_out, r_lse = binding.jfa_forward_cross(q, k, v, oq, ok, max_q, 599)
    r_dq, r_dk, r_dv, _ = binding.jfa_backward_cross(q, k, v, r_out, dout, r_lse, oq, ok, max_q, 599)
    torch.cuda.synchronize()
    for name, a, b in (("out", out, r_out), ("dq", qa.grad, r_dq), ("dk", ka.grad, r_dk), ("dv", va.grad, r_dv)):
        assert torch.equal(a.detach().view(torch.int16), b.view(torch.int16)), name


def test_gradients_through_the_wrapper_match_the_oracle():
    """A scalar loss sum(out * w) differentiated by torch through the wrapper against the oracle's gradients for dout = w."""
    import oracle
    from paper_2409_15373_amd.autograd import jagged_flash_attention
    w = make_custom("autograd", [70, 1, 33, 130, 300], H=2, D=128, dtype="bf16", seed=11, dout=True)
    d = to_device(w)
    qa, ka, va = (d[n].clone().requires_grad_(True) for n in ("q", "k", "v"))
    out = jagged_flash_attention(qa, ka, va, d["offsets"], w.max_len)
    (out.float() * d["dout"].float()).sum().backward()
    torch.cuda.synchronize()
    r_out, _ = oracle.forward(w.q, w.k, w.v, w.offsets)
    r_dq, r_dk, r_dv, _ = oracle.backward(w.q, w.k, w.v, w.dout, w.offsets)
    gate_bf16("out", f64(out), r_out)
    gate_bf16("dq", f64(qa.grad), r_dq)
    gate_bf16("dk", f64(ka.grad), r_dk)
    gate_bf16("dv", f64(va.grad), r_dv)


def _call(mode, dtype, node):
    """Loss-free step of one attention with a strided dout: outputs, gradients and what the graph saved."""
    from paper_2409_15373_amd import autograd
    H, D = 2, 64
    lq, lk = [70, 1, 0, 130, 33], [40, 5, 64, 0, 129]
    oq, ok = (torch.from_numpy(offsets_from_lengths(np.array(x))).cuda() for x in (lq, lk))
    gen = torch.Generator(device="cuda").manual_seed(3)
    q = _rand(sum(lq), H, D, dtype, gen).requires_grad_(True)
    k, v = (_rand(sum(lk if mode == "cross" else lq), H, D, dtype, gen).requires_grad_(True) for _ in range(2))
    dout = _rand(sum(lq), D, H, dtype, gen).transpose(1, 2)
    args = (q, k, v, oq, ok, 200, 200) if mode == "cross" else (q, k, v, oq, 200, mode == "causal")
    wrapper, function = ((autograd.jagged_flash_cross_attention, autograd._CrossAttention) if mode == "cross"
                         else (autograd.jagged_flash_attention, autograd._SelfAttention))
    packed = []
    with torch.autograd.graph.saved_tensors_hooks(lambda t: packed.append(tuple(t.shape)) or t, lambda t: t):
        out = wrapper(*args) if node == "native" else function.apply(*args)
    return (out.detach(),) + torch.autograd.grad(out, (q, k, v), dout), packed


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("mode", ["self", "causal", "cross"])
def test_native_nodes_equal_the_python_functions(mode, dtype):
    from paper_2409_15373_amd import autograd
    (got, saved), (ref, ref_saved) = _call(mode, dtype, "native"), _call(mode, dtype, "python")
    assert autograd._native
    assert all(torch.equal(a, b) for a, b in zip(got, ref)) and sorted(saved) == sorted(ref_saved)


def test_what_the_native_nodes_refuse_is_refused_as_before():
    from paper_2409_15373_amd.autograd import jagged_flash_attention as attention, jagged_flash_cross_attention as cross
    from paper_2409_15373_amd.binding import JfaError
    off = torch.tensor([0, 8], device="cuda")
    x = torch.randn(8, 2, 64, device="cuda", dtype=torch.bfloat16, requires_grad=True)
    with pytest.raises(AssertionError):
        attention(x.transpose(0, 1).contiguous().transpose(0, 1), x, x, off, 8)
    with pytest.raises(AssertionError):
        attention(x, x, x, off.int(), 8)
    with pytest.raises(AssertionError):
        attention(x, x[:4], x, off, 8)
    with pytest.raises(AssertionError):
        attention(x.cpu(), x, x, off, 8)
    with pytest.raises(TypeError):
        attention(*(x.half(),) * 3, off, 8)
    with pytest.raises(JfaError):
        attention(*(x[:, :, :48].contiguous(),) * 3, off, 8)
    with pytest.raises(JfaError):
        cross(x, x, x, off, off, -1, 8)
    with pytest.raises(RuntimeError):
        torch.func.grad(lambda t: attention(t, t, t, off, 8).float().sum())(x.detach())
    with torch.autograd.forward_ad.dual_level(), pytest.raises(NotImplementedError):   # a Python function's; the C++ one's is a RuntimeError
        attention(torch.autograd.forward_ad.make_dual(x.detach(), x.detach()), x, x, off, 8)
    out = attention(x, x, x, off, 8)
    with torch.no_grad():
        x.mul_(2)
    with pytest.raises(RuntimeError):   # a saved tensor has changed
        out.sum().backward()


class _Raised(Exception):
    pass


def _raise(t):
    raise _Raised("from a hook")


def _step(mode):
    """(wrapper call, inputs) of a small attention that goes through the native nodes."""
    from paper_2409_15373_amd import autograd
    off = torch.tensor([0, 8, 20], device="cuda")
    q, k, v = (torch.randn(20, 2, 64, device="cuda", requires_grad=True) for _ in range(3))
    if mode == "cross":
        return (lambda: autograd.jagged_flash_cross_attention(q, k, v, off, off, 12, 12)), (q, k, v)
    return (lambda: autograd.jagged_flash_attention(q, k, v, off, 12)), (q, k, v)


@pytest.mark.parametrize("mode", ["self", "cross"])
def test_hooks_on_saved_tensors(mode):
    """What a hook gives back is checked before a kernel reads it: the Python function's error for a tensor that is not on the GPU or not
    contiguous, an error for one of another size or type.  What a hook raises reaches the caller (a recomputation by
    torch.utils.checkpoint is stopped that way)."""
    from torch.utils.checkpoint import checkpoint
    call, inputs = _step(mode)

    def step_with(unpack, pack=lambda t: t):
        with torch.autograd.graph.saved_tensors_hooks(pack, unpack):
            out = call()
        return torch.autograd.grad(out.square().sum(), inputs)
    expected = torch.autograd.grad(call().square().sum(), inputs)
    assert all(torch.equal(a, b) for a, b in zip(step_with(lambda t: t.cuda(), lambda t: t.cpu()), expected))
    got = torch.autograd.grad(checkpoint(lambda *_: call(), *inputs, use_reentrant=False).square().sum(), inputs)
    assert all(torch.equal(a, b) for a, b in zip(got, expected))
    floats = lambda f: lambda t: f(t) if t.dim() == 3 else t
    for unpack in (lambda t: t.cpu(), floats(lambda t: t.cpu()), lambda t: t.cpu() if t.dim() == 1 else t,
                   floats(lambda t: t.transpose(0, 1).contiguous().transpose(0, 1))):
        with pytest.raises(AssertionError):
            step_with(unpack)
    for unpack in (floats(lambda t: t[:8]), floats(lambda t: t.bfloat16()), floats(lambda t: t.half()), lambda t: t.int() if t.dim() == 1 else t,
                   lambda t: t[:2] if t.dim() == 1 else t, lambda t: t[:, :4].contiguous() if t.dim() == 2 else t):
        with pytest.raises(RuntimeError, match="was saved"):
            step_with(unpack)
    with pytest.raises(_Raised):
        step_with(_raise)
    with pytest.raises(_Raised):
        step_with(lambda t: t, _raise)


@pytest.mark.parametrize("mode", ["self", "cross"])
def test_native_nodes_on_a_stream_of_their_own(mode):
    """Both directions run on the stream that is current in the forward: behind a long wait on it, on inputs and a dout that are only
    written after that wait."""
    call, inputs = _step(mode)
    expected = torch.autograd.grad(call().square().sum(), inputs)
    values = [x.detach().clone() for x in inputs]
    stream = torch.cuda.Stream()
    with torch.no_grad():
        for x in inputs:
            x.fill_(float("nan"))
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        torch.cuda._sleep(50_000_000)
        with torch.no_grad():
            for x, y in zip(inputs, values):
                x.copy_(y)
        out = call()
        dout = torch.full_like(out, float("nan"))
        torch.cuda._sleep(50_000_000)
        dout.copy_(2 * out.detach())
        got = torch.autograd.grad(out, inputs, dout)
    stream.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, expected))
