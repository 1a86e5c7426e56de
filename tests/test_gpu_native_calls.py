"""Calls that go through C++ (results allocated there) against the same calls through ctypes, bit for bit, and what the C++ side
leaves to the Python functions: their errors stay."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def inputs(dtype=torch.bfloat16, B=5, rows=150, H=2, D=64):
    g = torch.Generator().manual_seed(5)
    offsets = torch.tensor([0, 40, 40, 41, 110, rows], dtype=torch.int64).cuda()
    q, k, v = (torch.randn(rows, H, D, generator=g).to(dtype).cuda() for _ in range(3))
    return q, k, v, offsets


def both(monkeypatch, call, answered=True):
    from paper_2409_15373_amd import binding
    assert binding._load_calls(), "the C++ calls are not built"
    answers, ask = [], binding._native
    with monkeypatch.context() as m:
        m.setattr(binding, "_native", lambda *args: answers.append(ask(*args)) or answers[-1])
        native = call(binding)
    assert [a is not None for a in answers] == [True] * answered, "the C++ function did not answer, or was asked where it is not to be"
    with monkeypatch.context() as m:
        m.setattr(binding, "_calls", False)
        python = call(binding)
    native, python = (x if isinstance(x, tuple) else (x,) for x in (native, python))
    assert len(native) == len(python)
    for a, b in zip(native, python):
        assert a.shape == b.shape and a.dtype == b.dtype and a.device == b.device and a.is_contiguous() and a.requires_grad == b.requires_grad
        assert torch.equal(a, b)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_forward(monkeypatch, dtype):
    q, k, v, offsets = inputs(dtype)
    q.requires_grad_()
    both(monkeypatch, lambda b: b.jfa_forward(q, k, v, offsets, 70))
    both(monkeypatch, lambda b: b.jfa_forward(q, k, v, offsets, 70, causal=True))
    both(monkeypatch, lambda b: b.jfa_forward_cross(q, k, v, offsets, offsets, 70, 70))


def test_conversions_and_feature_operators(monkeypatch):
    q, _, _, offsets = inputs()
    both(monkeypatch, lambda b: b.jfa_jagged_to_dense(q, offsets, 72))
    both(monkeypatch, lambda b: b.jfa_jagged_to_dense(q, offsets, 72, pad=-0.0), answered=False)   # not a pattern of zeros
    dense = torch.randn(5, 72, 2, 64, device="cuda").bfloat16()
    both(monkeypatch, lambda b: b.jfa_dense_to_jagged(dense, offsets, torch.zeros_like(q)))
    x, y, w = q[:, 0].contiguous(), q[:, 1, :32].contiguous(), torch.randn(5, 64, 32, device="cuda").bfloat16()
    both(monkeypatch, lambda b: b.jfa_jagged_dense_bmm(x, w, offsets, 70))
    both(monkeypatch, lambda b: b.jfa_jagged_jagged_bmm(x, y, offsets, 70))
    both(monkeypatch, lambda b: b.jfa_jagged_softmax(x, offsets, 70))
    both(monkeypatch, lambda b: b.jfa_jagged_softmax_backward(x, x, offsets, 70))


def test_errors_stay():
    from paper_2409_15373_amd import binding
    q, k, v, offsets = inputs()
    for call, error in [(lambda: binding.jfa_forward(q, k[1:], v, offsets, 70), AssertionError),
                        (lambda: binding.jfa_forward(q.half(), k.half(), v.half(), offsets, 70), TypeError),
                        (lambda: binding.jfa_forward(q.cpu(), k, v, offsets, 70), AssertionError),
                        (lambda: binding.jfa_forward(q.transpose(0, 1), k.transpose(0, 1), v.transpose(0, 1), offsets, 70), AssertionError),
                        (lambda: binding.jfa_forward(q, k, v, offsets.int(), 70), AssertionError),
                        (lambda: binding.jfa_forward(q, k, v, offsets, -1), binding.JfaError),
                        (lambda: binding.jfa_forward(q[..., :16].contiguous(), k[..., :16].contiguous(), v[..., :16].contiguous(), offsets, 70), binding.JfaError),
                        (lambda: binding.jfa_forward_cross(q, k, v, offsets, offsets[1:], 70, 70), AssertionError),
                        (lambda: binding.jfa_jagged_to_dense(q, offsets, -1), RuntimeError),
                        (lambda: binding.jfa_dense_to_jagged(q[None], offsets, q), AssertionError)]:
        with pytest.raises(error):
            call()


def test_a_dispatch_mode_sees_the_allocations():
    from torch.utils._python_dispatch import TorchDispatchMode
    from paper_2409_15373_amd import binding

    class Seen(TorchDispatchMode):
        ops = ()

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            self.ops += (str(func),)
            return func(*args, **(kwargs or {}))

    q, k, v, offsets = inputs()
    with Seen() as seen:
        binding.jfa_forward(q, k, v, offsets, 70)
        assert binding._native("forward", q, k, v, offsets, 70, False) is None
    assert any("empty" in op for op in seen.ops)
    assert binding._native("forward", q, k, v, offsets, 70, False) is not None


def test_a_function_mode_sees_the_allocations():
    from torch.overrides import TorchFunctionMode
    from paper_2409_15373_amd import binding

    class Seen(TorchFunctionMode):
        functions = ()

        def __torch_function__(self, func, types, args=(), kwargs=None):
            self.functions += (func,)
            return func(*args, **(kwargs or {}))

    q, k, v, offsets = inputs()
    x, w = q[:, 0].contiguous(), torch.randn(5, 64, 32, device="cuda").bfloat16()
    for call, allocation in [(lambda: binding.jfa_forward(q, k, v, offsets, 70), torch.empty),
                             (lambda: binding.jfa_forward_cross(q, k, v, offsets, offsets, 70, 70), torch.empty),
                             (lambda: binding.jfa_jagged_to_dense(q, offsets, 70), torch.empty),
                             (lambda: binding.jfa_jagged_dense_bmm(x, w, offsets, 70), torch.empty),
                             (lambda: binding.jfa_jagged_softmax(x, offsets, 70), torch.empty_like)]:
        with Seen() as seen:
            call()
        assert allocation in seen.functions


def test_listeners_have_the_python_function_called(monkeypatch):
    """Function transforms (their own tensors and others inside them), the tracer, fake tensors, both kinds of mode and compilation:
    the C++ call leaves the call to the Python function."""
    from torch._subclasses.fake_tensor import FakeTensorMode
    from torch.overrides import BaseTorchFunctionMode
    from torch.utils._python_dispatch import TorchDispatchMode
    from paper_2409_15373_amd import binding

    class Pass(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    q, _, _, offsets = inputs()
    native, answers = binding._load_calls(), []

    def ask(t):
        answers.append(native.forward(t, t, t, offsets, 70, False))
        answers.append(native.to_dense(t, offsets, 70))
        return t.float().sum()

    ask(q)
    assert all(a is not None for a in answers)
    answers.clear()
    torch.func.vmap(lambda t: (ask(t), ask(q))[0])(q[None])
    torch.func.grad(lambda t: (ask(t), ask(q))[0])(q)
    torch.jit.trace(ask, q, check_trace=False)
    for mode in (FakeTensorMode(allow_non_fake_inputs=True), BaseTorchFunctionMode(), Pass()):
        with mode:
            ask(q)
    assert len(answers) == 2 * 8 and all(a is None for a in answers)
    monkeypatch.setattr(torch.compiler, "is_compiling", lambda: True)
    assert binding._native("forward", q, q, q, offsets, 70, False) is None
