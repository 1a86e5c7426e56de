"""Table 1's jagged feature operators on the GPU vs oracle/feature_ops.py on the same seeded bf16 inputs.

Outputs are bf16 roundings of fp32 accumulations of bf16 products: the gate is the bf16 gate of the attention
tests, max |gpu - oracle| <= 1e-2 * max |oracle| (and 2e-2 absolute, scaled up with the output's magnitude where
sums over hundreds of rows exceed 1).  Guard rows after sum_B must stay untouched.
"""
import numpy as np
import pytest
import torch

from oracle import feature_ops as fo
from paper_2409_15373_amd.synthetic import offsets_from_lengths, round_to_bf16_bits, bf16_bits_to_f32, lengths_for
from helpers import f64, gate_bf16

pytestmark = pytest.mark.gpu

LENGTHS = [300, 1, 0, 129, 128, 127, 64, 33, 257, 2, 65, 0]
GUARD = 2


def bf16_pair(rng, shape, sigma=1.0):
    """(float32 array holding exact bf16 values, the same as a CUDA bf16 tensor)."""
    bits = round_to_bf16_bits((rng.standard_normal(shape) * sigma).astype(np.float32))
    return bf16_bits_to_f32(bits), torch.from_numpy(bits.view(np.int16)).view(torch.bfloat16).cuda()


def guarded(t, value=777.0):
    """t with GUARD extra rows of `value` appended; returns (whole buffer, view of the first rows)."""
    buf = torch.cat([t, torch.full((GUARD,) + tuple(t.shape[1:]), value, dtype=t.dtype, device=t.device)])
    return buf, buf[:t.shape[0]]


def scaled_gate(name, got, ref):
    gate_bf16(name, got, ref, abs_tol=2e-2 * max(1.0, float(np.abs(ref).max())))


@pytest.mark.parametrize("D,T", [(64, 64), (128, 128), (32, 128), (128, 32), (64, 32), (32, 32)])
def test_bmm_pair_matches_the_oracle(D, T):
    from paper_2409_15373_amd import binding
    rng = np.random.default_rng(D * 7 + T)
    off = offsets_from_lengths(np.array(LENGTHS)); n = int(off[-1]); B = len(LENGTHS)
    offd = torch.from_numpy(off).cuda()
    x, xd = bf16_pair(rng, (n, D)); y, yd = bf16_pair(rng, (n, T)); w, wd = bf16_pair(rng, (B, D, T), 0.5)
    xbuf, _ = guarded(xd, float("nan")); ybuf, _ = guarded(yd, float("nan"))
    obuf = torch.full((n + GUARD, T), 777.0, dtype=torch.bfloat16, device="cuda")
    binding.jfa_jagged_dense_bmm(xbuf, wd, offd, 512, out=obuf)
    torch.cuda.synchronize()
    assert (obuf[n:] == 777.0).all(), "guard rows of out were written"
    scaled_gate("jagged_dense_bmm", f64(obuf[:n]), fo.jagged_dense_bmm(x, w, off))
    got = binding.jfa_jagged_jagged_bmm(xbuf, ybuf, offd, 512)
    torch.cuda.synchronize()
    ref = fo.jagged_jagged_bmm(x, y, off)
    scaled_gate("jagged_jagged_bmm", f64(got), ref)
    assert (f64(got)[[2, 11]] == 0).all(), "empty samples give zero blocks"


@pytest.mark.parametrize("D", [32, 64, 128])
def test_softmax_and_backward_match_the_oracle(D):
    from paper_2409_15373_amd import binding
    rng = np.random.default_rng(D)
    off = offsets_from_lengths(np.array(LENGTHS)); n = int(off[-1])
    offd = torch.from_numpy(off).cuda()
    x, xd = bf16_pair(rng, (n, D), 2.0)
    xbuf, _ = guarded(xd, float("nan"))
    ybuf = torch.full((n + GUARD, D), 777.0, dtype=torch.bfloat16, device="cuda")
    binding.jfa_jagged_softmax(xbuf, offd, 512, y=ybuf)
    torch.cuda.synchronize()
    assert (ybuf[n:] == 777.0).all()
    y_ref = fo.jagged_softmax(x, off)
    gate_bf16("jagged_softmax", f64(ybuf[:n]), y_ref)
    # backward on the probabilities the GPU really produced (bf16) and a bf16 dy
    dy, dyd = bf16_pair(rng, (n, D))
    dybuf, _ = guarded(dyd, float("nan"))
    dxbuf = torch.full((n + GUARD, D), 555.0, dtype=torch.bfloat16, device="cuda")
    ybuf[n:] = float("nan")
    binding.jfa_jagged_softmax_backward(ybuf, dybuf, offd, 512, dx=dxbuf)
    torch.cuda.synchronize()
    assert (dxbuf[n:] == 555.0).all()
    gate_bf16("jagged_softmax_backward", f64(dxbuf[:n]), fo.jagged_softmax_backward(f64(ybuf[:n]), dy, off))


def test_softmax_large_values_and_long_sample():
    """Columns with values around +-80 (exp overflows without the running maximum) and one sample of 5000 rows."""
    from paper_2409_15373_amd import binding
    rng = np.random.default_rng(3)
    off = offsets_from_lengths(np.array([5000, 3, 40])); n = int(off[-1])
    x, xd = bf16_pair(rng, (n, 64), 30.0)
    y = binding.jfa_jagged_softmax(xd, torch.from_numpy(off).cuda(), 5000)
    torch.cuda.synchronize()
    assert np.isfinite(f64(y)).all()
    gate_bf16("jagged_softmax", f64(y), fo.jagged_softmax(x, off))


def test_feature_ops_on_a_table_sized_workload():
    """B = 1024 samples with lengths uniform on [1, 200], D = T = 64: every sample of jagged_jagged_bmm and sampled
    rows of the others against the oracle."""
    from paper_2409_15373_amd import binding
    rng = np.random.default_rng(11)
    L = lengths_for("uniform", 1024, 200, np.random.Generator(np.random.PCG64(5)))
    off = offsets_from_lengths(L); n = int(off[-1]); offd = torch.from_numpy(off).cuda()
    x, xd = bf16_pair(rng, (n, 64)); y, yd = bf16_pair(rng, (n, 64)); w, wd = bf16_pair(rng, (1024, 64, 64), 0.5)
    scaled_gate("jagged_dense_bmm", f64(binding.jfa_jagged_dense_bmm(xd, wd, offd, 200)), fo.jagged_dense_bmm(x, w, off))
    scaled_gate("jagged_jagged_bmm", f64(binding.jfa_jagged_jagged_bmm(xd, yd, offd, 200)), fo.jagged_jagged_bmm(x, y, off))
    gate_bf16("jagged_softmax", f64(binding.jfa_jagged_softmax(xd, offd, 200)), fo.jagged_softmax(x, off))


class Operators:
    """The four operators on one batch: every call writes into buffers that hold NaN before it, so that a row or block that is
    never written shows, whatever memory the allocator hands out."""

    def __init__(self, B, D, T, seed):
        rng = np.random.default_rng(seed)
        off = offsets_from_lengths(rng.integers(0, 40, size=B))
        if off[-1] == 0:
            off[-1] = 1
        self.B, n = B, int(off[-1])
        (x, self.x), (y, self.y), (w, self.w) = bf16_pair(rng, (n, D)), bf16_pair(rng, (n, T)), bf16_pair(rng, (B, D, T), 0.5)
        self.off = torch.from_numpy(off).cuda()
        self.shapes = [(n, D), (n, T), (B, D, T), (n, D)]
        self.ref = [fo.jagged_softmax(x, off), fo.jagged_dense_bmm(x, w, off), fo.jagged_jagged_bmm(x, y, off), fo.jagged_softmax_backward(x, x, off)]
        self.first = None

    def buffers(self):
        return [torch.full(shape, float("nan"), dtype=torch.bfloat16, device="cuda") for shape in self.shapes]

    def run(self, out):
        from paper_2409_15373_amd import binding
        binding.jfa_jagged_softmax(self.x, self.off, 64, y=out[0])
        binding.jfa_jagged_dense_bmm(self.x, self.w, self.off, 64, out=out[1])
        binding.jfa_jagged_jagged_bmm(self.x, self.y, self.off, 64, out=out[2])
        binding.jfa_jagged_softmax_backward(self.x, self.x, self.off, 64, dx=out[3])
        return out

    def check(self, out):
        """The first results against the oracle, all samples; later ones against them bit for bit."""
        if self.first is None:
            for name, got, ref in zip(("softmax", "dense_bmm", "jagged_bmm", "softmax_backward"), out, self.ref):
                scaled_gate(name, f64(got), ref)
            self.first = [t.clone() for t in out]
        return all(torch.equal(a, b) for a, b in zip(out, self.first))


# one workgroup, fewer samples than workgroups, more (claims decide who does what); D = T = 32: samples are claimed in pairs
@pytest.mark.parametrize("B,D,T", [(1, 32, 64), (37, 32, 64), (6001, 32, 64), (6001, 32, 32), (12000, 32, 32), (9001, 128, 128)])
def test_operators_follow_each_other_on_one_work_counter(B, D, T):
    """The operators share a work counter: back to back, behind other calls that use the same work table, after the table has
    grown, and replayed from a graph, every result equals the first one bit for bit and that one the oracle."""
    from paper_2409_15373_amd import binding
    ops = Operators(B, D, T, 58)
    big = torch.arange(20001, dtype=torch.int64, device="cuda")   # a larger batch: a new work table
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        for _ in range(2):
            assert ops.check(ops.run(ops.buffers()))
        binding.jfa_build_schedule(big, 128)
        for _ in range(2):
            assert ops.check(ops.run(ops.buffers()))
        graph, out = torch.cuda.CUDAGraph(), ops.buffers()
        s.synchronize()
        with torch.cuda.graph(graph, stream=s):
            ops.run(out)
    for _ in range(3):
        for t in out:
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert ops.check(out)
        with torch.cuda.stream(s):
            assert ops.check(ops.run(ops.buffers()))
        torch.cuda.synchronize()


@pytest.mark.parametrize("B", [37, 9001])
def test_a_work_table_that_is_new_under_capture(B):
    """A stream's first call under a relaxed capture allocates the work table and enqueues nothing that runs: operators on that
    stream before the first replay, and a replay of a second graph, must not depend on what the table's memory held."""
    import ctypes
    from paper_2409_15373_amd import binding
    ops = Operators(B, 64, 64, 60)
    hip = binding.load()   # the HIP runtime the library is linked with
    size = ctypes.c_size_t(binding.jfa_workspace_bytes(B, 64, 1, 64))
    p, handle = ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipMalloc(ctypes.byref(p), size) == 0 and hip.hipMemset(p, 0x11, size) == 0   # what the table may be given: past every claim
    torch.cuda.synchronize()
    assert hip.hipFree(p) == 0
    assert hip.hipStreamCreate(ctypes.byref(handle)) == 0
    s = torch.cuda.ExternalStream(handle.value)
    outs, graphs = [ops.buffers(), ops.buffers()], [torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()]
    torch.cuda.synchronize()
    for graph, out in zip(graphs, outs):
        with torch.cuda.graph(graph, stream=s, capture_error_mode="relaxed"):
            ops.run(out)
    for _ in range(2):
        with torch.cuda.stream(s):
            assert ops.check(ops.run(ops.buffers()))
        for i in (1, 0):
            for t in outs[i]:
                t.fill_(float("nan"))
            torch.cuda.synchronize()
            graphs[i].replay()
            torch.cuda.synchronize()
            assert ops.check(outs[i])


@pytest.mark.parametrize("B,D,T", [(37, 32, 64), (6001, 64, 32), (9001, 128, 128)])
def test_rows_stored_past_the_l2(B, D, T):
    """A large bound on the lengths makes the operators store past the L2 (and jagged_dense_bmm take the last samples first): the same bits."""
    from paper_2409_15373_amd import binding
    ops = Operators(B, D, T, 61)
    small = ops.run(ops.buffers())
    assert ops.check(small)
    bound = 10 ** 8   # rows: more than 256 MB with every B here
    out = ops.buffers()
    binding.jfa_jagged_softmax(ops.x, ops.off, bound, y=out[0])
    binding.jfa_jagged_dense_bmm(ops.x, ops.w, ops.off, bound, out=out[1])
    binding.jfa_jagged_jagged_bmm(ops.x, ops.y, ops.off, bound, out=out[2])
    binding.jfa_jagged_softmax_backward(ops.x, ops.x, ops.off, bound, dx=out[3])
    assert ops.check(out)
