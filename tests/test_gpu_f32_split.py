"""fp32 attention at head sizes 32 and 64 on the bf16 matrix instructions, where it can go wrong: lengths around its 32-row waves and
stages, 128-row tiles of queries and 64-row tiles of keys; work dealt, claimed and listed in the kernel; values that are not the sum
of three bf16 numbers.  A bound of 16384 rows on the lengths makes a batch of any lengths large enough for these kernels.  Errors are
held to those of fp32 arithmetic on the same inputs as in test_gpu_f32_large_scores.py: a quarter more, and five units of fp32's
roundoff (6e-8) for the exponential and the statistics, whose errors the host's arithmetic does not have."""
import numpy as np
import pytest
import torch

from paper_2409_15373_amd.synthetic import make_custom, offsets_from_lengths
import test_gpu_causal
import test_gpu_cross
import test_gpu_f32
from test_gpu_f32_large_scores import evaluate
from test_gpu_f32_tiles import EDGES

pytestmark = pytest.mark.gpu
LARGE = 16384


@pytest.mark.parametrize("copies", [1, 60])   # a tile or two per workgroup; more than four, claimed
@pytest.mark.parametrize("D", [32, 64])
def test_self(oracle, D, copies):
    test_gpu_f32.run_case(oracle, make_custom("edges", EDGES * copies, 2, D, dtype="f32", seed=41 + D, max_len=LARGE))


@pytest.mark.parametrize("D", [32, 64])
def test_schedule_in_the_kernel(oracle, D):
    lengths = np.random.default_rng(40 + D).integers(0, 151, 130)   # 520 tiles of 128 rows at most, 780 of 64
    test_gpu_f32.run_case(oracle, make_custom("small", lengths.tolist(), 2, D, dtype="f32", seed=40 + D, max_len=150))


@pytest.mark.parametrize("D", [32, 64])
def test_causal(D):
    test_gpu_causal.run(make_custom("edges", EDGES, 2, D, dtype="f32", seed=42 + D), LARGE)


@pytest.mark.parametrize("D", [32, 64])
def test_cross(D):
    keys = EDGES[4:] + EDGES[:4]
    got, ref, oq, ok = test_gpu_cross.run(EDGES, keys, 2, D, "f32", 43 + D, LARGE, LARGE)
    test_gpu_cross.compare(got, ref, "f32", oq, ok, EDGES, keys)


def evaluate_by_rows(q, k, v, do, causal, rounded):
    """evaluate() a query at a time with the keys that it sees: what causal masking hides takes no part, not even as 0 times infinity."""
    if not causal:
        return evaluate(q, k, v, do, False, rounded)
    out, dq, dk, dv = (np.zeros(x.shape) for x in (q, q, k, v))
    for i in range(len(q)):
        one = slice(i, i + 1)
        out[one], dq[one], dk_i, dv_i = evaluate(q[one], k[:i + 1], v[:i + 1], do[one], False, rounded)
        dk[:i + 1] += dk_i
        dv[:i + 1] += dv_i
    return out, dq, dk, dv


def run(lengths, H, D, sigma, causal, seed, change, evaluate=evaluate):
    """GPU results and their fp64 and rounded host values (out, dq, dk, dv), inputs changed by `change` first."""
    from paper_2409_15373_amd import binding
    rng = np.random.default_rng(seed)
    off = offsets_from_lengths(np.array(lengths))
    q, k, v, do = ((rng.standard_normal((int(off[-1]), H, D)) * s).astype(np.float32) for s in (sigma, sigma, 1.0, 1.0))
    change(q, k, v, do)
    d = [torch.from_numpy(x).cuda() for x in (q, k, v, do)]
    o = torch.from_numpy(off).cuda()
    out, lse = binding.jfa_forward(d[0], d[1], d[2], o, LARGE, causal=causal)
    got = [x.double().cpu().numpy() for x in (out,) + binding.jfa_backward(d[0], d[1], d[2], out, d[3], lse, o, LARGE, causal=causal)[:3]]
    exact, plain = ([np.empty(x.shape) for x in got] for _ in range(2))
    with np.errstate(all="ignore"):
        for b in range(len(lengths)):
            r = slice(off[b], off[b + 1])
            for h in range(H):
                for dest, rounded in ((exact, False), (plain, True)):
                    for x, y in zip(dest, evaluate(q[r, h], k[r, h], v[r, h], do[r, h], causal, rounded)):
                        x[r, h] = y
    return got, exact, plain


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("D", [32, 64])
@pytest.mark.parametrize("sigma", [1.0, 4.0])
def test_error_is_that_of_fp32(D, causal, sigma):
    got, exact, plain = run([200, 64, 33, 150, 1] * 8, 1, D, sigma, causal, D, lambda *x: None)
    norm = np.linalg.norm
    for name, g, e, p in zip(("out", "dq", "dk", "dv"), got, exact, plain):
        error, bound = norm(g - e) / norm(e), 1.25 * norm(p - e) / norm(e) + 3e-7
        print(f"D {D} sigma {sigma} {name}: {error:.2e}, bound {bound:.2e}", flush=True)
        assert error <= bound, f"{name}: {error:.2e} > {bound:.2e}"


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("D", [32, 64])
@pytest.mark.parametrize("small", ["q", "k", "v", "dout"])
def test_small_factors_keep_their_bits(D, causal, small):
    """One factor of the products around 2^-118 (with v or dout, dS below that), where a float still has 24 bits but the last of three
    bf16 pieces would lie below bf16's smallest number: the error stays that of fp32.  (The bound's host arithmetic rounds small
    differences and products, some of them below 2^-126, to fp32 as well.)"""
    def change(q, k, v, do):
        x = dict(q=q, k=k, v=v, dout=do)[small]
        x *= np.float32(2.0 ** -118)
    got, exact, plain = run([200, 64, 33, 150, 1] * 2, 1, D, 1.0, causal, D, change)
    norm = np.linalg.norm
    for name, g, e, p in zip(("out", "dq", "dk", "dv"), got, exact, plain):
        error, bound = norm(g - e) / norm(e), 1.25 * norm(p - e) / norm(e) + 3e-7
        print(f"D {D} {small} {name}: {error:.2e}, bound {bound:.2e}", flush=True)
        assert error <= bound, f"{name}: {error:.2e} > {bound:.2e}"


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("D", [32, 64])
@pytest.mark.parametrize("what", ["inf in v", "-inf in dout", "-inf score", "near the largest float", "nan in k", "nan in v", "nan in q", "nan in dout",
                                  "inf and nan"])
def test_values_without_a_split(D, causal, what):
    """Where the sums have a value, infinite or not, it is the result; what is NaN there is NaN here.  Relative error per element."""
    rows = [7, 150]   # one row of the first sample, one of the second

    def change(q, k, v, do):
        if what == "inf in v":
            v[rows, :, 3] = np.inf
        elif what == "-inf in dout":
            do[rows, :, 5] = -np.inf
        elif what == "-inf score":   # q > 0: the key is invisible
            np.abs(q, out=q)
            k[rows, :, 2] = -np.inf
        elif what == "near the largest float":   # rounds to infinity in bf16
            v[rows, :, 1] = 3.4e38
            do[:] = 0
        elif what == "inf and nan":   # one column of out and dv infinite, one NaN
            v[rows, :, 3], v[rows, :, 6] = np.inf, np.nan
            do[rows, :, 5], do[rows, :, 6] = -np.inf, np.nan
        else:
            dict(k=k, v=v, q=q, dout=do)[what.split()[-1]][rows, :, 4] = np.nan
    got, exact, _ = run([100, 129, 64], 2, D, 1.0, causal, 7, change, evaluate_by_rows)
    for name, g, e in zip(("out", "dq", "dk", "dv"), got, exact):
        known = ~np.isnan(e)
        assert (np.isnan(g) == np.isnan(e)).all(), name
        assert (np.isinf(g) == np.isinf(e))[known].all() and (g[known & np.isinf(e)] == e[known & np.isinf(e)]).all(), name
        f = known & np.isfinite(e)
        assert np.isfinite(g[f]).all() and (np.abs(g[f] - e[f]) <= 2e-5 * np.maximum(np.abs(e[f]), 1.0)).all(), name


@pytest.mark.parametrize("where", ["everywhere", "k", "v", "q", "dout"])
def test_nan_costs_little(where):
    """Rows with NaN are not taken again: looking for the NaN costs a wave less than its products (1.0 to 1.6 times the ordinary call was
    measured), taking every row again some thirty times as much."""
    from paper_2409_15373_amd import binding
    gen = torch.Generator(device="cuda").manual_seed(8)
    off = torch.from_numpy(offsets_from_lengths(np.random.default_rng(8).integers(1, 513, 256))).cuda()
    names = ("q", "k", "v", "dout")
    ordinary = [torch.randn(int(off[-1]), 2, 64, device="cuda", generator=gen) for _ in names]
    odd = [x.clone() for x in ordinary]
    for name, x in zip(names, odd):
        if where == "everywhere":
            x.fill_(float("nan"))
        elif where == name:
            x[off[1:] - 1, :, 3] = float("nan")   # the last row of every sample

    def time(q, k, v, do):
        def call():
            out, lse = binding.jfa_forward(q, k, v, off, 512)
            binding.jfa_backward(q, k, v, out, do, lse, off, 512)
        call()
        times = []
        for _ in range(7):
            start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            for _ in range(3):
                call()
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end))
        return sorted(times)[3]
    ratio = time(*odd) / time(*ordinary)
    print(f"NaN in {where}: {ratio:.2f} times", flush=True)
    assert ratio < 3
