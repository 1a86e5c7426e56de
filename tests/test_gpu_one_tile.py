"""The bf16 kernels for samples of at most 128 queries and keys, one workgroup each, where they can go wrong: lengths around their
32-row tiles with one, two and four tiles per sample, batches that do not fill the last round of dies, empty sides, batches in which
only some samples are theirs and the others go to the kernels for longer ones, and batches done in two launches."""
import numpy as np
import pytest
import torch

from paper_2409_15373_amd import binding
from paper_2409_15373_amd.synthetic import make_custom, offsets_from_lengths
import test_gpu_causal
import test_gpu_cross
from test_gpu_narrow_heads import run_self

pytestmark = pytest.mark.gpu
ONE = [1, 31, 32, 0, 16, 17, 2, 32, 0, 15, 29]           # one tile of 32 rows
TWO = ONE + [33, 63, 64, 48, 0, 64, 47, 1]               # up to two
FOUR = TWO + [65, 96, 127, 128, 0, 97, 128, 1]           # up to four
LENGTHS = [pytest.param(ONE, id="one"), pytest.param(TWO, id="two"), pytest.param(FOUR, id="four")]


@pytest.mark.parametrize("lengths", LENGTHS)
@pytest.mark.parametrize("D", [32, 64, 128])
def test_self(oracle, D, lengths):
    run_self(oracle, make_custom("tiles", lengths, 3, D, dtype="bf16", seed=71 + D, max_len=max(lengths)))


@pytest.mark.parametrize("lengths", LENGTHS)
@pytest.mark.parametrize("D", [32, 64, 128])
def test_causal(D, lengths):
    test_gpu_causal.run(make_custom("tiles", lengths, 3, D, dtype="bf16", seed=72 + D), max(lengths))


@pytest.mark.parametrize("lengths", LENGTHS)
@pytest.mark.parametrize("D", [32, 64, 128])
def test_cross(D, lengths):
    keys = lengths[3:] + lengths[:3]
    got, ref, oq, ok = test_gpu_cross.run(lengths, keys, 3, D, "bf16", 73 + D, max(lengths), max(lengths))
    test_gpu_cross.compare(got, ref, "bf16", oq, ok, lengths, keys)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("D,B,H,max_len", [(128, 1030, 4, 200), (128, 1030, 4, 300), (64, 2050, 8, 200)])
def test_only_some_samples(D, B, H, max_len, causal):
    """Large batches of mixed lengths: the short samples come here, the others' schedule skips them.  Both halves give the bits of
    calls on those samples alone, which the tests above and those of the other kernels hold to the oracle."""
    lengths = np.random.default_rng(74).integers(0, 9, size=B)
    for first, length in ((10, 63), (11, 64), (12, 65), (13, 66)):
        lengths[first:B:100] = length
    lengths[[0, 500, B - 1]] = [max_len, 97, 129]
    gen = torch.Generator(device="cuda").manual_seed(75)
    q, k, v, do = (torch.randn(int(lengths.sum()), H, D, device="cuda", generator=gen).bfloat16() for _ in range(4))

    compare_parts((q, k, v, do), lengths, lengths, max_len, causal, "self")


def compare_parts(tensors, lq, lk, max_len, causal, mode):
    """A call on all samples and calls on those of at most 64 rows and on the others, bit for bit."""
    q, k, v, do = tensors

    def everything(q, k, v, do, lq, lk, max_len):
        oq, ok = (torch.from_numpy(offsets_from_lengths(x)).cuda() for x in (lq, lk))
        if mode == "cross":
            out, lse = binding.jfa_forward_cross(q, k, v, oq, ok, max_len, max_len)
            dq, dk, dv, delta = binding.jfa_backward_cross(q, k, v, out, do, lse, oq, ok, max_len, max_len)
        else:
            out, lse = binding.jfa_forward(q, k, v, oq, max_len, causal=causal)
            dq, dk, dv, delta = binding.jfa_backward(q, k, v, out, do, lse, oq, max_len, causal=causal)
        assert delta.shape == lse.shape
        return dict(out=out, dq=dq, lse=lse.T, delta=delta.T), dict(dk=dk, dv=dv)   # by queries, by keys

    got = everything(q, k, v, do, lq, lk, max_len)
    short = (lq <= 64) & (lk <= 64)
    for part, bound in ((short, 64), (~short, max_len)):
        rows = [torch.from_numpy(np.repeat(part, x)).cuda() for x in (lq, lk)]
        mine = [x[r].contiguous() for x, r in ((q, rows[0]), (k, rows[1]), (v, rows[1]), (do, rows[0]))]
        ref = everything(*mine, lq[part], lk[part], bound)
        for g, r, at in zip(got, ref, rows):
            for name in g:
                assert torch.equal(g[name][at], r[name]), f"{name}, samples of at most {bound} rows"


@pytest.mark.parametrize("mode", ["self", "causal", "cross"])
@pytest.mark.parametrize("D", [32, 64, 128])
def test_two_launches(D, mode):
    """At most 128 rows and so many (sample, head) pairs that samples of at most 64 rows are done in a launch of their own: 64 per compute
    unit (head size 32 and cross attention take one launch in some directions; the bits are the same).  Both parts alone are too small for
    that and are held to the oracle above."""
    B, H = 2051, 8
    rng = np.random.default_rng(76)
    lq, lk = rng.integers(0, 9, size=B), rng.integers(0, 9, size=B)
    for first, length in ((10, 63), (11, 64), (12, 65), (13, 128), (14, 96), (15, 127)):
        lq[first:B:100] = length
        lk[first + 3:B:100] = length
    lk = lk if mode == "cross" else lq
    assert B * H >= 64 * torch.cuda.get_device_properties(0).multi_processor_count
    gen = torch.Generator(device="cuda").manual_seed(77)
    q, do = (torch.randn(int(lq.sum()), H, D, device="cuda", generator=gen).bfloat16() for _ in range(2))
    k, v = (torch.randn(int(lk.sum()), H, D, device="cuda", generator=gen).bfloat16() for _ in range(2))
    compare_parts((q, k, v, do), lq, lk, 128, mode == "causal", mode)


def test_more_items_than_one_launch_holds():
    """530001 x 8 (sample, head) pairs are more than the 2^22 workgroups of a launch.  A sample of one row is its own softmax: out is v
    and dv is dout, bit for bit; dq and dk are zero up to the rounding of two sums of 32 products that are the same (delta and dO . v)."""
    B, H, D = 530001, 8, 32
    gen = torch.Generator(device="cuda").manual_seed(78)
    q, k, v, do = (torch.randn(B, H, D, device="cuda", generator=gen).bfloat16() for _ in range(4))
    off = torch.arange(B + 1, device="cuda")
    out, lse = binding.jfa_forward(q, k, v, off, 1)
    dq, dk, dv, _ = binding.jfa_backward(q, k, v, out, do, lse, off, 1)
    assert torch.equal(out, v) and torch.equal(dv, do)
    # each sum's error is at most 32 * 2^-24 of the sum of the products' sizes, (|dO| . |v|); times |k| or |q| and 1 / sqrt(D)
    bound = 2 * 32 * 2.0 ** -24 * (do.float().abs() * v.float().abs()).sum(2, keepdim=True) / D ** 0.5 * 1.01
    assert bool((dq.float().abs() <= bound * k.float().abs()).all()) and bool((dk.float().abs() <= bound * q.float().abs()).all())
    s = (q.float() * k.float()).sum(2).T / D ** 0.5
    assert bool(((lse - s).abs() <= 1e-5 * (1 + s.abs())).all())
