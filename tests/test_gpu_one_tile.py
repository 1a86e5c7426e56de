"""The bf16 kernels for samples of at most 64 queries and keys, one workgroup each, where they can go wrong: lengths around their
32-row tiles with one and two tiles per sample, batches that do not fill the last round of dies, empty sides, and batches in which
only some samples are theirs and the others go to the kernels for longer ones."""
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

    def everything(tensors, lengths, max_len):
        off = torch.from_numpy(offsets_from_lengths(lengths)).cuda()
        out, lse = binding.jfa_forward(*tensors[:3], off, max_len, causal=causal)
        dq, dk, dv, delta = binding.jfa_backward(*tensors[:3], out, tensors[3], lse, off, max_len, causal=causal)
        return out, dq, dk, dv, lse.T, delta[0].T

    got = everything((q, k, v, do), lengths, max_len)
    for part, bound in ((lengths <= 64, 64), (lengths > 64, max_len)):
        rows = torch.from_numpy(np.repeat(part, lengths)).cuda()
        ref = everything([x[rows].contiguous() for x in (q, k, v, do)], lengths[part], bound)
        for name, g, r in zip(("out", "dq", "dk", "dv", "lse", "delta"), got, ref):
            assert torch.equal(g[rows], r), f"{name}, samples of at most {bound} rows"
