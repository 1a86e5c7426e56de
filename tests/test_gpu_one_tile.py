"""The bf16 kernels for samples of at most 64 queries and keys, one workgroup each, where they can go wrong: lengths around their
32-row tiles with one and two tiles per sample, batches that do not fill the last round of dies, empty sides, and batches in which
only some samples are theirs and the others go to the kernels for longer ones."""
import numpy as np
import pytest

from paper_2409_15373_amd.synthetic import make_custom
import test_gpu_causal
import test_gpu_cross
from test_gpu_narrow_heads import run_self

pytestmark = pytest.mark.gpu
ONE = [1, 31, 32, 0, 16, 17, 2, 32, 0, 15, 29]           # one tile of 32 rows
TWO = ONE + [33, 63, 64, 48, 0, 64, 47, 1]               # up to two
LENGTHS = [pytest.param(ONE, id="one"), pytest.param(TWO, id="two")]


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
