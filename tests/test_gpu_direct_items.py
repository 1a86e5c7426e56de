"""Calls without a schedule, every block of rows a workgroup of its own: at both sides of the lines up to which they are made (one
block per sample in fp32, as many blocks as compute units), with samples that have fewer blocks than the bound admits, none, and no
keys.  Checked against the oracle, forward and backward, with the gates of the causal and cross parity tests (fp32 2e-5 relative to
max(1, |ref|), bf16 2e-2 absolute and 1e-2 of the tensor's maximum)."""
import numpy as np
import pytest

from test_gpu_causal import run as run_causal
from test_gpu_cross import compare, run as run_cross
from paper_2409_15373_amd.synthetic import make_custom

pytestmark = pytest.mark.gpu


def lengths(B, longest, seed):
    rng = np.random.default_rng(seed)
    L = rng.integers(0, longest + 1, B)
    L[rng.integers(0, B)] = longest
    return L.tolist()


@pytest.mark.parametrize("B,H,longest", [(1, 1, 1), (3, 1, 32), (3, 2, 33), (5, 1, 64), (300, 1, 64), (5, 1, 65), (9, 2, 128), (64, 2, 65), (65, 2, 65), (4, 1, 700)])
@pytest.mark.parametrize("D", [32, 128])
def test_fp32(B, H, longest, D):
    run_causal(make_custom("direct", lengths(B, longest, B + longest), H, D, dtype="f32", seed=B), longest)


@pytest.mark.parametrize("q_longest,k_longest", [(1, 128), (64, 64), (20, 129), (65, 30), (200, 70)])
def test_fp32_cross(q_longest, k_longest):
    Lq, Lk = lengths(7, q_longest, 1), lengths(7, k_longest, 2)
    got, ref, oq, ok = run_cross(Lq, Lk, 2, 64, "f32", 3, q_longest, k_longest)
    compare(got, ref, "f32", oq, ok, Lq, Lk)


@pytest.mark.parametrize("B,H,longest", [(1, 1, 257), (5, 2, 300), (64, 2, 300), (43, 3, 300), (7, 1, 1030), (128, 2, 140), (129, 2, 140)])
@pytest.mark.parametrize("D", [32, 64, 128])
def test_bf16(B, H, longest, D):
    run_causal(make_custom("direct", lengths(B, longest, B + longest), H, D, dtype="bf16", seed=B), longest)


@pytest.mark.parametrize("q_longest,k_longest", [(33, 300), (300, 40), (513, 257)])
@pytest.mark.parametrize("D", [32, 64, 128])
def test_bf16_cross(q_longest, k_longest, D):
    Lq, Lk = lengths(7, q_longest, 1), lengths(7, k_longest, 2)
    got, ref, oq, ok = run_cross(Lq, Lk, 2, D, "bf16", 3, q_longest, k_longest)
    compare(got, ref, "bf16", oq, ok, Lq, Lk)
