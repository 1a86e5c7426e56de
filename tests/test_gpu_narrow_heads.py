"""The direct-to-LDS kernels for head sizes 32 and 64 where they can go wrong: lengths around their 32-row waves, 64-row
stages and 128-row tiles (odd and even numbers of stages, ragged ones, idle waves), every way in which their work is dealt
(schedule built in the kernel; scheduler kernel with the schedule copied to LDS and with batches too large for that, claimed
dynamically), a reference maximum that goes stale, and rows too wide for 32-bit offsets inside a stage."""
import numpy as np
import pytest
import torch

from paper_2409_15373_amd.synthetic import make_custom, round_to_bf16_bits
import test_gpu_bf16_bwd
import test_gpu_bf16_fwd
import test_gpu_causal
import test_gpu_cross
from helpers import f64, gate_bf16

pytestmark = pytest.mark.gpu
EDGES = [1, 31, 32, 33, 0, 63, 64, 65, 127, 128, 129, 191, 192, 193, 256, 257, 321, 449]
SIZES = [pytest.param(449, id="schedule in the kernel"), pytest.param(16384, id="scheduler kernel")]


def run_self(oracle, w):
    dq, dk, dv, delta, out, lse = test_gpu_bf16_bwd.gpu_forward_backward(w, with_forward=True)
    r_out, r_lse = oracle.forward(w.q, w.k, w.v, w.offsets)
    r_dq, r_dk, r_dv, r_delta = oracle.backward(w.q, w.k, w.v, w.dout, w.offsets)
    # delta = rowsum(dO o O) of the bf16 output: rounding O costs 2^-9 |O|, rounding the probabilities (each up to 2^-9 of
    # itself, in the numerator and in the row sum) at most 2 * 2^-9 of the same average over |V|.
    bound = 2.0 ** -9 * (np.abs(r_out) + 2 * oracle.forward(w.q, w.k, np.abs(w.v), w.offsets)[0])
    bound = (np.abs(w.dout) * bound).sum(axis=2).T + 1e-4
    assert (np.abs(f64(delta) - r_delta) <= bound).all()
    for name, g, r in (("out", out, r_out), ("lse", lse, r_lse), ("dq", dq, r_dq), ("dk", dk, r_dk), ("dv", dv, r_dv)):
        # bf16 costs |x| / 512 by itself: the absolute gate follows the tensor's scale above 4, the relative one stays
        gate_bf16(name, f64(g), r, abs_tol=2e-2 * max(1.0, float(np.abs(r).max()) / 4))


@pytest.mark.parametrize("max_len", SIZES)
@pytest.mark.parametrize("D", [32, 64])
def test_self(oracle, D, max_len):
    run_self(oracle, make_custom("edges", EDGES, 2, D, dtype="bf16", seed=51 + D, max_len=max_len))


@pytest.mark.parametrize("max_len", SIZES)
@pytest.mark.parametrize("D", [32, 64])
def test_causal(D, max_len):
    test_gpu_causal.run(make_custom("edges", EDGES, 2, D, dtype="bf16", seed=52 + D), max_len)


@pytest.mark.parametrize("max_len", SIZES)
@pytest.mark.parametrize("D", [32, 64])
def test_cross(D, max_len):
    keys = EDGES[4:] + EDGES[:4]
    got, ref, oq, ok = test_gpu_cross.run(EDGES, keys, 2, D, "bf16", 53 + D, max_len, max_len)
    test_gpu_cross.compare(got, ref, "bf16", oq, ok, EDGES, keys)


@pytest.mark.parametrize("B", [900, 1100])   # at most, and more than, the samples whose schedule is copied to LDS
@pytest.mark.parametrize("D", [32, 64])
def test_dynamic_claims(oracle, D, B):
    # at least 8 x 900 tiles: more than four per workgroup at five workgroups per compute unit
    lengths = np.random.default_rng(54).integers(1, 140, size=B)
    run_self(oracle, make_custom("many", lengths, 8, D, dtype="bf16", seed=55 + D, max_len=2048))


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("D", [32, 64])
def test_stale_reference_maximum(oracle, D, causal):
    """Keys from 70 on score 8 * 8 * D / sqrt(D) >= 362 above the first 64, which set the reference: their exponentials
    overflow and the tile has to be redone maximum first; a sample of 60 rows has no such keys."""
    from oracle import causal as causal_oracle
    from paper_2409_15373_amd import binding
    lengths = [300, 500, 60]
    w = make_custom("stale", lengths, 1, D, dtype="bf16", seed=56, dout=False, max_len=512)
    w.q, w.k = np.full_like(w.q, 8.0), np.zeros_like(w.k)
    for b, L in enumerate(lengths):
        w.k[int(w.offsets[b]) + 70: int(w.offsets[b]) + L] = 8.0
    w.bits["q"], w.bits["k"] = round_to_bf16_bits(w.q), round_to_bf16_bits(w.k)
    if causal:
        d = test_gpu_bf16_fwd.to_device(w, names=("q", "k", "v"))
        out, lse = binding.jfa_forward(d["q"], d["k"], d["v"], d["offsets"], w.max_len, causal=True)
        r_out, r_lse = causal_oracle.forward(w.q, w.k, w.v, w.offsets)
    else:
        out, lse = test_gpu_bf16_fwd.gpu_forward(w)
        r_out, r_lse = oracle.forward(w.q, w.k, w.v, w.offsets)
    gate_bf16("out", f64(out), r_out)
    gate_bf16("lse", f64(lse), r_lse, abs_tol=2e-2 * max(1.0, float(np.abs(r_lse).max()) / 4))


def test_rows_wider_than_32_bit_offsets():
    """H * D just past 2^24: offsets inside a 64-row stage no longer fit the copies' 32 bits.  First, last and a middle head
    against float64 on the host; every element finite."""
    from paper_2409_15373_amd import binding
    D, H, lengths = 64, (1 << 18) + 1, [2, 66]
    n = sum(lengths)
    gen = torch.Generator(device="cuda").manual_seed(57)
    q, k, v, dout = (torch.randn(n, H, D, device="cuda", generator=gen, dtype=torch.bfloat16) for _ in range(4))
    off = torch.tensor([0, 2, 68], dtype=torch.int64, device="cuda")
    out, lse = binding.jfa_forward(q, k, v, off, 66)
    dq, dk, dv, _ = binding.jfa_backward(q, k, v, out, dout, lse, off, 66)
    for x in (out, dq, dk, dv):
        assert torch.isfinite(x).all()
    # gated per head over both samples: in a sample of two rows alone dS is a small difference of large numbers, and dk is
    # off by the bf16 rounding of `out` relative to a maximum that small (1.3e-2 seen, also from the register-staged kernels)
    for h in (0, 12345, H - 1):
        ref = []
        for s0, s1 in ((0, 2), (2, 68)):
            a = [x[s0:s1, h].double().cpu().requires_grad_(i < 3) for i, x in enumerate((q, k, v, dout))]
            o = torch.softmax(a[0] @ a[1].T / D ** 0.5, dim=1) @ a[2]
            o.backward(a[3])
            ref.append((o.detach(), a[0].grad, a[1].grad, a[2].grad))
        for name, g, r in zip(("out", "dq", "dk", "dv"), (out, dq, dk, dv), zip(*ref)):
            r = torch.cat(r).numpy()
            gate_bf16(name, f64(g[:, h]), r, abs_tol=2e-2 * max(1.0, float(np.abs(r).max()) / 2))
