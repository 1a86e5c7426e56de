"""The direct-to-LDS forward (D = 128, samples longer than 256 rows admitted) at the edges of its rounds: one to nine 64-key
stages, a last stage with one or two 32-key blocks, 256-query tiles with waves that have no rows, and under the mask waves whose
last stage is any of the tile's four.  One sample each is a tile per workgroup, without a schedule; repeated, a workgroup goes through
several tiles, with the schedule copied to LDS or, beyond 1024 samples, in memory.  Gates as for the other bf16 forward tests (2e-2 absolute, 1e-2 of the tensor's maximum)."""
import numpy as np
import pytest
import torch

import oracle
from oracle import causal, cross
from paper_2409_15373_amd.synthetic import bf16_bits_to_f32, offsets_from_lengths, round_to_bf16_bits
from helpers import f64, gate_bf16, launched

pytestmark = pytest.mark.gpu
LENGTHS = [1, 31, 32, 33, 63, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 255, 256, 257, 288, 289, 320, 321, 384, 385, 449, 513, 0]


def forward_of(mode, host, dev, oq, ok, max_len, out, lse):
    """The GPU's call into out and lse, and the oracle's results."""
    from paper_2409_15373_amd import binding
    oqd, okd = torch.from_numpy(oq).cuda(), torch.from_numpy(ok).cuda()
    if mode == "cross":
        return lambda: binding.jfa_forward_cross(*dev, oqd, okd, max_len, max_len, out=out, lse=lse), cross.forward(*host, oq, ok)
    ref = (causal if mode == "causal" else oracle).forward(*host, oq)
    return lambda: binding.jfa_forward(*dev, oqd, max_len, out=out, lse=lse, causal=mode == "causal"), ref


def both_sides(mode, lengths):
    """(queries, keys) per sample; cross: of different samples"""
    return (lengths if mode != "cross" else lengths[5:] + lengths[:5]), lengths


@pytest.mark.parametrize("mode", ["self", "causal", "cross"])
@pytest.mark.parametrize("repeats", [1, 12, 40])
def test_every_number_of_stages(mode, repeats):
    H, D, max_len = 2, 128, 513
    Lq, Lk = both_sides(mode, LENGTHS * repeats)
    oq, ok = offsets_from_lengths(np.array(Lq)), offsets_from_lengths(np.array(Lk))
    rng = np.random.default_rng(31)
    host, dev = [], []
    for n in (oq[-1], ok[-1], ok[-1]):
        bits = round_to_bf16_bits(rng.standard_normal((int(n), H, D)).astype(np.float32))
        host.append(bf16_bits_to_f32(bits))
        t = torch.from_numpy(bits.view(np.int16)).view(torch.bfloat16)
        dev.append(torch.cat([t, torch.full((2, H, D), float("nan"), dtype=t.dtype)]).cuda())   # rows past the end: never read
    out = torch.full_like(dev[0], 777.0)
    lse = torch.full((H, int(oq[-1])), 777.0, dtype=torch.float32, device="cuda")
    call, (r_out, r_lse) = forward_of(mode, host, dev, oq, ok, max_len, out, lse)
    _, names = launched(call)
    assert "fwd_bf16_dma" in names and ("schedule" in names) == (repeats > 1)
    n = int(oq[-1])
    assert (out[n:] == 777.0).all(), "rows past the end were written"
    got_lse, has_keys = f64(lse), np.isfinite(r_lse)
    assert (got_lse[~has_keys] == -np.inf).all()
    gate_bf16("out", f64(out[:n]), r_out)
    gate_bf16("lse", got_lse[has_keys], r_lse[has_keys])


@pytest.mark.parametrize("mode", ["self", "causal", "cross"])
def test_restarted_tiles_among_others(mode):
    """Every third sample's keys from 40 on score 8 * 8 * 128 / sqrt(128) = 724 above its first 32, which set the reference: its tiles are
    redone maximum first (but for samples of at most 40 keys), between tiles of ordinary samples in the same workgroup."""
    H, D, max_len = 2, 128, 513
    Lq, Lk = both_sides(mode, [300, 257, 500, 129, 513, 280, 40] * 40)   # seven lengths, every third sample: each meets both kinds
    oq, ok = offsets_from_lengths(np.array(Lq)), offsets_from_lengths(np.array(Lk))
    rng = np.random.default_rng(33)
    q, k, v = (rng.standard_normal((int(n), H, D)).astype(np.float32) for n in (oq[-1], ok[-1], ok[-1]))
    for b in range(0, len(Lk), 3):
        q[oq[b]:oq[b + 1]] = 8.0
        k[ok[b]:ok[b + 1]] = 0.0
        k[min(ok[b] + 40, ok[b + 1]):ok[b + 1]] = 8.0
    host, dev = [], []
    for x in (q, k, v):
        bits = round_to_bf16_bits(x)
        host.append(bf16_bits_to_f32(bits))
        dev.append(torch.from_numpy(bits.view(np.int16)).view(torch.bfloat16).cuda())
    out, lse = torch.full_like(dev[0], float("nan")), torch.full((H, int(oq[-1])), float("nan"), dtype=torch.float32, device="cuda")
    call, (r_out, r_lse) = forward_of(mode, host, dev, oq, ok, max_len, out, lse)
    _, names = launched(call)
    assert {"fwd_bf16_dma", "schedule"} <= names
    gate_bf16("out", f64(out), r_out)
    gate_bf16("lse", f64(lse), r_lse, abs_tol=2e-2 * max(1.0, float(np.abs(r_lse).max()) / 4))
