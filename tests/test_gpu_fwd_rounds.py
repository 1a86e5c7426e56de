"""The direct-to-LDS forward (D = 128, samples longer than 256 rows admitted) at the edges of its rounds: one to nine 64-key
stages, a last stage with one or two 32-key blocks, 256-query tiles with waves that have no rows, and under the mask waves whose
last stage is any of the tile's four.  Gates as for the other bf16 forward tests (2e-2 absolute, 1e-2 of the tensor's maximum)."""
import numpy as np
import pytest
import torch

import oracle
from oracle import causal, cross
from paper_2409_15373_amd.synthetic import bf16_bits_to_f32, offsets_from_lengths, round_to_bf16_bits
from helpers import f64, gate_bf16

pytestmark = pytest.mark.gpu
LENGTHS = [1, 31, 32, 33, 63, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 255, 256, 257, 288, 289, 320, 321, 384, 385, 449, 513, 0]


@pytest.mark.parametrize("mode", ["self", "causal", "cross"])
def test_every_number_of_stages(mode):
    from paper_2409_15373_amd import binding
    H, D, max_len = 2, 128, 513
    Lq = LENGTHS if mode != "cross" else LENGTHS[5:] + LENGTHS[:5]
    oq, ok = offsets_from_lengths(np.array(Lq)), offsets_from_lengths(np.array(LENGTHS))
    rng = np.random.default_rng(31)
    host, dev = [], []
    for n in (oq[-1], ok[-1], ok[-1]):
        bits = round_to_bf16_bits(rng.standard_normal((int(n), H, D)).astype(np.float32))
        host.append(bf16_bits_to_f32(bits))
        t = torch.from_numpy(bits.view(np.int16)).view(torch.bfloat16)
        dev.append(torch.cat([t, torch.full((2, H, D), float("nan"), dtype=t.dtype)]).cuda())   # rows past the end: never read
    oqd, okd = torch.from_numpy(oq).cuda(), torch.from_numpy(ok).cuda()
    out = torch.full_like(dev[0], 777.0)
    lse = torch.full((H, int(oq[-1])), 777.0, dtype=torch.float32, device="cuda")
    if mode == "cross":
        binding.jfa_forward_cross(*dev, oqd, okd, max_len, max_len, out=out, lse=lse)
        r_out, r_lse = cross.forward(*host, oq, ok)
    else:
        binding.jfa_forward(*dev, oqd, max_len, out=out, lse=lse, causal=mode == "causal")
        r_out, r_lse = (causal if mode == "causal" else oracle).forward(*host, oq)
    n = int(oq[-1])
    assert (out[n:] == 777.0).all(), "rows past the end were written"
    got_lse, has_keys = f64(lse), np.isfinite(r_lse)
    assert (got_lse[~has_keys] == -np.inf).all()
    gate_bf16("out", f64(out[:n]), r_out)
    gate_bf16("lse", got_lse[has_keys], r_lse[has_keys])
