"""The fp32 matrix-core kernels at the edges of their tiles: a workgroup's four waves are the quarters of a 64 x 64 square,
so lengths around 32, 64, 96 and 128 leave waves idle, blocks ragged, or one wave of a pair without anything to add.  With a tight
max_len there is no schedule (D = 128, backward: the kernels build it), with 4096 the kernels build it, with 8192 the scheduler kernel
does, for the fp32 instructions at D = 128 and the split products at D = 32 and 64."""
import pytest

from paper_2409_15373_amd.synthetic import make_custom
import test_gpu_causal
import test_gpu_cross
import test_gpu_f32

pytestmark = pytest.mark.gpu
EDGES = [1, 31, 32, 33, 0, 63, 64, 65, 95, 96, 97, 127, 128, 129, 200]


@pytest.mark.parametrize("max_len", [200, 4096, 8192])
@pytest.mark.parametrize("D", [32, 64, 128])
def test_self(oracle, D, max_len):
    test_gpu_f32.run_case(oracle, make_custom("edges", EDGES, 1, D, dtype="f32", seed=31 + D, max_len=max_len))


@pytest.mark.parametrize("max_len", [200, 4096, 8192])
@pytest.mark.parametrize("D", [32, 64, 128])
def test_causal(D, max_len):
    test_gpu_causal.run(make_custom("edges", EDGES, 1, D, dtype="f32", seed=32 + D), max_len)


@pytest.mark.parametrize("max_len", [200, 4096, 8192])
@pytest.mark.parametrize("D", [32, 64, 128])
def test_cross(D, max_len):
    keys = EDGES[4:] + EDGES[:4]
    got, ref, oq, ok = test_gpu_cross.run(EDGES, keys, 1, D, "f32", 33 + D, max_len, max_len)
    test_gpu_cross.compare(got, ref, "f32", oq, ok, EDGES, keys)


@pytest.mark.parametrize("mode", ["self", "cross"])
@pytest.mark.parametrize("D", [32, 64, 128])
def test_an_infinity_in_the_last_row_stays_in_its_column(D, mode):
    """Stages of a sample's last rows are filled up by repeating its last one, with probability 0.  An infinite value there
    makes its column of `out` infinite, and an infinite dout its column of dv, with every probability above 0; no other
    column changes, and nothing becomes NaN (an infinity times 0)."""
    import numpy as np
    import torch
    from paper_2409_15373_amd import binding
    w = make_custom("inf", [33, 64, 1, 40, 100, 127, 200], 2, D, dtype="f32", seed=34, max_len=200)
    d = test_gpu_f32.to_device(w)
    last = torch.from_numpy(w.offsets[1:] - 1).cuda()

    def run():
        if mode == "cross":
            out, lse = binding.jfa_forward_cross(d["q"], d["k"], d["v"], d["offsets"], d["offsets"], 200, 200)
            return out, binding.jfa_backward_cross(d["q"], d["k"], d["v"], plain_out, d["dout"], lse, d["offsets"], d["offsets"], 200, 200)[2]
        out, lse = binding.jfa_forward(d["q"], d["k"], d["v"], d["offsets"], 200)
        return out, binding.jfa_backward(d["q"], d["k"], d["v"], plain_out, d["dout"], lse, d["offsets"], 200)[2]

    plain_out = binding.jfa_forward(d["q"], d["k"], d["v"], d["offsets"], 200)[0]
    out, dv = run()
    d["v"][last, :, 3] = float("inf")
    d["dout"][last, :, 5] = float("-inf")
    inf_out, inf_dv = run()
    assert (inf_out[:, :, 3] == float("inf")).all() and (inf_dv[:, :, 5] == float("-inf")).all()
    others = lambda x, c: torch.cat([x[:, :, :c], x[:, :, c + 1:]], dim=2)
    assert torch.equal(others(inf_out, 3), others(out, 3)) and torch.equal(others(inf_dv, 5), others(dv, 5))
    assert np.isfinite(test_gpu_f32.f64(others(inf_out, 3))).all()


@pytest.mark.parametrize("B", [300, 5000, 13000])   # no schedule but for the backward at D = 128: built in the kernel, then claimed
@pytest.mark.parametrize("D", [32, 64, 128])
def test_many_short_samples(oracle, D, B):
    import numpy as np
    lengths = np.random.default_rng(35).integers(0, 21, size=B)
    test_gpu_f32.run_case(oracle, make_custom("many", lengths, 2, D, dtype="f32", seed=36 + D, max_len=20))


# (samples, heads, longest, bound) on the fp32 instructions, where a bound of more than one block and more blocks than compute units keep a
# schedule, and whether the scheduler kernel makes it.  Workgroups: 256 x 1 to 12 by registers; four, at D <= 64 sixteen, items each
# are dealt without claims.
WALKS = [pytest.param(200, 2, 65, 65, False, id="schedule in the kernel"),
         pytest.param(300, 2, 100, 100, True, id="dealt"),
         pytest.param(5000, 2, 20, 33, True, id="one wave, dealt"),          # D = 128: claimed
         pytest.param(30000, 2, 6, 33, True, id="one wave, claimed")]


@pytest.mark.parametrize("B,H,longest,bound,scheduler", WALKS)
@pytest.mark.parametrize("D", [32, 64, 128])
def test_walks_through_a_schedule(oracle, D, B, H, longest, bound, scheduler):
    import numpy as np
    from helpers import launched
    lengths = np.random.default_rng(42).integers(0, longest + 1, size=B)
    w = make_custom("walk", lengths, H, D, dtype="f32", seed=43 + D, max_len=bound)
    _, names = launched(lambda: test_gpu_f32.run_case(oracle, w))
    assert names == {"fwd_f32", "bwd_f32"} | ({"schedule"} if scheduler else set())


@pytest.mark.parametrize("B,scheduler", [(100, False), (300, True), (4000, True)])   # built in the kernel; dealt; claimed
@pytest.mark.parametrize("D", [32, 64, 128])
def test_walks_of_four_wave_workgroups_against_longer_streams(D, B, scheduler):
    """At most 64 queries against at most 128 keys: blocks of 64 queries that keep a schedule, longest stream first."""
    import numpy as np
    from helpers import launched
    rng = np.random.default_rng(44)
    lq, lk = rng.integers(0, 9, size=B), np.where(rng.random(B) < 0.1, rng.integers(65, 129, size=B), rng.integers(0, 20, size=B))
    lq[0], lk[0], lq[1], lk[1] = 64, 128, 0, 0
    (got, ref, oq, ok), names = launched(lambda: test_gpu_cross.run(lq, lk, 4, D, "f32", 45 + D, 64, 128))
    test_gpu_cross.compare(got, ref, "f32", oq, ok, lq, lk)
    assert names == {"fwd_f32", "bwd_f32"} | ({"schedule"} if scheduler else set())



SHORT = [1, 31, 32, 0, 7, 8, 9, 16, 30, 2]
LONG = [70, 5, 0, 33, 64, 96, 1, 200, 31, 32]


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("form", ["causal", "short queries", "short keys", "both short"])
def test_one_wave_workgroups(D, form):
    """Streams of at most 32 rows: one-wave workgroups for the kernels they stream through (the keys through forward and dQ, the
    queries through dK / dV), the others as before, in one call."""
    if form == "causal":
        return test_gpu_causal.run(make_custom("short", SHORT, 2, D, dtype="f32", seed=37 + D), 32)
    lq, lk = (LONG if form == "short keys" else SHORT), (LONG if form == "short queries" else SHORT[::-1])
    got, ref, oq, ok = test_gpu_cross.run(lq, lk, 2, D, "f32", 38 + D, max(lq), max(lk))
    test_gpu_cross.compare(got, ref, "f32", oq, ok, lq, lk)


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("form", ["self", "causal", "cross"])
def test_one_wave_workgroups_of_two_stages(oracle, D, form):
    """Streams of at most 64 rows in a batch of more tiles than are dealt in the kernel: one-wave workgroups with up to two
    stages, blocks of 32 rows, the schedule kernel."""
    import numpy as np
    rng = np.random.default_rng(39)
    lengths = rng.integers(0, 65, size=700)
    if form == "cross":
        other = rng.integers(0, 65, size=700)
        got, ref, oq, ok = test_gpu_cross.run(lengths, other, 2, D, "f32", 40 + D, 64, 64)
        return test_gpu_cross.compare(got, ref, "f32", oq, ok, lengths, other)
    w = make_custom("two", lengths, 2, D, dtype="f32", seed=41 + D, max_len=64)
    test_gpu_causal.run(w, 64) if form == "causal" else test_gpu_f32.run_case(oracle, w)
