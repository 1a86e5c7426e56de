"""The direct-to-LDS kernels for head sizes 32 and 64 where they can go wrong: lengths around their 32-row waves, 64-row
stages and 128-row tiles (odd and even numbers of stages, ragged ones, idle waves), every way in which their work is dealt
(no schedule; schedule built in the kernel; scheduler kernel with the schedule copied to LDS and with batches too large for that, claimed
dynamically), a reference maximum that goes stale, and rows too wide for 32-bit offsets inside a stage."""
import numpy as np
import pytest
import torch

from paper_2409_15373_amd.synthetic import bf16_bits_to_f32, make_custom, round_to_bf16_bits
import test_gpu_bf16_bwd
import test_gpu_bf16_fwd
import test_gpu_causal
import test_gpu_cross
from helpers import f64, gate_bf16

pytestmark = pytest.mark.gpu
EDGES = [1, 31, 32, 33, 0, 63, 64, 65, 127, 128, 129, 191, 192, 193, 256, 257, 321, 449]
SIZES = [pytest.param(449, id="no schedule"), pytest.param(1024, id="schedule in the kernel"), pytest.param(16384, id="scheduler kernel")]


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


@pytest.mark.parametrize("B", [500, 700])   # static deal of a scheduler kernel's schedule, with and without an LDS copy of it
@pytest.mark.parametrize("D", [32, 64])
def test_static_deal(oracle, D, B):
    lengths = np.random.default_rng(63).integers(0, 140, size=B)
    run_self(oracle, make_custom("static", lengths, 2, D, dtype="bf16", seed=64 + D, max_len=2048))


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


def forward_of(mode, w):
    """(out, lse) of the GPU and of the oracle; cross: the sample's rows as its keys and again as its queries."""
    from oracle import causal as causal_oracle, cross as cross_oracle
    from paper_2409_15373_amd import binding
    d = test_gpu_bf16_fwd.to_device(w, names=("q", "k", "v"))
    if mode == "cross":
        got = binding.jfa_forward_cross(d["q"], d["k"], d["v"], d["offsets"], d["offsets"], w.max_len, w.max_len)
        ref = cross_oracle.forward(w.q, w.k, w.v, w.offsets, w.offsets)
    else:
        got = binding.jfa_forward(d["q"], d["k"], d["v"], d["offsets"], w.max_len, causal=mode == "causal")
        ref = causal_oracle.forward(w.q, w.k, w.v, w.offsets) if mode == "causal" else cross_oracle.forward(w.q, w.k, w.v, w.offsets, w.offsets)
    return [f64(x) for x in got], ref


def rising_scores(D, rise, lengths, v_scale=1.0, seed=61):
    """Queries along one direction (plus noise), keys whose score along it is rise(j) for key j: maxima that go up on the way."""
    w = make_custom("rising", lengths, 2, D, dtype="bf16", seed=seed, dout=False, max_len=512)
    rng = np.random.default_rng(seed)
    w.q, w.k = rng.standard_normal(w.q.shape).astype(np.float32) * 0.25, rng.standard_normal(w.k.shape).astype(np.float32) * 0.25
    w.q[:, :, 0] = 8.0
    for b, L in enumerate(lengths):
        w.k[int(w.offsets[b]):int(w.offsets[b]) + L, :, 0] = np.array([rise(j) for j in range(L)], dtype=np.float32)[:, None] * D ** 0.5 / 8
    w.v = w.v * np.float32(v_scale)
    for n in ("q", "k", "v"):
        w.bits[n] = round_to_bf16_bits(getattr(w, n))
        setattr(w, n, bf16_bits_to_f32(w.bits[n]))
    return w


@pytest.mark.parametrize("mode", ["self", "causal", "cross"])
@pytest.mark.parametrize("step", [1.5, 4.0, 7.0])   # per 64-key stage; e^5.5 = 2^8 is where the reference goes stale
@pytest.mark.parametrize("D", [32, 64])
def test_maxima_that_rise_from_stage_to_stage(D, step, mode):
    """Rescale factors between 0 and 1 at every rise, row sums of many sizes, samples with and without a ragged last stage."""
    w = rising_scores(D, lambda j: step * (j / 64.0), [300, 500, 60, 448, 1])
    (out, lse), (r_out, r_lse) = forward_of(mode, w)
    gate_bf16("out", out, r_out)
    gate_bf16("lse", lse, r_lse, abs_tol=2e-2 * max(1.0, float(np.abs(r_lse).max()) / 4))


@pytest.mark.parametrize("mode", ["self", "causal", "cross"])
@pytest.mark.parametrize("D", [32, 64])
def test_large_values_behind_a_stale_maximum(D, mode):
    """Values of 1e25, and keys from 70 on that score 34 above the first 64: against the first stage's maximum their
    probabilities are up to e^37, and those times the values are beyond fp32."""
    w = rising_scores(D, lambda j: 34.0 * (j >= 70), [300, 500, 60], v_scale=1e25)
    (out, lse), (r_out, r_lse) = forward_of(mode, w)
    assert np.isfinite(out).all()
    gate_bf16("out", out / 1e25, r_out / 1e25)
    gate_bf16("lse", lse, r_lse, abs_tol=2e-2 * max(1.0, float(np.abs(r_lse).max()) / 4))


@pytest.mark.parametrize("D", [32, 64])
def test_row_sums_of_large_scores(D):
    """Scores of standard deviation 16, where one key has most of a row's weight: its probability is rounded to bf16 unless
    the reference is that very score, so how closely the reference follows shows in the log-sum-exp.  The bound is the error
    of a reference that is raised, for the 32 queries of a wave together, where a stage's maximum exceeds it by 2^8,
    evaluated on the host in fp64 but for that rounding; 1.2 times for the few rows whose sums are rounded elsewhere."""
    L = 960
    w = make_custom("large", [L], 2, D, dtype="bf16", seed=62, sigma=4.0, dout=False, max_len=1024)
    (_, lse), (_, exact) = forward_of("self", w)
    err = np.empty_like(exact)
    for h in range(2):
        s = w.q[:, h].astype(np.float64) @ w.k[:, h].astype(np.float64).T / (D ** 0.5 * np.log(2.0))
        for q0 in range(0, L, 32):
            m, l = np.full(32, -np.inf), np.zeros(32)
            for j in range(0, L, 64):
                x = s[q0:q0 + 32, j:j + 64]
                if (x.max(axis=1) > m + 8).any():
                    n = np.maximum(m, x.max(axis=1))
                    m, l = n, l * np.exp2(m - n)
                l += bf16_bits_to_f32(round_to_bf16_bits(np.exp2(x - m[:, None]).astype(np.float32))).astype(np.float64).sum(axis=1)
            err[h, q0:q0 + 32] = (m + np.log2(l)) * np.log(2.0) - exact[h, q0:q0 + 32]
    rms = lambda x: float(np.sqrt(np.mean(x * x)))
    print(f"D {D}: {rms(lse - exact):.2e}, bound {1.2 * rms(err):.2e}", flush=True)
    assert rms(lse - exact) <= 1.2 * rms(err)


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


SHORT = [1, 31, 32, 33, 0, 63, 64, 65, 95, 96, 97, 127, 128]


def everything(form, D, lq, lk, max_q, max_k, seed):
    """out, lse, dq, dk, dv and delta of a call with these bounds on the lengths; the inputs are a function of the seed."""
    from paper_2409_15373_amd import binding
    from paper_2409_15373_amd.synthetic import offsets_from_lengths
    gen = torch.Generator(device="cuda").manual_seed(seed)
    oq, ok = (torch.from_numpy(offsets_from_lengths(np.array(x))).cuda() for x in (lq, lk))
    q, do = (torch.randn(sum(lq), 2, D, device="cuda", generator=gen).bfloat16() for _ in range(2))
    k, v = (torch.randn(sum(lk), 2, D, device="cuda", generator=gen).bfloat16() for _ in range(2))
    if form == "cross":
        out, lse = binding.jfa_forward_cross(q, k, v, oq, ok, max_q, max_k)
        return (out, lse) + tuple(binding.jfa_backward_cross(q, k, v, out, do, lse, oq, ok, max_q, max_k))
    out, lse = binding.jfa_forward(q, k, v, oq, max_q, causal=form == "causal")
    return (out, lse) + tuple(binding.jfa_backward(q, k, v, out, do, lse, oq, max_q, causal=form == "causal"))


# few queries, few keys: no schedule; one built in the kernel; scheduler kernel, and a fixed deal of several rounds
@pytest.mark.parametrize("copies", [1, 10, 400])
@pytest.mark.parametrize("form", ["few queries", "few keys", "keys in shorter blocks", "causal, keys in shorter blocks"])
@pytest.mark.parametrize("D", [32, 64])
def test_two_wave_workgroups(D, form, copies):
    """64-row tiles do the same arithmetic in the same order as 128-row ones, which a large bound on the lengths selects and which
    the tests above hold to the oracle.  They take at most 64 rows against at most 256 in large batches, and the keys of a small
    backward at D = 64 with samples of up to 256 rows whose 128-row tiles could be more than 512 (two per compute unit)."""
    lq = lk = SHORT * copies
    if form.startswith("few"):
        lq, lk = [min(x, 64) for x in lq], ([200, 256, 129] + lk)[:len(lk)]
        lq, lk = (lq, lk) if form == "few queries" else (lk, lq)
    elif form.endswith("shorter blocks"):
        lq = lk = [256, 1, 130, 64, 0, 193, 65, 200] * (24 if copies == 1 else copies)   # 768 tiles of 128 rows at most, 1536 of 64
    mode = "causal" if form.startswith("causal") else "self" if form == "keys in shorter blocks" else "cross"
    got = everything(mode, D, lq, lk, max(lq), max(lk), 65 + D)
    ref = everything(mode, D, lq, lk, 4096, 4096, 65 + D)
    for name, g, r in zip(("out", "lse", "dq", "dk", "dv", "delta"), got, ref):
        assert torch.equal(g, r) and not bool(torch.isnan(g).any()), name
