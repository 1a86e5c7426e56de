"""fp32 attention where scores are large: queries and keys of standard deviation 4, so that scaled scores have standard
deviation 16 and a relative error e of a score is an error of up to 70 e of its probability.

The bound is the error of the same formulas evaluated on the host with every score, difference and probability rounded to
fp32 (scores as four chains of D / 4 sequential additions) and everything behind the probabilities in fp64, on the same
inputs: the 2-norm of the GPU's error may be 1.25 times that one (the two round at different places, so that the errors are
two samples of one distribution; products are rounded by themselves here and not on the GPU) plus 6e-7 for the sums behind
the probabilities, which the host does not round (measured alone, at scores of standard deviation 1: 2.5e-7 to 4.3e-7).
"""
import numpy as np
import pytest
import torch

from paper_2409_15373_amd.synthetic import offsets_from_lengths

pytestmark = pytest.mark.gpu
f32 = np.float32
LQ, LK, H = [200, 64, 33, 150, 1], [150, 70, 200, 31, 40], 2


def chained(a, b):
    """a b^T of fp32 arrays in four chains of D / 4, every product and sum rounded to fp32."""
    D = a.shape[1]
    total = None
    for c in range(4):
        chain = np.zeros((a.shape[0], b.shape[0]), dtype=f32)
        for d in range(c * D // 4, (c + 1) * D // 4):
            chain = chain + a[:, d, None] * b[None, :, d]
        total = chain if total is None else total + chain
    return total


def evaluate(q, k, v, do, causal, rounded):
    """out, dq, dk, dv of one sample and head; rounded: scores, differences and probabilities in fp32, else all in fp64."""
    D = q.shape[1]
    r = (lambda x: np.asarray(x, dtype=f32).astype(np.float64)) if rounded else (lambda x: x)
    product = (lambda a, b: chained(a, b).astype(np.float64)) if rounded else (lambda a, b: a.astype(np.float64) @ b.astype(np.float64).T)
    scale = float(r(1.0 / np.sqrt(np.float64(D))))
    q64, k64, v64, do64 = (x.astype(np.float64) for x in (q, k, v, do))
    s = product(q, k)
    if causal:
        s[np.triu_indices(s.shape[0], 1, s.shape[1])] = -np.inf
    m = r(s.max(axis=1, keepdims=True) * scale)
    p = r(np.exp(r(s * scale - m)))
    l = p.sum(axis=1, keepdims=True)
    out = r(p @ v64 / l)
    p = r(np.exp(r(s * scale - r(m + np.log(l)))))
    ds = r(p * r(product(do, v) - r((do64 * out).sum(axis=1, keepdims=True))))
    return out, ds @ k64 * scale, ds.T @ q64 * scale, p.T @ do64


@pytest.mark.parametrize("mode", ["self", "causal", "cross"])
@pytest.mark.parametrize("D", [32, 64, 128])
def test_error_is_that_of_fp32_scores(D, mode):
    from paper_2409_15373_amd import binding
    rng = np.random.default_rng(D)
    oq = offsets_from_lengths(np.array(LQ))
    ok = offsets_from_lengths(np.array(LK)) if mode == "cross" else oq
    draw = lambda n, sigma: (rng.standard_normal((int(n), H, D)) * sigma).astype(f32)
    q, do, k, v = draw(oq[-1], 4.0), draw(oq[-1], 1.0), draw(ok[-1], 4.0), draw(ok[-1], 1.0)
    qd, kd, vd, dod, oqd, okd = (torch.from_numpy(x).cuda() for x in (q, k, v, do, oq, ok))
    if mode == "cross":
        out, lse = binding.jfa_forward_cross(qd, kd, vd, oqd, okd, 200, 200)
        grads = binding.jfa_backward_cross(qd, kd, vd, out, dod, lse, oqd, okd, 200, 200)
    else:
        out, lse = binding.jfa_forward(qd, kd, vd, oqd, 200, causal=mode == "causal")
        grads = binding.jfa_backward(qd, kd, vd, out, dod, lse, oqd, 200, causal=mode == "causal")
    got = [x.double().cpu().numpy() for x in (out,) + grads[:3]]
    exact, plain = ([np.empty(x.shape) for x in got] for _ in range(2))
    for b in range(len(LQ)):
        rq, rk = slice(oq[b], oq[b + 1]), slice(ok[b], ok[b + 1])
        for h in range(H):
            for dest, rounded in ((exact, False), (plain, True)):
                res = evaluate(q[rq, h], k[rk, h], v[rk, h], do[rq, h], mode == "causal", rounded)
                for x, y, rows in zip(dest, res, (rq, rq, rk, rk)):
                    x[rows, h] = y
    norm = np.linalg.norm
    for name, g, e, p in zip(("out", "dq", "dk", "dv"), got, exact, plain):
        error, bound = norm(g - e) / norm(e), 1.25 * norm(p - e) / norm(e) + 6e-7
        print(f"{mode} D {D} {name}: {error:.2e}, bound {bound:.2e}", flush=True)
        assert error <= bound, f"{name}: {error:.2e} > {bound:.2e}"
