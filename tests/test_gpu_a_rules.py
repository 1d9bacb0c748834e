"""Edges of the kernels' internal rules, each against the fp64 oracle: the
sign and zero of the scale, rows whose entries come late in their window,
masked scores that overflow."""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_08098_amd import workloads as W

pytestmark = pytest.mark.gpu

# fp16 probabilities: rounding 2^-11 each, the parity bar of the forward tests
MAX_ABS, REL = 5e-3, 1e-3


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _check(got, ref):
    got = got.double().cpu().numpy()
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= MAX_ABS * max(1.0, np.abs(ref).max())
    assert np.linalg.norm(got - ref) <= REL * np.linalg.norm(ref)


@pytest.mark.parametrize("scale", [-0.125, 0.0, -0.0, 3.0, 1e-30])
@pytest.mark.parametrize("d,N,deg", [(64, 77, 40), (32, 16, 3), (96, 600, 400), (256, 33, 17)])
def test_any_scale(gpu, scale, d, N, deg):
    rng = np.random.default_rng(d + N)
    rp, ci = W.random_csr(rng, N, deg, empty_frac=0.1)
    Q, K, V = W.features(rng, N, d)
    plan = gpu.Plan(_dev(rp), _dev(ci), N)
    O, lse = gpu.forward(plan, _dev(Q), _dev(K), _dev(V), scale=scale)
    _check(O, oracle.attention_f64(rp, ci, Q, K, V, scale))
    deg_row = np.array([len(set(ci[rp[i]:rp[i + 1]])) for i in range(N)])
    if abs(scale) < 1e-20:
        want = np.log(np.where(deg_row > 0, deg_row, 1))
        got = lse.cpu().numpy()
        assert np.allclose(got[deg_row > 0], want[deg_row > 0], atol=1e-5)
    assert (lse.cpu().numpy()[deg_row == 0] == -np.inf).all()


def test_rows_that_start_late_and_maxima_that_grow(gpu):
    """Row r of a window has entries from column block r on only, and its
    scores grow along the row, so every pair moves some row's maximum."""
    N, d = 512, 64
    rng = np.random.default_rng(5)
    rows = [np.arange(16 * (i % 16), N, dtype=np.int32) for i in range(N)]
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    ci = np.concatenate(rows).astype(np.int32)
    Q, K, V = W.features(rng, N, d)
    Q[:, 0] = 4.0
    K[:, 0] = np.linspace(-60, 60, N).astype(np.float16)
    plan = gpu.Plan(_dev(rp), _dev(ci), N)
    _check(gpu.run(plan, _dev(Q), _dev(K), _dev(V), scale=1.0),
           oracle.attention_f64(rp, ci, Q, K, V, 1.0))


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_masked_overflow_stays_with_its_row(gpu, dtype):
    """Scores of key 3 overflow for every query but only row 3 attends to it:
    the other rows of its window do not see them."""
    N, d = 48, 64
    rng = np.random.default_rng(9)
    rows = [np.array([j for j in range(N) if j != 3], dtype=np.int32) for _ in range(N)]
    rows[3] = np.arange(N, dtype=np.int32)
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    ci = np.concatenate(rows).astype(np.int32)
    Q, K, V = (torch.from_numpy(rng.standard_normal((N, d)).astype(np.float32)) for _ in range(3))
    big = float("inf") if dtype == "f16" else 3e38
    K[3] = big
    t = torch.float16 if dtype == "f16" else torch.bfloat16
    Q, K, V = Q.to(t), K.to(t), V.to(t)
    plan = gpu.Plan(_dev(rp), _dev(ci), N)
    O, _ = gpu.forward_typed(plan, Q.cuda(), K.cuda(), V.cuda(), scale=0.125)
    K[3] = 0
    keep = [i for i in range(N) if i != 3]
    rows[3] = np.zeros(0, dtype=np.int32)
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    ci = np.concatenate(rows).astype(np.int32)
    q, k, v = (x.double().numpy() for x in (Q, K, V))
    ref = oracle.attention_f64(rp, ci, q.astype(np.float16), k.astype(np.float16),
                               v.astype(np.float16), 0.125)
    if dtype == "bf16":
        ref = np.zeros((N, d))
        for i in keep:
            s = 0.125 * (k[rows[i]] @ q[i])
            p = np.exp(s - s.max())
            ref[i] = (p / p.sum()) @ v[rows[i]]
    _check(O[keep], ref[keep])
