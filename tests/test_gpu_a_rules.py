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


def _skewed(rng, N, hubs, hub_deg, deg):
    """Rows of up to ``deg`` random entries, the rows of every ``hubs``-th
    window of up to ``hub_deg``: a heavy-first list with both kinds of item."""
    rows = []
    for i in range(N):
        top = hub_deg if (i // 16) % hubs == 0 else deg
        rows.append(np.sort(rng.choice(N, size=int(rng.integers(1, top + 1)), replace=False)))
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    return rp, np.concatenate(rows).astype(np.int32)


# windows on either side of the waves' grouping: a last workgroup of one, two
# and three single-wave items; hub windows below and above the piece size
@pytest.mark.parametrize("N,hubs,hub_deg", [(16 * 61, 7, 300), (16 * 62 + 5, 9, 900),
                                            (16 * 150 + 1, 40, 1500)])
@pytest.mark.parametrize("H,d,dtype", [(1, 64, "f16"), (3, 32, "bf16"), (2, 128, "f16")])
def test_heavy_items_shared_by_four_waves(gpu, N, hubs, hub_deg, H, d, dtype, monkeypatch):
    """Heavy items shared by a workgroup's waves beside light ones of one wave
    each, forward and backward, against the oracle and one wave per item."""
    rng = np.random.default_rng(N + d)
    rp, ci = _skewed(rng, N, hubs, hub_deg, 6)
    t = torch.float16 if dtype == "f16" else torch.bfloat16
    Q, K, V, G = (torch.from_numpy(rng.standard_normal((N, H, d)).astype(np.float32)).to(t)
                  for _ in range(4))
    q, k, v, g = (x.cuda() for x in (Q, K, V, G))
    plan = gpu.Plan(_dev(rp), _dev(ci), N)
    plan_t = plan.transpose()
    i = plan.info
    assert i["max_blocks"] * i["n_items"] > 2 * i["n_blocks"]   # a skewed plan
    assert i["max_blocks"] > 8                                  # with items to share

    def both():
        O, lse = gpu.forward_typed(plan, q, k, v, scale=0.1, want_lse=True)
        return (O, lse) + gpu.backward(plan, plan_t, q, k, v, O, g, lse, scale=0.1)

    got = both()
    monkeypatch.setenv("F3S_WAVES_PER_ITEM", "1")
    one = both()
    monkeypatch.delenv("F3S_WAVES_PER_ITEM")
    # fp32 sums in another order: about sqrt(terms) roundings of 2^-24, and
    # 16-bit roundings of P and dS that may fall the other way (2^-11 / 2^-16)
    bound = 1e-3 if dtype == "f16" else 2e-5
    for a, b in zip(got, one):
        assert float((a - b).norm()) <= bound * float(b.norm())
    if dtype == "f16":
        for h in range(H):
            q1, k1, v1 = (x[:, h].numpy() for x in (Q, K, V))
            _check(got[0][:, h], oracle.attention_f64(rp, ci, q1, k1, v1, 0.1))
    # results and gradients of both types against fp64 (f16: probabilities and
    # score gradients in 11 bits; bf16: in two 8-bit terms)
    for h in range(H):
        ref = _attention_f64(rp, ci, *(x[:, h].double() for x in (q, k, v, g)), 0.1)
        for a, b in zip(got, ref):
            assert float((a[:, h] - b).norm()) <= (REL if dtype == "f16" else 2e-5) * float(b.norm())


def test_uniform_windows_stay_whole(gpu):
    """Windows of about the same size are not split for being a little above
    the mean; one far above it is."""
    rng = np.random.default_rng(3)
    N = 4096
    rows = [np.sort(rng.choice(N, size=90 + int(rng.integers(0, 8)), replace=False))
            for _ in range(N)]
    for heavy in (False, True):
        if heavy:
            for i in range(16):
                rows[i] = np.arange(N)
        rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
        ci = np.concatenate(rows).astype(np.int32)
        plan = gpu.Plan(_dev(rp), _dev(ci), N)
        assert plan.info["n_split"] == (1 if heavy else 0)
        Q, K, V = W.features(rng, N, 64)
        _check(gpu.run(plan, _dev(Q), _dev(K), _dev(V)),
               oracle.attention_f64(rp, ci, Q, K, V, 0.125))


@pytest.mark.parametrize("N,H,d,dtype", [(20479, 1, 64, "f16"), (20465, 3, 32, "f16"),
                                         (1280 * 16 + 1, 3, 32, "bf16"),
                                         (24000, 2, 128, "f16"), (8000, 2, 64, "bf16"),
                                         (12300, 2, 256, "f16"), (12100, 1, 32, "f16")])
def test_sequences_around_the_wave_and_order_rules(gpu, N, H, d, dtype):
    """Uniform windows around 1,280 of them (window order), and launches whose
    waves are about one per SIMD, one and a half, or leave their last round
    nearly empty: forward and gradients against the fp64 oracle."""
    rng = np.random.default_rng(N + d)
    far = rng.integers(0, N, size=(N, 6))
    band = np.arange(N)[:, None] + np.arange(-60, 60)
    rows = np.sort(np.concatenate([np.clip(band, 0, N - 1), far], 1), 1)
    keep = np.ones(rows.shape, dtype=bool)
    keep[:, 1:] = rows[:, 1:] != rows[:, :-1]
    rp = np.concatenate([[0], np.cumsum(keep.sum(1))]).astype(np.int32)
    ci = rows[keep].astype(np.int32)
    t = torch.float16 if dtype == "f16" else torch.bfloat16
    Q, K, V, G = (torch.from_numpy(rng.standard_normal((N, H, d)).astype(np.float32)).to(t)
                  for _ in range(4))
    q, k, v, g = (x.cuda() for x in (Q, K, V, G))
    plan = gpu.Plan(_dev(rp), _dev(ci), N)
    plan_t = plan.transpose()
    assert plan.info["n_split"] == 0
    assert bool(plan.info["flags"] & 1) == ((N + 15) // 16 >= 1280)
    O, lse = gpu.forward_typed(plan, q, k, v, scale=0.1, want_lse=True)
    grads = gpu.backward(plan, plan_t, q, k, v, O, g, lse, scale=0.1)
    h = H - 1
    qh, kh, vh, gh = (x[:, h].float().double().cuda() for x in (Q, K, V, G))
    want = _attention_f64(rp, ci, qh, kh, vh, gh, 0.1)
    for got, ref in zip((O, lse) + grads, want):
        ref = ref.cpu().numpy()
        bar = REL if dtype == "f16" else 2e-5  # two bf16 terms: 2^-17 each
        got = got[:, h].double().cpu().numpy()
        assert np.linalg.norm(got - ref) <= bar * np.linalg.norm(ref)


def _attention_f64(rp, ci, q, k, v, g, scale):
    """O, lse, dQ, dK, dV of one head, entry by entry in fp64."""
    N, d = q.shape
    dev = q.device
    rows = torch.repeat_interleave(torch.arange(N, device=dev),
                                   torch.from_numpy(np.diff(rp)).to(dev))
    cols = torch.from_numpy(ci).to(dev).long()

    def spread(to, w, X):
        return torch.zeros((N, d), dtype=torch.float64, device=dev).index_add_(
            0, to, X * w[:, None])

    x = (q[rows] * k[cols]).sum(1) * scale
    top = torch.full((N,), -float("inf"), dtype=torch.float64, device=dev)
    top = top.scatter_reduce(0, rows, x, "amax")
    p = torch.exp(x - top[rows])
    total = torch.zeros(N, dtype=torch.float64, device=dev).index_add_(0, rows, p)
    p = p / total[rows]
    O = spread(rows, p, v[cols])
    ds = p * ((g[rows] * v[cols]).sum(1) - (g * O).sum(1)[rows]) * scale
    return (O, top + torch.log(total), spread(rows, ds, k[cols]), spread(cols, ds, q[rows]),
            spread(cols, p, g[rows]))


# windows on either side of what one workgroup shapes and sorts (1,024,
# 4,096, 8,192, 17,408 and 32,768 windows), of the digits the one-workgroup
# sort covers (pieces of 2,048 blocks), and of the per-window paths (64, 128,
# 256, 512, 1,024 and 4,096 entries)
@pytest.mark.parametrize("T,deg,hub", [(1023, 5, 40), (1025, 5, 0), (4097, 3, 900),
                                       (8193, 2, 0), (17409, 1, 300), (32769, 1, 70)])
@pytest.mark.parametrize("order", [None, "0", "1"])
def test_plan_shape_paths(gpu, T, deg, hub, order, monkeypatch):
    from test_gpu_1_plan import _check_plan_against_oracle as check_plan
    if order is not None:
        monkeypatch.setenv("F3S_NO_REORDER", order)
    rng = np.random.default_rng(T)
    N = 16 * T - 3
    counts = rng.integers(0, deg + 1, size=N)
    if hub:
        counts[rng.choice(N, size=24, replace=False)] = hub
    rp = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    ci = rng.integers(0, N, size=int(rp[-1])).astype(np.int32)
    check_plan(gpu, oracle, rp, ci, N)


@pytest.mark.parametrize("T", [64, 65, 1024, 1500, 8192, 16385, 20001])
def test_ranks_of_windows_with_few_distinct_keys(gpu, T):
    """Windows of zero to three blocks in any order, some keys absent from
    whole runs: equal keys within 64 windows, across them and across waves
    keep their window order, and every window has its item."""
    from test_gpu_1_plan import _check_plan_against_oracle as check_plan
    rng = np.random.default_rng(T)
    N = 16 * T
    counts = np.zeros(N, dtype=np.int64)
    counts[::16] = 16 * rng.integers(0, 4, size=T)
    counts[:16 * (T // 4)] //= 3
    counts[16 * (T // 2):16 * (T // 2 + 70):16] = 40
    counts = np.minimum(counts, N)
    rp = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    ci = rng.integers(0, N, size=int(rp[-1])).astype(np.int32)
    check_plan(gpu, oracle, rp, ci, N)


def test_plan_with_pieces_beyond_the_one_workgroup_sort(gpu, monkeypatch):
    from test_gpu_1_plan import _check_plan_against_oracle as check_plan
    rng = np.random.default_rng(1)
    N = 40000
    counts = np.full(N, 2)
    counts[:16] = 39000         # one window of 2,500 blocks
    counts[64:80] = 3000
    rows = [np.sort(rng.choice(N, size=c, replace=False)) for c in counts]
    rp = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    ci = np.concatenate(rows).astype(np.int32)
    for piece in ("2300", "2046", "2048"):
        monkeypatch.setenv("F3S_PIECE_BLOCKS", piece)
        check_plan(gpu, oracle, rp, ci, N)


@pytest.mark.parametrize("n", [64, 65, 128, 129, 256, 257, 512, 513, 1024, 1025, 4096, 4097])
def test_window_entry_classes(gpu, n):
    """One window of n entries among small ones, duplicates included."""
    from test_gpu_1_plan import _check_plan_against_oracle as check_plan
    rng = np.random.default_rng(n)
    N = 300
    counts = np.full(N, 1)
    counts[32:48] = n // 16
    counts[47] += n % 16
    rp = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    ci = rng.integers(0, N, size=int(rp[-1])).astype(np.int32)
    check_plan(gpu, oracle, rp, ci, N)


def test_symmetry_of_patterns_that_differ_in_one_entry(gpu):
    """The transposed plan shares a symmetric pattern's arrays and builds its own
    when one entry, in a dense or a sparse block, lacks its mirror."""
    rng = np.random.default_rng(4)
    N = 530
    dense = rng.random((N, N)) < 0.02
    dense[:40, :40] = True
    dense |= dense.T
    for drop in (None, (3, 17), (39, 0), (529, int(np.flatnonzero(dense[529])[0]))):
        a = dense.copy()
        if drop:
            a[drop] = False
        ref = a.T
        rp = np.concatenate([[0], np.cumsum(a.sum(1))]).astype(np.int32)
        ci = np.nonzero(a)[1].astype(np.int32)
        plan = gpu.Plan(_dev(rp), _dev(ci), N)
        t = plan.transpose().export()
        win, mask, cols = t["blk_off"], t["mask"].reshape(-1, 8), t["cols"].reshape(-1, 16)
        got = np.zeros((N, N), dtype=bool)
        for w in range(len(win) - 1):
            for b in range(win[w], win[w + 1]):
                for k in range(256):
                    if (int(mask[b, k // 32]) >> (k % 32)) & 1:
                        q, r = k // 4, k % 4
                        got[16 * w + q % 16, cols[b, 4 * (q // 16) + r]] = True
        assert np.array_equal(got, ref)


def test_symmetric_plans_share_their_arrays(gpu):
    """Either of a plan and its transposed plan may be destroyed first."""
    rng = np.random.default_rng(6)
    N = 200
    m = rng.random((N, N)) < 0.1
    m |= m.T
    rp = np.concatenate([[0], np.cumsum(m.sum(1))]).astype(np.int32)
    ci = np.nonzero(m)[1].astype(np.int32)
    Q, K, V = W.features(rng, N, 32)
    q, k, v = _dev(Q), _dev(K), _dev(V)
    g = q.clone()
    for first in (True, False):
        plan = gpu.Plan(_dev(rp), _dev(ci), N)
        plan_t = plan.transpose()
        O, lse = gpu.forward(plan, q, k, v)
        want = gpu.backward(plan, plan_t, q, k, v, O, g, lse)
        second = plan.transpose()
        (plan_t if first else second).close()
        left = second if first else plan_t
        got = gpu.backward(plan, left, q, k, v, O, g, lse)
        assert all(torch.equal(a, b) for a, b in zip(got, want))
        plan.close()
        assert left.export()["cols"].min() >= -1
        left.close()


@pytest.mark.parametrize("N,H,d,dtype", [(9_000_000, 1, 128, "f16"), (16_777_213, 1, 128, "bf16"),
                                         (50_000, 88, 256, "f16")])
def test_rows_between_2_and_4_gib(gpu, N, H, d, dtype):
    """32-bit row offsets with the top bit set: a few rows attend to keys all
    over Q, K and V of 2.1 to 4 GiB each; outputs and gradients of these rows
    and keys against fp64, everything else zero."""
    t = torch.float16 if dtype == "f16" else torch.bfloat16
    size = 2 * N * H * d
    assert 2**31 < size <= 0xFFFFFFF0
    if torch.cuda.mem_get_info()[0] < 14 * size:
        pytest.skip("not enough device memory")
    rng = np.random.default_rng(N)
    rows = np.unique(np.concatenate([rng.integers(0, N, size=60), [0, N - 1, N // 2]]))
    cols = [np.unique(np.concatenate([rng.integers(0, N, size=12), [N - 1 - i % 7, i % 5]]))
            for i in range(len(rows))]
    counts = np.zeros(N, dtype=np.int64)
    counts[rows] = [len(c) for c in cols]
    rp = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    ci = np.concatenate(cols).astype(np.int32)
    shape = (N, d) if H == 1 else (N, H, d)
    gen = torch.Generator(device="cuda").manual_seed(N)
    q, k, v, g = (torch.randn(shape, generator=gen, device="cuda", dtype=t) for _ in range(4))
    plan = gpu.Plan(_dev(rp), _dev(ci), N)
    plan_t = plan.transpose()
    print("2 to 4 GiB", N, H, d, dtype, flush=True)
    O, lse = gpu.forward_typed(plan, q, k, v, scale=0.1, want_lse=True)
    dQ, dK, dV = gpu.backward(plan, plan_t, q, k, v, O, g, lse, scale=0.1)
    keys = np.unique(ci)
    r, c = torch.from_numpy(rows).cuda(), torch.from_numpy(keys).cuda()
    sub_rp = np.zeros(max(len(rows), len(keys)) + 1, dtype=np.int32)
    sub_rp[1:len(rows) + 1] = np.cumsum([len(x) for x in cols])
    sub_rp[len(rows) + 1:] = sub_rp[len(rows)]
    sub_ci = np.searchsorted(keys, ci).astype(np.int32)
    n = len(sub_rp) - 1

    def part(x, ids, h):
        out = torch.zeros((n, d), dtype=torch.float64, device="cuda")
        out[:len(ids)] = x.view(N, H, d)[ids, h].double()
        return out

    bar = REL if dtype == "f16" else 2e-5
    for h in sorted({0, H // 2, H - 1}):
        want = _attention_f64(sub_rp, sub_ci, part(q, r, h), part(k, c, h), part(v, c, h),
                              part(g, r, h), 0.1)
        for got, ids, ref in ((O, r, want[0]), (dQ, r, want[2]), (dK, c, want[3]),
                              (dV, c, want[4])):
            x = got.view(N, H, d)[ids, h].double()
            ref = ref[:len(ids)]
            assert float((x - ref).norm()) <= bar * float(ref.norm())
        x = lse.view(N, H)[r, h].double()
        assert float((x - want[1][:len(rows)]).abs().max()) <= 1e-3
    for got, ids in ((O, r), (dQ, r), (dK, c), (dV, c)):
        got[ids] = 0
        assert not got.any()
