"""The calls whose speed counts: sparse attention as programs use it.

Kinds of pattern (all drawn on the GPU from the seed alone):

er      a small undirected random graph, self-loops (a citation-sized graph)
mol     a batch of small molecule-like graphs, block-diagonal: every training
        step has a new one, so its plan is part of the step
cl      a Chung-Lu power-law graph, self-loops: hubs, uneven windows
seq     a token sequence: a local band plus random keys per query

Kinds of call:

forward  one attention layer on a graph whose plan is kept
train    forward with the log-sum-exp and backward, plans kept
fresh    forward on a graph seen for the first time: the plan is built first
step     a training step on a new batch: plan, forward, transposed plan,
         backward
"""
import math

import torch

import paper_2505_08098_amd as f3s

_TYPES = {"f16": torch.float16, "bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn}
_OUTS = {"f32": torch.float32, "f16": torch.float16}


def _case(name, call, kind, heads=1, d=64, dtype="f16", out="f32", **sizes):
    c = dict(call=call, kind=kind, heads=heads, d=d, dtype=dtype, out=out, **sizes)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # inference on one small graph: launch and latency, nothing else
        _case("er_1k_forward", "forward", "er", n=1021, degree=15.0),
        # full-batch training on a citation-sized graph with a layer's heads
        _case("er_2k7_train", "train", "er", n=2708, degree=4.0, heads=8),
        # a training step on a small batch of molecules, new graphs each step
        _case("mol_256_step", "step", "mol", graphs=256, segments=False, heads=4, d=32),
        # inference on a batch of ordinary size
        _case("mol_1024_forward", "forward", "mol", graphs=1024, segments=False),
        # a training step on a large batch of molecules, new graphs each step
        _case("mol_4096_step", "step", "mol", graphs=4096, segments=False),
        # a layer on a hub-heavy graph that the caches hold
        _case("cl21_64k_forward", "forward", "cl", n=65536, gamma=2.1, degree=20.0),
        # training on the same graph with several bfloat16 heads
        _case("cl21_64k_train", "train", "cl", n=65536, gamma=2.1, degree=20.0, heads=4,
              dtype="bf16"),
        # first inference on a graph of middle size: plan and one layer
        _case("cl25_256k_fresh", "fresh", "cl", n=262147, gamma=2.5, degree=16.0, d=128),
        # the large graph, where memory bandwidth counts
        _case("cl25_1m_forward", "forward", "cl", n=1048576, gamma=2.5, degree=16.0, d=128),
        # the same with 8-bit inputs and a 16-bit result
        _case("cl25_1m_fp8", "forward", "cl", n=1048576, gamma=2.5, degree=16.0, d=128,
              dtype="fp8", out="f16"),
        # inference over a long sequence with a layer's heads
        _case("seq_32k_forward", "forward", "seq", n=32768, band=256, rand=64, heads=8,
              dtype="bf16", out="f16"),
        # training over a sequence of odd length, larger heads
        _case("seq_16k_train", "train", "seq", n=16001, band=256, rand=64, heads=2, d=128),
    ]


# entries x heads x d of the listed case that takes longest; gradients count
# 2.5 times a forward pass, a sequence's entries (which share their rows of K
# and V) a quarter
_MOST = 1048576 * 17 * 128


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choice(("er", "mol", "cl", "seq"))
        call = rng.choice(("forward", "train", "step" if kind == "mol" else "fresh"))
        if kind == "er":
            sizes = dict(n=_log_int(rng, 500, 20000), degree=round(rng.uniform(3, 24), 1))
        elif kind == "mol":
            sizes = dict(graphs=_log_int(rng, 64, 8192), segments=rng.random() < 0.3)
        elif kind == "cl":
            sizes = dict(n=_log_int(rng, 10000, 1000000), gamma=round(rng.uniform(2.1, 2.7), 2),
                         degree=round(rng.uniform(8, 24), 1))
        else:
            sizes = dict(n=_log_int(rng, 2000, 65536), band=rng.choice((64, 128, 256, 512)),
                         rand=rng.choice((0, 16, 64)))
        dtype = rng.choice(("f16", "f16", "bf16", "fp8") if call in ("forward", "fresh")
                           else ("f16", "bf16"))
        out = rng.choice(("f32", "f32", "f16")) if call in ("forward", "fresh") else "f32"
        c = _case(None, call, kind, heads=rng.choice((1, 1, 2, 3, 4, 8)),
                  d=rng.choice((32, 64, 64, 96, 128, 160, 256)), dtype=dtype, out=out, **sizes)
        cost = _entries(c) * c["heads"] * c["d"] * (3.5 if call in ("train", "step") else 1)
        if cost * (0.25 if kind == "seq" else 1) <= _MOST:
            return c


# ---- patterns -----------------------------------------------------------------

def _mol_sizes(graphs):
    """Nodes of each graph of a batch: 15 to 45, the same number of each."""
    return 15 + torch.arange(graphs, dtype=torch.int64) % 31


def _rows(c):
    return int(_mol_sizes(c["graphs"]).sum()) if c["kind"] == "mol" else c["n"]


def _entries(c):
    """Entries of the pattern, as expected from its sizes."""
    N = _rows(c)
    if c["kind"] == "mol":
        return int(N * 3.1)
    if c["kind"] == "seq":
        return N * min(N, c["band"] + c["rand"])
    return int(N * (c["degree"] + 1))


def _csr(N, src, dst, loops=True, symmetric=True):
    if symmetric:
        src, dst = torch.cat([src, dst]), torch.cat([dst, src])
    if loops:
        ids = torch.arange(N, device=src.device)
        src, dst = torch.cat([src, ids]), torch.cat([dst, ids])
    key = torch.unique(src * N + dst)
    row_ptr = torch.zeros(N + 1, dtype=torch.int64, device=src.device)
    row_ptr[1:] = torch.cumsum(torch.bincount(key // N, minlength=N), 0)
    return row_ptr.to(torch.int32), (key % N).to(torch.int32)


def _pattern(c, gen):
    """(row_ptr, col_idx, graph offsets or None) on the GPU."""
    dev = gen.device
    N = _rows(c)

    def rand(n):
        return torch.rand(n, generator=gen, device=dev, dtype=torch.float64)

    if c["kind"] == "er":
        m = int(N * c["degree"] / 2)
        return _csr(N, (rand(m) * N).long(), (rand(m) * N).long()) + (None,)
    if c["kind"] == "mol":
        # a random tree per graph (each node hangs on an earlier one), and one
        # more edge for every tenth node
        G = c["graphs"]
        size = _mol_sizes(G).to(dev)[torch.argsort(rand(G))]
        seg = torch.zeros(G + 1, dtype=torch.int64, device=dev)
        seg[1:] = torch.cumsum(size, 0)
        first = torch.repeat_interleave(seg[:-1], size)
        ids = torch.arange(N, device=dev)
        tree = ids > first
        parent = first + (rand(N) * (ids - first)).long()
        other = first + (rand(N) * torch.repeat_interleave(size, size)).long()
        more = rand(N) < 0.1
        src = torch.cat([ids[tree], ids[more]])
        dst = torch.cat([parent[tree], other[more]])
        return _csr(N, src, dst) + (seg.to(torch.int32).cpu().numpy(),)
    if c["kind"] == "cl":
        # expected degrees from a power law capped at 4096, their mean set by
        # bisection; both ends of an edge drawn with these weights; node ids
        # sorted by degree below exponent 2.3, else permuted
        x = 1.0 - (torch.arange(N, device=dev, dtype=torch.float64) + 0.5) / N
        base = x ** (-1.0 / (c["gamma"] - 1.0))
        lo, hi = 1e-6, c["degree"]
        for _ in range(40):
            mid = 0.5 * (lo + hi)
            if float((mid * base).clamp_(max=4096.0).mean()) < c["degree"]:
                lo = mid
            else:
                hi = mid
        cdf = torch.cumsum((hi * base).clamp_(max=4096.0), 0)
        cdf /= cdf[-1].clone()
        m = int(N * c["degree"] / 2)
        a = torch.searchsorted(cdf, rand(m)).clamp_(max=N - 1)
        b = torch.searchsorted(cdf, rand(m)).clamp_(max=N - 1)
        if c["gamma"] >= 2.3:
            perm = torch.argsort(rand(N))
            a, b = perm[a], perm[b]
        return _csr(N, a, b) + (None,)
    # a token attends to the band around it and to random tokens
    ids = torch.arange(N, device=dev)[:, None]
    band = ids + torch.arange(-(c["band"] // 2), c["band"] - c["band"] // 2, device=dev)
    far = (rand(N * c["rand"]) * N).long().view(N, c["rand"])
    dst = torch.cat([band, far], 1)
    src = ids.expand_as(dst)
    ok = (dst >= 0) & (dst < N)
    return _csr(N, src[ok], dst[ok], loops=False, symmetric=False) + (None,)


def _inputs(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000003 * int(seed) + 17)
    row_ptr, col_idx, seg = _pattern(c, gen)
    N = len(row_ptr) - 1
    shape = (N, c["d"]) if c["heads"] == 1 else (N, c["heads"], c["d"])
    n = 4 if c["call"] in ("train", "step") else 3
    x = [torch.randn(shape, generator=gen, device="cuda").to(_TYPES[c["dtype"]])
         for _ in range(n)]
    return dict(N=N, row_ptr=row_ptr, col_idx=col_idx, seg=seg, Q=x[0], K=x[1], V=x[2],
                dO=x[3] if n == 4 else None)


def _plan(s):
    if s["case"].get("segments"):
        return f3s.Plan.segments(s["row_ptr"], s["col_idx"], s["N"], s["seg"])
    return f3s.Plan(s["row_ptr"], s["col_idx"], s["N"])


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    if case["call"] in ("forward", "train"):
        s["plan"] = _plan(s)
    if case["call"] == "train":
        s["plan_t"] = s["plan"].transpose()
    return s


# ---- one pass -------------------------------------------------------------------

def _forward(s, plan):
    c = s["case"]
    if c["dtype"] == "f16" and c["out"] == "f32":
        return f3s.run(plan, s["Q"], s["K"], s["V"])
    return f3s.forward_typed(plan, s["Q"], s["K"], s["V"], out_dtype=_OUTS[c["out"]])[0]


def _train(s, plan, plan_t):
    """plan_t: the transposed plan, or None where it is still to be built."""
    Q, K, V = s["Q"], s["K"], s["V"]
    if s["case"]["dtype"] == "f16":
        O, lse = f3s.forward(plan, Q, K, V)
    else:
        O, lse = f3s.forward_typed(plan, Q, K, V, want_lse=True)
    if plan_t is None:
        plan_t = plan.transpose()
    return (O, lse) + f3s.backward(plan, plan_t, Q, K, V, O, s["dO"], lse)


def run(state):
    call = state["case"]["call"]
    if call == "forward":
        return _forward(state, state["plan"])
    if call == "train":
        return _train(state, state["plan"], state["plan_t"])
    if call == "fresh":
        return _forward(state, _plan(state))
    return _train(state, _plan(state), None)


# ---- what a pass cannot do without ------------------------------------------------

def work(case):
    N, nnz = _rows(case), _entries(case)
    width = N * case["heads"] * case["d"]
    eb = 1 if case["dtype"] == "fp8" else 2
    ob = 2 if case["out"] == "f16" else 4
    # the pattern, Q, K and V in, O out
    nbytes = 4 * (N + 1) + 4 * nnz + 3 * width * eb + width * ob
    flops = 4 * nnz * case["heads"] * case["d"]
    if case["call"] in ("train", "step"):
        # lse out; dO in, dQ, dK and dV out
        nbytes += 4 * N * case["heads"] + width * eb + 3 * width * 4
        flops += 10 * nnz * case["heads"] * case["d"]
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Relative 2-norm, about four times what the path shows against 64 bits
    (forward, then with gradients): 0.9e-4 and 2.3e-4 where probabilities and
    score gradients are rounded to binary16 (binary16 and 8-bit inputs),
    1.1e-6 and 2.6e-6 where they are two bfloat16 terms, 2.3e-4 where the
    result is rounded to binary16.  "max": one value against the result's
    root mean square, whose tail is some tens of the 2-norm's figure."""
    if case["out"] == "f16":
        return {"rel": 1e-3, "max": 1e-2}
    if case["dtype"] == "bf16":
        return {"rel": 1.2e-5, "max": 5e-4}
    if case["call"] in ("train", "step"):
        return {"rel": 1e-3, "max": 2e-2}
    return {"rel": 4e-4, "max": 1e-2}


def exact(case, seed):
    """The same outputs from plain torch in 64 bits, entry by entry."""
    s = _inputs(case, seed)
    N, H, d = s["N"], case["heads"], case["d"]
    deg = (s["row_ptr"][1:] - s["row_ptr"][:-1]).long()
    rows = torch.repeat_interleave(torch.arange(N, device="cuda"), deg)
    cols = s["col_idx"].long()
    scale = 1.0 / math.sqrt(d)
    step = max(1, (1 << 27) // d)
    chunks = [slice(k, min(k + step, len(cols))) for k in range(0, len(cols), step)]
    train = case["call"] in ("train", "step")

    def products(A, B):  # A[row] . B[column] of every entry
        return torch.cat([(A[rows[k]] * B[cols[k]]).sum(-1) for k in chunks])

    def spread(to, frm, w, X):  # sum of w * X[frm] over the entries of each `to`
        out = torch.zeros((N, d), dtype=torch.float64, device="cuda")
        for k in chunks:
            out.index_add_(0, to[k], X[frm[k]] * w[k][:, None])
        return out

    outs = []
    for h in range(H):
        Q, K, V = (s[n].view(N, H, d)[:, h].float().double() for n in "QKV")
        x = products(Q, K) * scale
        top = torch.full((N,), -math.inf, dtype=torch.float64, device="cuda")
        top = top.scatter_reduce(0, rows, x, "amax")
        p = torch.exp(x - top[rows])
        total = torch.zeros(N, dtype=torch.float64, device="cuda").index_add_(0, rows, p)
        p = p / total[rows]
        O = spread(rows, cols, p, V)
        if not train:
            outs.append((O,))
            continue
        G = s["dO"].view(N, H, d)[:, h].float().double()
        ds = p * (products(G, V) - (G * O).sum(-1)[rows]) * scale
        outs.append((O, top + torch.log(total), spread(rows, cols, ds, K),
                     spread(cols, rows, ds, Q), spread(cols, rows, p, G)))
    whole = [o[0] if H == 1 else torch.stack(o, 1) for o in zip(*outs)]
    return tuple(whole) if train else whole[0]
