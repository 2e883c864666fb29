"""The calls that a user of this library makes, as cases to be timed.

A case is one call (or the refresh + top-k pair of one step) of
paper_1506_03872_amd on GPU-resident inputs:

* ``oneshot``    -- ``topk(A, B, ...)``: plan, sample, verify, release.
* ``dense``      -- a step on a kept dense plan: ``refresh`` (the inputs
                    changed) and ``topk_raw``.
* ``sparse``     -- the same on a kept CSR plan of unchanged sparsity.
* ``sparse_new`` -- a CSR plan made from new inputs, one top-k, release.
* ``bf``         -- ``bruteforce_topk``: the exact answer on dense inputs.
* ``bf_csr``     -- ``bruteforce_topk_csr``: the exact answer on sparse ones.
* ``mips``       -- ``batch_raw`` on a kept database plan: a batch of queries
                    with a sample budget each.

Sizes are those of the library's own workloads (dense 1000 x 1000 x 64,
1e5 x 1e5 x 100 and 1e5 x 1e6 x 256, sparse 1e6 x 1e6 over 1e5 coordinates,
a MIPS batch of 4096 queries on 1e6 x 128) and the rating-factor sizes
65,133 x 71,567 x 150 of the paper's dense experiments.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1506_03872_amd as mad

PRECISIONS = {"fp32": mad.MAD_FP32, "bf16": mad.MAD_BF16,
              "fp8": mad.MAD_FP8_E4M3}


def listed():
    return [
        # The smallest one-shot call: 1000 x 1000 vectors, everything from
        # plan to result; launches, allocations and latency count.
        dict(name="oneshot_1k", kind="oneshot", m=1000, n=1000, d=64,
             s=100_000, tp=100, t=10),
        # Online serving: a handful of queries against the movie factors of
        # a rating matrix with the small budgets of the paper's MIPS runs
        # (64 to 512 samples per query, t' = s, top 10).
        dict(name="mips_online", kind="mips", m=65_133, d=150, nq=16,
             s_lo=64.0, s_hi=512.0, t=10, precision="fp32"),
        # The benchmark's dense step: new vectors of a known shape, s = 1e7.
        dict(name="dense_100k", kind="dense", m=100_000, n=100_000, d=100,
             s=10_000_000, tp=10_000, t=100, precision="fp32", check=False,
             decay=0.0, planted=50),
        # Rating factors of odd sizes (movies x users, d = 150, decaying
        # spectrum), inputs checked, bf16 screen before the verification of
        # many candidates, more results.
        dict(name="dense_factors", kind="dense", m=65_133, n=71_567, d=150,
             s=10_000_000, tp=100_000, t=1000, precision="bf16", check=True,
             decay=0.5, planted=0),
        # The largest dense step: a long sampling run (more than one
        # ordering chunk) on 1e5 x 1e6 vectors of 256 coordinates.
        dict(name="dense_1m", kind="dense", m=100_000, n=1_000_000, d=256,
             s=300_000_000, tp=200_000, t=1000, precision="fp32", check=False,
             decay=0.0, planted=1000),
        # Item-item similarity of a new sparse rating matrix (A^T A, Gram
        # scores): the plan is made for one question and thrown away.
        dict(name="sparse_new_50k", kind="sparse_new", variant="gram",
             m=50_000, n=50_000, d=100_000, nnz=20, s=10_000_000,
             tp=100_000, t=1000),
        # The sparse step at full size: new values of a known sparsity.
        dict(name="sparse_1m", kind="sparse", m=1_000_000, n=1_000_000,
             d=100_000, nnz=20, s=100_000_000, tp=100_000, t=1000),
        # Exact answers: fp32 on the rating factors ...
        dict(name="bf_fp32_factors", kind="bf", m=65_133, n=71_567, d=150,
             precision="fp32", t=1000, t_screen=0, decay=0.5, planted=0),
        # ... bf16 with the certified bound at the largest dense size ...
        dict(name="bf_bf16_1m", kind="bf", m=100_000, n=1_000_000, d=256,
             precision="bf16", t=1000, t_screen=0, decay=0.0, planted=1000),
        # ... and fp8 screening (20 t values re-ranked) at the benchmark's.
        dict(name="bf_fp8_100k", kind="bf", m=100_000, n=100_000, d=100,
             precision="fp8", t=100, t_screen=2000, decay=0.0, planted=50),
        # The exact sparse answer, heavy coordinates filtered in bf16.
        dict(name="bf_csr_30k", kind="bf_csr", m=30_000, n=30_000, d=100_000,
             nnz=20, precision="bf16", t=1000),
        # The large MIPS batch: 4096 queries, uneven budgets 1e3 to 1e5.
        dict(name="mips_4096", kind="mips", m=1_000_000, d=128, nq=4096,
             s_lo=1e3, s_hi=1e5, t=10, precision="fp32"),
    ]


def _size(rng, lo, hi):
    """A whole number, spread over the logarithm of [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(
        rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["oneshot", "dense", "dense", "sparse", "sparse_new",
                       "bf", "bf", "bf_csr", "mips", "mips"])
    if kind == "oneshot":
        t = _size(rng, 1, 100)
        return dict(kind=kind, m=_size(rng, 300, 20_000),
                    n=_size(rng, 300, 20_000), d=_size(rng, 8, 256),
                    s=_size(rng, 10_000, 2_000_000),
                    tp=_size(rng, t, 10_000), t=t)
    if kind == "dense":
        t = _size(rng, 10, 1000)
        return dict(kind=kind, m=_size(rng, 2_000, 100_000),
                    n=_size(rng, 2_000, 500_000), d=_size(rng, 16, 256),
                    s=_size(rng, 200_000, 100_000_000),
                    tp=_size(rng, t, 100_000), t=t,
                    precision=rng.choice(["fp32", "fp32", "bf16", "fp8"]),
                    check=rng.random() < 0.5, decay=rng.choice([0.0, 0.5]),
                    planted=rng.choice([0, 50]))
    if kind in ("sparse", "sparse_new"):
        t = _size(rng, 10, 1000)
        gram = rng.random() < 0.5
        m = _size(rng, 5_000, 500_000 if kind == "sparse" else 100_000)
        n = m if gram else _size(rng, 5_000, m)
        c = dict(kind=kind, variant="gram" if gram else "plain", m=m, n=n,
                 d=_size(rng, 2_000, 100_000), nnz=rng.randint(5, 24),
                 s=_size(rng, 500_000,
                         50_000_000 if kind == "sparse" else 20_000_000),
                 tp=_size(rng, t, 100_000), t=t)
        return c
    if kind == "bf":
        p = rng.choice(["fp32", "bf16", "fp8"])
        t = _size(rng, 10, 1000)
        return dict(kind=kind, m=_size(rng, 1_000, 100_000),
                    n=_size(rng, 1_000, 100_000), d=_size(rng, 16, 256),
                    precision=p, t=t,
                    t_screen=0 if p == "fp32" or
                    (p == "bf16" and rng.random() < 0.5) else 20 * t,
                    decay=rng.choice([0.0, 0.5]),
                    planted=rng.choice([0, 50]))
    if kind == "bf_csr":
        return dict(kind=kind, m=_size(rng, 3_000, 40_000),
                    n=_size(rng, 3_000, 40_000), d=_size(rng, 2_000, 100_000),
                    nnz=rng.randint(5, 24),
                    precision=rng.choice(["fp32", "bf16"]),
                    t=_size(rng, 10, 1000))
    lo = 10.0 ** rng.uniform(1.5, 3.0)
    return dict(kind="mips", m=_size(rng, 10_000, 1_000_000),
                d=_size(rng, 16, 160), nq=_size(rng, 1, 2048), s_lo=lo,
                s_hi=lo * 10.0 ** rng.uniform(0.2, 2.0), t=10,
                precision=rng.choice(["fp32", "fp32", "bf16"]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed, role):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 16 + role)
    return g


def _dense_inputs(case, seed):
    """A (m x d), B (n x d) N(0,1); with ``decay`` > 0 coordinate k is
    scaled by (k + 1)^-decay (factors ordered by their singular values);
    ``planted`` pairs get a_i . b_j = 8 to 10 sqrt(d)."""
    m, n, d = case["m"], case["n"], case["d"]
    A = torch.randn(m, d, generator=_gen(seed, 0), device="cuda")
    B = torch.randn(n, d, generator=_gen(seed, 1), device="cuda")
    if case.get("decay", 0.0):
        k = torch.arange(1, d + 1, device="cuda", dtype=torch.float32)
        A *= k ** -case["decay"]
        B *= k ** -case["decay"]
    p = min(case.get("planted", 0), m, n)
    if p:
        g = _gen(seed, 2)
        ii = torch.randperm(m, generator=g, device="cuda")[:p]
        jj = torch.randperm(n, generator=g, device="cuda")[:p]
        want = (8.0 + 2.0 * torch.rand(p, generator=g, device="cuda"))
        want *= math.sqrt(d)
        a, b = A[ii], B[jj]
        lam = (want - (a * b).sum(1)) / (a * a).sum(1)
        B[jj] = b + lam[:, None] * a
    return A, B


def _sparse_side(rows, d, nnz, seed, role):
    """CSR of ``rows`` vectors: coordinates are the first ``nnz`` distinct
    ones of a run of Zipf(1.5) draws over [0, d) (fewer when the run holds
    fewer), through a permutation of the coordinates; lognormal(0,1) values
    with random signs."""
    g = _gen(seed, role)
    perm = torch.randperm(d, generator=_gen(seed, 15), device="cuda")
    p = torch.arange(1, d + 1, device="cuda", dtype=torch.float64) ** -1.5
    cdf = torch.cumsum(p, 0)
    cdf /= cdf[-1].clone()
    width, counts, cols = 12 * nnz, [], []
    for r0 in range(0, rows, 1 << 17):
        r = min(1 << 17, rows - r0)
        u = torch.rand(r, width, generator=g, device="cuda",
                       dtype=torch.float64)
        z = torch.searchsorted(cdf, u).clamp_(max=d - 1)
        # first occurrence of each value, in draw order
        zs, order = torch.sort(z, dim=1, stable=True)
        first = torch.ones_like(zs, dtype=torch.bool)
        first[:, 1:] = zs[:, 1:] != zs[:, :-1]
        keep = torch.zeros_like(first).scatter_(1, order, first)
        keep &= torch.cumsum(keep, 1) <= nnz
        c = torch.where(keep, perm[z], d).sort(dim=1).values[:, :nnz]
        live = c < d
        counts.append(live.sum(1))
        cols.append(c[live].to(torch.int32))
    ptr = torch.zeros(rows + 1, dtype=torch.int64, device="cuda")
    ptr[1:] = torch.cumsum(torch.cat(counts), 0)
    idx = torch.cat(cols)
    val = torch.randn(idx.numel(), generator=g, device="cuda").exp_()
    sign = torch.rand(idx.numel(), generator=g, device="cuda") < 0.5
    return ptr, idx, torch.where(sign, -val, val)


def _sparse_inputs(case, seed):
    a = _sparse_side(case["m"], case["d"], case["nnz"], seed, 0)
    if case.get("variant") == "gram":
        return a, a
    return a, _sparse_side(case["n"], case["d"], case["nnz"], seed, 1)


def _budgets(case, seed):
    e = np.random.default_rng([5, int(seed)]).uniform(
        math.log10(case["s_lo"]), math.log10(case["s_hi"]), size=case["nq"])
    return np.round(10.0 ** e).astype(np.int64)


def _out(rows):
    return (torch.zeros((rows, 3), dtype=torch.int64, device="cuda"),
            torch.zeros(1, dtype=torch.int64, device="cuda"))


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case, seed=int(seed) & 0xffff)
    if kind in ("oneshot", "dense", "bf"):
        st["A"], st["B"] = _dense_inputs(case, seed)
    elif kind in ("sparse", "sparse_new", "bf_csr"):
        st["a"], st["b"] = _sparse_inputs(case, seed)
    flags = mad.MAD_FLAG_GRAM if case.get("variant") == "gram" else 0
    if kind == "dense":
        if not case["check"]:
            flags |= mad.MAD_FLAG_NO_CHECK
        st["plan"] = mad.Plan.dense(st["A"], st["B"], flags=flags)
        if case["precision"] != "fp32":
            st["plan"].set_verify_precision(PRECISIONS[case["precision"]])
    elif kind == "sparse":
        # the structure was checked once; each step brings new values
        st["plan"] = mad.Plan.csr(st["a"], st["b"], case["m"], case["n"],
                                  case["d"],
                                  flags=flags | mad.MAD_FLAG_NO_CHECK)
    elif kind == "sparse_new":
        st["flags"] = flags
    elif kind == "mips":
        A = torch.randn(case["m"], case["d"], generator=_gen(seed, 0),
                        device="cuda")
        st["Q"] = torch.randn(case["nq"], case["d"], generator=_gen(seed, 1),
                              device="cuda")
        st["s"] = _budgets(case, seed)
        st["tp"] = np.maximum(st["s"], case["t"])
        st["plan"] = mad.MipsPlan.create(A)
        if case["precision"] != "fp32":
            st["plan"].set_verify_precision(PRECISIONS[case["precision"]])
        st["out"] = _out(case["nq"] * case["t"])[0]
        st["n_out"] = torch.zeros(case["nq"], dtype=torch.int64,
                                  device="cuda")
    if kind in ("dense", "sparse"):
        st["out"], st["n_out"] = _out(case["t"])
    return st


def _records(out, n_out):
    """The mad_pair records as i, j and (c, x), without waiting for them."""
    return dict(i=out[:, 0], j=out[:, 1],
                cx=out.view(torch.float32)[:, 4:6], n=n_out)


def run(state):
    c, kind = state["case"], state["case"]["kind"]
    if kind == "oneshot":
        return mad.topk(state["A"], state["B"], c["t"], c["s"], c["tp"],
                        seed=state["seed"])
    if kind in ("dense", "sparse"):
        plan = state["plan"]
        plan.refresh()
        plan.topk_raw(c["t"], c["s"], c["tp"], state["seed"], state["out"],
                      state["n_out"])
        return _records(state["out"], state["n_out"])
    if kind == "sparse_new":
        plan = mad.Plan.csr(state["a"], state["b"], c["m"], c["n"], c["d"],
                            flags=state["flags"])
        r = plan.topk(c["t"], c["s"], c["tp"], seed=state["seed"])
        plan.close()
        return r
    if kind == "bf":
        r, _ = mad.bruteforce_topk(state["A"], state["B"], c["t"],
                                   precision=PRECISIONS[c["precision"]],
                                   t_screen=c["t_screen"])
        return dict(i=r["i"], j=r["j"], c=r["c"])
    if kind == "bf_csr":
        r, _ = mad.bruteforce_topk_csr(state["a"], state["b"], c["m"],
                                       c["n"], c["d"], c["t"],
                                       precision=PRECISIONS[c["precision"]])
        return dict(i=r["i"], j=r["j"], c=r["c"])
    state["plan"].batch_raw(state["Q"], state["s"], state["tp"], c["t"],
                            state["seed"], state["out"], state["n_out"])
    return _records(state["out"], state["n_out"])


# ---------------------------------------------------------------------------
# what a pass cannot do without, and exact answers
# ---------------------------------------------------------------------------
def work(case):
    """Inputs read once, results written once; a sample reads three table
    entries of 8 bytes and a 4-byte fourth edge; verification multiplies
    the rows of the candidates; the exact answer multiplies every pair."""
    kind, t = case["kind"], case["t"]
    if kind in ("oneshot", "dense"):
        m, n, d = case["m"], case["n"], case["d"]
        return {"bytes": 4.0 * (m + n) * d + 28.0 * case["s"] + 24.0 * t,
                "flops": 2.0 * case["tp"] * d}
    if kind in ("sparse", "sparse_new"):
        sides = 1 if case.get("variant") == "gram" else 2
        nnz = (case["m"] + (case["n"] if sides == 2 else 0)) * case["nnz"]
        return {"bytes": 8.0 * nnz + 28.0 * case["s"] + 24.0 * t,
                "flops": 2.0 * case["tp"] * case["nnz"]}
    if kind == "bf":
        m, n, d = case["m"], case["n"], case["d"]
        return {"bytes": 4.0 * (m + n) * d + 24.0 * t,
                "flops": 2.0 * m * n * d}
    if kind == "bf_csr":
        # wedges: pairs of entries that share a coordinate
        p = np.arange(1, case["d"] + 1, dtype=np.float64) ** -1.5
        p /= p.sum()
        share = 1.0 - np.exp(-p * 4.0 * case["nnz"])  # P(vector holds k)
        share *= case["nnz"] / share.sum()
        share = np.minimum(share, 1.0)
        return {"bytes": 8.0 * (case["m"] + case["n"]) * case["nnz"] +
                24.0 * t,
                "flops": 2.0 * case["m"] * case["n"] * float(
                    (share * share).sum())}
    mean = (case["s_hi"] - case["s_lo"]) / math.log(case["s_hi"] /
                                                    case["s_lo"])
    s = case["nq"] * mean
    # three words of a sample, and the row of each candidate (t' = s)
    return {"bytes": 20.0 * s + 4.0 * case["nq"] * case["d"] +
            4.0 * case["d"] * min(s, case["m"]),
            "flops": 2.0 * s * case["d"]}


def _exact_top(blocks, t):
    """The t largest |c| (descending, with their signs) over blocks of FP64
    products."""
    best = torch.empty(0, dtype=torch.float64, device="cuda")
    for block in blocks:
        flat = block.reshape(-1)
        if best.numel() == t:
            flat = flat[flat.abs() >= best[-1].abs()]
        best = torch.cat([best, flat])
        best = best[torch.topk(best.abs(), min(t, best.numel())).indices]
    return best


def exact(case, seed):
    """Exhaustive products in 64 bits for the exact answers.  The sampled
    calls have none: which pairs they return, and their scores, are a
    function of the random stream."""
    kind = case["kind"]
    if kind == "bf":
        m, n, d = case["m"], case["n"], case["d"]
        if m * n * d > 3e13:
            return None
        A, B = _dense_inputs(case, seed)
        B = B.double().t().contiguous()
        step = max(1, 200_000_000 // n)
        return dict(i=None, j=None, c=_exact_top(
            (A[r:r + step].double() @ B for r in range(0, m, step)),
            case["t"]))
    if kind == "bf_csr":
        m, n, d = case["m"], case["n"], case["d"]
        a, b = _sparse_inputs(case, seed)
        used, inv = torch.unique(torch.cat([a[1], b[1]]),
                                 return_inverse=True)
        if m * n * used.numel() > 6e13:
            return None
        dense = []
        for (ptr, idx, val), col, rows in (
                (a, inv[:a[1].numel()], m), (b, inv[a[1].numel():], n)):
            X = torch.zeros(rows, used.numel(), dtype=torch.float64,
                            device="cuda")
            r = torch.repeat_interleave(
                torch.arange(rows, device="cuda"), ptr[1:] - ptr[:-1])
            X[r, col] = val.double()
            dense.append(X)
        Bt = dense[1].t().contiguous()
        step = max(1, 200_000_000 // n)
        return dict(i=None, j=None, c=_exact_top(
            (dense[0][r:r + step] @ Bt for r in range(0, m, step)),
            case["t"]))
    return None
