"""Cases by which the speed of the library is measured: what a training program has it do, over the range of sizes.

A case is one call (or one short sequence of calls) through the package's public entry points on seeded synthetic
inputs.  Four kinds:

  tree   one `grow_tree` call on fp32 derivatives that the caller computed (its own loss);
  boost  `iterations` calls of `boost_iteration` in a row, binary cross-entropy (derivatives, tree, score update);
  rank   the same with the lambdarank loss over queries of `group` rows;
  steps  one split done by hand with the step functions (quantize, build, search, partition, build the child,
         subtract, search both children, refit), as a program does that grows its trees by its own rules.

Inputs: the bins of independent features cut at their quantiles are uniform over 0..bins-1; ranking matrices are
mostly one default bin.  Labels depend on ten features, linearly and through interactions, with noise, and the scores
are those of a partly fitted model, so trees are as deep and as unbalanced as in the middle of a boosting run.
"""
from __future__ import annotations

import math

import torch

from paper_2207_09682_amd import binding as qb

SEED_SALT = 7919


def listed():
    return [
        # the smallest ordinary call: a small table, few leaves, the matrix used once and not bound; launches count
        dict(name="tree_10k_x28_15_leaves", kind="tree", rows=10_000, features=28, bins=63, bin_bytes=1, bits_g=2,
             bits_h=2, leaves=15, bound=False),
        # an ordinary table with an odd row and feature count
        dict(name="tree_100k_x50_31_leaves", kind="tree", rows=100_003, features=50, bins=255, bin_bytes=1, bits_g=4,
             bits_h=4, leaves=31, bound=True),
        # a boosting run on a table that the caches hold
        dict(name="boost_1m_x28", kind="boost", rows=1_000_000, features=28, bins=255, bin_bytes=1, bits_g=3, bits_h=3,
             leaves=255, bound=True, iterations=3),
        # the headline workload of the benchmark: many rows, few features
        dict(name="tree_10m5_x28", kind="tree", rows=10_500_000, features=28, bins=255, bin_bytes=1, bits_g=3, bits_h=3,
             leaves=255, bound=True),
        # one tree on a matrix that is not bound (rows are kept in leaf order), wider gradients
        dict(name="tree_2m5_x28_unbound_5bit", kind="tree", rows=2_500_003, features=28, bins=255, bin_bytes=1, bits_g=5,
             bits_h=5, leaves=127, bound=False),
        # squared error: constant hessians, a feature count that is no multiple of four
        dict(name="tree_464k_x90_l2", kind="tree", rows=463_715, features=90, bins=255, bin_bytes=1, bits_g=3, bits_h=0,
             leaves=255, bound=True),
        # few rows, many features
        dict(name="tree_400k_x2000", kind="tree", rows=400_000, features=2000, bins=63, bin_bytes=1, bits_g=3, bits_h=3,
             leaves=63, bound=True),
        # 16-bit bins
        dict(name="tree_2m_x40_600_bins", kind="tree", rows=2_000_000, features=40, bins=600, bin_bytes=2, bits_g=3,
             bits_h=3, leaves=127, bound=True),
        # ranking, an ordinary size
        dict(name="rank_200k_x136", kind="rank", rows=200_000, features=136, bins=255, bin_bytes=1, bits_g=3, bits_h=8,
             leaves=63, bound=True, iterations=1, group=100),
        # ranking, the largest workload of the benchmark
        dict(name="rank_20m_x200", kind="rank", rows=20_000_000, features=200, bins=255, bin_bytes=1, bits_g=3, bits_h=8,
             leaves=511, bound=True, iterations=1, group=100),
        # a program with growth rules of its own: the step functions one after the other
        dict(name="steps_3m_x28", kind="steps", rows=3_000_000, features=28, bins=255, bin_bytes=1, bits_g=3, bits_h=3,
             leaves=31, bound=False),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["tree", "boost", "rank", "steps"], [6, 2, 2, 1])[0]
    while True:
        rows = _log_uniform(rng, 8_000, 20_000_000)
        features = _log_uniform(rng, 12, 2000)
        if rng.random() < 0.5:
            features = max(12, features // 4 * 4)
        bin_bytes = 2 if kind in ("tree", "boost") and rng.random() < 0.1 else 1
        bins = rng.randint(300, 1000) if bin_bytes == 2 else rng.choice([15, 31, 63, 63, 127, 255, 255, 255])
        leaves = _log_uniform(rng, 8, 511)
        if rows * features * bin_bytes <= 2_000_000_000 and features * bins * leaves <= 40_000_000 and leaves * 100 <= rows:
            break
    bits = rng.choice([2, 3, 3, 3, 4, 5])
    c = dict(kind=kind, rows=rows, features=features, bins=bins, bin_bytes=bin_bytes, bits_g=bits, bits_h=bits,
             leaves=leaves, bound=rng.random() < 0.75)
    if kind == "tree" and rng.random() < 0.2:
        c["bits_h"] = 0
    if kind in ("boost", "rank"):
        c["iterations"] = 1 if rows * features > 50_000_000 else rng.randint(1, 3)
    if kind == "rank":
        c["bits_h"] = rng.choice([bits, 8])
        c["group"] = rng.randint(20, 150)
    return c


# ---- inputs ------------------------------------------------------------------------------------


def _matrix(case, gen, dev):
    """Bins [rows, features] and the target values z [rows] that depend on ten of the features."""
    n, f, nb = case["rows"], case["features"], case["bins"]
    skewed = case["kind"] == "rank"  # the default bin 0 holds 70 % of every feature
    dtype = torch.int16 if case["bin_bytes"] == 2 else torch.uint8
    bins = torch.empty((n, f), dtype=dtype, device=dev)
    z = torch.empty(n, dtype=torch.float32, device=dev)
    w = torch.randn(10, generator=gen, device=dev)
    cols = torch.randperm(f, generator=gen, device=dev)[:10].sort().values
    step = max(1, min(n, 400_000_000 // f))
    for a in range(0, n, step):
        b = min(n, a + step)
        blk = torch.randint(0, nb, (b - a, f), generator=gen, device=dev, dtype=dtype)
        if skewed:
            blk *= (torch.randint(0, 10, (b - a, f), generator=gen, device=dev, dtype=torch.uint8) >= 7).to(dtype)
        bins[a:b] = blk
        x = blk[:, cols].float() / nb - 0.5
        m = x.shape[1]
        s = x @ w[:m]
        for k in range(0, m - 1, 2):  # interactions: products and steps
            s += 4.0 * w[k + 1] * x[:, k] * x[:, k + 1] + 0.5 * w[k] * ((x[:, k] > 0.1) & (x[:, k + 1] < -0.1)).float()
        z[a:b] = s
    z = (z - z.mean()) / z.std()
    return (bins.view(torch.uint16) if case["bin_bytes"] == 2 else bins), z


def prepare(case, seed):
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed) * SEED_SALT + 17)
    n, kind = case["rows"], case["kind"]
    bins, z = _matrix(case, gen, dev)
    noise = lambda: torch.randn(n, generator=gen, device=dev)  # noqa: E731
    fitted = 0.5 * z + 0.3 * noise()  # the scores of a partly fitted model
    s = dict(case=case, bins=bins, seed=int(seed) & 0xffffffff)
    if kind == "rank":
        zn = z + 0.5 * noise()
        edges = torch.tensor([0.0, 0.75, 1.43, 2.1], device=dev)  # grades 0..4, each rarer than the one below
        s["label"] = torch.bucketize(zn, edges).float()
        s["start"] = fitted.contiguous()
        s["score"] = fitted.clone()
    elif kind == "tree" and case["bits_h"] == 0:
        s["g"] = (fitted - (z + 0.5 * noise())).contiguous()
        s["h"] = torch.ones(n, device=dev)
    else:
        y = (torch.rand(n, generator=gen, device=dev) < torch.sigmoid(2.0 * z)).float()
        if kind == "boost":
            s["label"], s["start"], s["score"] = y, fitted.contiguous(), fitted.clone()
        else:
            p = torch.sigmoid(fitted)
            s["g"], s["h"] = (p - y).contiguous(), (p * (1.0 - p)).contiguous()
    flags = (qb.WS_BIND if case["bound"] else qb.WS_ROW_COPIES) | (qb.WS_BOOST if kind in ("boost", "rank") else 0)
    ctx = qb.Context(n, case["features"], case["bins"], max_leaves=case["leaves"], bin_bytes=case["bin_bytes"],
                     device=dev, workspace_flags=flags)
    if case["bound"]:
        ctx.bind_bins(bins)
    s["ctx"] = ctx
    if kind == "steps":
        s["rows"] = torch.empty(n, dtype=torch.int32, device=dev)
        s["hists"] = torch.empty((2, case["features"] * case["bins"]), dtype=torch.int64, device=dev)
        s["root"] = torch.empty(case["features"] * case["bins"], dtype=torch.int64, device=dev)
    else:
        s["tree"] = ctx.new_tree()
    return s


# ---- one pass ----------------------------------------------------------------------------------


def _tree_outputs(t):
    return {k: getattr(t, k) for k in ("n_leaves", "split_leaf", "split_feature", "split_bin", "split_gain", "split_stats",
                                       "split_n_left", "leaf_begin", "leaf_count", "leaf_sum_g", "leaf_sum_h",
                                       "leaf_value", "leaf_value_quant", "delta", "hist_units", "row_idx")}


def _run_steps(s):
    c, ctx, bins, rows = s["case"], s["ctx"], s["bins"], s["rows"]
    n, bg, bh = c["rows"], c["bits_g"], c["bits_h"]
    dev = bins.device
    torch.arange(n, dtype=torch.int32, out=rows)
    gh, delta = ctx.quantize_gradients(s["g"], s["h"], bg, bh, s["seed"], 0)
    root = ctx.build_histograms(bins, gh, bits_g=bg, bits_h=bh, hist_out=s["root"])
    first = root.view(c["bins"], c["features"])[:, 0]  # any one feature holds every row
    stats = torch.stack([torch.full((), n, dtype=torch.int64, device=dev), (first >> 32).sum(),
                         (first & 0xffffffff).sum()]).view(1, 3)
    found = ctx.find_best_splits(root, stats, delta)
    best = qb.unpack_splits(found)[0]  # the program decides on the host
    n_left = ctx.partition_rows(bins, rows, 0, n, best["feature"], best["bin"])
    nl = int(n_left.item())
    left_small = nl <= n - nl
    begin, count = (0, nl) if left_small else (nl, n - nl)
    small, large = (0, 1) if left_small else (1, 0)
    ctx.build_histograms(bins, gh, row_idx=rows, begin=begin, count=count, bits_g=bg, bits_h=bh, hist_out=s["hists"][small])
    ctx.subtract_histograms(root, s["hists"][small], out=s["hists"][large])
    sides = torch.tensor([[nl, best["GL"], best["HL"]], [n - nl, best["GR"], best["HR"]]], dtype=torch.int64, device=dev)
    both = ctx.find_best_splits(s["hists"], sides, delta)
    begins = torch.tensor([0, nl], dtype=torch.int64, device=dev)
    counts = torch.tensor([nl, n - nl], dtype=torch.int64, device=dev)
    value = ctx.refit_leaves(s["g"], s["h"], rows, begins, counts)
    return dict(gh=gh, delta=delta, root=root, found=found, rows=rows, n_left=n_left, hists=s["hists"], both=both, value=value)


def run(state):
    c, ctx = state["case"], state["ctx"]
    kind = c["kind"]
    if kind == "steps":
        return _run_steps(state)
    if kind == "tree":
        t = ctx.grow_tree(state["bins"], state["g"], state["h"], c["bits_g"], c["bits_h"], state["seed"], 0, c["leaves"],
                          tree=state["tree"])
        return _tree_outputs(t)
    # a boosting program continues from its scores: every pass starts at the same ones
    state["score"].copy_(state["start"])
    for it in range(c["iterations"]):
        t = ctx.boost_iteration(state["bins"], state["label"], state["score"], c["bits_g"], c["bits_h"], state["seed"], it,
                                c["leaves"], 0.1, tree=state["tree"], group_size=c.get("group", 0))
    out = _tree_outputs(t)
    out["score"] = state["score"]
    return out


# ---- what a pass cannot do without, and how far right results may differ -------------------------


def work(case):
    n, f, nb = case["rows"], case["features"], case["bins"]
    matrix = n * f * case["bin_bytes"]
    k = case.get("iterations", 1)
    if case["kind"] == "steps":
        # matrix, derivatives and row list read; packed gradients, row list and three histograms written
        return {"bytes": matrix + 8 * n + 2 * n + 8 * n + 3 * 8 * f * nb, "flops": 2.0 * n * f}
    if case["kind"] == "tree":
        return {"bytes": matrix + 8 * n + 4 * n, "flops": 2.0 * n * f}  # matrix and derivatives in, row list out
    # per iteration: matrix, labels and scores in, scores and row list out
    return {"bytes": k * (matrix + 4 * n + 4 * n + 4 * n + 4 * n), "flops": 2.0 * k * n * f}


def tolerance(case):
    # Whole numbers are exact.  Leaf values are quotients of fp64 sums of fp32 values (another order of the sums moves
    # them by about 1e-15 of the sum of magnitudes), split gains fp64 with a fixed order of operations; the scores are
    # fp32 and take one rounded addition per iteration.
    if case["kind"] in ("boost", "rank"):
        return {"rel": 1e-7, "max": 1e-6}
    return {"rel": 1e-12, "max": 1e-10}
