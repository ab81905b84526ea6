"""Growth of whole trees on inputs made for particular branches of the growth kernels, against the oracle (bit-exact)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2207_09682_amd.binding import describe_counting, describe_hist_plan

pytestmark = pytest.mark.gpu


def _check(t, e, N):
    n = e.n_leaves
    assert int(t.n_leaves.item()) == n
    for name in ("split_leaf", "split_feature", "split_bin", "split_n_left"):
        assert np.array_equal(getattr(t, name).cpu().numpy()[: n - 1], getattr(e, name)[: n - 1]), name
    assert np.array_equal(t.leaf_begin.cpu().numpy()[:n], e.leaf_begin[:n])
    assert np.array_equal(t.leaf_count.cpu().numpy()[:n], e.leaf_count[:n])
    assert np.array_equal(t.leaf_sum_g.cpu().numpy()[:n], e.leaf_G[:n])
    assert np.array_equal(t.leaf_sum_h.cpu().numpy()[:n], e.leaf_H[:n])
    assert np.array_equal(t.row_idx.cpu().numpy(), e.row_idx)


@pytest.mark.parametrize("N,F,nb,L", [(4000, 7, 16, 31), (30_000, 7, 32, 255), (3000, 300, 8, 63), (2000, 5, 4, 100)])
def test_equal_gains_take_the_lowest_leaf(N, F, nb, L):
    # two mirror images: the second half of the rows repeats the first half's bins with the gradients negated, and one
    # feature tells the halves apart; below that split every node has a twin with exactly the same gain
    rng = np.random.default_rng(N + F)
    half = N // 2
    b = rng.integers(0, nb, (half, F)).astype(np.uint8)
    b[:, 0] = 0
    g = (1 + (b[:, 1] > nb // 2) + (b[:, 2] > nb // 3)).astype(np.float32) * (rng.random(half) < 0.9)
    bins = np.concatenate([b, b]); bins[half:, 0] = 1
    g = np.concatenate([g, -g]).astype(np.float32)
    h = np.ones(N, np.float32)
    from paper_2207_09682_amd import Context
    ctx = Context(N, F, nb, max_leaves=L)
    t = ctx.grow_tree(torch.from_numpy(bins).cuda(), torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda(), 3, 0, 5, 0, L,
                      min_data_in_leaf=5, rounding=1)
    e = oracle.grow_tree(bins, nb, g, h, 3, 0, 5, 0, L, min_data=5, rounding=1)
    assert e.n_leaves > 4 and len(set(e.split_gain[1:].tolist())) < e.n_leaves - 2, "the input makes no ties"
    _check(t, e, N)


def test_tied_leaf_the_selection_stops_at_is_expanded_first():
    # Four blocks of 2 m rows, split by feature 0 (gain 2.25 m, in units of delta_g^2), then by feature 1 (4.5 m on the right,
    # 2 m on the left); two of the four leaves have a last split by feature 2, of gain m exactly.  The one on the right comes
    # first by node number, the one on the left by leaf id: the fifth leaf is the left one's, and nothing else is expanded.
    m, gl = 64, [(3, 1), (0, 0), (-3, -1), (1, 1)]       # left: 2 +- 1 and 0, right: -2 +- 1 and 1
    bins = np.array([[b >> 1, b & 1, k, 0] for b in range(4) for k in range(2) for _ in range(m)], np.uint8)
    g = np.array([gl[b][k] for b in range(4) for k in range(2) for _ in range(m)], np.float32) * 0.25   # delta_g = 1/4
    h = np.ones(len(g), np.float32)
    from paper_2207_09682_amd import Context
    ctx = Context(len(g), 4, 4, max_leaves=5)
    t = ctx.grow_tree(torch.from_numpy(bins).cuda(), torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda(), 3, 0, 5, 0, 5,
                      min_data_in_leaf=5, rounding=1)
    e = oracle.grow_tree(bins, 4, g, h, 3, 0, 5, 0, 5, min_data=5, rounding=1)
    assert e.split_gain.tolist() == [2.25 * m / 16, 4.5 * m / 16, 2.0 * m / 16, m / 16] and e.split_leaf.tolist() == [0, 1, 0, 0]
    _check(t, e, len(g))
    assert ctx.tree_stats() == (3, 4, 4, 9)   # rounds, nodes expanded, splits, nodes


# Splits whose descendants have larger gains, several levels in a row (parity of features with a slight lead), and splits that
# peel a few rows off a large node: what is expanded ahead of the commits, and whose rows have to outlive it.
@pytest.mark.parametrize("kind,N,L", [("parity", 6000, 40), ("parity", 60_000, 255), ("peel", 20_000, 63), ("peel", 300_000, 255)])
def test_growth_ahead_of_the_commits(kind, N, L):
    F, nb = 16, 64
    rng = np.random.default_rng(N + L)
    bins = rng.integers(0, nb, (N, F)).astype(np.uint8)
    hi = bins >= nb // 2
    if kind == "parity":
        g = sum((-1.0) ** hi[:, 4 * k: 4 * k + 4].sum(1) * (1.0 + 0.1 * hi[:, 4 * k]) for k in range(3)) + 0.05 * hi[:, 0]
    else:
        g = np.exp(0.3 * (bins[:, :8] > nb - 6).sum(1) ** 2) - 0.05 * (bins[:, 8:12].sum(1) / nb) ** 2
    g = (g + 0.1 * rng.normal(size=N)).astype(np.float32)
    h = rng.uniform(0.2, 0.25, N).astype(np.float32)
    from paper_2207_09682_amd import Context
    ctx = Context(N, F, nb, max_leaves=L)
    dbins = torch.from_numpy(bins).cuda()
    e = oracle.grow_tree(bins, nb, g, h, 4, 4, 5, 0, L, min_data=20)
    n = e.n_leaves
    assert n > L // 2 and (np.diff(e.split_gain[: n - 1]) > 0).sum() > n // 10
    for bound, layout in ((True, 1), (True, 2), (False, 3)):
        ctx.bind_bins(dbins if bound else None)
        t = ctx.grow_tree(dbins, torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda(), 4, 4, 5, 0, L, min_data_in_leaf=20,
                          row_layout=layout)
        _check(t, e, N)
        assert np.allclose(t.leaf_value.cpu().numpy()[:n], e.leaf_value[:n], rtol=1e-9, atol=1e-13)


# row lists whose entries carry the row's quantized gradients: id and gradients fill the 32 bits, miss them by one, constant
# hessians; on the element-wise, the dword, the 16-byte-piece and both wide-row kernels
@pytest.mark.parametrize("N,bits_g,bits_h", [(65_536, 8, 8), (65_537, 8, 8), (131_072, 8, 0), (16_385, 2, 8), (40_000, 8, 2)])
@pytest.mark.parametrize("F,nb,bb", [(3, 64, 1), (13, 64, 1), (28, 64, 1), (36, 255, 1), (45, 300, 2), (68, 255, 1), (72, 255, 1), (80, 63, 1)])
def test_row_entries_with_gradients(N, bits_g, bits_h, F, nb, bb):
    L = 24
    rng = np.random.default_rng(N + F + bits_g)
    bins = rng.integers(0, nb, (N, F)).astype(np.uint16 if bb == 2 else np.uint8)
    x = bins[:, :3].astype(np.float64) / nb - 0.5
    g = (2 * x[:, 0] + 3 * x[:, 1] * x[:, 2] + 0.5 * rng.normal(size=N)).astype(np.float32)
    h = np.full(N, 0.25, np.float32) if bits_h == 0 else rng.uniform(0.0, 0.25, N).astype(np.float32)
    from paper_2207_09682_amd import Context
    ctx = Context(N, F, nb, max_leaves=L, bin_bytes=bb)
    dbins = torch.from_numpy(bins).cuda()
    e = oracle.grow_tree(bins, nb, g, h, bits_g, bits_h, 5, 0, L, min_data=20)
    assert e.n_leaves == L
    ctx.bind_bins(dbins)
    t = ctx.grow_tree(dbins, torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda(), bits_g, bits_h, 5, 0, L, min_data_in_leaf=20)
    _check(t, e, N)
    assert np.allclose(t.leaf_value.cpu().numpy()[:L], e.leaf_value[:L], rtol=1e-9, atol=1e-13)


# Trees whose histogram launches count the left rows themselves: row ids sorted by the split feature, so that whole stretches of a
# parent's list go one way, and hessians by which the child of more rows is taken for the smaller one; rows on both sides of a segment
# (512 rows, 2048 above 2^18) and of the 4096 that a workgroup reads at a time, work items of two such stretches (1.2 M rows), several tiles and
# fewer lanes than nodes, 8- and 16-byte pieces, 16-bit bins, row ids without gradients, more than 64 nodes in a round, more candidates
# per histogram than the plan kernel reduces itself (256).
@pytest.mark.parametrize("N,F,nb,bb,L,bits,layout", [
    (511, 16, 64, 1, 9, 3, 0), (4096, 28, 64, 1, 31, 3, 0), (4097, 17, 255, 1, 31, 3, 1), (8193, 33, 64, 1, 31, 5, 0),
    (262_144, 16, 64, 1, 127, 3, 0), (262_145, 16, 64, 1, 127, 3, 1), (100_000, 16, 64, 1, 658, 3, 0), (1_200_001, 16, 32, 1, 63, 3, 0),
    (30_000, 90, 255, 1, 127, 4, 0), (30_000, 72, 255, 1, 63, 8, 0), (20_000, 800, 63, 1, 63, 3, 0), (3000, 4096, 16, 1, 31, 3, 0),
    (50_001, 40, 300, 2, 63, 3, 0), (40_000, 9, 300, 2, 63, 3, 1), (6000, 520, 300, 2, 31, 3, 0), (2000, 4112, 16, 1, 15, 3, 0)])
def test_histogram_launches_that_count(N, F, nb, bb, L, bits, layout):
    rng = np.random.default_rng(N + F)
    bins = rng.integers(0, nb, (N, F)).astype(np.uint16 if bb == 2 else np.uint8)
    bins[:, 0] = np.arange(N, dtype=np.int64) * nb // N
    x = bins[:, :4].astype(np.float64) / nb - 0.5
    g = (3 * x[:, 0] + 2 * x[:, 1] * x[:, 2] + x[:, 0] * x[:, 3] + 0.2 * rng.normal(size=N)).astype(np.float32)
    h = (np.where((x[:, 0] < 0.3) & (x[:, 1] < 0.3), 0.01, 0.25) * rng.uniform(0.9, 1.0, N)).astype(np.float32)
    from paper_2207_09682_amd import Context
    ctx = Context(N, F, nb, max_leaves=L, bin_bytes=bb)
    dbins = torch.from_numpy(bins).cuda()
    e = oracle.grow_tree(bins, nb, g, h, bits, bits, 5, 0, L, min_data=3)
    n = e.n_leaves
    assert n > L // 2
    seg_rows = 512 if N <= 2 ** 18 else 2048
    c, p = describe_counting(N, F, nb, L, bb, bits, bits, segments=-(-N // seg_rows)), describe_hist_plan(N, F, nb, L, bb, bits, bits)
    assert c["seg_rows"] == seg_rows and (c["item_segs"] * seg_rows > 4096) == (N > 1_200_000)   # an item of two stretches
    assert (c["search_sums"] == 8) == (N * p["n_tiles"] > (2 ** 17 if p["n_tiles"] > 1 else 2 ** 14))   # the reduce kernel adds up
    assert (c["lanes"] < L) == ((F, L) in ((16, 658), (90, 127), (800, 63), (4096, 31), (520, 31), (4112, 15)))   # a round may have more nodes than lanes
    for bound in (True, False):
        ctx.bind_bins(dbins if bound else None)
        t = ctx.grow_tree(dbins, torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda(), bits, bits, 5, 0, L, min_data_in_leaf=3, row_layout=layout)
        assert ctx.tree_counting()
        _check(t, e, N)
        assert np.allclose(t.leaf_value.cpu().numpy()[:n], e.leaf_value[:n], rtol=1e-9, atol=1e-13)


# Trees beyond those whose histogram launches count: the counting pass in the order of the XCDs, in one step and in eight, with fewer and
# more than 64 nodes in a round, sorted rows (a node's rows in one place of the matrix), and gathered builds of few and many row groups
@pytest.mark.parametrize("N,F,nb,bb,L,bound", [(2_600_001, 16, 32, 1, 300, True), (1_100_003, 40, 600, 2, 63, False), (6_000_003, 5, 32, 1, 31, True),
                                                (2_500_003, 16, 32, 1, 127, False)])
def test_large_trees_of_row_lists(N, F, nb, bb, L, bound):
    rng = np.random.default_rng(N + F)
    bins = rng.integers(0, nb, (N, F), dtype=np.uint16 if bb == 2 else np.uint8)
    bins[:, 0] = np.arange(N, dtype=np.int64) * nb // N
    x = bins[:, :4].astype(np.float32) / nb - 0.5
    g = (3 * x[:, 0] + 2 * x[:, 1] * x[:, 2] + x[:, 0] * x[:, 3] + 0.2 * rng.normal(size=N)).astype(np.float32)
    h = rng.uniform(0.2, 0.25, N).astype(np.float32)
    from paper_2207_09682_amd import Context
    ctx = Context(N, F, nb, max_leaves=L, bin_bytes=bb)
    dbins = torch.from_numpy(bins).cuda()
    e = oracle.grow_tree(bins, nb, g, h, 3, 3, 5, 0, L, min_data=20)
    ctx.bind_bins(dbins if bound else None)
    t = ctx.grow_tree(dbins, torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda(), 3, 3, 5, 0, L, min_data_in_leaf=20, row_layout=0 if bound else 1)
    assert not ctx.tree_counting()
    _check(t, e, N)


# A bound matrix large enough for the copy whose rows begin on cache lines, in a workspace with and without room for it, and from an
# address that no wide load could use
@pytest.mark.parametrize("N,F,bits_h", [(2_300_003, 120, 3), (1_400_000, 200, 8)])
def test_trees_from_padded_rows(N, F, bits_h):
    nb, L = 32, 15
    gen = torch.Generator(device="cuda").manual_seed(N)
    store = torch.randint(0, nb, (N * F + 4,), generator=gen, device="cuda", dtype=torch.uint8)
    dbins = store[4:].view(N, F)
    bins = dbins.cpu().numpy()
    rng = np.random.default_rng(N)
    x = bins[:, :4].astype(np.float32) / nb - 0.5
    g = (3 * x[:, 0] + 2 * x[:, 1] * x[:, 2] + x[:, 0] * x[:, 3] + 0.2 * rng.normal(size=N)).astype(np.float32)
    h = rng.uniform(0.2, 0.25, N).astype(np.float32)
    from paper_2207_09682_amd import Context
    from paper_2207_09682_amd import binding as qb
    ctx = Context(N, F, nb, max_leaves=L, workspace_flags=qb.WS_BIND)
    e = oracle.grow_tree(bins, nb, g, h, 3, bits_h, 5, 0, L, min_data=20)
    dg, dh = torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda()
    ctx.bind_bins(dbins)
    _check(ctx.grow_tree(dbins, dg, dh, 3, bits_h, 5, 0, L, min_data_in_leaf=20), e, N)
    small = torch.empty(ctx.workspace_bytes - N * 128, dtype=torch.uint8, device="cuda")
    ctx.set_workspace(small, flags=qb.WS_BIND)
    ctx.bind_bins(dbins)
    _check(ctx.grow_tree(dbins, dg, dh, 3, bits_h, 5, 0, L, min_data_in_leaf=20), e, N)


def test_rounds_beyond_those_enqueued_up_front():
    # a tree of more rounds than the one before it: whatever is missing, at most one round too many is enqueued and the passes over
    # the leaves at most four times
    N, F, nb, L = 20_000, 12, 64, 255
    rng = np.random.default_rng(3)
    bins = rng.integers(0, nb, (N, F)).astype(np.uint8)
    g = np.exp(0.3 * (bins[:, :8] > nb - 6).sum(1) ** 2).astype(np.float32) + 0.1 * rng.normal(size=N).astype(np.float32)
    h = rng.uniform(0.2, 0.25, N).astype(np.float32)
    from paper_2207_09682_amd import Context
    ctx = Context(N, F, nb, max_leaves=L)
    dbins, dg, dh = torch.from_numpy(bins).cuda(), torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda()
    up_front = 10   # of a context's first tree
    seen = set()
    for i, l in enumerate((L, L, 2, L, 3, 5, 40, 2, 4, 6, 8, 10, 12, 2, 3, 2, 6, 2, 8)):
        t = ctx.grow_tree(dbins, dg, dh, 3, 3, 5, 0, l, min_data_in_leaf=20)
        _check(t, oracle.grow_tree(bins, nb, g, h, 3, 3, 5, 0, l, min_data=20), N)
        rounds = ctx.tree_stats()[0]
        assert i > 0 or rounds > up_front + 3
        missing = rounds - up_front
        assert ctx.tree_launches() == ((up_front, 1) if missing <= 0 else (rounds, missing + 1) if missing <= 2 else (rounds + 1, 4)), (i, l, rounds)
        seen.add(min(missing, 3))
        up_front = rounds
    assert {0, 1, 2, 3} <= seen, seen


# what the automatic choice takes for a matrix that is not bound, and that the choice does not change the tree
@pytest.mark.parametrize("N,F,L,layout", [(1_600_000, 20, 255, 4), (1_700_000, 20, 255, 3), (1_600_000, 16, 255, 4), (1_700_000, 16, 255, 3),
                                          (2_100_000, 16, 64, 4), (2_200_000, 20, 64, 3), (3_200_000, 16, 5, 4), (3_300_000, 16, 5, 3), (2_000_000, 24, 255, 4)])
def test_layout_of_an_unbound_matrix(N, F, L, layout):
    nb = 32
    rng = np.random.default_rng(F)
    bins = rng.integers(0, nb, (N, F)).astype(np.uint8)
    g = (bins[:, 0] / nb * (bins[:, 1] > 9) - 0.3 * (bins[:, 2] > 20) + 0.1 * rng.normal(size=N)).astype(np.float32)
    h = rng.uniform(0.2, 0.25, N).astype(np.float32)
    from paper_2207_09682_amd import Context
    ctx = Context(N, F, nb, max_leaves=L)
    dbins, dg, dh = torch.from_numpy(bins).cuda(), torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda()
    trees = []
    for asked, took in ((0, layout), (1, 1)):
        t = ctx.grow_tree(dbins, dg, dh, 3, 3, 5, 0, L, row_layout=asked)
        assert ctx.tree_layout() == took
        trees.append({k: getattr(t, k).cpu() for k in ("n_leaves", "split_feature", "split_bin", "split_gain", "leaf_sum_g", "leaf_sum_h", "leaf_value", "row_idx")})
    for k, v in trees[0].items():
        assert torch.equal(v, trees[1][k]), k


# 32-bit working words and 8-bit gradients: groups of 129 rows, on both sides of where the split search adds them all up itself
@pytest.mark.parametrize("N,F", [(4000, 28), (4400, 28), (2000, 100), (12_000, 100)])
def test_small_trees_of_many_short_row_groups(N, F):
    nb, L = 255, 31
    rng = np.random.default_rng(N)
    bins = rng.integers(0, nb, (N, F)).astype(np.uint8)
    g = (bins[:, 0] / nb * (bins[:, 1] > 99) - 0.3 + 0.1 * rng.normal(size=N)).astype(np.float32)
    h = rng.uniform(0.2, 0.25, N).astype(np.float32)
    from paper_2207_09682_amd import Context
    ctx = Context(N, F, nb, max_leaves=L)
    e = oracle.grow_tree(bins, nb, g, h, 8, 8, 5, 0, L, min_data=20)
    t = ctx.grow_tree(torch.from_numpy(bins).cuda(), torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda(), 8, 8, 5, 0, L, min_data_in_leaf=20, acc_width=16)
    _check(t, e, N)


def test_trees_of_very_different_depth_in_turn():
    # the number of rounds enqueued up front is the last tree's: too few and too many of them, on one context, without a
    # synchronisation of the caller's between the trees
    N, F, nb, L = 20_000, 12, 64, 127
    rng = np.random.default_rng(3)
    bins = rng.integers(0, nb, (N, F)).astype(np.uint8)
    x = bins.astype(np.float64) / nb
    h = rng.uniform(0.2, 0.25, N).astype(np.float32)
    gs = [(x[:, 0] - 0.5).astype(np.float32), np.exp(0.3 * (bins[:, :8] > nb - 6).sum(1) ** 2).astype(np.float32), np.zeros(N, np.float32),
          (x[:, 1] * x[:, 2] - x[:, 3] + 0.1 * rng.normal(size=N)).astype(np.float32)]
    from paper_2207_09682_amd import Context
    ctx = Context(N, F, nb, max_leaves=L)
    dbins, dh, dg = torch.from_numpy(bins).cuda(), torch.from_numpy(h).cuda(), [torch.from_numpy(g).cuda() for g in gs]
    order = [0, 1, 2, 3, 1, 0, 3, 2, 2, 1]
    leaves = [L, 2, L, L, L, L, 5, L, 3, L]
    trees = [ctx.grow_tree(dbins, dg[k], dh, 3, 3, 5, i, l, min_data_in_leaf=20) for i, (k, l) in enumerate(zip(order, leaves))]
    for i, (k, l, t) in enumerate(zip(order, leaves, trees)):
        e = oracle.grow_tree(bins, nb, gs[k], h, 3, 3, 5, i, l, min_data=20)
        _check(t, e, N)
        n = e.n_leaves
        assert np.allclose(t.leaf_value.cpu().numpy()[:n], e.leaf_value[:n], rtol=1e-9, atol=1e-13)


# both sides of the lines at which the partition takes other segments or sums its counts in two levels, ragged ends
@pytest.mark.parametrize("N,F,L,layout", [(511, 4, 6, 1), (262_144, 5, 63, 1), (262_145, 5, 63, 2), (262_147, 16, 40, 3),
                                          (3 * 2**20, 4, 31, 1), (3 * 2**20 + 1, 4, 255, 2), (3_300_001, 16, 31, 3),
                                          (5 * 2**20, 4, 15, 0), (5 * 2**20 + 1, 4, 15, 0)])
def test_partition_segments(N, F, L, layout):
    rng = np.random.default_rng(N)
    nb = 32
    bins = rng.integers(0, nb, (N, F)).astype(np.uint8)
    x = bins[:, :3].astype(np.float64) / nb - 0.5
    y = (rng.random(N) < 1 / (1 + np.exp(-(4 * x[:, 0] + 6 * x[:, 1] * x[:, 2])))).astype(np.float32)
    p = rng.uniform(0.2, 0.8, N).astype(np.float32)
    g = (p - y).astype(np.float32); h = (p * (1 - p)).astype(np.float32)
    from paper_2207_09682_amd import Context
    ctx = Context(N, F, nb, max_leaves=L)
    dbins = torch.from_numpy(bins).cuda()
    e = oracle.grow_tree(bins, nb, g, h, 3, 3, 5, 0, L, min_data=20)
    for bound in (False, True):
        ctx.bind_bins(dbins if bound else None)
        t = ctx.grow_tree(dbins, torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda(), 3, 3, 5, 0, L, min_data_in_leaf=20,
                          row_layout=layout)
        _check(t, e, N)


# both sides of the 256 candidates per histogram (a tile has 2 features above 256 bins, 16 for such wide 8-bit matrices) up to
# which the plan kernel reduces them itself; above, a launch of its own does; columns that repeat tie between far tiles
@pytest.mark.parametrize("F,nb,bb", [(512, 300, 2), (513, 300, 2), (1000, 300, 2), (4096, 12, 1), (4097, 12, 1)])
def test_growth_with_candidates_reduced_apart(F, nb, bb):
    N, L = 3001, 31
    rng = np.random.default_rng(F)
    bins = rng.integers(0, nb, (N, F)).astype(np.uint16 if bb == 2 else np.uint8)
    bins[:, F - 1] = bins[:, 3]; bins[:, F // 2] = bins[:, F - 2]
    x = bins[:, [3, F - 2, 40, F // 3]].astype(np.float64) / nb - 0.5
    g = (x[:, 0] + 1.5 * x[:, 1] * (x[:, 0] > 0) + 2 * x[:, 2] * x[:, 3] + 0.1 * rng.normal(size=N)).astype(np.float32)
    h = rng.uniform(0.1, 0.25, N).astype(np.float32)
    from paper_2207_09682_amd import Context
    ctx = Context(N, F, nb, max_leaves=L, bin_bytes=bb)
    dbins = torch.from_numpy(bins).cuda()
    e = oracle.grow_tree(bins, nb, g, h, 3, 3, 5, 0, L, min_data=20)
    used = e.split_feature[: e.n_leaves - 1]
    assert e.n_leaves > 8 and F - 1 not in used and {3, F // 2} <= set(used.tolist())
    for bound in (False, True):
        ctx.bind_bins(dbins if bound else None)
        for _ in range(2):  # the second tree with the first one's number of rounds
            t = ctx.grow_tree(dbins, torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda(), 3, 3, 5, 0, L, min_data_in_leaf=20)
            _check(t, e, N)
        assert np.array_equal(t.split_gain.cpu().numpy()[: e.n_leaves - 1], e.split_gain[: e.n_leaves - 1])
    assert ctx.tree_stats()[0] > 2


def _split_cases():
    # bins and features around the edges of the search's tiles and of the bins a thread takes
    return [(F, nb) for F, nb in [(1, 2), (3, 64), (4, 65), (5, 63), (7, 128), (29, 129), (63, 255), (64, 256), (66, 100), (255, 9),
                                  (256, 64), (257, 65), (260, 129), (271, 255), (3, 257), (9, 512), (6, 513), (33, 1023), (2, 1024)]]


@pytest.mark.parametrize("F,nb", _split_cases())
def test_split_search_edges(F, nb):
    from paper_2207_09682_amd import Context, binding
    rng = np.random.default_rng(1000 * F + nb)
    n = 5
    G = rng.integers(-300, 300, (n, nb, F)).astype(np.int64)
    H = rng.integers(0, 400, (n, nb, F)).astype(np.int64) * (rng.random((n, nb, F)) < 0.8)
    tg = G.sum(axis=1).max(axis=1) + 10; th = H.sum(axis=1).max(axis=1) + 10
    last = nb // 2  # every feature of a leaf sums to the leaf's totals
    G[:, last, :] += tg[:, None] - G.sum(axis=1)
    H[:, last, :] += th[:, None] - H.sum(axis=1)
    rows = (th // 3 + 1).astype(np.int64)
    hist = torch.from_numpy(((G << 32) + H).reshape(n, nb * F)).cuda()
    stats = torch.from_numpy(np.stack([rows, tg, th], axis=1)).cuda()
    d = np.array([0.25, 0.125], np.float32)
    ctx = Context(1000, F, nb, max_leaves=3, bin_bytes=2 if nb > 256 else 1)   # batches of 6 histograms, an odd number here
    for min_data, min_h in ((0, 0.0), (20, 0.0), (int(rows.min()) // 3, 5.0), (10**6, 0.0)):
        got = binding.unpack_splits(ctx.find_best_splits(hist, stats, torch.from_numpy(d).cuda(), min_data, min_h))
        for i in range(n):
            o = np.stack([G[i].T, H[i].T], axis=-1).copy()
            e = oracle.find_best_split(o, int(rows[i]), int(tg[i]), int(th[i]), d[0], d[1], min_data, min_h)
            assert got[i]["feature"] == e.feature and got[i]["gain"] == e.gain, (min_data, i)
            if e.feature >= 0:
                assert all(got[i][k] == getattr(e, k) for k in ("bin", "GL", "HL", "GR", "HR", "cnt_left"))


# both sides of the lines between a whole pair of histograms per XCD and tiles spread over all of them: more than 256 wavefronts per
# pair (257 features of 255 bins, 65 of 300 and more), fewer than 32 pairs; numbers of tiles and shares that are no multiples of 8
@pytest.mark.parametrize("F,nb", [(1000, 65), (271, 255), (256, 255), (64, 300), (65, 300), (67, 600)])
def test_split_search_spread_over_xcds(F, nb):
    from paper_2207_09682_amd import Context, binding
    rng = np.random.default_rng(F)
    most = 70
    G = rng.integers(-300, 300, (most, nb, F)).astype(np.int64)
    H = rng.integers(0, 400, (most, nb, F)).astype(np.int64)
    tg = G.sum(axis=1).max(axis=1) + 10; th = H.sum(axis=1).max(axis=1) + 10
    G[:, -1, :] += tg[:, None] - G.sum(axis=1)
    H[:, -1, :] += th[:, None] - H.sum(axis=1)
    rows = (th // 3 + 1).astype(np.int64)
    hist = torch.from_numpy(((G << 32) + H).reshape(most, nb * F)).cuda()
    stats = torch.from_numpy(np.stack([rows, tg, th], axis=1)).cuda()
    d = np.array([0.25, 0.125], np.float32)
    exp = [oracle.find_best_split(np.stack([G[i].T, H[i].T], axis=-1).copy(), int(rows[i]), int(tg[i]), int(th[i]), d[0], d[1], 20, 0.0)
           for i in range(most)]
    ctx = Context(1000, F, nb, max_leaves=most // 2, bin_bytes=2 if nb > 256 else 1)
    for n in (1, 2, 3, 15, 16, 17, 32, 33, 62, 63, 64, most):
        got = binding.unpack_splits(ctx.find_best_splits(hist[:n], stats[:n], torch.from_numpy(d).cuda()))
        for i in range(n):
            assert all(got[i][k] == getattr(exp[i], k) for k in ("feature", "gain", "bin", "GL", "HL", "GR", "HR", "cnt_left")), (n, i)


# leaves as units of work: one leaf, empty leaves, one that holds nearly all rows, both sides of the lines at which the row
# order is cut into more parts, and more rows than the largest number of parts is made for
@pytest.mark.parametrize("N,counts", [(1, [1]), (7, [0, 7, 0]), (5000, [1, 4990, 0, 9]), (2**20, [2**19] * 2),
                                      (2**20 + 1, [2**20 - 600, 601]), (2**20 + 9, [3] * 657 + [2**20 - 1962]),
                                      (2**25 + 5, [2**25 - 70_000, 70_000, 0, 5])])
def test_refit_and_update_over_leaf_layouts(N, counts):
    rng = np.random.default_rng(N)
    L = len(counts)
    g = rng.normal(size=N).astype(np.float32); h = rng.uniform(0.1, 0.25, N).astype(np.float32)
    owner = np.repeat(np.arange(L, dtype=np.int16), counts); rng.shuffle(owner)
    rows = np.argsort(owner, kind="stable").astype(np.int32)
    count = np.asarray(counts, np.int64); begin = np.cumsum(count) - count
    from paper_2207_09682_amd import Context
    ctx = Context(N, 4, 4, max_leaves=L)
    drows, dbegin, dcount = (torch.from_numpy(a).cuda() for a in (rows, begin, count))
    got = ctx.refit_leaves(torch.from_numpy(g).cuda(), torch.from_numpy(h).cuda(), drows, dbegin, dcount).cpu().numpy()
    G = np.bincount(owner, g.astype(np.float64), L); H = np.bincount(owner, h.astype(np.float64), L)
    A = np.bincount(owner, np.abs(g.astype(np.float64)), L)
    exp = np.where(H > 0, -G / np.where(H > 0, H, 1), 0.0)
    # fp64 sums of n terms in another order: at most n 2^-53 of the sum of magnitudes
    bound = 2.0**-52 * count * (A / np.where(H > 0, H, 1) + np.abs(exp)) + 1e-300
    assert (np.abs(got - exp) <= bound).all()
    score = rng.normal(size=N).astype(np.float32); value = rng.normal(size=L)
    d = torch.from_numpy(score.copy()).cuda()
    ctx.update_scores(d, drows, dbegin, dcount, torch.from_numpy(value).cuda(), 0.1)
    assert np.array_equal(d.cpu().numpy(), score + (0.1 * value).astype(np.float32)[owner])


# leaves on both sides of the 64 that a wavefront looks through at a time, the most leaves, lists that share rows (their counts
# add up to more than the matrix has), empty leaves in front, at the end and between
@pytest.mark.parametrize("L", [1, 2, 63, 64, 65, 128, 129, 320, 658])
@pytest.mark.parametrize("N", [900, 40_001])
def test_refit_over_lists_that_share_rows(N, L):
    rng = np.random.default_rng(N + L)
    g = rng.normal(size=N).astype(np.float32); h = rng.uniform(0.1, 0.25, N).astype(np.float32)
    count = rng.integers(0, N // 2, L) * (rng.random(L) < 0.7); count[L // 2] = N
    begin = np.array([rng.integers(0, N - c + 1) for c in count])
    rows = rng.permutation(N).astype(np.int32)
    from paper_2207_09682_amd import Context
    got = Context(N, 4, 4, max_leaves=L).refit_leaves(*(torch.from_numpy(a).cuda() for a in (g, h, rows, begin, count))).cpu().numpy()
    for l in range(L):
        r = rows[begin[l]:begin[l] + count[l]]
        G, H, A = (float(a[r].astype(np.float64).sum()) for a in (g, h, np.abs(g)))
        exp = -G / H if count[l] else 0.0
        assert abs(got[l] - exp) <= 2.0**-52 * count[l] * (A / H + abs(exp)) if count[l] else got[l] == 0.0, l  # bound as above


# one and several queries per workgroup, ragged last queries, group sizes around multiples of a wavefront and of the four
# pairs that share a reciprocal, and the largest
@pytest.mark.parametrize("n,group", [(5, 1), (7, 3), (131, 2), (1000, 5), (333, 20), (2001, 63), (2000, 64), (2600, 65), (3000, 127),
                                     (3001, 150), (60_001, 100), (2049, 256), (2060, 257), (5111, 511), (2049, 513), (2500, 1000), (3333, 1024)])
def test_lambdarank_group_sizes(n, group):
    from paper_2207_09682_amd import Context
    rng = np.random.default_rng(n * 7 + group)
    s = np.round(rng.normal(size=n) * 8).astype(np.float32) / 8      # ties, and zeros of both signs
    s[s == 0] *= rng.choice([-1.0, 1.0], int((s == 0).sum())).astype(np.float32)
    rel = rng.choice([0, 0, 0, 1, 2, 4], n).astype(np.float32)
    nq = (n + group - 1) // group
    q = np.arange(n) // group
    if nq > 8:  # score ranges on both sides of the line between the two forms, gains beyond 1e100, no relevant row
        for at, width in ((1, 330.0), (3, 350.0), (5, 5000.0)):
            s[q == at] = rng.uniform(-width / 2, width / 2, int((q == at).sum())).astype(np.float32)
        rel[np.flatnonzero(q == 6)[0]] = 400.0
        rel[q == 2] = 0.0
    g, h = (a.cpu().numpy() for a in Context(n, 4, 16).lambdarank_gradients(torch.from_numpy(s).cuda(), torch.from_numpy(rel).cuda(), group))
    eg, eh = oracle.lambdarank_gradients(s, rel, group)
    # fp64 sums of at most `group` terms in another order, each term to a few 2^-52 (exp of |x| <= 170: 170 * 2^-53), and one
    # rounding to fp32 (2^-24); sums of both signs cancel, so the bound is on the magnitudes, at most the query's largest h + |g|
    top = np.zeros(nq); np.maximum.at(top, q, np.abs(eg)); tol = 2.0**-23
    assert (np.abs(g - eg) <= tol * np.abs(eg) + group * 2.0**-43 * top[q]).all()
    assert (np.abs(h - eh) <= tol * np.abs(eh) + group * 2.0**-43 * top[q]).all()


# score ranges and gains on both sides of the lines between the three forms of a pair (340, 690; 1e100, that is grade 332),
# queries whose last pairs are not four, one and several queries per workgroup
@pytest.mark.parametrize("group", [2, 37, 100, 150, 1023])
def test_lambdarank_forms_of_a_pair(group):
    from paper_2207_09682_amd import Context
    rng = np.random.default_rng(group)
    widths = [339.9, 340.1, 500.0, 689.9, 690.1, 2000.0, 1.0, 1.0, 500.0]
    grades = [4, 4, 4, 4, 4, 4, 331, 333, 1000]
    s = np.empty((len(widths), group), np.float32); rel = np.empty((len(widths), group), np.float32)
    for i, (w, top) in enumerate(zip(widths, grades)):
        s[i] = rng.uniform(-w / 2, w / 2, group); s[i, 0] = -w / 2; s[i, -1] = w / 2
        rel[i] = rng.integers(0, 5, group); rel[i, 0] = top; rel[i, -1] = 0
    s, rel = s.ravel(), rel.ravel()
    g, h = (a.cpu().numpy() for a in Context(len(s), 4, 16).lambdarank_gradients(torch.from_numpy(s).cuda(), torch.from_numpy(rel).cuda(), group))
    eg, eh = oracle.lambdarank_gradients(s, rel, group)
    # as for the group sizes above; exp of |x| <= 345 here, and the largest magnitude of the query is that of its sums' terms
    top = np.repeat(np.abs(eg).reshape(-1, group).max(axis=1), group); tol = 2.0**-23
    assert (top > 0).all()
    assert (np.abs(g - eg) <= tol * np.abs(eg) + group * 2.0**-42 * top).all()
    assert (np.abs(h - eh) <= tol * np.abs(eh) + group * 2.0**-42 * top).all()


def test_lambdarank_with_more_work_items_than_a_launch_may_have():
    # queries of one row leave half of the lanes idle: 2^32 work-items for the largest number of rows; with three rows per
    # query the second launch begins inside the rows and not at their last workgroup
    from paper_2207_09682_amd import Context
    n, period = 2**31 - 1, 3 * 2**16
    ctx = Context(n, 1, 2, max_leaves=1, workspace_flags=0)
    gen = torch.Generator(device="cuda"); gen.manual_seed(1)
    s0 = torch.randn(period, generator=gen, device="cuda"); r0 = torch.randint(0, 5, (period,), generator=gen, device="cuda").float()
    times = n // period + 1
    s, r = s0.repeat(times)[:n], r0.repeat(times)[:n]
    for group in (1, 3):
        eg, eh = ctx.lambdarank_gradients(s0, r0, group)
        assert group == 1 or float(eg.abs().max()) > 0
        g = torch.full((n,), float("nan"), device="cuda"); h = torch.full((n,), float("nan"), device="cuda")
        ctx._chk(ctx.lib.qgbdt_lambdarank_gradients(ctx._h, s.data_ptr(), r.data_ptr(), n, group, g.data_ptr(), h.data_ptr()))
        for got, exp in ((g, eg), (h, eh)):
            whole = (times - 1) * period
            assert bool((got[:whole].view(times - 1, period) == exp).all())
            rest = (n - whole) // 3 * 3                     # (the last query may be a part of one)
            assert torch.equal(got[whole:whole + rest], exp[:rest]) and bool(got[whole + rest:].isfinite().all())
        del g, h, got
    ctx.close()
    del s, r
    torch.cuda.empty_cache()


def test_lambdarank_nan_score_stays_in_its_query():
    from paper_2207_09682_amd import Context
    rng = np.random.default_rng(3)
    n, group = 700, 100
    s = rng.normal(size=n).astype(np.float32); rel = rng.integers(0, 5, n).astype(np.float32)
    eg, eh = oracle.lambdarank_gradients(s, rel, group)
    s[250] = np.nan; s[503] = -np.float32(np.nan)
    g, h = (a.cpu().numpy() for a in Context(n, 4, 16).lambdarank_gradients(torch.from_numpy(s).cuda(), torch.from_numpy(rel).cuda(), group))
    bad = np.isin(np.arange(n) // group, (2, 5))
    assert np.isnan(g[bad]).all() and np.isnan(h[bad]).all()
    assert np.allclose(g[~bad], eg[~bad], rtol=1e-6, atol=1e-7) and np.allclose(h[~bad], eh[~bad], rtol=1e-6, atol=1e-7)


# tiles of 2048 rows, at most 512 segments of them: around one tile, around the size from which segments hold more than one, a slice
# that starts at an odd row, a list in no order, everything to one side
@pytest.mark.parametrize("N,begin,count,bin_", [(2100, 3, 2047, 30), (2100, 0, 2048, 30), (2100, 1, 2049, 30), (300, 7, 257, 0),
                                                (2**20 + 9, 0, 2**20, 31), (2**20 + 9, 5, 2**20 + 1, 31), (2_100_003, 1, 2_100_001, 12),
                                                (2_100_003, 0, 2_100_003, 63)])
def test_partition_rows_tiles(N, begin, count, bin_):
    from paper_2207_09682_amd import Context
    rng = np.random.default_rng(count)
    bins = rng.integers(0, 64, (N, 5)).astype(np.uint8)
    idx = rng.permutation(N).astype(np.int32)
    exp, nl = oracle.partition_rows(bins, idx, begin, count, 3, bin_)
    didx = torch.from_numpy(idx.copy()).cuda()
    got = Context(N, 5, 64, max_leaves=2).partition_rows(torch.from_numpy(bins).cuda(), didx, begin, count, 3, bin_)
    assert int(got.item()) == nl
    assert np.array_equal(didx.cpu().numpy(), exp)
