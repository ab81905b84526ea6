"""Growth of whole trees on inputs made for particular branches of the growth kernels, against the oracle (bit-exact)."""
import numpy as np
import pytest
import torch

import oracle

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


# both sides of the lines at which the partition takes other segments or sums its counts in two levels, ragged ends
@pytest.mark.parametrize("N,F,L,layout", [(511, 4, 6, 1), (262_144, 5, 63, 1), (262_145, 5, 63, 2), (262_147, 16, 40, 3),
                                          (3 * 2**20, 4, 31, 1), (3 * 2**20 + 1, 4, 255, 2), (3_300_001, 16, 31, 3)])
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
