"""ppo_solve_cluster on the nodes and cuts that can matter: batches large enough for that are compared element by element
with the same instances one at a time, which are searched whole.  The number of cuts left decides how many sets share a
wave, so it is set here: `cheap` of the transfer sizes are 1, the rest far above."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import ppo_cluster_oracle as O
from paper_2210_12219_amd import workloads as W


def check(w, oracle=0, segments=None):
    import torch
    from paper_2210_12219_amd import binding as ppo
    dev = ppo.to_device(w)

    def solve(a):
        out = ppo.ppo_solve_cluster(*a) if segments is None else ppo.ppo_solve_cluster_few(*a, max_segments=segments)
        return [x.cpu().numpy() for x in out]

    got = solve(dev)
    for i in range(w.n_inst):
        one = [x[0] for x in solve([x[i:i + 1].contiguous() for x in dev])]
        assert got[0][i].view(np.uint32) == one[0].view(np.uint32) and got[1][i] == one[1], i
        assert np.array_equal(got[2][i], one[2]) and np.array_equal(got[3][i], one[3]), i
    for i in range(oracle):
        b, p, cuts, order = O.subset_dp(w.t[i], w.m[i], w.M[i], w.B[i], segments)
        assert got[0][i].view(np.uint32) == np.float32(b).view(np.uint32) and got[1][i] == p
        assert np.array_equal(got[2][i], cuts) and np.array_equal(got[3][i], order)
    return got


def batch(n):
    """instances of n nodes that are searched on what can matter"""
    return -(-800000 // (n << (n - 1)))


@pytest.mark.parametrize("cheap", [1, 5, 14, 15, 18, 19, 22, 23, 30, 31, 32, 60, 61, 62, 63, 99])
def test_cuts_left(cheap):
    w = W.cluster_mixed(13, L=100, n_inst=batch(13), seed=900 + cheap, capacity_factor=0.4)
    rng = np.random.default_rng(cheap)
    for i in range(w.n_inst):
        w.t[i] = 1e6 * (1 + rng.random(w.L))
        w.t[i, rng.permutation(w.L - 1)[:cheap]] = 1.0 + (rng.random(cheap) if i % 2 else 0.0)
        w.m[i] = 1.0
        w.M[i] = rng.choice([12.0, 25.0, 50.0], w.k) if i % 3 else 30.0
        if i % 4 < 2:
            w.B[i] = np.where(np.eye(w.k, dtype=bool), 0, 2.0)
    check(w, oracle=1)


@pytest.mark.parametrize("n,L", [(13, 13), (11, 24), (11, 64), (12, 128), (13, 63), (14, 127), (15, 17)])
def test_ties_zeros_and_capacities(n, L):
    w = W.random_instances(950 + n, batch(n), L, n, capacity_factor=1.5, quantised=L % 2 == 0)
    rng = np.random.default_rng(n)
    w.M[...] *= np.exp(rng.uniform(np.log(0.1), np.log(20.0), (w.n_inst, 1))).astype(np.float32)   # from none that fits to any
    for i in range(0, w.n_inst, 3):
        w.t[i, rng.random(L) < 0.4] = 0.0
        w.t[i, rng.random(L) < 0.2] = -0.0
    check(w, oracle=2 if n < 13 else 0)


def test_paper_shaped_clusters():
    """one capacity, many ties: nine nodes may be too few to hold the chain, and no node is left out"""
    for capacity in (10.0, 16.0, 64.0, 200.0):
        check(W.cluster_geometric(12, capacity, n_inst=batch(12), seed=int(capacity)), oracle=1)
    check(W.cluster_mixed(16, L=100, n_inst=2, seed=3), oracle=1)   # from 16 nodes on one instance is confined as well


def few_batch(n, segments):
    """instances that ppo_solve_cluster_few searches on what can matter"""
    from math import comb
    return -(-(300000 if n >= 30 else 1200000) // sum(comb(n, c) * c for c in range(1, segments)))


@pytest.mark.parametrize("n,L,segments", [(12, 100, 6), (14, 33, 5), (30, 100, 5), (30, 17, 5), (50, 64, 4), (50, 128, 4), (64, 40, 4),
                                          (64, 100, 3)])
def test_few_segments(n, L, segments):
    batch = few_batch(n, segments)
    w = W.cluster_mixed(n, L=L, n_inst=batch, seed=n + L, capacity_factor=0.8 / segments)
    rng = np.random.default_rng(n + L)
    for i in range(w.n_inst):
        if i % 4 == 1:
            w.t[i, rng.random(L) < 0.3] = -0.0 if i % 8 == 1 else 0.0
        if i % 4 == 2:   # ties
            w.t[i] = np.round(w.t[i]) + 1
            w.B[i] = np.where(np.eye(n, dtype=bool), 0, np.round(w.B[i]) + 1)
        if i % 4 == 3:   # short of memory, down to none that fits
            w.M[i] *= np.float32(rng.uniform(0.2, 0.9))
    check(w, oracle=2 if n < 15 else 0, segments=segments)


def test_few_segments_of_one_capacity():
    check(W.cluster_geometric(40, 32.0, n_inst=few_batch(40, 4), seed=4), segments=4)


def equal_links(n):
    return np.where(np.eye(n, dtype=bool), 0.0, 1.0)


def vanishing(kind, n, L, n_inst, segments, seed):
    """Quotients t / B that round to 0 or to a value below the normal range, in clusters whose optimum is such a value: what
    counts as within the bound has to be told by the rounded quotient, not by t against bound * B."""
    w = W.random_instances(seed, n_inst, L, n, capacity_factor=1.0)
    rng = np.random.default_rng(seed)
    w.m[...] = 1.0
    w.M[...] = np.ceil(1.2 * L / segments)
    if kind == "to zero":   # the last node holds everything: 0 without a link, and every link is 0
        w.M[:, -1] = L
        w.t[...], w.B[...] = 1e-16, 1e30 * equal_links(n)
    elif kind == "some to zero":   # zero transfers beside those that vanish and those that do not
        w.t[...] = rng.choice([0.0, -0.0, 3e-16, 6e-16, 1e-14], w.t.shape)
        w.B[...] = 1e30 * equal_links(n)
    elif kind == "one value below the normal range":   # 2^-133 for every t, which differ by less than its rounding
        w.t[...] = 2.0 ** -123 * (1.0 + rng.choice([0.0, 3e-6, 6e-6], w.t.shape))
        w.B[...] = 1024.0 * equal_links(n)
    else:   # few values each, from 2^-149 on
        w.t[...] = 2.0 ** -139 * rng.integers(1, 2000, w.t.shape) * (1.0 + rng.choice([0.0, 1e-4], w.t.shape))
        w.B[...] = 2.0 ** np.triu(rng.integers(4, 11, w.B.shape), 1)
        w.B[...] = np.triu(w.B, 1) + np.triu(w.B, 1).transpose(0, 2, 1)
    assert np.isfinite(w.t).all()
    return w


VANISHING = ["to zero", "some to zero", "one value below the normal range", "few values below it"]


@pytest.mark.parametrize("kind", VANISHING)
def test_quotients_that_vanish(kind):
    check(vanishing(kind, 11, 24, batch(11), 6, 5), oracle=6)
    check(vanishing(kind, 16, 8, 1, 5, 6), oracle=1)


@pytest.mark.parametrize("kind", VANISHING)
def test_quotients_that_vanish_few_segments(kind):
    check(vanishing(kind, 12, 24, few_batch(12, 6), 5, 7), oracle=6, segments=6)
