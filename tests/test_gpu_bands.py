"""Search by subsets on the ranges of cuts that a set can meet (ppo_bands.hip): ranges of every class (up to 16, 32, 64 and
128 entries, set by the capacities), with rows in LDS and in global memory.  ppo_solve takes that form for 1024 instances
and more on six to eight nodes and chains of more than 64 layers (six nodes: up to 80); the staged search always does.  Against the oracle's subset
route for some instances, and against batches small enough for the other form for all of them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import ppo_oracle as O
from paper_2210_12219_amd import workloads as W


def mixed_capacities(w, seed):
    """from none that fits (0.6 of the model together) over tight ones to nodes that hold all of it"""
    rng = np.random.default_rng(seed)
    total = w.m.astype(np.float64).sum(axis=1, keepdims=True)
    factor = np.exp(rng.uniform(np.log(0.6), np.log(4.0 * w.k), (w.n_inst, 1)))
    factor[rng.random((w.n_inst, 1)) < 0.6] = 1.0
    factor = np.where(factor == 1.0, rng.uniform(1.02, 1.5, factor.shape), factor)
    w.M[...] = (w.M / w.M.sum(axis=1, keepdims=True) * total * factor).astype(np.float32)
    return w


def same(got, ref):
    assert np.array_equal(got[0].view(np.uint32), ref[0].view(np.uint32))
    assert np.array_equal(got[2], ref[2]) and np.array_equal(got[1], ref[1])


@pytest.mark.parametrize("L,k", [(65, 6), (66, 8), (96, 7), (80, 6), (128, 8), (128, 7)])
@pytest.mark.parametrize("quantised", [False, True])
def test_many_long_chains(L, k, quantised):
    import torch
    from paper_2210_12219_amd import binding as ppo
    n = 1030
    w = mixed_capacities(W.random_instances(7000 + L + k, n, L, k, capacity_factor=1.3, quantised=quantised), L + k)
    w.t[::7, ::5] = 0.0
    w.t[3::11, ::3] = -0.0
    dev = ppo.to_device(w)
    got = [x.cpu().numpy() for x in ppo.ppo_solve(*dev)]
    ws = ppo.alloc_workspace(L, k, n)
    same([x.cpu().numpy() for x in ppo.ppo_solve(*dev, workspace=ws)], got)
    halves = [[x.cpu().numpy() for x in ppo.ppo_solve(*(a[i:i + 515].contiguous() for a in dev))] for i in (0, 515)]
    same(got, [np.concatenate([a, b]) for a, b in zip(*halves)])
    some = slice(0, 40)
    same([x[some] for x in got], O.subset_dp(w.t[some], w.m[some], w.M[some], w.B[some]))
    assert np.isinf(got[0]).any() and np.isfinite(got[0]).any()


@pytest.mark.parametrize("L,k,n", [(1, 1, 3), (5, 5, 4), (128, 2, 3), (64, 4, 1100), (17, 8, 40), (32, 8, 9), (100, 7, 20), (128, 8, 9),
                                   (9, 9, 4), (40, 9, 9), (128, 9, 3), (33, 10, 270), (100, 10, 5), (64, 11, 2), (30, 12, 2)])
def test_staged(L, k, n):
    import torch
    from paper_2210_12219_amd import binding as ppo
    for quantised in (False, True):
        w = mixed_capacities(W.random_instances(7500 + 3 * L + k, n, L, k, capacity_factor=1.3, quantised=quantised), n)
        ref = O.subset_dp(w.t, w.m, w.M, w.B) if n < 300 else [x.cpu().numpy() for x in ppo.ppo_solve(*ppo.to_device(w))]
        ws = ppo.alloc_workspace(L, k, n)
        keys = torch.empty(n, dtype=torch.int64, device="cuda:0")
        ppo.ppo_prepare(*ppo.to_device(w), ws)
        ppo.ppo_solve_subsets(L, k, n, ws, keys)
        same([x.cpu().numpy() for x in ppo.ppo_finalize(L, k, n, ws, keys)], ref)


def ample(w, seed):
    """1.2 to 4 times what the chain needs: from ranges of a part of the chain to all that leave every node a layer, so that some
    instances are searched on whole rows and others are not"""
    rng = np.random.default_rng(seed)
    total = w.m.astype(np.float64).sum(axis=1, keepdims=True)
    w.M[...] = (w.M / w.M.sum(axis=1, keepdims=True) * total * np.exp(rng.uniform(np.log(1.2), np.log(4.0), (w.n_inst, 1)))).astype(np.float32)
    w.t[::5, ::4] = 0.0
    return w


@pytest.mark.parametrize("L,k", [(68, 6), (69, 6), (79, 6), (70, 7), (71, 7), (128, 7), (72, 8), (127, 8), (128, 8)])
def test_ample_memory(L, k):
    """Ranges of up to 64 entries and one more, first cuts even and odd, rows in LDS and in global memory, the longest."""
    from paper_2210_12219_amd import binding as ppo
    w = ample(W.random_instances(7700 + L + k, 1030, L, k, quantised=L % 2 == 1), L)
    dev = ppo.to_device(w)
    got = [x.cpu().numpy() for x in ppo.ppo_solve(*dev)]
    halves = [[x.cpu().numpy() for x in ppo.ppo_solve(*(a[i:i + 515].contiguous() for a in dev))] for i in (0, 515)]
    same(got, [np.concatenate([a, b]) for a, b in zip(*halves)])
    same([x[:20] for x in got], O.subset_dp(w.t[:20], w.m[:20], w.M[:20], w.B[:20]))


@pytest.mark.parametrize("L,k,n", [(64, 1, 2), (64, 2, 3), (65, 2, 3), (128, 3, 40), (128, 6, 20), (71, 7, 5), (72, 8, 5), (128, 8, 12), (100, 8, 300),
                                   (73, 9, 4), (128, 9, 6), (100, 10, 6), (128, 10, 4), (70, 10, 270), (100, 11, 2), (80, 12, 2)])
def test_ample_memory_staged(L, k, n):
    """The same with the tables of ppo_prepare: one workgroup an instance of 8 or 16 waves, levels over many, with room for the
    table of whole rows and without."""
    import torch
    from paper_2210_12219_amd import binding as ppo
    w = ample(W.random_instances(7800 + L + k, n, L, k, quantised=k % 2 == 1), n)
    dev = ppo.to_device(w)
    ws = ppo.alloc_workspace(L, k, n)
    keys = torch.empty(n, dtype=torch.int64, device="cuda:0")
    ppo.ppo_prepare(*dev, ws)
    ppo.ppo_solve_subsets(L, k, n, ws, keys)
    got = [x.cpu().numpy() for x in ppo.ppo_finalize(L, k, n, ws, keys)]
    same(got, [x.cpu().numpy() for x in ppo.ppo_solve(*dev)])
    if k <= 10:
        same([x[:4] for x in got], O.subset_dp(w.t[:4], w.m[:4], w.M[:4], w.B[:4]))
