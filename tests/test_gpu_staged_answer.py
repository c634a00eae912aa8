"""The final stage (ppo_finalize) where its windows change form: up to 14 candidates (20 or 12 on longer chains) two at a time,
longer ones by minima over runs.  Equal layers and nodes of a given number of layers make every window that long."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import ppo_oracle as O
from paper_2210_12219_amd import workloads as W


@pytest.mark.parametrize("L,k,longest", [(30, 5, 7), (30, 5, 8), (30, 5, 9), (64, 9, 8), (65, 9, 16), (128, 12, 17), (128, 2, 127), (128, 3, 64),
                                         (12, 12, 8), (16, 2, 9), (64, 9, 14), (64, 9, 15), (65, 9, 20), (67, 9, 21), (68, 9, 12), (68, 9, 13),
                                         (128, 12, 12), (128, 12, 13)])
def test_windows(L, k, longest):
    import torch
    from paper_2210_12219_amd import binding as ppo
    w = W.random_instances(8100 + L + k, 3, L, k, quantised=True)
    w.m[...] = 1.0
    w.M[...] = longest
    w.M[1, 0] = 1.0   # windows of two kinds in one search
    w.t[2, ::4] = 0.0
    ref = O.subset_dp(w.t, w.m, w.M, w.B)
    ws = ppo.alloc_workspace(L, k, 3)
    keys = torch.empty(3, dtype=torch.int64, device="cuda:0")
    ppo.ppo_prepare(*ppo.to_device(w), ws)
    ppo.ppo_solve_subsets(L, k, 3, ws, keys)
    got = [x.cpu().numpy() for x in ppo.ppo_finalize(L, k, 3, ws, keys)]
    assert np.array_equal(got[0].view(np.uint32), ref[0].view(np.uint32))
    assert np.array_equal(got[1], ref[1]) and np.array_equal(got[2], ref[2])
    assert np.isfinite(got[0]).any()
