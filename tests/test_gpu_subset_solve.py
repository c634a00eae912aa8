"""ppo_solve by subsets of nodes: the shapes at which the kernel changes form (64 layers: two sets to a wave or one; rows
in LDS or in global memory; beyond 8 nodes a launch per level), and quotients so close that codes are shared and the
search is repeated on a narrower range.  Bit for bit against the oracle's subset route."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import ppo_oracle as O
from paper_2210_12219_amd import workloads as W


def check(w, static=False):
    import torch
    from paper_2210_12219_amd import binding as ppo
    dev = ppo.to_device(w)
    ref = O.subset_dp(w.t, w.m, w.M, w.B)
    ws = ppo.alloc_workspace(w.L, w.k, w.n_inst)
    forms = {"own scratch": lambda: ppo.ppo_solve(*dev), "given scratch": lambda: ppo.ppo_solve(*dev, workspace=ws)}
    if static:
        forms["static scratch"] = lambda: ppo.ppo_solve_static(*dev, out=ppo.alloc_outputs(w.n_inst, w.k))
    for name, call in forms.items():
        got = [x.cpu().numpy() for x in call()]
        torch.cuda.synchronize()
        assert np.array_equal(got[0].view(np.uint32), ref[0].view(np.uint32)), name
        assert np.array_equal(got[2], ref[2]) and np.array_equal(got[1], ref[1]), name
    return ref


@pytest.mark.parametrize("L,k,n", [(1, 1, 3), (128, 1, 2), (2, 2, 5), (63, 6, 7), (64, 6, 7), (65, 6, 7), (128, 6, 3), (62, 7, 3),
                                   (64, 7, 3), (128, 7, 3), (30, 8, 9), (64, 8, 3), (65, 8, 3), (128, 8, 2), (9, 9, 4),
                                   (64, 9, 3), (65, 9, 3), (127, 9, 2), (40, 10, 19), (64, 11, 1), (20, 12, 3)])
def test_shapes_where_the_kernel_changes_form(L, k, n):
    for quantised in (False, True):
        check(W.random_instances(5000 + 13 * L + k, n, L, k, capacity_factor=1.4, quantised=quantised), static=True)


@pytest.mark.parametrize("L,k", [(40, 5), (50, 7), (100, 8), (48, 9), (70, 9)])
def test_quotients_a_few_units_apart(L, k):
    """Sizes that differ in the last bits beside a few that are far away: the range of the quotients is wide, so those
    near the optimum share a code (and, at nine nodes, a bucket of the counting sort that is too large to be told apart)."""
    w = W.random_instances(6000 + L, 6, L, k, capacity_factor=1.5)
    rng = np.random.default_rng(L)
    near = (np.float32(1.0).view(np.uint32) + rng.integers(0, 3000, w.t.shape).astype(np.uint32)).view(np.float32)
    w.t[:] = near
    w.t[:, :: 9] = np.float32(1e-6)
    w.t[:, 5] = np.float32(1e6)
    w.B[:] = np.where(np.eye(k, dtype=bool), 0, np.float32(3.0))
    ref = check(w)
    assert np.isfinite(ref[0]).any()
    w.t[:, 1::2] = 0.0                   # an optimum of 0 or not, and zeros of both signs
    w.t[:, 3::4] = -0.0
    check(w)


def test_more_instances_than_row_areas():
    """With the static scratch 27 of these share 16 MiB: several rounds of launches."""
    check(W.random_instances(6500, 27, 30, 11, capacity_factor=1.3), static=True)


@pytest.mark.parametrize("L,k,n", [(70, 7, 1100), (22, 8, 300)])
def test_a_workgroup_with_several_instances(L, k, n):
    """Rows in global memory, fewer areas than instances (1024 of ppo_solve's own, fewer in the least scratch): a workgroup
    takes another instance on the tables and rows of the last, with capacities from none that fits to all that fit."""
    import torch
    from paper_2210_12219_amd import binding as ppo
    w = W.random_instances(6600 + L, n, L, k, capacity_factor=1.4)
    w.M[...] *= np.exp(np.random.default_rng(n).uniform(np.log(0.4), np.log(30.0), (n, 1))).astype(np.float32)
    ref = check(w)
    least, area = ppo.ppo_workspace_bytes(L, k, n), ppo.ppo_solve_workspace_bytes(L, k, 1)
    areas = least // area
    assert 1 <= areas < min(n, 1024) and np.isinf(ref[0][areas:]).any() and np.isfinite(ref[0][areas:]).any()
    out = ppo.ppo_solve(*ppo.to_device(w), workspace=torch.empty(least, dtype=torch.uint8, device="cuda:0"))
    got = [x.cpu().numpy() for x in out]
    assert np.array_equal(got[0].view(np.uint32), ref[0].view(np.uint32))
    assert np.array_equal(got[2], ref[2]) and np.array_equal(got[1], ref[1])
