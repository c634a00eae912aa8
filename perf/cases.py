"""The work that a user of this package has it do, as cases that can be timed and compared.

A case is one call (or one sequence of staged calls) of the public entry points on a batch of instances that is
already on the GPU.  `path` names the entry points:

    solve       ppo_solve: the exact optimum of every instance (the call of the README); with `keep` the caller
                brings its own workspace and outputs, as a serving loop does
    enumerate   ppo_prepare, ppo_init_keys, ppo_solve_range over every rank, ppo_finalize: the staged search with
                every ordering evaluated in full (the step of bench.py)
    subsets     ppo_prepare, ppo_solve_subsets, ppo_finalize (bench.py --subsets)
    cluster     ppo_solve_cluster: hosting nodes and number of segments free, up to 20 nodes
    few         ppo_solve_cluster_few: up to 64 nodes, few segments
    ct          ppo_solve_ct: with the compute-time term
    kpath       ppo_place_kpath: the paper's own placement algorithm

`inputs` names the distribution (package module `workloads`); chains and clusters of other sizes are drawn from its
generic generator.  The data type is fixed by the entry points (binary32 in, binary32 and 32-bit integers out).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2210_12219_amd import binding as ppo
from paper_2210_12219_amd import workloads


def listed():
    return [
        # smallest call: many tiny problems, where launches and allocation are all there is
        {"name": "solve_tiny", "path": "solve", "inputs": "tiny", "L": 12, "k": 4, "n": 256, "keep": False},
        # ordinary batch of 50-layer convolutional chains on six nodes, in a loop that keeps its buffers
        {"name": "solve_resnet50", "path": "solve", "inputs": "resnet50_shaped", "L": 50, "k": 6, "n": 1024, "keep": True},
        # large batch of transformer chains on eight nodes; almost every ordering ties
        {"name": "solve_transformer", "path": "solve", "inputs": "transformer_encoder", "L": 96, "k": 8, "n": 4096,
         "keep": False},
        # long chains of an odd length, few instances
        {"name": "solve_long_odd", "path": "solve", "inputs": "random", "L": 127, "k": 9, "n": 37, "keep": True},
        # one large problem with tight memory
        {"name": "solve_large", "path": "solve", "inputs": "large", "L": 64, "k": 11, "n": 1, "keep": False},
        # the step of bench.py: every ordering's own dynamic programme
        {"name": "enumerate_headline", "path": "enumerate", "inputs": "headline", "L": 100, "k": 10, "n": 64},
        # the same instances by subsets of nodes, staged (bench.py --subsets)
        {"name": "subsets_headline", "path": "subsets", "inputs": "headline", "L": 100, "k": 10, "n": 64},
        # largest cluster of the subset form (bench.py --cluster 20)
        {"name": "cluster_mixed_20", "path": "cluster", "inputs": "cluster_mixed", "L": 100, "k": 20, "n": 1, "keep": True},
        # the paper's cluster: devices of one capacity at random places (bench.py --approx)
        {"name": "cluster_geometric_15", "path": "cluster", "inputs": "cluster_geometric", "L": 50, "k": 15, "n": 32,
         "capacity": 16.0, "keep": False},
        # the paper's largest cluster with a handful of partitions (bench.py --cluster 50)
        {"name": "few_mixed_50", "path": "few", "inputs": "cluster_mixed", "L": 100, "k": 50, "n": 1, "segments": 5, "keep": True},
        # compute-time term on the convolutional chains (bench.py --ct)
        {"name": "ct_resnet50", "path": "ct", "inputs": "resnet50_shaped", "L": 50, "k": 6, "n": 1024},
        # the paper's own algorithm on its largest cluster, its 50 runs at a time
        {"name": "kpath_geometric_50", "path": "kpath", "inputs": "cluster_geometric", "L": 50, "k": 50, "n": 50,
         "capacity": 32.0},
    ]


def _log_int(rng, lo, hi):
    """An integer in [lo, hi], evenly spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _batch(rng, most):
    return _log_int(rng, 1, max(1, min(4096, int(most))))


def draw(rng):
    path = rng.choice(["solve", "solve", "solve", "enumerate", "subsets", "cluster", "few", "ct", "kpath"])
    inputs = rng.choice(["random", "random", "quantised"])
    keep = rng.random() < 0.5
    if path in ("solve", "enumerate", "subsets"):
        k = rng.randint(6 if path == "enumerate" else 3, 10)
        L = rng.randint(max(k + 1, 10), 128)
        # orderings that stay below the largest listed case; chains whose rows exceed 96 entries cost more each
        most = 1.5e8 if L - k + 2 <= 96 else 1.2e7
        return {"path": path, "inputs": inputs, "L": L, "k": k, "n": _batch(rng, most / math.factorial(k)), "keep": keep}
    if path == "ct":
        k = rng.randint(3, 7)
        L = rng.randint(max(k + 1, 10), 100)
        return {"path": path, "inputs": inputs, "L": L, "k": k, "n": _batch(rng, 7e5 * (50.0 / L) ** 2 / math.factorial(k))}
    if path == "cluster":
        k = rng.randint(5, 19)
        geometric = rng.random() < 0.5
        L = 50 if geometric else rng.randint(20, 128)
        n = _batch(rng, min(256.0, 8e8 / (k * 2.0 ** (k - 1) * L)))
        c = {"path": path, "inputs": "cluster_geometric" if geometric else "cluster_mixed", "L": L, "k": k, "n": n, "keep": keep}
        if geometric:
            c["capacity"] = rng.choice([16.0, 32.0, 64.0])
        return c
    if path == "few":
        k = rng.randint(21, 64)
        segments = rng.randint(3, 5 if k <= 50 else 4)
        L = rng.randint(20, 128)
        rows = math.comb(k, segments - 1) * (segments - 1)
        return {"path": path, "inputs": "cluster_mixed", "L": L, "k": k, "n": _batch(rng, min(32.0, 9e7 / (rows * L))),
                "segments": segments, "keep": keep}
    k = rng.randint(5, 64)
    return {"path": path, "inputs": "cluster_geometric", "L": 50, "k": k, "n": _batch(rng, 128),
            "capacity": rng.choice([16.0, 32.0, 64.0])}


def _workload(case, seed):
    name, L, k, n = case["inputs"], case["L"], case["k"], case["n"]
    if name == "cluster_mixed":
        # clusters for few segments have nodes just large enough that the chain needs what it is allowed
        factor = 0.8 / case["segments"] if "segments" in case else 0.25
        return workloads.cluster_mixed(k, L=L, n_inst=n, seed=seed, capacity_factor=factor)
    if name == "cluster_geometric":
        return workloads.cluster_geometric(k, case["capacity"], n_inst=n, seed=seed)
    if name in ("random", "quantised"):
        return workloads.random_instances(seed, n, L, k, capacity_factor=1.3, quantised=name == "quantised")
    return workloads.WORKLOADS[name](n_inst=n, seed=seed)


def prepare(case, seed):
    w = _workload(case, seed)
    assert (w.L, w.k, w.n_inst) == (case["L"], case["k"], case["n"])
    path, L, k, n = case["path"], w.L, w.k, w.n_inst
    s = {"case": case, "dev": ppo.to_device(w), "out": None, "ws": None}
    if path in ("enumerate", "subsets"):
        s["ws"] = ppo.alloc_workspace(L, k, n)
        s["keys"] = torch.empty(n, dtype=torch.int64, device="cuda:0")
        s["out"] = ppo.alloc_outputs(n, k)
    elif path == "solve" and case["keep"]:
        s["ws"], s["out"] = ppo.alloc_workspace(L, k, n), ppo.alloc_outputs(n, k)
    elif path in ("cluster", "few") and case["keep"]:
        size = (ppo.ppo_cluster_workspace_bytes(L, k, n) if path == "cluster"
                else ppo.ppo_cluster_few_workspace_bytes(L, k, case["segments"], n))
        s["ws"] = torch.empty(size, dtype=torch.uint8, device="cuda:0")
    elif path == "ct":
        work, speed = workloads.compute_terms(w, seed=seed + 1, seconds=10.0, quantised=case["inputs"] == "quantised")
        s["work"], s["speed"] = torch.from_numpy(work).cuda(), torch.from_numpy(speed).cuda()
    elif path == "kpath":
        s["kappa"] = torch.from_numpy(np.ascontiguousarray(w.M[:, 0])).cuda()
    return s


def run(s):
    case, (t, m, M, B) = s["case"], s["dev"]
    path, L, k, n = case["path"], case["L"], case["k"], case["n"]
    if path == "solve":
        return ppo.ppo_solve(t, m, M, B, out=s["out"], workspace=s["ws"])
    if path in ("enumerate", "subsets"):
        ws, keys = s["ws"], s["keys"]
        ppo.ppo_prepare(t, m, M, B, ws)
        if path == "enumerate":
            ppo.ppo_init_keys(keys)
            ppo.ppo_solve_range(L, k, n, ws, 0, math.factorial(k), keys)
        else:
            ppo.ppo_solve_subsets(L, k, n, ws, keys)
        return (keys,) + ppo.ppo_finalize(L, k, n, ws, keys, out=s["out"])
    if path == "cluster":
        return ppo.ppo_solve_cluster(t, m, M, B, workspace=s["ws"])
    if path == "few":
        return ppo.ppo_solve_cluster_few(t, m, M, B, max_segments=case["segments"], workspace=s["ws"])
    if path == "ct":
        return ppo.ppo_solve_ct(t, m, s["work"], M, s["speed"], B)
    return ppo.ppo_place_kpath(t, m, s["kappa"], B, 5)


def _subset_ops(k, L, sizes):
    """One maximum and one minimum per entry and pair (node outside a set of c nodes, node of the set), one minimum
    per entry of the window of every row."""
    return sum(math.comb(k, c) * (k - c) * (2 * c + 1) * L for c in sizes)


def work(case):
    path, L, k, n = case["path"], case["L"], case["k"], case["n"]
    ins = 4 * (2 * L + k + k * k)
    outs = 4 * (1 + (k - 1) + k)
    if path in ("solve", "subsets"):
        ops = _subset_ops(k, L, range(k))
    elif path == "enumerate":
        # every ordering's k - 1 rows of L - k + 1 entries: a maximum with the link and at least one minimum each
        ops = math.factorial(k) * (k - 1) * (L - k + 1) * 2
        outs += 8
    elif path == "cluster":
        ops = _subset_ops(k, L, range(k))
        outs += 4
    elif path == "few":
        # the last level keeps one entry per row, which takes the whole row below it
        ops = _subset_ops(k, L, range(1, case["segments"]))
        outs += 4
    elif path == "ct":
        # the window minimum takes a maximum and a minimum per pair of ends that fit: a quarter of the chain, about
        ops = _subset_ops(k, L, range(k)) + 2 * sum(math.comb(k, c) * (k - c) for c in range(k)) * L * (L // 4)
        ins += 4 * (L + k)
    else:
        ins = 4 * (2 * L + 1 + k * k)
        outs = 4 * (1 + 1 + (L - 1) + k + 1)
        ops = L * L + k * k * math.ceil(math.log2(k * k))   # the partitioning step and the order of the links
    return {"bytes": float(n * (ins + outs)), "flops": float(n * ops)}


def tolerance(case):
    # one binary32 division per latency, exact minima and maxima, ties broken by a stated rule: every result is unique
    return "exact"
