"""Cluster form (ppo_solve_cluster): number of segments, hosting nodes and cuts, compared bit for bit with
the CPU oracle of the cluster form; at sizes the oracle cannot reach, with what holds at any size."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import ppo_cluster_oracle as CO
from oracle import ppo_oracle as O
from paper_2210_12219_amd import workloads as W


@pytest.fixture(scope="module")
def ppo():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2210_12219_amd import binding
    binding.load()
    return binding


def bits(x):
    return np.asarray(x, dtype=np.float32).view(np.uint32)


def solve(ppo, w, pmax=None, workspace_bytes=None):
    import torch
    dev = ppo.to_device(w)
    ws = None
    if workspace_bytes is not None:
        ws = torch.empty(workspace_bytes, dtype=torch.uint8, device="cuda:0")
    out = ppo.ppo_solve_cluster(*dev, max_segments=pmax, workspace=ws)
    torch.cuda.synchronize()
    return tuple(x.cpu().numpy() for x in out)


def oracle(w, pmax, route):
    n = w.k
    beta = np.zeros(w.n_inst, np.float32)
    segs = np.zeros(w.n_inst, np.int32)
    cuts = np.zeros((w.n_inst, max(n - 1, 0)), np.int32)
    order = np.zeros((w.n_inst, n), np.int32)
    for i in range(w.n_inst):
        beta[i], segs[i], cuts[i], order[i] = route(w.t[i], w.m[i], w.M[i], w.B[i], pmax)
    return beta, segs, cuts, order


def assert_same(got, ref, what):
    bad = np.nonzero(bits(got[0]) != bits(ref[0]))[0]
    assert bad.size == 0, f"{what}: beta differs at instances {bad[:8]}: {got[0][bad[:4]]} vs {ref[0][bad[:4]]}"
    assert np.array_equal(got[1], ref[1]), f"{what}: number of segments differs"
    assert np.array_equal(got[3], ref[3]), f"{what}: node sequence differs"
    assert np.array_equal(got[2], ref[2]), f"{what}: cuts differ"


def test_cluster_small_shapes_ties_and_infeasible(ppo):
    """Random shapes from n = 1 and L = 1 up, clusters larger than the chain included, capacities from
    'nothing fits' to 'one node holds everything', values with few distinct levels every other seed."""
    for seed in range(40):
        rng = np.random.default_rng(7000 + seed)
        L = int(rng.integers(1, 15))
        n = int(rng.integers(1, 8))
        cf = float(rng.uniform(0.5, 1.0) * n) if seed % 3 else float(rng.uniform(0.8, 1.3))
        w = W.random_instances(seed, 24, L, n, capacity_factor=cf, quantised=bool(seed % 2))
        for pmax in sorted({1, max(1, n // 2), n}):
            print(f"cluster small seed={seed} L={L} n={n} pmax={pmax}", flush=True)
            ref = oracle(w, pmax, CO.exhaustive)
            assert_same(solve(ppo, w, pmax), ref, f"cluster L={L} n={n} pmax={pmax} seed={seed}")


def test_cluster_memory_rule_in_binary64(ppo):
    """Weights near 2^24: a segment of 2^24 + 1 does not fit a node of 2^24 (binary64 sums and comparison)."""
    big = np.float32(2.0 ** 24)
    rng = np.random.default_rng(78)
    L, n, cnt = 6, 4, 48
    t = rng.integers(1, 9, (cnt, L)).astype(np.float32)
    m = rng.choice(np.array([1, 2, 3, big, big + np.float32(2)], np.float32), (cnt, L), p=[0.3, 0.2, 0.2, 0.2, 0.1])
    M = rng.choice(np.array([big, big + np.float32(2), big + np.float32(4), 4], np.float32), (cnt, n))
    B = np.ones((cnt, n, n), np.float32)
    w = W.Workload("near 2^24", L, n, cnt, 78, t, m, M, B)
    for pmax in (2, 4):
        ref = oracle(w, pmax, CO.bruteforce)
        assert np.isfinite(ref[0]).sum() >= 6 and np.isinf(ref[0]).sum() >= 6
        assert_same(solve(ppo, w, pmax), ref, f"cluster near 2^24, pmax={pmax}")


def test_cluster_brute_force_definition(ppo):
    w = W.random_instances(11, 16, 9, 5, capacity_factor=2.0, quantised=True)
    print("cluster brute force L=9 n=5", flush=True)
    assert_same(solve(ppo, w), oracle(w, 5, CO.bruteforce), "cluster vs the definition")


@pytest.mark.parametrize("n,cap", [(5, 32), (5, 64), (10, 32), (10, 64), (10, 128), (12, 24), (15, 32)])
def test_cluster_paper_shaped(ppo, n, cap):
    """Sec. IV clusters: equal capacities, Shannon-rate bandwidths (few distinct values, many ties)."""
    w = W.cluster_geometric(n, cap, n_inst=2 if n >= 15 else 6)
    print(f"cluster geometric n={n} capacity={cap}", flush=True)
    assert_same(solve(ppo, w), oracle(w, n, CO.subset_dp), f"geometric n={n} cap={cap}")


def test_cluster_mixed_capacities_several_tiles(ppo):
    """L = 100 (two lanes-of-64 passes per row, ragged tail), n = 12 and 14, every max_segments."""
    w = W.cluster_mixed(12, L=100, n_inst=5)
    for pmax in (1, 2, 3, 5, 8, 12):
        print(f"cluster mixed n=12 pmax={pmax}", flush=True)
        assert_same(solve(ppo, w, pmax), oracle(w, pmax, CO.subset_dp), f"mixed n=12 pmax={pmax}")
    w = W.cluster_mixed(14, L=100, n_inst=2, seed=9)
    print("cluster mixed n=14", flush=True)
    assert_same(solve(ppo, w), oracle(w, 14, CO.subset_dp), "mixed n=14")
    w = W.random_instances(5, 3, 128, 11, capacity_factor=3.0)
    print("cluster L=128 n=11", flush=True)
    assert_same(solve(ppo, w), oracle(w, 11, CO.subset_dp), "L=128 n=11")


def test_cluster_batches_follow_the_workspace(ppo):
    """A workspace sized for four instances solves seven in batches of three; results do not depend on it."""
    w = W.cluster_mixed(9, L=60, n_inst=7, seed=3)
    full = solve(ppo, w)
    four = ppo.ppo_cluster_workspace_bytes(60, 9, 4)
    assert ppo.ppo_cluster_workspace_bytes(60, 9, 1) < four < ppo.ppo_cluster_workspace_bytes(60, 9, 7)
    print("cluster smaller workspace", flush=True)
    batched = solve(ppo, w, workspace_bytes=four)
    for a, b in zip(full, batched):
        assert np.array_equal(a, b)
    assert_same(full, oracle(w, 9, CO.subset_dp), "mixed n=9")
    with pytest.raises(ppo.PpoError) as err:
        solve(ppo, w, workspace_bytes=1 << 16)
    assert err.value.code == ppo.PPO_ENOSPC


def check_solution(w, i, got, pmax, rng, samples=300):
    """What must hold at any size: the reported solution is feasible with exactly the reported bottleneck
    (fixed-k evaluator on its nodes), and no other sequence tried does better or ties with a smaller one."""
    beta, p, cuts, order = got[0][i], int(got[1][i]), got[2][i], got[3][i]
    t, m, M, B = w.t[i], w.m[i], w.M[i], w.B[i]
    n = w.k
    assert 1 <= p <= pmax and list(order[p:]) == [-1] * (n - p) and list(cuts[p - 1:]) == [-1] * (n - p)
    idx = order[:p]
    assert len(set(idx.tolist())) == p
    b, feas = O.evaluate(t, m, M[idx], B[np.ix_(idx, idx)], np.arange(p), cuts[:p - 1])
    assert feas and bits(b) == bits(beta)
    assert bits(CO.sequence_beta(t, m, M, B, idx)) == bits(beta)
    mine = tuple(int(x) for x in idx)
    for s in range(samples):
        if s % 3 == 0:      # a random sequence
            q = int(rng.integers(1, pmax + 1))
            seq = rng.permutation(n)[:q]
        elif s % 3 == 1:    # the solution with one node replaced
            seq = idx.copy()
            free = np.setdiff1d(np.arange(n), idx)
            if free.size == 0:
                continue
            seq[int(rng.integers(0, p))] = int(rng.choice(free))
        else:               # the solution with two nodes swapped, or its last node dropped
            seq = idx.copy()
            if p >= 2 and s % 2:
                a, c = rng.choice(p, 2, replace=False)
                seq[a], seq[c] = seq[c], seq[a]
            elif p >= 2:
                seq = seq[:-1]
        other = bits(CO.sequence_beta(t, m, M, B, seq))
        assert other >= bits(beta)
        if other == bits(beta):
            assert mine <= tuple(int(x) for x in seq)


def test_cluster_of_twenty(ppo):
    """n = 20: a million node sets per instance.  Exact against the oracle for up to three segments;
    properties for the unrestricted search."""
    rng = np.random.default_rng(20)
    for w in (W.cluster_geometric(20, 32, n_inst=2), W.cluster_mixed(20, L=100, n_inst=1)):
        print(f"cluster n=20 {w.name} pmax=3", flush=True)
        three = solve(ppo, w, 3)
        assert_same(three, oracle(w, 3, CO.exhaustive), f"{w.name} pmax=3")
        print(f"cluster n=20 {w.name} unrestricted", flush=True)
        full = solve(ppo, w)
        for i in range(w.n_inst):
            assert bits(full[0][i]) <= bits(three[0][i])
            check_solution(w, i, full, 20, rng)
        print(f"cluster n=20 {w.name} pmax=6", flush=True)
        six = solve(ppo, w, 6)
        for i in range(w.n_inst):
            assert bits(full[0][i]) <= bits(six[0][i]) <= bits(three[0][i])
            check_solution(w, i, six, 6, rng)


def embed_with_decoys(w, i, n_big, rng):
    """Instance i of w inside a cluster of n_big nodes: the real nodes keep their relative order (so the
    lexicographic tie rule carries over), the others hold less than the lightest layer and can host nothing."""
    n0 = w.k
    pos = np.sort(rng.choice(n_big, n0, replace=False))
    M = np.full(n_big, 0.5 * float(w.m[i].min()), np.float32)
    assert M[0] > 0 and (M[0] < w.m[i]).all()
    M[pos] = w.M[i]
    up = np.triu(np.exp(rng.uniform(np.log(1.0), np.log(100.0), (n_big, n_big))), 1)
    B = (up + up.T).astype(np.float32)
    B[np.ix_(pos, pos)] = w.B[i]
    return pos, M, B


def test_cluster_of_twenty_exact_through_decoy_nodes(ppo):
    """n = 20 with every segment count allowed, bit for bit: a cluster of 11 to 13 real nodes that the oracle
    solves, plus nodes too small for any layer, which change nothing (the oracle's own pins show that).
    Expected beta, segment count, cuts are the small cluster's; the node sequence is the small one's through
    the embedding.  (The nodes that hold no layer can be left out by the search; the next test is searched whole.)"""
    import torch
    rng = np.random.default_rng(2020)
    cases = [(W.random_instances(311, 2, 100, 12, capacity_factor=1.7), "L=100, eight segments or so"),
             (W.cluster_mixed(13, L=100, n_inst=1, seed=21), "L=100 mixed"),
             (W.random_instances(312, 2, 128, 11, capacity_factor=2.5), "L=128"),
             (W.cluster_geometric(12, 16, n_inst=2, seed=23), "paper-shaped, ties")]
    for w, what in cases:
        n0 = w.k
        t = np.ascontiguousarray(w.t)
        m = np.ascontiguousarray(w.m)
        Ms, Bs, poss = [], [], []
        for i in range(w.n_inst):
            pos, M, B = embed_with_decoys(w, i, 20, rng)
            poss.append(pos); Ms.append(M); Bs.append(B)
        big = W.Workload(w.name + "+decoys", w.L, 20, w.n_inst, w.seed, t, m, np.stack(Ms), np.stack(Bs))
        print(f"cluster n=20 through decoys: {what}", flush=True)
        got = solve(ppo, big)
        for i in range(w.n_inst):
            beta, p, cuts, order = CO.subset_dp(w.t[i], w.m[i], w.M[i], w.B[i])
            assert bits(got[0][i]) == bits(beta) and got[1][i] == p, (what, i, got[0][i], beta, got[1][i], p)
            want_order = np.full(20, -1, np.int32)
            want_order[:p] = poss[i][order[:p]]
            want_cuts = np.full(19, -1, np.int32)
            want_cuts[:max(p - 1, 0)] = cuts[:max(p - 1, 0)]
            assert np.array_equal(got[3][i], want_order), (what, i, got[3][i], want_order)
            assert np.array_equal(got[2][i], want_cuts), (what, i)
        assert max(int(x) for x in got[1]) >= 2


@pytest.mark.parametrize("n0,L,cf", [(12, 100, 1.7), (11, 128, 2.5), (13, 70, 1.4)])
def test_cluster_of_twenty_searched_whole(ppo, n0, L, cf):
    """The same with a million node sets, 32-bit row numbers and every level of the DP for sure: transfer sizes and
    bandwidths differ by less than a part in a thousand, so that any bound within 2^-8 of the optimum lets all of the
    69 to 127 cuts pass, which is more than a search can be confined to."""
    rng = np.random.default_rng(n0 + L)
    w = W.random_instances(400 + L, 2, L, n0, capacity_factor=cf)
    poss, Ms, Bs = [], [], []
    w.t[...] = 1.503 + 1e-3 * rng.random(w.t.shape)
    for i in range(w.n_inst):
        pos, M, B = embed_with_decoys(w, i, 20, rng)
        up = np.triu(1.0 + 1e-4 * rng.random((20, 20)), 1).astype(np.float32)
        B = up + up.T
        w.B[i] = B[np.ix_(pos, pos)]
        poss.append(pos); Ms.append(M); Bs.append(B)
    big = W.Workload(w.name + "+decoys", L, 20, w.n_inst, w.seed, w.t, w.m, np.stack(Ms), np.stack(Bs))
    print(f"cluster n=20 whole, {n0} real nodes, L={L}", flush=True)
    got = solve(ppo, big)
    for i in range(w.n_inst):
        beta, p, cuts, order = CO.subset_dp(w.t[i], w.m[i], w.M[i], w.B[i])
        assert p >= 3
        assert bits(got[0][i]) == bits(beta) and got[1][i] == p, (i, got[0][i], beta, got[1][i], p)
        assert list(got[3][i]) == list(poss[i][order[:p]]) + [-1] * (20 - p)
        assert list(got[2][i]) == list(cuts[:p - 1]) + [-1] * (20 - p)


def test_cluster_seventeen_and_eighteen_against_the_oracle(ppo):
    """Above n = 16 with every segment count allowed and a short chain, where the oracle still finishes."""
    for n, L, seed, cf in ((17, 16, 927, 0.35), (18, 12, 927, 0.5), (17, 12, 920, 0.35), (17, 16, 917, 0.35)):
        w = W.random_instances(seed, 1, L, n, capacity_factor=cf * n)
        print(f"cluster n={n} L={L}", flush=True)
        ref = oracle(w, n, CO.subset_dp)
        assert ref[1][0] >= 5
        assert_same(solve(ppo, w), ref, f"n={n} L={L}")


def test_cluster_sixteen_against_the_oracle(ppo):
    w = W.cluster_mixed(16, L=100, n_inst=1, seed=12)
    print("cluster n=16 L=100", flush=True)
    assert_same(solve(ppo, w), oracle(w, 16, CO.subset_dp), "mixed n=16")


def test_layer_graph_to_placement(ppo):
    """End to end as in the paper: a layer graph with shortcuts (Sec. III-A) -> chain -> exact partition and
    placement on a cluster.  The chain comes from the library's host front-end; the search from the GPU."""
    import torch
    rng = np.random.default_rng(3)
    edges, v = [], 0
    for _ in range(12):              # twelve residual blocks: in -> a -> b -> add, in -> add
        a, b, add = v + 1, v + 2, v + 3
        edges += [(v, a), (a, b), (b, add), (v, add)]
        v = add
    n_vertices = v + 1
    weight = rng.uniform(0.5, 12.0, n_vertices).astype(np.float32)
    out = rng.uniform(1.0, 30.0, n_vertices).astype(np.float32)
    t, m, point = ppo.ppo_chain_from_dag(n_vertices, edges, weight, out)
    assert list(point) == [3 * i for i in range(13)] and len(t) == 13      # the block boundaries, nothing inside
    n = 7
    M = np.full(n, 0.3 * float(m.sum()), np.float32)
    w = W.cluster_geometric(n, 1.0, n_inst=1, seed=11)                      # for its bandwidth matrix
    dev = [torch.tensor(x[None], device="cuda:0") for x in (t, m, M)] + [torch.tensor(w.B, device="cuda:0")]
    print("layer graph -> chain -> cluster", flush=True)
    got = tuple(x.cpu().numpy() for x in ppo.ppo_solve_cluster(*dev))
    torch.cuda.synchronize()
    beta, p, cuts, order = CO.exhaustive(t, m, M, w.B[0])
    assert bits(got[0][0]) == bits(beta) and got[1][0] == p >= 4
    assert np.array_equal(got[2][0], cuts) and np.array_equal(got[3][0], order)


def test_more_instances_than_one_launch_takes(ppo):
    """40,000 instances: the tables, the level launches and the trace all go in several pieces (a launch
    covers 32,768 instances at most); sampled instances against the oracle."""
    import torch
    w = W.random_instances(77, 40000, 10, 4, capacity_factor=2.0)
    print("cluster, 40000 instances", flush=True)
    out = solve(ppo, w)
    rng = np.random.default_rng(0)
    for i in list(rng.choice(w.n_inst, 200, replace=False)) + [0, 32767, 32768, w.n_inst - 1]:
        b, p, cu, o = CO.subset_dp(w.t[i], w.m[i], w.M[i], w.B[i])
        assert bits(out[0][i]) == bits(b) and out[1][i] == p, i
        assert np.array_equal(out[2][i], cu) and np.array_equal(out[3][i], o), i
    # the fixed-k routes on as many
    w3 = W.random_instances(78, 40000, 8, 3, capacity_factor=1.6)
    dev = ppo.to_device(w3)
    print("fixed k, 40000 instances", flush=True)
    full = tuple(x.cpu().numpy() for x in ppo.ppo_solve(*dev))
    ws = ppo.alloc_workspace(8, 3, w3.n_inst)
    keys = torch.empty(w3.n_inst, dtype=torch.int64, device="cuda:0")
    ppo.ppo_prepare(*dev, ws)
    ppo.ppo_init_keys(keys)
    ppo.ppo_solve_subsets(8, 3, w3.n_inst, ws, keys)
    sub = tuple(x.cpu().numpy() for x in ppo.ppo_finalize(8, 3, w3.n_inst, ws, keys))
    torch.cuda.synchronize()
    for a, b in zip(full, sub):
        assert np.array_equal(a.view(np.uint32) if a.dtype == np.float32 else a, b.view(np.uint32) if b.dtype == np.float32 else b)
    for sl in (slice(0, 150), slice(32700, 32850), slice(-150, None)):
        ref = O.bruteforce(w3.t[sl], w3.m[sl], w3.M[sl], w3.B[sl])
        assert np.array_equal(bits(full[0][sl]), bits(ref[0])) and np.array_equal(full[2][sl], ref[2])
        assert np.array_equal(full[1][sl], ref[1])


@pytest.mark.parametrize("L", [2, 3, 33, 62, 63, 64, 65, 127, 128])
def test_cluster_rows_at_the_edges_of_a_wave(ppo, L):
    """Chain lengths around the ones at which the layout of rows over lanes changes, windows from one layer to the whole
    chain, an odd number of sets per wave, and a bounded number of segments."""
    for n, cf, quantised in ((3, 3.5, False), (5, 1.3, True), (6, 2.5, False)):
        w = W.random_instances(900 + L + n, 6, L, min(n, L), capacity_factor=cf, quantised=quantised)
        for pmax in (2, w.k):
            print(f"cluster edges L={L} n={w.k} pmax={pmax}", flush=True)
            assert_same(solve(ppo, w, pmax), oracle(w, pmax, CO.exhaustive), f"cluster edges L={L} n={w.k} pmax={pmax}")


@pytest.mark.parametrize("n,L", [(2, 2), (5, 12), (7, 70), (9, 128)])
def test_links_that_take_no_time_tie_with_none(ppo, n, L):
    """Transfers of size 0 and nodes that hold the whole chain: a segment more costs nothing, and the smaller node sequence
    wins whether it crosses links or not."""
    rng = np.random.default_rng(100 * n + L)
    w = W.random_instances(40 + n, 6, L, n, capacity_factor=1.5)
    w.t[:, rng.random(L) < 0.5] = 0.0
    w.t[:, :1] = -0.0
    for i in range(w.n_inst):
        w.M[i, rng.integers(1, n):] = 1.01 * w.m[i].sum()
    for pmax in (1, n):
        ref = oracle(w, pmax, CO.subset_dp)
        assert_same(solve(ppo, w, pmax), ref, f"no time n={n} L={L} pmax={pmax}")
    assert (ref[0] == 0).all() and (ref[1] > 1).any()
