"""What a call asks of the HIP runtime: allocations, kernels, launch sizes.  The library runs in a process of its own on a
runtime that only writes its requests down (fake_hip.c), so no GPU is needed; device pointers are never looked at."""
import json
import os
import subprocess
import sys

import pytest

from paper_2210_12219_amd import binding

HERE = os.path.dirname(os.path.abspath(__file__))

CHILD = r"""
import ctypes as C, json, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
fake.fake_reset.argtypes = [C.c_size_t, C.c_int]
fake.fake_log.restype = C.c_char_p
lib = C.CDLL(sys.argv[2])
for f in ("ppo_workspace_bytes", "ppo_solve_workspace_bytes"):
    if hasattr(lib, f):
        getattr(lib, f).restype = C.c_size_t
p, s = C.c_void_p(0x10000000), C.c_void_p(0)
out = []
for call in json.loads(sys.argv[3]):
    L, k, n = call["L"], call["k"], call["n"]
    fake.fake_reset(call.get("limit", 2**64 - 1), int(call.get("capturing", False)))
    head, res = (p, p, L, p, p, k, n, p, p, p), {}
    if call["entry"] == "sizes":
        res = {"least": lib.ppo_workspace_bytes(L, k, n), "whole": lib.ppo_solve_workspace_bytes(L, k, n)}
    elif call["entry"] == "ws":
        size = call["bytes"] if "bytes" in call else getattr(lib, call["size"])(L, k, n)
        res["rc"] = lib.ppo_solve_ws(*head, p, C.c_size_t(size), s)
    elif call["entry"] == "ct":
        res["rc"] = lib.ppo_solve_ct(p, p, p, L, p, p, p, k, n, p, p, p, s)
    else:
        res["rc"] = getattr(lib, call["entry"])(*head, s)
    res["log"] = [x.split() for x in fake.fake_log().decode().splitlines()]
    out.append(res)
print(json.dumps(out))
"""


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    if not os.path.exists(binding.LIB_PATH):
        from paper_2210_12219_amd import build
        build.build()
    fake = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-o", fake, os.path.join(HERE, "fake_hip.c")])

    def run(*calls):
        done = subprocess.run([sys.executable, "-c", CHILD, fake, binding.LIB_PATH, json.dumps(calls)],
                              capture_output=True, text=True, timeout=300)
        assert done.returncode == 0, done.stderr
        return json.loads(done.stdout)
    return run


def kernels(res):
    return [x[1] for x in res["log"] if x[0] == "launch"]


def allocations(res):
    return [int(x[1]) for x in res["log"] if x[0] == "malloc"]


# rows in LDS; in the scratch with 7 and 8 nodes; a launch per level; the largest shape; one instance of many nodes
SHAPES = [(50, 6, 1024), (128, 7, 1000), (100, 8, 300), (127, 9, 37), (100, 10, 64), (64, 11, 1), (128, 12, 150)]


@pytest.mark.parametrize("L,k,n", SHAPES)
@pytest.mark.parametrize("capturing", [False, True])
def test_solve_ws_works_on_the_given_scratch_alone(record, L, k, n, capturing):
    base = {"entry": "ws", "L": L, "k": k, "n": n, "capturing": capturing}
    least, whole = record({**base, "size": "ppo_workspace_bytes"}, {**base, "size": "ppo_solve_workspace_bytes"})
    for res in (least, whole):
        assert res["rc"] == 0 and not allocations(res)
    assert all("subset" in x for x in kernels(whole)), "the whole scratch is for the search by subsets"
    launches = [x for x in whole["log"] if x[0] == "launch"]
    assert len(launches) == (1 if k <= 8 else 1 + k), "all instances at once: tables, k - 1 levels, answer"


def test_sizes_of_the_scratch(record):
    for (L, k, n), res in zip(SHAPES, record(*({"entry": "sizes", "L": L, "k": k, "n": n} for L, k, n in SHAPES))):
        assert res["whole"] >= res["least"] > 0 and res["whole"] % 256 == 0
        assert res["whole"] <= max(res["least"], 1 << 30)
        rows = k * 2 ** (k - 1) * 2 * L
        areas = min(n, 1024, (1 << 30) // (rows + 65536))
        assert k <= 6 or res["whole"] >= areas * rows
    for L, k, n in ((0, 1, 1), (4, 5, 1), (129, 4, 1), (100, 13, 1), (4, 2, -1)):
        assert record({"entry": "sizes", "L": L, "k": k, "n": n})[0] | {"log": 0} == {"least": 0, "whole": 0, "log": 0}


def test_a_scratch_without_room_for_one_area(record):
    """64 layers on 11 nodes: the least scratch of one instance is smaller than its rows; the enumeration answers."""
    res, = record({"entry": "ws", "L": 64, "k": 11, "n": 1, "size": "ppo_workspace_bytes"})
    assert res["rc"] == 0 and not allocations(res) and not any("subset" in x for x in kernels(res))
    short, = record({"entry": "ws", "L": 64, "k": 11, "n": 1, "bytes": 256})
    assert short["rc"] == binding.PPO_ENOSPC and not short["log"]


@pytest.mark.parametrize("entry,L,k,n", [("ppo_solve", 127, 9, 37), ("ppo_solve", 100, 8, 300), ("ppo_solve", 128, 12, 150),
                                         ("ct", 100, 8, 64), ("ct", 50, 6, 1024)])
def test_less_scratch_where_memory_is_short(record, entry, L, k, n):
    """The areas wanted, then half as many, and so on to one; ppo_solve does without any."""
    base = {"entry": entry, "L": L, "k": k, "n": n}
    wanted, = allocations(record(base)[0])
    assert wanted <= 1 << 30
    one, = allocations(record({**base, "n": 1})[0])
    assert wanted % one == 0 and wanted // one == min(n, 1024, (1 << 30) // one)
    for most in (wanted - 1, wanted // 3, one):
        res, = record({**base, "limit": most})
        got, = allocations(res)
        assert res["rc"] == 0 and one <= got <= most < 2 * got + one and kernels(res)
        assert [x[0] for x in res["log"]].count("free") == 1
    res, = record({**base, "limit": one - 1})
    if entry == "ct":
        assert res["rc"] == binding.PPO_EHIP and not kernels(res) and not allocations(res)
        return
    # every ordering enumerated, on the least scratch; where there is no memory for that either, an error
    least = record({"entry": "sizes", "L": L, "k": k, "n": n})[0]["least"]
    assert (res["rc"] == 0) == (least < one) and (least < one) == bool(kernels(res))
    few = {**base, "n": 1, "limit": one - 1}
    res, = record(few)
    assert res["rc"] == 0 and kernels(res) and not any("subset" in x for x in kernels(res))


def test_a_shape_with_its_rows_in_lds_allocates_nothing(record):
    res, = record({"entry": "ppo_solve", "L": 50, "k": 6, "n": 1024})
    assert res["rc"] == 0 and not allocations(res) and len(kernels(res)) == 1


@pytest.mark.parametrize("entry", ["ppo_solve", "ws"])
@pytest.mark.parametrize("L,k,n", [(10, 8, 4_200_000), (3, 2, 70_000_000), (1, 1, 2**31 - 1)])
def test_millions_of_small_instances(record, entry, L, k, n):
    """A launch may have fewer than 2^32 threads."""
    res, = record({"entry": entry, "L": L, "k": k, "n": n, "bytes": 2**62})
    assert res["rc"] == 0, "a launch beyond the documented limits"
    grids = [int(x[2]) for x in res["log"] if x[0] == "launch"]
    assert sum(grids) == n and all("subset" in x for x in kernels(res))
