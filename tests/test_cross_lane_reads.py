"""Reads of other lanes' registers stand where those lanes are active.  v_readlane reads a lane whether it is active or
not, but inside a branch that only one lane takes, the compiler may as well compute what is read there, for that lane
alone: what the others' registers hold then is anyone's guess."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2210_12219_amd", "csrc")
CROSS_LANE = re.compile(r"readlane|readfirstlane|__shfl|__ballot|_dpp|ds_bpermute")
ONE_LANE = re.compile(r"if\s*\(\s*(?:lane|tid|threadIdx\.x)\s*==\s*\w+\s*\)")


def branch(text, at):
    """the statement or block that follows the condition ending at `at`"""
    while text[at].isspace():
        at += 1
    depth, start = 0, at
    for i in range(at, len(text)):
        depth += text[i] in "({"
        depth -= text[i] in ")}"
        if depth == 0 and text[i] in ";}" and (text[i] == "}" or ";" in text[start:i + 1]):
            return text[start:i + 1]
    raise AssertionError("unbalanced braces")


def findings(text):
    text = re.sub(r"//[^\n]*", "", text)
    for m in ONE_LANE.finditer(text):
        body = branch(text, m.end())
        if CROSS_LANE.search(body):
            yield text[:m.start()].count("\n") + 1, body


def test_no_cross_lane_read_in_a_branch_of_one_lane():
    found = []
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h"))):
        found += [f"{os.path.basename(path)}:{line}" for line, _ in findings(open(path).read())]
    assert not found, found


def test_the_check_sees_what_it_should():
    assert list(findings("if (lane == 0) { for (;;) { x += readlane(w, i); } }"))
    assert list(findings("if (tid == 0)\n  y = __shfl(x, 3, 64);"))
    assert not list(findings("if (lane == 0) { a = 1; } x = __shfl(x, 3, 64);"))
    assert not list(findings("if (lane == s) a = x;\n y = readlane(x, 1); // if (lane == 0) readlane"))
