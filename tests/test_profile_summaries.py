"""Figures from profiles/ are quoted only while the kernel they were measured on is the one in the tree."""
import os
import shutil

from paper_2210_12219_amd import profile_summary as P

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_a_summary_counts_while_the_code_is_the_one_profiled(tmp_path):
    csrc = tmp_path / "csrc"
    csrc.mkdir()
    shutil.copy(os.path.join(P.CSRC, "ppo_cluster.hip"), csrc)
    source = csrc / "ppo_cluster.hip"
    summary = tmp_path / "cluster.md"
    text = "# cluster\n\nsource: ppo_cluster.hip\nsource_digest: {}\ntraffic_bytes_per_launch: 12.5\n"
    summary.write_text(text.format(P.source_digest(["ppo_cluster.hip"], str(csrc))))
    code = source.read_text()
    assert P.current_summary(str(summary), str(csrc))["traffic_bytes_per_launch"] == 12.5
    source.write_text("// another comment\n" + code.replace("\n", "\n\n", 40))
    assert P.current_summary(str(summary), str(csrc))["traffic_bytes_per_launch"] == 12.5
    source.write_text(code.replace("cl_pk_min(v, x[C - 1])", "cl_pk_max(v, x[C - 1])"))
    assert source.read_text() != code and P.current_summary(str(summary), str(csrc)) == {}
    # a summary that does not say what code it is of, whatever version it names
    source.write_text(code)
    summary.write_text("ppo_version: 205\ntraffic_bytes_per_launch: 12.5\n")
    assert P.current_summary(str(summary), str(csrc)) == {}


def test_bench_quotes_current_summaries_only():
    import bench
    for name in os.listdir(os.path.join(ROOT, "profiles")):
        path = os.path.join(ROOT, "profiles", name)
        assert bench.profiled(name[:-3]) == P.current_summary(path)
    assert bench.profiled("no_such_summary") == {}
    # the headline's own
    assert bench.profiled("enumerate_paired_headline")["valu_issue"] > 0.0
