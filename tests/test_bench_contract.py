"""bench.py and the entry points keep their contract (no GPU needed for these checks)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_bench_refuses_more_than_one_gpu():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode != 0
    assert "one GPU" in r.stderr


def test_entry_points_exist():
    sys.path.insert(0, ROOT)
    import __graft_entry__ as g
    assert callable(g.build) and callable(g.smoke)


def test_traffic_figures_end_with_the_sources_of_the_kernels_they_were_read_from():
    """Every kernel that a launch of the two kinds of layers can be sent to counts."""
    import re
    sys.path.insert(0, ROOT)
    import bench
    csrc = os.path.join(ROOT, "paper_2310_19509_amd", "csrc")
    for own, sources in (("sbn_conv1x1.hip", bench.SOURCES_1X1), ("sbn_conv3x3.hip", bench.SOURCES_3X3)):
        called = set(re.findall(r"\b(launch_\w+)\(p, ", open(os.path.join(csrc, own)).read()))
        assert "launch_few" in called
        for f in os.listdir(csrc):
            text = open(os.path.join(csrc, f)).read()
            if f.endswith(".hip") and any(re.search(rf"^int {name}\([^;]*\n{{", text, re.M) for name in called):
                assert f in sources, (own, f)


def test_launches_counted_by_the_rule_of_the_library():
    """One image has 196 tiles of 8 x 8 pixels in the first block and 49 in the second and third, on 256 compute units."""
    sys.path.insert(0, ROOT)
    import bench
    import workloads as W
    assert bench.fused_pairs(W, 64, 256) == [0, 1, 2] and bench.fused_pairs(W, 2, 256) == [0, 1, 2]
    assert bench.fused_pairs(W, 1, 256) == [0]


def test_product_never_imports_the_oracle():
    """The library and its binding must not route through the CPU oracle."""
    pkg = os.path.join(ROOT, "paper_2310_19509_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".cpp", ".hip", ".h")):
                text = open(os.path.join(dirpath, f)).read()
                assert "oracle" not in text.lower(), os.path.join(dirpath, f)
