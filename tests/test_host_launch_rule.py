"""The rules that choose a launch's kernel and layout (launch_rule.h), without a GPU."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2605_02224_amd", "csrc")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("rule") / "launch_rule_check")
    subprocess.run([gxx, "-O1", "-std=c++17", "-I", CSRC,
                    os.path.join(HERE, "native", "launch_rule_check.cpp"), "-o", exe], check=True)

    def ask(*launches):
        """launches: dicts; the answers (kernel, bucketed, lanes, queries per wavefront)."""
        text = ""
        for l in launches:
            n = l.get("n", 400000)
            text += "%d %d %d %d %d %d %d\n" % (l["nq"], l["k"], l.get("var", 0), l.get("m", n), n,
                                                l.get("longest", 300), l.get("planes", 0))
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [(a, int(b), int(c), int(d)) for a, b, c, d in (s.split() for s in out.splitlines())]
    return ask


SIZES = [1, 24, 300, 4096, 4097, 8191, 8192, 8193, 12288, 16384, 16385, 32768, 65536, 65537, 98304,
         98305, 131072, 131073, 196608, 262143, 262144, 262145, 1000000]


def test_layout_fits_the_wavefront(rule):
    """Lanes per query times queries fit 64 lanes, for every launch."""
    launches = [dict(nq=nq, k=k, var=v, m=m, longest=g) for nq in SIZES for k in (1, 2, 8, 16, 17, 32, 33, 64)
                for v in (0, 1) for m in (400000, 100000, 300) for g in (300, 3000, 60000)]
    for l, (walk, _, lanes, per) in zip(launches, rule(*launches)):
        assert lanes in (8, 16) and 1 <= per <= 64 // lanes, (l, lanes, per)
        assert lanes == 16 or l["k"] <= 32, l


def test_hubs(rule):
    """A list that is a good part of the cloud: larger launches go by rows, as small ones and
    single neighbours, bucketed and with 16 lanes, need not."""
    hub = dict(n=60000, longest=17096)
    ask = [dict(nq=nq, k=k, **hub) for nq, k in ((300, 64), (8192, 32), (8193, 17), (16384, 32), (65536, 64),
                                                 (200000, 20), (65536, 16), (65537, 8))]
    assert [a[0] for a in rule(*ask)] == ["waves", "waves", "rows", "rows", "rows", "rows", "waves", "rows"]
    assert [a[0] for a in rule(*[dict(nq=nq, k=k, var=1, **hub) for nq in (10000, 70000, 500000)
                                 for k in (4, 32)])] == ["rows"] * 6
    assert [a[0] for a in rule(*[dict(nq=nq, k=32, m=20000, **hub) for nq in (10000, 70000, 500000)])] == ["rows"] * 3
    assert rule(dict(nq=200000, k=1, **hub)) == [("waves", 1, 16, 4)]
    # (a sheet's longest list, n / 32, is none)
    assert rule(dict(nq=200000, k=32, n=400000, longest=12366)) == [("waves", 0, 16, 4)]
    assert [a[:2] for a in rule(*[dict(nq=nq, k=1, **hub) for nq in (16385, 32767, 32768)])] == [
        ("waves", 0), ("waves", 0), ("waves", 1)]


def test_long_lists(rule):
    """Longer lists than most clouds have, but none that many queries meet (a height field): 16
    lanes for single neighbours, and no scan of one list at a time for a k and prefix per query."""
    sheet = dict(n=400000, longest=2755)
    assert rule(dict(nq=200000, k=1, **sheet)) == [("waves", 0, 16, 4)]
    assert rule(dict(nq=200000, k=1)) == [("waves", 0, 8, 8)]
    assert [a[0] for a in rule(*[dict(nq=nq, k=k, var=1, **sheet) for nq in (70000, 200000)
                                 for k in (4, 32)])] == ["waves"] * 4


def test_few_queries_in_prefixes(rule):
    """One short query to a wavefront: rows where a prefix leaves the waves' batches half empty; four
    descents to a wavefront for single neighbours."""
    ask = [dict(nq=nq, k=k, m=m) for nq, k, m in (
        (5001, 2, 100000), (8191, 4, 200000), (8191, 8, 12000), (6501, 5, 4000))]
    assert [a[0] for a in rule(*ask)] == ["rows"] * 4
    ask = [dict(nq=nq, k=k, m=m) for nq, k, m in (
        (5000, 2, 100000), (8192, 4, 200000), (8191, 8, 13000), (6500, 8, 4000), (8191, 9, 4000),
        (16384, 17, 100000), (16384, 64, 200000), (8191, 1, 4000), (8191, 2, 400000), (8191, 5, 100000))]
    assert [a[0] for a in rule(*ask)] == ["waves"] * 10
    assert rule(*[dict(nq=nq, k=1) for nq in (3072, 3073, 8191, 16384, 65535, 65536)]) == [
        ("waves", 0, 16, 1), ("waves", 0, 16, 4), ("waves", 0, 16, 4), ("waves", 0, 16, 4),
        ("waves", 0, 16, 4), ("waves", 0, 8, 8)]


def test_a_k_and_prefix_per_query(rule):
    """Waves while they are not bucketed, the scan kernel only for long rows of many queries, rows
    for short rows of many."""
    ask = [dict(nq=nq, k=k, var=1) for nq, k in (
        (65536, 64), (65537, 32), (98304, 32), (98304, 17), (131072, 16), (262143, 4), (262143, 1))]
    assert [a[0] for a in rule(*ask)] == ["waves"] * 7
    assert [a[0] for a in rule(*[dict(nq=nq, k=k, var=1) for nq, k in (
        (98305, 17), (65537, 33), (131072, 64), (1000000, 32))])] == ["scan"] * 4
    assert [a[0] for a in rule(*[dict(nq=nq, k=k, var=1) for nq, k in (
        (131073, 5), (262144, 16), (262144, 2), (262144, 1), (1000000, 8))])] == ["rows"] * 5
