"""The choice of a batch's captured graph (batch_graphs.h), without a GPU: a graph launches no
class by rows and by waves both, whatever came before."""
import os
import random
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2605_02224_amd", "csrc")


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("graphs") / "batch_graphs_check")
    subprocess.run([gxx, "-O1", "-std=c++17", "-I", CSRC,
                    os.path.join(HERE, "native", "batch_graphs_check.cpp"), "-o", exe], check=True)

    def ask(batches):
        text = "".join("%d %d %d\n" % b for b in batches)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, s.split())) for s in out.splitlines()]
    return ask


def test_sides_do_not_pile_up(choose):
    """Whole clouds, prefixes, whole clouds: the third batch replays the first one's graph."""
    full, prefix = (0, 0b1110, 0b1110), (0, 0b1110, 0)
    got = choose([full, prefix, full, prefix])
    assert got == [(7, 1, 0b1110 << 4), (0, 1, 0b1110), (7, 0, 0b1110 << 4), (0, 0, 0b1110)]


@pytest.mark.parametrize("seed", range(4))
def test_any_sequence(choose, seed):
    """Each graph launches every class with work on its side, no class twice, and is captured again
    only when it gains one: at most once a class."""
    rng = random.Random(seed)
    batches = []
    for _ in range(400):
        work = rng.randrange(16)
        batches.append((rng.randrange(2), work, work & rng.randrange(16) & 0b1110))
    grown = {}
    for (v, work, by_wave), (graph, again, launch) in zip(batches, choose(batches)):
        rows, waves = launch & 15, launch >> 4
        assert rows & waves == 0
        assert work & ~by_wave & ~rows == 0 and by_wave & ~waves == 0
        grown[(v, graph)] = grown.get((v, graph), 0) + again
    assert all(n <= 4 for n in grown.values()) and len(grown) <= 16
