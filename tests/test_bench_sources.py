"""The traffic figure of the benchmark holds for the sources that it was taken with:
those it names are the ones that choose, set up and run the register tile kernel's
launches, on the host too (which tiles a pass visits decides what it moves)."""
import glob
import os

import bench

CSRC = os.path.join(bench.ROOT, "paper_1612_08091_amd", "csrc")


def test_every_source_of_a_launch_is_covered():
    named = {os.path.join(bench.ROOT, s) for s in bench.TRAFFIC_SOURCES}
    assert all(os.path.exists(s) for s in named)
    for path in glob.glob(os.path.join(CSRC, "*")):
        with open(path) as f:
            text = f.read()
        if "launch_tile_reg(" in text or "plan_passes_relabel(" in text or "compile_pass(const" in text:
            assert path in named, path
