"""The benchmark's kernel meter: algorithmic bytes do not depend on how many
launches a kernel's work was reported as."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _stats(lib, binning_launches):
    timed = [0] * lib.NTIMED
    timed[lib.TIME_BINNING] = binning_launches
    ms = [0.0] * lib.NTIMED
    ms[lib.TIME_BINNING] = 0.25
    return {"timed_launches": timed, "timed_ms": ms, "bin_arcs": [7] * lib.NBINS, "bin_vertices": [3] * lib.NBINS,
            "iterations": [4, 2], "communities": [1000, 90]}


@pytest.mark.parametrize("launches", [6, 190])
def test_binning_bytes_are_one_walk_per_iteration(launches):
    sys.path.insert(0, ROOT)
    import bench
    from paper_2404_19634_amd import lib
    m = bench.KernelMeter(lib, 100_000)
    m.add(_stats(lib, launches))
    walks = 4 * ((100_000 + 31) // 32) + 2 * ((1000 + 31) // 32)
    want = bench.BIN_BYTES_PER_WORD * walks + bench.BIN_BYTES_PER_VERTEX * 3 * lib.NBINS
    assert m.bytes[lib.TIME_BINNING] == want
    assert m.launches[lib.TIME_BINNING] == launches and m.ms[lib.TIME_BINNING] == 0.25
