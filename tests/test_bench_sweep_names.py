"""The benchmark looks up the counters of the kernels that a solve's sweeps
launch (no GPU: the names are those of the built library's kernels)."""
import json
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402

STORED = {"edge_state": 1}
CHUNKED = {"edge_state": 2, "stateless_depth": 3, "series_reciprocal": 3, "tile_chunk": 2}
TILES = dict(CHUNKED, tile_chunk=1, stateless_depth=2, series_reciprocal=1)


@pytest.mark.parametrize("plan,count", [(STORED, 3), (CHUNKED, 1), (TILES, 1)])
@pytest.mark.parametrize("prec", ["mixed", "fp32"])
def test_names_are_kernels_of_the_library(plan, count, prec):
    lib = os.path.join(ROOT, "paper_0810_1648_amd", "libgabp_svm.so")
    nm = shutil.which("nm")
    if nm is None or not os.path.exists(lib):
        pytest.skip("needs nm and the built library")
    symbols = subprocess.run([nm, "-D", "-C", lib], capture_output=True, text=True, check=True).stdout
    names = bench.launched_sweep_names(prec, plan)
    assert len(names) == len(set(names)) == count
    for n in names:
        assert n + "(gabp::SweepArgs)" in symbols, n


def test_traffic_is_the_mean_over_a_period(tmp_path):
    names = bench.launched_sweep_names("mixed", STORED)
    entries = {"void " + n + "(gabp::SweepArgs)": {"traffic_bytes": b} for n, b in zip(names, (1e9, 2e9, 6e9))}
    path = tmp_path / "traffic.json"
    path.write_text(json.dumps({"kernel_source_sha256": bench.device_source_hash(), "entries": entries}))
    assert bench.sweep_traffic(str(path), "mixed", STORED) == 3.0
    assert bench.sweep_traffic(str(path), "mixed", CHUNKED) is None
    del entries["void " + names[1] + "(gabp::SweepArgs)"]
    path.write_text(json.dumps({"kernel_source_sha256": bench.device_source_hash(), "entries": entries}))
    assert bench.sweep_traffic(str(path), "mixed", STORED) is None
