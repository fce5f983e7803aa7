"""bench.py reports counter traffic only while the kernel source and the headers
it is built from are those the counters were taken on."""
from __future__ import annotations

import hashlib
import os
import re
import shutil

import pytest

import bench

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2106_02858_amd", "csrc")
CASES = [("k_stage_col<3,false,false>", 48000, bench.MEASURED_TRAFFIC, "kernels.hip"),
         ("k_stage_tile<3,false,false>", 48000, bench.MEASURED_TRAFFIC_FP64, "kernels.hip"),
         ("k_stage_col<2,false,false>", 1572864, bench.MEASURED_TRAFFIC_Q2, "kernels.hip"),
         ("k_stage2d<float,3,true>", 22500, bench.MEASURED_TRAFFIC_2D, "kernels2d.hip")]


def test_headers_of_the_kernels_are_the_measured_ones():
    h = hashlib.sha256(b"".join(open(os.path.join(CSRC, n), "rb").read() for n in bench.KERNEL_HEADERS)).hexdigest()
    for _, _, table, _ in CASES:
        for t in table if isinstance(table, list) else [table]:
            assert t["headers_sha256"] == h
    for _, _, _, source in CASES:  # every header that a kernel source includes is among them
        mine = re.findall(r'^#include "([^"]+)"', open(os.path.join(CSRC, source)).read(), re.M)
        assert set(mine) <= set(bench.KERNEL_HEADERS)


@pytest.mark.parametrize("kernel,K,table,source", CASES)
@pytest.mark.parametrize("changed", [None, *bench.KERNEL_HEADERS, "source"])
def test_a_changed_file_takes_the_traffic_back(tmp_path, monkeypatch, kernel, K, table, source, changed):
    csrc = tmp_path / "paper_2106_02858_amd" / "csrc"
    csrc.mkdir(parents=True)
    for n in (source, *bench.KERNEL_HEADERS):
        shutil.copy(os.path.join(CSRC, n), csrc / n)
    if changed:
        with open(csrc / (source if changed == "source" else changed), "a") as f:
            f.write("// changed\n")
    monkeypatch.setattr(bench, "__file__", str(tmp_path / "bench.py"))
    got = bench.measured_traffic(kernel, K, table, source)
    assert (got is None) == (changed is not None)
