"""Host-side checks of the benchmark's accounting (no GPU): committed counter
traffic is taken only for the sources the kernels are compiled from, headers
included, and launches of several steps are charged all of them."""
import json
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


def test_traffic_is_tied_to_every_source(tmp_path):
    names = [os.path.basename(p) for p in bench.KERNEL_SOURCE]
    assert {"k_fused.hip", "wave_dev.h", "fwi2d_internal.h"} <= set(names)
    files = []
    for n in names:
        p = tmp_path / n
        p.write_text(n)
        files.append(str(p))
    dec = {"band_rows": 8, "workload": "w"}
    table = tmp_path / "traffic.json"
    table.write_text(json.dumps({"source_sha256": bench.source_sha256(files), "kernels": {
        "adj_pair@w": {"decomposition": dec, "bytes_per_launch": 7}}}))
    assert bench.measured_traffic("adj_pair", dec, str(table), files) == 7
    for f in files:
        text = open(f).read()
        open(f, "w").write(text + "x")
        assert bench.measured_traffic("adj_pair", dec, str(table), files) is None
        open(f, "w").write(text)
    assert bench.measured_traffic("adj_pair", dec, str(table), files) == 7


def test_included_headers_are_hashed():
    """Every header of the project that a hashed source includes."""
    for group in (bench.KERNEL_SOURCE, bench.BORN_SOURCE):
        here = {os.path.basename(p) for p in group}
        for p in group:
            for line in open(p):
                if line.startswith('#include "') and "fwi2d.h" not in line:
                    assert line.split('"')[1] in here, (p, line)


def test_tile_launches_are_charged_their_steps():
    info = {"Nz": 141, "Nx": 141, "pml_cells": 9680, "ckpt_every": 16, "segments": 4}
    ab = bench.algorithmic_bytes(info, 2, 16)
    one = 141 * 141 * 2
    # 4 segments of 16, 16, 16 and 2 steps in launches of 8: 7 launches forward,
    # 6 again for the three recomputed, 7 in the adjoint
    got = bench.step_launches(ab, {"fwd_step": (13, 1.0), "adj_step": (7, 1.0)}, info, 50)
    assert got["cell_steps"]["fwd_step"] == round(one * 98 / 13)
    assert got["cell_steps"]["adj_step"] == round(one * 50 / 7)
    # strips: pairs and a leftover step
    got = bench.step_launches(ab, {"fwd_step": (3, 1.0), "fwd_pair": (40, 1.0),
                                   "adj_pair": (25, 1.0)}, info, 50)
    assert got["cell_steps"] == ab["cell_steps"]
    # one-step strips
    got = bench.step_launches(ab, {"fwd_step": (98, 1.0), "adj_step": (50, 1.0)}, info, 50)
    assert got["cell_steps"] == ab["cell_steps"]
