"""The counter summary finds the sweeps by the kernel names of the built library: a column sweep's name
ends with the number of zero states its first iterations do not read, and only the iterations'
kernels (0) are counted."""

import json
import os
import subprocess

import pytest

import bench
from paper_2503_20146_amd import build


@pytest.mark.parametrize("side,w", [(1024, 16), (2048, 8)])
def test_column_sweeps_are_found(tmp_path, monkeypatch, side, w):
    os.makedirs(tmp_path / "profiles")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    monkeypatch.setattr(bench, "kernel_source_hash", lambda: "h")
    px, copy_kib = 2 * side * side, bench.COPY_BYTES / 1024.0
    row, first, s11 = (f"void pwf::{k}(pwf::Sweep)" for k in (f"row_sweep<{side}, 4, 1, true>",
                                                              f"col_sweep<{side}, {w}, 6, 2>",
                                                              f"col_sweep<{side}, {w}, 6, 0>"))
    for name, counter, scale in (("f", "FETCH_SIZE", 0.5), ("w", "WRITE_SIZE", 1.0)):
        rows = [("copyBuffer", copy_kib * scale), (row, 8.0 * px / 1024 * scale), (first, 1.0),
                (s11, 20.0 * px / 1024 * scale)]
        with open(tmp_path / f"{name}.csv", "w") as fh:
            fh.write("Dispatch_Id,Kernel_Name,Counter_Name,Counter_Value\n")
            fh.writelines(f'{i},"{k}",{counter},{v}\n' for i, (k, v) in enumerate(rows))
    assert bench.ingest_counters(str(tmp_path / "f.csv"), str(tmp_path / "w.csv"), 2, side) == 0
    name = "traffic_counters.json" if side == 1024 else f"traffic_counters_{side}.json"
    sweeps = json.load(open(tmp_path / "profiles" / name))["sweeps"]
    assert set(sweeps) == {"4", f"11:{w}"}
    assert abs(sweeps[f"11:{w}"]["hbm_bytes_per_px"] - 40.0) < 1e-9
    assert abs(sweeps["4"]["hbm_bytes_per_px"] - 16.0) < 1e-9


def test_every_sweep_of_the_library_has_a_name():
    if not os.path.exists(build.LIB):
        pytest.skip("library not built")
    names = subprocess.run(["c++filt"], input=subprocess.run(["nm", build.LIB], capture_output=True, text=True,
                                                             check=True).stdout, capture_output=True, text=True,
                           check=True).stdout.split("\n")
    for side, widths in ((1024, (8, 16)), (2048, (8, 16))):
        for pattern in bench.SWEEP_KERNELS:
            for w in widths:
                assert any(bench.re.search(pattern.format(side=side, w=w), n) for n in names), (side, w, pattern)
