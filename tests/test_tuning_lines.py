"""Lines of the tuning cache, read without a GPU (the architecture is then "unknown"): widths of 0 and
plans of -1 leave a sweep unset, in a line beside set ones, also where it was set before; lines with
every sweep set are read as before, and lines with an unsupported width or plan are not applied."""

import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = """
import ctypes, sys
from paper_2503_20146_amd import _lib
lib = _lib.load()
p = _lib.pwf_problem()
p.geom.nx, p.geom.ny, p.geom.pixel_m, p.geom.wavelength_m, p.geom.z1_m, p.geom.z2_m = 1024, 512, 1e-6, 5e-11, 5e-3, .2
p.source.kind = _lib.PWF_SRC_GAUSS
p.params.eta, p.params.precondition = 0.5, 0
p.diffuser = 256          # (never read: nothing is launched)
lib.pwf_set_column_tile(1024, 11, 8)
lib.pwf_set_row_plan(512, 4, 0)
tuned = ctypes.c_int32(7)
arr = (_lib.pwf_problem * 1)(p)
rc = lib.pwf_autotune_cached(arr, 1, 1, sys.argv[1].encode(), 0, ctypes.byref(tuned), None, 0, None)
print(rc, tuned.value)
for n in (512, 1024):
    print([lib.pwf_column_tile(n, s) for s in range(1, 12, 2)], [lib.pwf_row_plan(n, s) for s in range(0, 12, 2)])
"""


def read_back(tmp_path, lines):
    path = tmp_path / "cache.txt"
    path.write_text("".join(f"unknown 1024x512*1 {l}\n" for l in lines))
    out = subprocess.run([sys.executable, "-c", CODE, str(path)], cwd=ROOT, capture_output=True, text=True,
                         timeout=120, env={**os.environ, "HIP_VISIBLE_DEVICES": "-1"})
    assert out.returncode == 0, out.stderr
    return out.stdout.split("\n")


def test_unset_sweeps_stay_unset(tmp_path):
    built_in = read_back(tmp_path, ["512 c 0 0 0 0 0 0 r -1 -1 -1 -1 -1 -1", "1024 c 0 0 0 0 0 0 r -1 -1 -1 -1 -1 -1"])
    assert built_in[0] == "0 0"
    assert built_in[2].startswith("[16, 16, 16, 16, 16, 16]")   # (11: set to 8 before)
    mixed = read_back(tmp_path, ["512 c 16 32 16 16 32 16 r -1 -1 -1 -1 -1 -1", "1024 c 0 0 0 0 0 0 r 2 1 0 2 1 0"])
    assert mixed[0] == "0 0"
    assert mixed[1] == "[16, 32, 16, 16, 32, 16] " + built_in[1].split("] ")[1]
    assert mixed[2] == "[16, 16, 16, 16, 16, 16] [2, 1, 0, 2, 1, 0]"


@pytest.mark.parametrize("line,want", [("1024 c 8 16 16 8 16 8 r 2 1 0 2 1 0", "[8, 16, 16, 8, 16, 8] [2, 1, 0, 2, 1, 0]"),
                                       ("1024 c 4 16 16 8 16 8 r 2 1 0 2 1 0", None),
                                       ("1024 c 8 16 16 8 16 8 r -2 1 0 2 1 0", None),
                                       ("1024 c 8 16 16 8 16 8 r 3 1 0 2 1 0", None)])
def test_lines_with_every_sweep_set(tmp_path, line, want):
    out = read_back(tmp_path, ["512 c 16 16 16 16 16 16 r 0 0 0 0 0 0", line])
    assert out[0] == "0 0"
    # not applied: what was set before the call stays (S11 at 8 columns, plans built in)
    assert out[2] == want if want else out[2].startswith("[16, 16, 16, 16, 16, 8] ") and "[2, 1, 0" not in out[2]


def test_shipped_entries_are_of_this_version():
    from paper_2503_20146_amd import _lib
    path = os.path.join(ROOT, "paper_2503_20146_amd", "tuning_cache.txt")
    lines = [l.split() for l in open(path).read().splitlines()]
    assert lines and {l[0] for l in lines} == {f"gfx950/v{_lib.load().pwf_version()}"}
    assert all(len(l) == 17 and l[3] == "c" and l[10] == "r" for l in lines)
