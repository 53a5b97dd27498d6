"""A grid that is not square: the autotuner times rows of one side and columns of the other, the cache
says so, and a process that reads it back makes the choices of the one that wrote it."""

import dataclasses

import numpy as np
import pytest

import synthetic as S
from gpu_helpers import device, gpu_problem, say

pytestmark = pytest.mark.gpu


def test_lines_of_a_wide_grid(tmp_path):
    from paper_2503_20146_amd import PWF, _lib, set_column_tile, set_row_plan
    dev = device()
    lib = _lib.load()
    geo = dataclasses.replace(S.config_geometry(0), ny=512, nx=1024)
    batch = PWF([gpu_problem(geo, np.ones((512, 1024)), dev)])
    path = tmp_path / "tuning.txt"
    say("tuning lines of 512 x 1024")

    def state():
        return [(lib.pwf_column_tile(n, s), lib.pwf_row_plan(n, s - 1)) for n in (512, 1024) for s in range(1, 12, 2)]

    def reset():
        for n in (512, 1024):
            set_column_tile(n, 0)
            for s in range(0, 12, 2):
                set_row_plan(n, s, -1)
    try:
        assert batch.autotune(2, path) is True
        tuned = state()
        lines = {int(l.split()[2]): l.split() for l in path.read_text().splitlines()}
        assert sorted(lines) == [512, 1024]
        assert "0" not in lines[512][4:10] and lines[512][11:] == ["-1"] * 6
        assert lines[1024][4:10] == ["0"] * 6 and "-1" not in lines[1024][11:]
        reset()
        assert batch.autotune(2, path) is False
        assert state() == tuned
    finally:
        reset()
