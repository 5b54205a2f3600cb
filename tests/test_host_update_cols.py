"""CPU test of the block update's column rule (csrc/update_cols.h): which column
of a slab of 1 to 8 input columns each lane loads.  A column at or past the
slab's width would be read outside the term, and in the block's last row
outside the allocation, without any trace in the result (it is multiplied as
zero)."""
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parents[1]


@pytest.fixture(scope="module")
def columns(tmp_path_factory):
    exe = tmp_path_factory.mktemp("cols") / "harness"
    subprocess.run(["g++", "-O1", "-std=c++17", f"-I{ROOT / 'paper_1506_06829_amd' / 'csrc'}",
                    str(ROOT / "tests" / "host_update_cols_harness.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    return {tuple(map(int, l.split()[:4])): int(l.split()[4]) for l in out.splitlines()}


@pytest.mark.parametrize("lim,pairs", [(l, 0) for l in range(1, 9)] + [(l, 1) for l in (2, 4, 6, 8)])
def test_update_reads_inside_its_columns(columns, lim, pairs):
    # (pairs are loaded from even widths only)
    for lk in range(4):
        for h in range(2):
            c = columns[lim, lk, h, pairs]
            assert 0 <= c < lim, (lk, h)
            if 2 * lk + h < lim:
                assert c == 2 * lk + h
        if pairs:       # one load of two columns from h = 0's on
            assert columns[lim, lk, 1, 1] == columns[lim, lk, 0, 1] + 1
