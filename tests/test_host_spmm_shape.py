"""CPU tests of the sparse product's row schedule (csrc/spmm_shape.h): every row
belongs to one workgroup in every order, and the eighths of the rows go one to
an XCD only where they hold about the same number of entries."""
import subprocess
from pathlib import Path

import numpy as np
import pytest

ROOT = Path(__file__).resolve().parents[1]


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    exe = tmp_path_factory.mktemp("shape") / "harness"
    subprocess.run(["g++", "-O1", "-std=c++17", f"-I{ROOT / 'paper_1506_06829_amd' / 'csrc'}",
                    str(ROOT / "tests" / "host_spmm_shape_harness.cpp"), "-o", str(exe)], check=True)

    def run(lines):
        return subprocess.run([str(exe)], input="\n".join(lines) + "\n", check=True, capture_output=True,
                              text=True).stdout.splitlines()
    return run


@pytest.mark.parametrize("n,plane", [(1, 0), (7, 0), (64, 0), (1031, 0), (20000, 0), (4096, 512), (4800, 600),
                                     (8 * 13 * 9, 104), (16, 8), (27000, 1080)])
def test_every_row_once(shapes, n, plane):
    for b in (1, 2, 5, 10, 16, 33, 64):
        for cols in (1, 2):
            if cols == 2 and b % 2:
                continue
            for row_len in (0, 5, 17, 40, 300):
                for cut in (0, 1):
                    if plane and n % plane:
                        continue
                    out = shapes([f"x {n} {b} {cols} {cols} {plane} {row_len} {256 if cols == 1 else 320} {cut} 1"])
                    _, grid, lpr, rpw, rpb, sp, order = out[0].split()
                    assert int(lpr) * int(rpw) <= 64 and int(rpb) <= 4 * int(rpw)
                    for l in out[1:]:
                        seen = np.zeros(n, int)
                        for r0, nr in (map(int, w.split(":")) for w in l.split()[2:]):
                            if nr > 0:
                                assert 0 <= r0 and r0 + nr <= n and nr <= int(rpb)
                                seen[r0:r0 + nr] += 1
                        assert (seen == 1).all(), (b, cols, row_len, l[:6])


@pytest.mark.parametrize("pattern,even", [("uniform", 1), ("grid", 1), ("ragged", 1), ("first", 0), ("last", 0),
                                          ("sorted", 0), ("rising", 0), ("empty", 1)])
def test_eighths_only_where_they_are_even(shapes, pattern, even):
    rng = np.random.default_rng(1)
    n = 32000
    cnt = np.full(n, 7)
    if pattern == "grid":
        cnt[:1600] = cnt[-1600:] = 6
    elif pattern == "ragged":
        cnt = rng.integers(1, 36, n)
    elif pattern == "first":
        cnt[:n // 8] = 70
    elif pattern == "last":
        cnt[-n // 8:] = 8
    elif pattern == "sorted":
        cnt = np.sort(rng.integers(1, 36, n))
    elif pattern == "rising":
        cnt = np.linspace(10, 14, n).astype(int)
    elif pattern == "empty":
        cnt[:] = 0
    rp = np.concatenate([[0], np.cumsum(cnt)])
    _, grid, _, _, rpb, _, order = shapes([f"x {n} 10 1 1 0 7 256 1 0"])[0].split()
    assert order == "2"                      # the row pointers decide
    per = int(grid) // 8 * int(rpb)
    at = rp[np.minimum(np.arange(9) * per, n)]
    most = int(np.diff(at).max())
    assert int(most <= at[8] // 8 + at[8] // 128) == even
    assert shapes([f"eighths {most} {at[8]}"])[-1] == str(even)


def test_no_check_where_it_cannot_pay(shapes):
    # few workgroups; one row to a wavefront; rows beyond 32 bits
    for n, b, want in ((12 ** 3, 16, "0"), (262144, 33, "1"), (1 << 31, 4, "1"), (262144, 32, "2")):
        assert shapes([f"x {n} {b} 1 1 0 7 320 1 0"])[0].split()[-1] == want


def test_slabs_keep_their_lanes_busy(shapes):
    # a plane whose slabs hold fewer than four workgroups' rows runs in natural order;
    # where slabs are kept, no more than a quarter of the lanes wait at their ends
    for plane in (512, 520, 1024, 2048, 4096, 25600):
        n = plane * 64
        for b in (1, 2, 4, 5, 10, 16, 33, 64):
            grid, _, _, _, sp, _ = map(int, shapes([f"x {n} {b} 1 1 {plane} 7 256 1 0"])[0].split()[1:])
            full = int(shapes([f"x {n} {b} 1 1 0 7 256 1 0"])[0].split()[4])
            assert (sp == plane) == (plane // 8 >= 4 * full), (plane, b)
            if sp:
                assert grid * full <= 1.25 * n


def test_launches_below_2_to_the_32_threads(shapes):
    def run(n, b, cols, most, plane):
        grid, lpr, rpw, rpb, sp, order = map(int, shapes([f"x {n} {b} {cols} {most} {plane} 7 256 1 0"])[0].split()[1:])
        assert grid < 1 << 24
        return grid, rpb, order
    rows = (1 << 24) - 1
    # rows in turn take the last few, whose eighths would round up to 2^24 workgroups
    assert run(4 * rows, 33, 1, 1, 0) == (rows, 4, 1)
    assert run(4 * (rows - 8), 33, 1, 1, 0)[0] == rows - 7
    assert run(4 * rows + 1, 33, 1, 1, 0)[0] == 0           # refused
    assert run(4 * rows + 1, 64, 1, 2, 0)[1:] == (8, 2)     # two columns to a lane
    assert run(8 * ((1 << 21) + 5), 2, 1, 2, 8)[2] == 2     # tiny planes: natural order
