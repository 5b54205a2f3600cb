"""CPU test of a Gram's scratch (csrc/gram_split.h): it holds the partials of the
row blocks the launch asks for, and a call that allocates it (gplhr_proj_orth,
which pays for mapping it every time) takes no more than its rows need."""
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parents[1]


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    exe = tmp_path_factory.mktemp("split") / "harness"
    subprocess.run(["g++", "-O1", "-std=c++17", f"-I{ROOT / 'paper_1506_06829_amd' / 'csrc'}",
                    str(ROOT / "tests" / "host_gram_split_harness.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    return [(l[0], tuple(map(int, l[1:].split()))) for l in out.splitlines()]


@pytest.fixture(scope="module")
def split(lines):
    return ({v[:3]: v[3] for k, v in lines if k == "s"}, {v[:3]: v[3:] for k, v in lines if k == "t"})


def _tiles(bx, by):
    """Tile counts a call of these widths can run with: X and Y apart (either as
    the wider one), or Y the last by columns of X; with each, the count that
    decides the row blocks."""
    u = lambda w: (w + 7) // 8
    yield u(bx) * u(by), u(bx) * u(by)
    if bx >= by:
        a, m = u(bx - by), u(by)
        t = a * m + m * (m + 1) // 2
        yield t, (t if a else m * m)


def test_scratch_holds_the_wanted_row_blocks(split):
    scratch, blocks = split
    for (n, bx, by), have in scratch.items():
        for tiles, rule in _tiles(bx, by):
            for c64 in (0, 1):
                few, want = blocks[n, rule, c64]
                assert few or have >= 128 * tiles * want, (n, bx, by, tiles)


def test_scratch_of_a_projection_follows_its_rows(split):
    # a tile's partial is 128 entries; one row block per 128 rows, but 128 of them
    # from 4096 rows on and no more than 512
    scratch, _ = split
    for (n, wg, w), have in scratch.items():
        if w > 48 or wg < w or wg - w > 48:
            continue
        tiles = ((wg + 7) // 8 + 1) * ((w + 7) // 8)
        if n <= 1024:
            assert have == 0
        assert have <= 128 * tiles * max(128, n // 128), (n, wg, w)
        assert have <= 128 * 512 * tiles, (n, wg, w)


def test_row_blocks_fill_the_cus_evenly(split):
    # beyond one block per CU (256) each CU takes the same number, or the CUs with
    # one more set the time; all rows are covered, by at least 32 per block
    _, blocks = split
    for (n, tiles, c64), (_, nblk) in blocks.items():
        assert 1 <= nblk <= 256 or nblk % 256 == 0, (n, tiles, c64, nblk)
        assert nblk == 1 or n // nblk >= 32


def test_kept_scratch_never_costs_row_blocks(split, lines):
    # gplhr_gram_noalloc of two blocks runs with the row blocks of gplhr_gram
    _, blocks = split
    kept, = [v[0] for k, v in lines if k == "c"]
    for (n, tiles, c64), (few, want) in blocks.items():
        assert few or tiles > 64 or kept >= 128 * tiles * want, (n, tiles, c64)
