"""Which kernel a layer is given, asked from the library's own host functions (no GPU): the rules that choose by size have their lines
where the comments beside them say, and the shapes that the tests on the GPU use lie on the sides that those tests are named for."""
import ctypes as C

import pytest

from paper_2105_00619_amd import binding as B
from paper_2105_00619_amd import workloads as W


def _function(name, *argtypes):
    f = getattr(B.load_library(), name)
    f.argtypes, f.restype = argtypes, C.c_int
    return f


def test_grouping_blocks_by_xcd_adds_no_round():
    """256 CUs in 8 XCDs: blocks renumbered so that the channel blocks of a row tile share one are no more rounds of an XCD's 32 CUs
    than all blocks are of 256."""
    rows_per_xcd = _function("_ZN4oseq28conv_patch_wide_rows_per_xcdEii", C.c_int, C.c_int)
    grouped = 0
    for blocks in range(1, 9):
        for tiles in range(1, 1500):
            rows = rows_per_xcd(tiles, blocks)
            if rows:
                grouped += 1
                assert blocks > 1 and rows == -(-tiles // 8)
                assert -(-rows * blocks // 32) <= -(-tiles * blocks // 256), (tiles, blocks)
    assert grouped > 1000
    assert rows_per_xcd(84, 3) == 0 and rows_per_xcd(80, 3) == 10 and rows_per_xcd(127, 2) == 16
