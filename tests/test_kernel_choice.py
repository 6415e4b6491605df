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


class ConvGeom(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("N", "H", "W", "C", "K", "R", "S", "stride", "pad", "P", "Q")]


def _conv3x3(n, h, w, cin, cout):
    return C.byref(ConvGeom(n, h, w, cin, cout, 3, 3, 1, 1, h, w))


def _forward_rows(dt, *layer):
    """Rows of channel sums of a forward pass: row tiles of 256 pixels where it takes the wide tiles, of 128 and less elsewhere."""
    return _function("_ZN4oseq25conv_mfma_fwd_stat_blocksEiRKNS_8ConvGeomEb", C.c_int, C.c_void_p, C.c_bool)(dt, _conv3x3(*layer), False)


def _data_gradient_rows(dt, *layer):
    return _function("_ZN4oseq21conv_dgrad_sum_blocksEiRKNS_8ConvGeomE", C.c_int, C.c_void_p)(dt, _conv3x3(*layer))


@pytest.mark.parametrize("dt", [W.BF16, W.FP16])
@pytest.mark.parametrize("layer,rows", [
    # the layers of test_wide_tiles_of_3x3_layers and of the bit comparison (test_gpu_parity.py); 218 images against 217
    ((256, 16, 16, 128, 128), 256), ((1024, 8, 8, 256, 256), 256), ((254, 15, 17, 256, 256), 254), ((1279, 7, 7, 256, 256), 256),
    ((8, 64, 128, 128, 128), 256), ((4091, 4, 4, 128, 128), 256), ((4096, 4, 4, 256, 256), 256), ((511, 8, 8, 512, 512), 128),
    ((507, 8, 8, 512, 512), 127), ((320, 8, 8, 384, 384), 80), ((336, 8, 8, 384, 384), 84), ((8190, 4, 4, 128, 128), 512),
    ((217, 16, 16, 128, 128), 434), ((218, 16, 16, 128, 128), 218),
    # up to three rounds of 256 where rows of a tile are short, not with least depth; beyond that only where the narrow tiles fit the map badly
    ((512, 16, 16, 128, 128), 512), ((440, 16, 16, 128, 128), 440), ((768, 16, 16, 128, 128), 768), ((1024, 16, 16, 128, 128), 2048),
    ((512, 16, 16, 96, 128), 512), ((64, 32, 64, 128, 128), 1024), ((509, 15, 17, 128, 128), 509), ((512, 16, 16, 32, 128), 1024), ((256, 16, 16, 32, 128), 256),
    ((512, 16, 16, 32, 256), 1024), ((508, 16, 16, 64, 256), 508), ((450, 16, 16, 64, 256), 900), ((450, 16, 16, 128, 256), 450),
    ((645, 7, 7, 128, 128), 323), ((1210, 7, 7, 128, 128), 242), ((2360, 7, 7, 128, 128), 472),
    # 256 channels that tiles of 256 do not fit, in tiles of 128: up to three rounds, beyond that 93 % of the products
    ((384, 16, 16, 256, 256), 384), ((550, 16, 16, 256, 256), 1100), ((600, 16, 16, 256, 256), 600), ((750, 16, 16, 384, 384), 750)])
def test_wide_tiles_are_taken_where_they_are_faster(dt, layer, rows):
    n, h, w, cin, cout = layer
    assert _forward_rows(dt, *layer) == rows
    # the data gradient goes by the same rule (0: too many rows to be worth it)
    assert _data_gradient_rows(dt, n, h, w, cout, cin) in (rows, 0)
    assert _forward_rows(W.FP32, *layer) != rows or rows > n * h * w // 200


@pytest.mark.parametrize("dt", [W.BF16, W.FP16])
@pytest.mark.parametrize("channels,h,w,b,swaps", [
    # layers of test_weight_gradient_of_64_channels_by_rows (test_gpu_parity.py): blocks of 64 channels, and 128 with too few sub-tiles for wider ones
    (64, 8, 8, 257, False), (64, 32, 32, 17, False), (192, 16, 16, 70, False), (128, 16, 16, 70, False),
    # blocks of 128 channels on maps whose width is a multiple of eight, and on others
    (128, 16, 16, 256, True), (256, 8, 8, 1024, True), (256, 24, 24, 114, True), (384, 9, 40, 182, True), (256, 14, 14, 512, False),
    (256, 7, 7, 1279, False), (512, 4, 4, 1024, False)])
def test_weight_gradients_whose_parts_are_exchanged(dt, channels, h, w, b, swaps):
    f = _function("_ZN4oseq19conv_wgrad3x3_swapsEiRKNS_8ConvGeomE", C.c_int, C.c_void_p)
    f.restype = C.c_bool
    assert f(dt, _conv3x3(b, h, w, channels, channels)) == swaps
    assert not f(W.FP32, _conv3x3(b, h, w, channels, channels))


def test_padded_patch_rows_leave_a_cu_its_blocks():
    """Rows of a staged patch are padded against bank conflicts only where that leaves a CU the blocks that its registers hold and the
    grid has: three of 64 channels, two of 128."""
    blocks = _function("_ZN4oseq24conv_patch_blocks_per_cuEiRKNS_8ConvGeomEb", C.c_int, C.c_void_p, C.c_bool)
    seen = 0
    for h in range(5, 130, 3):
        for w in list(range(4, 66)) + [80, 96, 100, 112, 128]:
            for c, held in ((64, 3), (128, 2)):
                for dt in (W.BF16, W.FP32):
                    layer = _conv3x3(max(1, 70000 // (h * w)), h, w, c, c)
                    n = blocks(dt, layer, False)
                    seen += n > 0
                    assert n >= min(held, blocks(dt, layer, True)), (dt, c, h, w)
    assert seen > 10000
    assert blocks(W.FP16, _conv3x3(28, 50, 50, 64, 64), False) == 3
    # two blocks a CU: padded, though a third would fit without
    assert blocks(W.FP16, _conv3x3(256, 8, 8, 256, 256), False) == 2 and blocks(W.FP16, _conv3x3(256, 8, 8, 256, 256), True) == 3


@pytest.mark.parametrize("dt", [W.BF16, W.FP16])
@pytest.mark.parametrize("layer,padded", [
    # n, h, w, C_in, C_out in tiles of 64 pixels
    ((329, 15, 5, 704, 704), True), ((329, 15, 5, 768, 704), True), ((329, 15, 5, 768, 768), False), ((329, 15, 5, 896, 704), False),
    ((329, 15, 5, 1280, 640), True), ((329, 15, 5, 576, 1024), True), ((329, 15, 5, 640, 896), False), ((329, 15, 5, 1024, 1024), False),
    # few tiles; columns that were padded before
    ((42, 15, 5, 896, 896), True), ((80, 15, 5, 896, 896), False), ((80, 16, 8, 1024, 1024), True), ((400, 15, 4, 1024, 1024), True),
    # tiles of 128 pixels
    ((250, 7, 7, 1024, 1024), True), ((120, 10, 5, 1024, 1024), True)])
def test_rows_are_not_padded_where_weights_miss_the_cache(dt, layer, padded):
    f = _function("_ZN4oseq22conv_patch_rows_paddedEiRKNS_8ConvGeomE", C.c_int, C.c_void_p)
    f.restype = C.c_bool
    assert f(dt, _conv3x3(*layer)) == padded
