"""Which form a training step takes, on the CPU: two kernels where they were
measured to be the faster form (profiled steps of 1024 to 32,768 rows, both
forms), one kernel beyond.  Rows of 128 (width 128) or 64 (width 256) a tile."""
import ctypes

import pytest


@pytest.mark.parametrize("width,depth,faster,slower", [
    (128, 2, 8192, 9216), (128, 3, 12_288, 13_312), (128, 4, 16_384, 17_408), (128, 5, 16_384, 17_408),
    (128, 6, 16_384, 17_408), (128, 7, 16_384, 17_408), (128, 8, 24_576, 25_600), (128, 9, 24_576, 25_600),
    (256, 2, 16_384, None), (256, 4, 16_384, None), (256, 9, 16_384, None)])
def test_rule_follows_the_measurements(width, depth, faster, slower):
    from paper_2510_05100_amd import _abi
    rule = _abi.load().rwgt_mlp_train_rows_rule
    rule.argtypes, rule.restype = [ctypes.c_int, ctypes.c_int], ctypes.c_int
    tile = 128 if width == 128 else 64
    tiles = rule(width, depth)
    assert 1 <= tiles <= 256                     # every tile has a slot of its own
    assert faster <= tiles * tile
    assert slower is None or tiles * tile < slower
