"""Which forward products split their sums between two k groups (bf16_forward_splits: those in tiles of 64 columns), on either side of the
line between tiles of 128x128 and of 64x64.  The library's rule on the host."""
import ctypes

import pytest

from paper_2110_00625_amd import kavg

CASES = [
    # P, B, d_in, d_out, splits
    (12, 90, 1000, 3000, False),         # 288 tiles of 128x128 without padding; 1128 of 64x64
    (9, 130, 1024, 2048, True),          # 288, a quarter of their rows padding; 864 of 64x64, which fit the chip twice over
    (20, 150, 1024, 1024, True),         # 320 and 960
    (21, 140, 1024, 1024, True),         # 336 and 1008
    (22, 140, 3072, 1024, False),        # 352 and 1056
    (12, 192, 1024, 2048, False),        # 384 and 1152
    (7, 260, 1024, 2048, False),         # 336 and 1120
    (6, 290, 1024, 2048, True),          # 288 and 960
    (16, 128, 1024, 1024, True),         # 128 tiles
    (512, 100, 64, 64, False),           # 512 tiles of 128x128, half of their columns padding: 1024 of 64x64
    (32, 192, 1024, 1024, False),        # 512 of 128x128
]


@pytest.mark.parametrize("P,B,d_in,d_out,splits", CASES)
def test_forward_tiles(P, B, d_in, d_out, splits):
    rule = kavg.load_library()._ZN4kavg19bf16_forward_splitsEiiii
    rule.restype = ctypes.c_bool
    rule.argtypes = [ctypes.c_int] * 4
    assert rule(P, B, d_in, d_out) is splits
