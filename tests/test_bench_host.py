"""The helpers of bench.py that decide what its figures count (CPU only)."""
import pytest
import torch

import bench

CASES = [
    # keys, digit bits, rounds that move records
    ([5, 5, 5, 5], 8, [7]),                      # no digit varies: the last round runs
    ([0, 1, 255], 8, [0]),
    ([0, 1 << 20], 8, [2]),
    ([0, -1], 8, list(range(8))),
    ([1 << 63 - 1, 0, 3], 8, [0, 7]),
    ([-(1 << 63), 0], 8, [7]),                   # the top bit: an arithmetic shift
    ([0x0F, 0xFF, 0x0F0], 4, [0, 1]),
    ([0, 1 << 63 - 1], 11, [5]),                 # six rounds, the last of 9 bits
]


@pytest.mark.parametrize("keys,bits,want", CASES, ids=lambda x: str(x)[:24])
def test_moving_rounds(keys, bits, want):
    assert bench.moving_rounds(torch.tensor(keys, dtype=torch.int64), bits) == want


def test_moving_rounds_of_32_bit_keys():
    keys = torch.tensor([7, 7 + (1 << 24), -(1 << 31) + 7], dtype=torch.int32)
    assert bench.moving_rounds(keys, 8) == [3]
