"""The packed FC1 weights are allocated as far as the fused kernels read them.

Each wave loads the weights of its next pairs of map positions before it is
known whether there are any.  The fragment's place is the scalar offset of a
buffer load, which the resource's bounds check does not cover, so the
allocation has to hold what the last wave of the last position range loads.
The pairs that a wave takes and loads are enumerated here, independently of the
kernels' loops (CPU only)."""

import ctypes

import pytest

PAIRS = 44 * 44 // 2            # of map positions
GROUPS = PAIRS // 4             # 242 steps of 4 pairs in all


def _bytes(name):
    from paper_2009_04509_amd import binding
    f = getattr(binding.lib, f"_ZN7pointid{len(name)}{name}Ev")
    f.restype = ctypes.c_int64
    return f()


def _last_pair(ranges, waves, ahead):
    """The last pair that any wave loads: wave g of a range takes pairs first + g,
    first + g + waves, ... below the range's end, and with each loads the pair
    `ahead` of its turns later."""
    last = 0
    for a, b in ranges:
        for g in range(waves):
            last = max([last] + [p + ahead * waves for p in range(a + g, b, waves)])
    return last


def _ranges(unit, count, splits=8):
    return [(unit * (count * s // splits), unit * (count * (s + 1) // splits)) for s in range(splits)]


@pytest.mark.parametrize("name, pair_bytes, waves, ahead", [
    ("conv_fc1_16_weight_bytes", 3 * 8 * 1024, 4, 1),
    ("conv_fc1_f32_weight_bytes", 3 * 3 * 8 * 1024, 8, 1),
    ("conv_fc1_8_weight_bytes", 8 * 1536, 4, 4),
])
def test_allocation_holds_every_load(name, pair_bytes, waves, ahead):
    ranges = _ranges(4, GROUPS)
    assert ranges[0][0] == 0 and ranges[-1][1] == PAIRS
    assert (_last_pair(ranges, waves, ahead) + 1) * pair_bytes <= _bytes(name)
