"""The grouped order of the tile kernels, on the CPU: a permutation of [0, n) for every n, groups whole on one XCD."""
import numpy as np
import pytest

XCDS = 8  # dev_types.h kXcds


def _xcd_group(b, n, G):
    if b >= (n & ~(XCDS * G - 1)):
        return b
    x, i = b % XCDS, b // XCDS
    return (i // G * XCDS + x) * G + i % G


@pytest.mark.parametrize("G", [32, 64])  # kPartGroup (reshard.hip), kTileGroup (stage.hip, moment_sums.hip)
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 511, 512, 513, 1023, 1024, 1025, 1536, 4099, 8192, 10000])
def test_grouped_order_is_a_permutation(n, G):
    t = np.array([_xcd_group(b, n, G) for b in range(n)])
    assert np.array_equal(np.sort(t), np.arange(n))
    full = n & ~(XCDS * G - 1)
    for g in range(full // G):  # the workgroups of a group share an XCD
        assert len({b % XCDS for b in np.flatnonzero(t // G == g) if b < full}) == 1


@pytest.mark.parametrize("groups", [1, 255, 511, 512, 513, 1023, 1024, 5000])
def test_reshard_parts_cover_a_tile(groups):
    """reshard_kernel moves a tile in one part of 512 groups where a chunk holds no more, else in two:
    the largest tile (at most a chunk, at most 1024 groups) is covered, and no part of it is empty."""
    parts = 1 if groups <= 512 else 2
    tile = min(groups, 1024)
    assert parts * 512 >= tile > (parts - 1) * 512
