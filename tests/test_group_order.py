"""The grouped order of the tile kernels, on the CPU: a permutation of [0, n) for every n, groups whole on one XCD."""
import numpy as np
import pytest

XCDS, G = 8, 64  # dev_types.h kXcds; kTileGroup (stage.hip), kPartGroup (reshard.hip)


def _xcd_group(b, n):
    if b >= (n & ~(XCDS * G - 1)):
        return b
    x, i = b % XCDS, b // XCDS
    return (i // G * XCDS + x) * G + i % G


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 511, 512, 513, 1023, 1024, 1025, 1536, 4099, 8192, 10000])
def test_grouped_order_is_a_permutation(n):
    t = np.array([_xcd_group(b, n) for b in range(n)])
    assert np.array_equal(np.sort(t), np.arange(n))
    full = n & ~(XCDS * G - 1)
    for g in range(full // G):  # the workgroups of a group share an XCD
        assert len({b % XCDS for b in np.flatnonzero(t // G == g) if b < full}) == 1


@pytest.mark.parametrize("groups,parts", [(1, 1), (255, 1), (256, 1), (257, 2), (512, 2), (513, 4), (1024, 4), (5000, 4)])
def test_reshard_parts_cover_a_tile(groups, parts):
    """reshard_kernel's parts per tile follow the chunk's groups: the largest tile (at most a chunk, at
    most 1024 groups) is covered by parts of 256 groups, and none is empty in it."""
    shift = 0 if groups <= 256 else 1 if groups <= 512 else 2
    assert 1 << shift == parts
    tile = min(groups, 1024)
    assert (parts << 8) >= tile and (parts == 1 or ((parts // 2) << 8) < tile)
