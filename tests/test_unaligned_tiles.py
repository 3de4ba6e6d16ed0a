"""The stage kernel's unaligned tiles, lane by lane, on the CPU.

Emulates which segment elements each lane of an unaligned tile loads, as one group or one by one,
and which it stores, and compares that with the segment's definition: element e of a segment comes
from source offset (e // cols) * stride + e % cols, and is stored once.  The 16-byte loads of a group
(one, and one more where its row ends inside it) must stay between the group's first and last
source element; a group stored with one 8-byte store must lie in the segment and on the
destination's 8-byte grid.
"""
import numpy as np
import pytest

THREADS, SCALAR_ITERS = 256, 8  # dev_types.h: kThreads, kScalarIters
PER = THREADS * SCALAR_ITERS


def _walk(units, lead, cols, stride):
    """Loads (element -> source offset) and the stored elements of every tile of a segment."""
    loaded = np.full(units, -1, dtype=np.int64)
    stored = np.zeros(units, dtype=np.int64)
    lane = np.arange(THREADS)
    for unit0 in range(0, units, PER):
        for k in range(SCALAR_ITERS // 4):
            for e in unit0 + 4 * (k * THREADS + lane) - lead:
                inside = [e + j for j in range(4) if 0 <= e + j < units]
                row, col = divmod(max(int(e), 0), cols)
                if e >= 0 and e + 4 <= units and cols >= 4:
                    p, j, cut = row * stride + col, np.arange(4), min(cols - col, 4)
                    last = (e + 3) // cols * stride + (e + 3) % cols
                    assert p + 3 <= last  # the first load
                    if cut < 4:
                        assert p + stride - cols + 3 == last  # the second, never before the first
                    loaded[e:e + 4] = np.where(j < cut, p + j, p + stride - cols + j)
                else:
                    for x in inside:
                        loaded[x] = x // cols * stride + x % cols
                if e >= 0 and e + 4 <= units:  # one 8-byte store
                    assert (lead + e) % 4 == 0
                stored[inside] += 1
        if unit0 + PER >= units:  # up to `lead` elements past the last tile's groups
            for x in range(unit0 + PER - lead, unit0 + PER):
                if x < units:
                    loaded[x] = x // cols * stride + x % cols
                    stored[x] += 1
    return loaded, stored


@pytest.mark.parametrize("lead", [0, 1, 2, 3])
@pytest.mark.parametrize("rows,cols,stride", [
    (1, 1, 1), (1, 3, 3), (1, 2045, 2045), (1, 2046, 2046), (1, 2047, 2047), (1, 2048, 2048), (1, 2049, 2049),
    (1, 4095, 4095), (1, 4096, 4096), (5, 1, 7), (700, 3, 5), (683, 3, 9), (1025, 2, 4), (2, 1024, 1030),
    (3, 1365, 2731), (2, 2047, 4094), (9, 683, 2049), (4097, 1, 3)])
def test_every_element_is_loaded_and_stored_once(rows, cols, stride, lead):
    units = rows * cols
    loaded, stored = _walk(units, lead, cols if rows > 1 else units, stride)
    e = np.arange(units)
    assert np.array_equal(loaded, e // cols * stride + e % cols)
    assert np.all(stored == 1)
