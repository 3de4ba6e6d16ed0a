"""The stage kernel's unaligned tiles, lane by lane, on the CPU.

Walks which segment elements each lane of an unaligned tile loads, as one group or one by one, and
which it stores, with the kernel's own compiled index functions (csrc/tile_index.h), and compares
that with the segment's definition: element e of a segment comes from source offset
(e // cols) * stride + e % cols, and is stored once.  The 16-byte loads of a group (one, and one more
where its row ends inside it) must stay between the group's first and last source element; a group
stored with one 8-byte store must lie in the segment and on the destination's 8-byte grid.
"""
import pytest

from tests.native_build import MISSING, native, run

pytestmark = pytest.mark.skipif(MISSING, reason="g++ or the HIP headers not available")


@pytest.fixture(scope="module")
def index_check(tmp_path_factory):
    return native(str(tmp_path_factory.mktemp("index") / "index_check"), "index_check.cpp")


@pytest.mark.parametrize("lead", [0, 1, 2, 3])
@pytest.mark.parametrize("rows,cols,stride", [
    (1, 1, 1), (1, 3, 3), (1, 2045, 2045), (1, 2046, 2046), (1, 2047, 2047), (1, 2048, 2048), (1, 2049, 2049),
    (1, 4095, 4095), (1, 4096, 4096), (5, 1, 7), (700, 3, 5), (683, 3, 9), (1025, 2, 4), (2, 1024, 1030),
    (3, 1365, 2731), (2, 2047, 4094), (9, 683, 2049), (4097, 1, 3)])
def test_every_element_is_loaded_and_stored_once(index_check, rows, cols, stride, lead):
    run(index_check, "unaligned", rows, cols, stride, lead)
