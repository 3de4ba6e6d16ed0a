"""The order in which the tile kernels' workgroups take tiles, and a reshard's parts of a tile, on the CPU: the
compiled index functions of the kernels (csrc/tile_index.h) over counts around their windows."""
import pytest

from tests.native_build import MISSING, native, run

pytestmark = pytest.mark.skipif(MISSING, reason="g++ or the HIP headers not available")


@pytest.fixture(scope="module")
def index_check(tmp_path_factory):
    return native(str(tmp_path_factory.mktemp("index") / "index_check"), "index_check.cpp")


@pytest.mark.parametrize("what", [
    "order",  # grouped and contiguous order are permutations, groups whole on one XCD
    "division",  # a row's division and an element's source offset
    "parts",  # parts cover every group of every segment once
])
def test_index_functions(index_check, what):
    run(index_check, what)
