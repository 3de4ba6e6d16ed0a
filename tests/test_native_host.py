"""The library's host code on the CPU: the launches, copies and waits that the calls enqueue, run by a stand-in
runtime (tests/native/fake_hip.h) in the latest order that the waits allow, with plain loops in place of the kernels."""
import pytest

from tests.native_build import MISSING, native, run
from tests.test_gpu_relay_pieces import RESHARD_PIECES, STAGE_PIECES

pytestmark = pytest.mark.skipif(MISSING, reason="g++ or the HIP headers not available")
SOURCES = ("plan.cpp", "capi.cpp", "staging.cpp", "reshard.cpp", "relay.cpp", "moments.cpp")


@pytest.fixture(scope="module")
def host_check(tmp_path_factory):
    return native(str(tmp_path_factory.mktemp("host") / "host_check"), "host_check.cpp", SOURCES)


@pytest.fixture(scope="module")
def host_check_fast(tmp_path_factory):
    return native(str(tmp_path_factory.mktemp("host") / "host_check_fast"), "host_check.cpp", SOURCES, ("-O2",))


@pytest.mark.parametrize("mode", ["copies", "sums", "destroy", "order"])
def test_host_code(host_check, mode):
    run(host_check, mode)


@pytest.mark.parametrize("model,w,to,b,depth,pieces", STAGE_PIECES + [(m, w, -w2, b, 0, n) for m, w, w2, b, n in RESHARD_PIECES])
def test_pieces_of_the_path_through_host_memory(host_check_fast, model, w, to, b, depth, pieces):
    """The layouts that the GPU test runs: they are cut into as many pieces as it claims, and put together again."""
    out = run(host_check_fast, "pieces", *model, w, to, b, depth)
    assert int(out.split()[1]) == pieces
