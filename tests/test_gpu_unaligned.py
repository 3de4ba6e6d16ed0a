"""Column slices that are no whole groups of 4 elements (odd widths per rank), on the GPU against the oracle.

The stage kernel's unaligned tiles move groups of 4 elements on the destination's 8-byte grid: a
segment may start or end inside a group, a row may end inside one, and the groups of a segment's
last tile end up to three elements before its last unit.  The listed widths put all of these at
tile boundaries: multi-tile column slices that start at each of the four positions in a group
(the widths of the layers and ranks before them shift it), rows shorter than a group, and segments
cut by shard and chunk boundaries.
"""
import numpy as np
import pytest
import torch

import oracle
from oracle import Model
from paper_2607_22614_amd import datagen, dr
from tests.gpu_helpers import as_u16, checksums_to_list, new_checksums, require_gpu, say, to_device_shards

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


# (model, W, T, B): ffn/T odd or 2 mod 4, head widths down to 1, rows of 1 to 1821 elements
_CASES = [
    ((2, 256, 3, 3, 6, 3 * 683, 96), 5, 3, 16 * 4099),
    ((1, 2056, 4, 2, 5, 2 * 1821, 64), 3, 2, 1 << 20),
    ((3, 64, 4, 4, 1, 4 * 1, 32), 2, 4, 48),
    ((2, 128, 6, 3, 7, 3 * 33, 48), 13, 3, 16 * 77),
    ((1, 512, 2, 2, 18, 2 * 1025, 40), 64, 2, 1 << 30),
    # segments whose last tile's groups end before its last unit (lead 3, 1 and 2 elements more)
    ((1, 160, 3, 3, 6, 3 * 2047, 24), 7, 3, 1 << 20),
    ((2, 280, 2, 2, 64, 2 * 2047, 16), 5, 2, 130896),
    ((3, 208, 2, 2, 6, 2 * 195, 16), 3, 2, 22592),
    ((1, 8, 8, 8, 3, 8 * 2047, 16), 7, 8, 4096 + 16),
]


@pytest.mark.parametrize("tile_depth", [2, 4])
@pytest.mark.parametrize("model,w,t,b", _CASES)
def test_odd_widths_against_the_oracle(model, w, t, b, tile_depth):
    say("unaligned stage", model, "W", w, "T", t, "B", b, "depth", tile_depth)
    flat = datagen.make_flat_numpy(model, w, seed=7, specials_frac=0.01)
    m = Model(*model)
    want = oracle.rollout_stream(oracle.training_views(flat.view(np.uint32), m), m, t)
    want_cks = oracle.chunk_checksums(want, b)
    shards, keep = to_device_shards(flat, w)
    plan = dr.dr_plan_create(model, w, t, b, tile_depth=tile_depth)
    info = dr.dr_plan_get_info(plan)
    segs = [dr.dr_plan_segment(plan, i) for i in range(info["num_segments"])]
    assert any(not s["flags"] & dr.DR_SEG_VEC4 for s in segs)
    guard = 64  # bytes around the stream that the kernel must leave alone
    buf = torch.full((info["rollout_bytes"] + 2 * guard,), 0xA5, dtype=torch.uint8, device="cuda")
    cks = new_checksums(info["num_chunks"])
    dr.dr_stage_all(plan, shards, buf[guard:guard + info["rollout_bytes"]], cks)
    torch.cuda.synchronize()
    got = as_u16(buf[guard:guard + info["rollout_bytes"]])
    bad = np.flatnonzero(got != want)
    assert bad.size == 0, f"{bad.size} elements differ, first {bad[:8]}"
    assert checksums_to_list(cks) == want_cks
    assert bool((buf[:guard] == 0xA5).all()) and bool((buf[-guard:] == 0xA5).all())
    del keep
