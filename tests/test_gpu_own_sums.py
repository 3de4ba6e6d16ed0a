"""Stage launches that sum their chunks themselves, on the GPU against the oracle: chunks of 1 to 128 tiles and one
more (which take the kernel behind the launch), launches around 2048 tiles, the same calls recorded into a graph (which
take the kernel) in turn with eager ones, chunk calls on several streams at once, and the shared static slots."""
import numpy as np
import pytest
import torch

import oracle
from oracle import Model
from paper_2607_22614_amd import datagen, dr
from tests.gpu_helpers import as_u16, checksums_to_list, new_checksums, require_gpu, say

pytestmark = pytest.mark.gpu

MODEL = (2, 256, 4, 4, 64, 688, 4096)  # 3.7 M rollout elements at T = 2


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _setup(b, depth, model=MODEL, w=3, t=2, seed=11):
    flat = datagen.make_flat_numpy(model, w, seed=seed, specials_frac=0.01)
    m = Model(*model)
    want = oracle.rollout_stream(oracle.training_views(flat.view(np.uint32), m), m, t)
    plan = dr.dr_plan_create(model, w, t, b, tile_depth=depth)
    S = plan.info["shard_elems"]
    shards = [torch.from_numpy(flat[i * S:(i + 1) * S].copy()).cuda() for i in range(w)]
    return plan, shards, want, oracle.chunk_checksums(want, b)


# bytes of a chunk of n whole tiles at a depth: 2048 * depth each
@pytest.mark.parametrize("depth", [2, 4])
@pytest.mark.parametrize("tiles", [9, 31, 32, 33, 63, 64, 65, 127, 128, 129, 500])
def test_chunks_by_tiles(tiles, depth):
    b = 2048 * depth * tiles
    say("own sums: chunks of", tiles, "tiles, depth", depth)
    plan, shards, want, cks_want = _setup(b, depth)
    info = plan.info
    for _ in range(3):  # slots and tickets are left ready for the next call
        dst = torch.full((info["rollout_bytes"],), 0xFF, dtype=torch.uint8, device="cuda")
        cks = new_checksums(info["num_chunks"])
        dr.dr_stage_all(plan, shards, dst, cks)
        torch.cuda.synchronize()
        assert np.array_equal(as_u16(dst), want) and checksums_to_list(cks) == cks_want
    dst.fill_(0xFF)
    cks.fill_(-1)
    for c in range(info["num_chunks"]):
        (dr.dr_stage_chunk, dr.dr_stage_chunk_noalloc)[c % 2](plan, c, shards, dst[c * b:], cks[c])
    torch.cuda.synchronize()
    assert np.array_equal(as_u16(dst), want) and checksums_to_list(cks) == cks_want


@pytest.mark.parametrize("vocab,tiles", [(4120, 2047), (4130, 2048), (4132, 2049)])
def test_launches_around_the_tile_limit(vocab, tiles):
    model = (1, 384, 4, 4, 64, 512, vocab)
    plan, shards, want, cks_want = _setup(256 << 10, 2, model=model)
    say("own sums: vocab", vocab, "tiles", tiles)
    assert plan.info["num_tiles"] == tiles  # up to 2048 tiles a launch sums its chunks itself
    dst = torch.full((plan.info["rollout_bytes"],), 0xFF, dtype=torch.uint8, device="cuda")
    cks = new_checksums(plan.info["num_chunks"])
    dr.dr_stage_all(plan, shards, dst, cks)
    torch.cuda.synchronize()
    assert np.array_equal(as_u16(dst), want) and checksums_to_list(cks) == cks_want


def test_graph_replays_between_eager_calls():
    b = 256 << 10
    plan, shards, want, cks_want = _setup(b, 4)
    info = plan.info
    dst = torch.empty(info["rollout_bytes"], dtype=torch.uint8, device="cuda")
    cks = new_checksums(info["num_chunks"])
    say("own sums: graph and eager in turn")
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        dr.dr_stage_all(plan, shards, dst, cks, torch.cuda.current_stream())
        dr.dr_stage_chunk_noalloc(plan, 1, shards, dst[b:], cks[1], torch.cuda.current_stream())
    eager = (lambda: dr.dr_stage_all(plan, shards, dst, cks), lambda: dr.dr_stage_chunk_noalloc(plan, 1, shards, dst[b:], cks[1]))
    for i in range(6):
        dst.fill_(0xFF)
        cks.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(as_u16(dst), want) and checksums_to_list(cks) == cks_want, i
        dst.fill_(0xFF)
        cks.fill_(-1)
        for call in eager:
            call()
        torch.cuda.synchronize()
        assert np.array_equal(as_u16(dst), want) and checksums_to_list(cks) == cks_want, i


def test_different_chunks_on_several_streams_at_once():
    b = 64 << 10
    plan, shards, want, cks_want = _setup(b, 2)
    info = plan.info
    streams = [torch.cuda.Stream() for _ in range(4)]
    dst = torch.full((info["rollout_bytes"],), 0xFF, dtype=torch.uint8, device="cuda")
    cks = new_checksums(info["num_chunks"])
    torch.cuda.synchronize()
    say("own sums: chunks of one plan on four streams")
    for c in range(info["num_chunks"]):
        dr.dr_stage_chunk(plan, c, shards, dst[c * b:], cks[c], stream=streams[c % 4])
    torch.cuda.synchronize()
    assert np.array_equal(as_u16(dst), want) and checksums_to_list(cks) == cks_want
