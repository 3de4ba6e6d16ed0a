"""The path through host memory where its launches meet: chunks of several pieces, pieces that end inside unaligned
column slices, reloads across destination shards, destinations reloaded by copies, calls in order on two streams."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2607_22614_amd import datagen, dr, workloads
from tests.gpu_helpers import checksums_to_list, new_checksums, require_gpu, say

pytestmark = pytest.mark.gpu

MiB = 1 << 20


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _stage_setup(model, w, t, b, depth=0, seed=5):
    plan = dr.dr_plan_create(model, w, t, b, tile_depth=depth)
    info = dr.dr_plan_get_info(plan)
    flat = datagen.make_flat_torch(model, w, seed)
    S = info["shard_elems"]
    shards = [flat[i * S:(i + 1) * S] for i in range(w)]
    return plan, info, shards, flat


def _out(info):
    return torch.full((info["rollout_bytes"],), 0xFF, dtype=torch.uint8, device="cuda"), new_checksums(info["num_chunks"])


# A chunk is cut into pieces of about 32 MiB, from 48 MiB on (two), 80 MiB on (three).  The numbers of pieces of
# these calls are checked against the library on the CPU (tests/test_native_host.py).
ODD, EVEN = (1024, 6, 3, 72, 3 * 1821, 3 * 401), (1024, 8, 4, 64, 4096, 4000)

# odd widths (pieces end inside unaligned segments) and aligned ones; chunks of one piece, of several, and of
# sizes around one and a half and two and a half pieces, several such chunks in a row
STAGE_PIECES = [  # model, W, T, B, tile depth, pieces of the whole call
    ((2,) + ODD, 5, 3, 1 << 30, 0, 3),
    ((2,) + ODD, 5, 3, 40 * MiB + 16, 2, 2),
    ((2,) + ODD, 5, 3, 16 * MiB, 4, 5),
    ((2,) + EVEN, 8, 4, 16 * MiB + 16, 0, 5),
    ((2,) + EVEN, 8, 4, 33 * MiB, 0, 3),
    ((6,) + ODD, 5, 3, 48 * MiB + 4096 + 16, 0, 9),
    ((6,) + ODD, 5, 3, 81 * MiB, 2, 8),
    # many shards: cuts inside the column slices, so that pieces end at any element
    ((6,) + ODD, 61, 3, 1 << 30, 0, 9),
    ((6,) + ODD, 64, 3, 48 * MiB + 4096 + 16, 2, 9),
    ((7,) + ODD, 53, 3, 100 * MiB, 4, 10),
    ((8,) + EVEN, 8, 4, 47 * MiB, 0, 5),
    ((8,) + EVEN, 8, 4, 49 * MiB, 0, 9),
    ((8,) + EVEN, 8, 4, 79 * MiB, 4, 6),
    ((8,) + EVEN, 8, 4, 81 * MiB, 4, 8),
]


@pytest.mark.parametrize("model,w,t,b,depth", [c[:5] for c in STAGE_PIECES])
def test_pieces_of_a_chunk(model, w, t, b, depth):
    say("stage_through_host pieces", model, "W", w, "T", t, "B", b, "depth", depth)
    rollout = dr.dr_plan_create_host(model, w, t, b).info["rollout_bytes"]
    plan, info, shards, flat = _stage_setup(model, w, t, min(b, 16 * -(-rollout // 16)), depth)
    want, want_cks = _out(info)
    dr.dr_stage_all(plan, shards, want, want_cks)
    for _ in range(2):
        dst, cks = _out(info)
        dr.dr_stage_through_host(plan, shards, dst, cks)
        torch.cuda.synchronize()
        assert torch.equal(dst, want) and torch.equal(cks, want_cks)


SMALL, LARGE = (1, 512, 4, 4, 64, 2048, 8000), (2, 1024, 8, 4, 64, 4096, 16000)
RESHARD_PIECES = [  # model, W, W', B, pieces of the whole call
    (SMALL, 5, 3, 64 * MiB, 1),
    (SMALL, 3, 64, 40 * MiB + 16, 2),
    (SMALL, 8, 1, 16 * MiB, 3),
    (SMALL, 1, 7, 16 * MiB + 16, 3),
    ((1, 64, 2, 2, 8, 96, 400), 2, 64, 4096, 80),
    (LARGE, 5, 3, 64 * MiB + 16, 7),
    (LARGE, 3, 64, 97 * MiB, 7),
    (LARGE, 8, 1, 47 * MiB, 5),
    (LARGE, 1, 7, 1 << 30, 7),
]


@pytest.mark.parametrize("model,w,w2,b", [c[:4] for c in RESHARD_PIECES])
def test_reshard_pieces_across_destination_shards(model, w, w2, b):
    say("reshard_through_host pieces", model, w, "->", w2, "B", b)
    plan = dr.dr_reshard_plan_create(model, w, w2, b)
    info = dr.dr_plan_get_info(plan)
    flat = datagen.make_flat_torch(model, w, 9)
    S, S2 = info["shard_elems"], info["dst_shard_elems"]
    src = [flat[i * S:(i + 1) * S] for i in range(w)]
    n = datagen.flat_sizes(model, w)[0]
    want = oracle.reshard(flat.cpu().numpy(), n, w2).view(np.uint32)
    for _ in range(2):
        dst = [torch.full((S2,), -1, dtype=torch.int32, device="cuda") for _ in range(w2)]
        cks = new_checksums(info["num_chunks"])
        dr.dr_reshard_through_host(plan, src, dst, cks)
        torch.cuda.synchronize()
        got = np.concatenate([d.cpu().numpy().view(np.uint32) for d in dst])
        assert np.array_equal(got, want)
        assert checksums_to_list(cks) == oracle.chunk_checksums(want, b)


def test_a_destination_that_is_not_this_devices_memory_is_reloaded_by_copies():
    """Pinned host memory as the destination (by address) takes the reload by copies; both routes on one plan."""
    wl = workloads.TINY
    plan, info, shards, flat = _stage_setup(wl.model, wl.train_shards, wl.tp, wl.chunk_bytes)
    want, want_cks = _out(info)
    dr.dr_stage_all(plan, shards, want, want_cks)
    for _ in range(2):
        host = torch.zeros(info["rollout_bytes"], dtype=torch.uint8).pin_memory()
        dst, cks = _out(info)
        say("relay into pinned host memory, then into device memory")
        dr.dr_stage_through_host(plan, shards, host.data_ptr(), cks)
        torch.cuda.synchronize()
        assert torch.equal(host, want.cpu()) and torch.equal(cks, want_cks)
        dr.dr_stage_through_host(plan, shards, dst, cks)
        torch.cuda.synchronize()
        assert torch.equal(dst, want) and torch.equal(cks, want_cks)


def test_calls_on_two_streams_of_one_plan_are_ordered():
    """Calls issued one after another on different streams share the pinned buffers: the plan orders them."""
    wl = workloads.TINY
    plan, info, shards, flat = _stage_setup(wl.model, wl.train_shards, wl.tp, wl.chunk_bytes)
    S = info["shard_elems"]
    other = torch.empty_like(flat).copy_(flat).mul_(2.0)
    shards2 = [other[i * S:(i + 1) * S] for i in range(wl.train_shards)]
    want = [_out(info) for _ in range(2)]
    for sh, (d, c) in zip((shards, shards2), want):
        dr.dr_stage_all(plan, sh, d, c)
    outs = [_out(info) for _ in range(8)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    say("relay calls alternating between two streams")
    for i, (d, c) in enumerate(outs):
        dr.dr_stage_through_host(plan, (shards, shards2)[i % 2], d, c, stream=streams[i % 2])
    torch.cuda.synchronize()
    for i, (d, c) in enumerate(outs):
        assert torch.equal(d, want[i % 2][0]) and torch.equal(c, want[i % 2][1]), i


def test_a_stream_that_is_gone_when_the_plan_is_used_again():
    """The plan orders its calls by an event recorded on the caller's stream, which may be destroyed by then."""
    wl = workloads.TINY
    plan, info, shards, flat = _stage_setup(wl.model, wl.train_shards, wl.tp, wl.chunk_bytes)
    want, want_cks = _out(info)
    dr.dr_stage_all(plan, shards, want, want_cks)
    torch.cuda.synchronize()
    hip = dr._lib  # the HIP runtime is among the library's dependencies
    for i in range(3):
        st = ctypes.c_void_p()
        assert hip.hipStreamCreateWithFlags(ctypes.byref(st), ctypes.c_uint(1)) == 0  # non-blocking
        dst, cks = _out(info)
        torch.cuda.synchronize()
        say("relay on a stream that is then destroyed", i)
        dr.dr_stage_through_host(plan, shards, dst, cks, stream=st.value)
        assert hip.hipStreamSynchronize(st) == 0
        assert hip.hipStreamDestroy(st) == 0
        assert torch.equal(dst, want) and torch.equal(cks, want_cks)
    plan.close()


def test_refused_while_the_stream_is_captured():
    wl = workloads.TINY
    plan, info, shards, flat = _stage_setup(wl.model, wl.train_shards, wl.tp, wl.chunk_bytes)
    want, want_cks = _out(info)
    dr.dr_stage_all(plan, shards, want, want_cks)
    dst, cks = _out(info)
    buf = torch.zeros(16, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    say("relay under capture")
    with torch.cuda.graph(g):
        buf.add_(1.0)
        with pytest.raises(dr.DrError) as e:
            dr.dr_stage_through_host(plan, shards, dst, cks, torch.cuda.current_stream())
    assert e.value.code == dr.DR_EHIP and "captured" in str(e.value)
    dr.dr_stage_through_host(plan, shards, dst, cks)
    torch.cuda.synchronize()
    assert torch.equal(dst, want) and torch.equal(cks, want_cks)
