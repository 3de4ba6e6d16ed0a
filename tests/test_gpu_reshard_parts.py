"""Reshard where its workgroups' parts of a tile and their grouped order can go wrong, on the GPU against the oracle:
chunks of one group, of one and two parts and one group around each, and counts of parts around a window of 256;
ragged shards whose segments end in any part."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_22614_amd import datagen, dr
from tests.gpu_helpers import checksums_to_list, new_checksums, require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("w,w2", [(1, 3), (5, 2)])
@pytest.mark.parametrize("b", [16, 4080, 4096, 4112, 8176, 8192, 8208, 16368, 16384, 16400, 256 * 8192, 257 * 8192 + 16])
def test_parts_and_order(b, w, w2):
    model = (1, 64, 2, 2, 8, 96, 40) if b == 16 else (1, 256, 4, 4, 64, 688, 1000 + (b // 16) % 7)
    say("reshard parts", model, w, "->", w2, "B", b)
    plan = dr.dr_reshard_plan_create(model, w, w2, b)
    info = dr.dr_plan_get_info(plan)
    flat = datagen.make_flat_numpy(model, w, seed=3, specials_frac=0.01)
    S, S2 = info["shard_elems"], info["dst_shard_elems"]
    n = datagen.flat_sizes(model, w)[0]
    src = [torch.from_numpy(flat[i * S:(i + 1) * S].copy()).cuda() for i in range(w)]
    want = oracle.reshard(flat, n, w2).view(np.uint32)
    for _ in range(2):  # the accumulators are back at zero after the first
        dst = [torch.full((S2,), -1, dtype=torch.int32, device="cuda") for _ in range(w2)]
        cks = new_checksums(info["num_chunks"])
        dr.dr_reshard(plan, src, dst, cks)
        torch.cuda.synchronize()
        got = np.concatenate([d.cpu().numpy().view(np.uint32) for d in dst])
        assert np.array_equal(got, want)
        assert checksums_to_list(cks) == oracle.chunk_checksums(want, b)


# more than 44 GiB read and written (a workgroup then moves a whole tile): ragged shards and chunks, and 64 shards
@pytest.mark.parametrize("w,w2,b,vocab", [(13, 7, (48 << 20) + 16, 725001), (1, 64, 1 << 30, 730001)])
def test_whole_tiles(w, w2, b, vocab):
    model = (0, 4096, 32, 8, 128, 14336, vocab)
    say("reshard whole tiles", model, w, "->", w2, "B", b)
    plan = dr.dr_reshard_plan_create(model, w, w2, b)
    info = dr.dr_plan_get_info(plan)
    assert 4 * info["n_elems"] + info["rollout_bytes"] > 44 << 30
    n, S, S2 = info["n_elems"], info["shard_elems"], info["dst_shard_elems"]
    flat = torch.empty(w * S, dtype=torch.int32, device="cuda").random_()
    src = [flat[i * S:(i + 1) * S] for i in range(w)]
    out = torch.full((w2 * S2,), -1, dtype=torch.int32, device="cuda")
    cks = new_checksums(info["num_chunks"])
    dr.dr_reshard(plan, src, [out[i * S2:(i + 1) * S2] for i in range(w2)], cks)
    torch.cuda.synchronize()
    assert torch.equal(out[:n], flat[:n]) and not out[n:].any()
    want = []
    for e in range(0, w2 * S2, b // 4):  # sums mod 2^64, as 64-bit integers wrap
        word = out[e:e + b // 4].to(torch.int64) & 0xFFFFFFFF
        at = torch.arange(1, word.numel() + 1, device="cuda")
        want.append(torch.stack([word.sum(), (at * word).sum()]))
    assert torch.equal(cks, torch.stack(want))
