"""The work that a user of the library has it do, as cases that can be timed and compared.

Every case is one pass through the public binding (paper_2607_22614_amd.dr): pack a whole rollout
stream, pack it chunk by chunk, send it through host memory, re-cut the training state to another
shard count, checksum, offload and restore the Adam moments.  Sizes are the repository's own
workloads (workloads.py), those shapes at another depth, and a generic ragged decoder whose
column slices are no whole groups of elements.

    op             call                        stands for
    stage          dr_stage_all                the weight path of a role switch
    chunks         dr_stage_chunk, each chunk  the same in bounded chunks that the caller ships
    stage_host     dr_stage_through_host       the same through two bounded pinned buffers
    reshard        dr_reshard                  training state to another number of shards
    reshard_host   dr_reshard_through_host     the same through two bounded pinned buffers
    moment_sums    dr_moment_checksums         checksums around an offload/restore round trip
    offload        dr_offload_moments          Adam moments to host memory
    restore        dr_restore_moments          and back
"""
import math

import numpy as np
import torch

from paper_2607_22614_amd import datagen, dr, workloads

KiB, MiB, GiB = 1 << 10, 1 << 20, 1 << 30

_SHAPE = ("n_layers", "hidden", "n_q_heads", "n_kv_heads", "head_dim", "ffn", "vocab")
_MOMENT_OPS = ("moment_sums", "offload", "restore")


def _case(name, op, wl, *, layers=None, to=0, chunk=None, moment_chunk=0, specials=False):
    c = dict(zip(_SHAPE, wl.model))
    if layers is not None:
        c["n_layers"] = layers
    c.update(name=name, op=op, w=wl.train_shards, tp=wl.tp, to=to, chunk_bytes=chunk or wl.chunk_bytes,
             moment_chunk_bytes=moment_chunk, specials=specials)
    return c


# A decoder whose width per rank is odd (ffn/tp = 1821), as an FFN of 8/3 x hidden easily is, on
# odd shard, rank and vocabulary counts: the down projection's column slices start at any element.
RAGGED = workloads.Workload("ragged", 0, 12, 2056, 12, 6, 72, 3 * 1821, 3 * 16753, train_shards=5, tp=3,
                            chunk_bytes=48 * MiB + 16)


def listed():
    tiny, half, eight = workloads.TINY, workloads.HALF_B, workloads.EIGHT_B
    return [
        # the smallest call: one pack of 5 MB, all launches and latency
        _case("tiny_stage", "stage", tiny),
        # the smallest bounded chunks (256 KiB), 21 calls in a row
        _case("tiny_chunks", "chunks", tiny),
        # an ordinary pack: 0.5B on one rank, weights with ties, subnormals, infinities and NaN
        _case("half_b_stage", "stage", half, specials=True),
        # the same bounded: 20 calls of 64 MiB
        _case("half_b_chunks", "chunks", half),
        # the large pack: 8B over 8 shards to 4 ranks, 48 GB moved
        _case("eight_b_stage", "stage", eight),
        # odd everything: column slices that are no whole groups, chunk budget no power of two
        _case("ragged_stage", "stage", RAGGED),
        # the 8B shape at 16 layers, 8 to 6 shards
        _case("eight_b_16_layers_reshard", "reshard", eight, layers=16, to=6),
        # its moments' checksums (36 GB read), in the 512 MiB chunks of the 8B + Adam workload
        _case("eight_b_16_layers_moment_sums", "moment_sums", eight, layers=16, moment_chunk=512 * MiB),
        # the host path: weights, training state, moments out and back
        _case("half_b_stage_host", "stage_host", half),
        _case("ragged_reshard_host", "reshard_host", RAGGED, to=3, chunk=8 * MiB),
        _case("half_b_offload", "offload", half, moment_chunk=128 * MiB),
        _case("half_b_restore", "restore", half, moment_chunk=128 * MiB),
    ]


# Training elements a drawn case has at most, by op: those of the largest listed case of that kind.
_MOST = {"stage": 8e9, "chunks": 8e9, "reshard": 4.4e9, "moment_sums": 4.4e9, "stage_host": 6e8, "reshard_host": 3e8,
         "offload": 6e8, "restore": 6e8}
_LEAST = 2e6
_MOST_CALLS = 200  # chunk calls, and chunks through host memory, in one pass


def _log_uniform(rng, a, b):
    return math.exp(rng.uniform(math.log(a), math.log(b)))


def _draw_shape(rng, tp, most):
    """A decoder whose size is spread over the logarithm of [_LEAST, most]; tp divides what it has to."""
    while True:
        target = _log_uniform(rng, _LEAST, most)
        kv = tp * rng.choice((1, 1, 2))
        q = kv * rng.choice((1, 2, 4, 7))
        d = rng.choice((32, 64, 64, 80, 96, 128, 128))
        hidden = 8 * round(_log_uniform(rng, 128, 6144) / 8)
        if rng.random() < 0.5:  # as configured models have it: whole groups per rank
            ffn = tp * 64 * max(1, round(hidden * rng.uniform(2, 5.5) / (64 * tp)))
        else:  # any width per rank
            ffn = tp * max(1, round(hidden * rng.uniform(2, 5.5) / tp))
        vocab = tp * max(1, round(_log_uniform(rng, 1000, 160000) / tp))
        one = (1, hidden, q, kv, d, ffn, vocab)
        none = (0, hidden, q, kv, d, ffn, vocab)
        n0 = datagen.flat_sizes(none, 1)[0]
        n1 = datagen.flat_sizes(one, 1)[0] - n0
        layers = round((target - n0) / n1)
        if not 1 <= layers <= 96:
            continue
        n = n0 + layers * n1
        if target / 1.5 <= n <= min(most, target * 1.5):
            return (layers,) + one[1:], n


def draw(rng):
    op = rng.choice(("stage", "stage", "stage", "chunks", "chunks", "reshard", "moment_sums", "stage_host",
                     "reshard_host", "offload", "restore"))
    tp = rng.choice((1, 2, 3, 4, 8))
    shape, n = _draw_shape(rng, tp, _MOST[op])
    out_bytes = (4 if op.startswith("reshard") else 2) * n
    c = dict(zip(_SHAPE, shape))
    c.update(op=op, w=rng.choice((1, 2, 3, 4, 5, 8, 8, 13, 16, 64)), tp=tp, to=0, moment_chunk_bytes=0,
             specials=op == "stage" and rng.random() < 0.25 and n < 1e9)
    most = 256 * MiB if op.endswith("_host") else GiB
    least = max(256 * KiB, out_bytes // _MOST_CALLS) if op == "chunks" or op.endswith("_host") else 256 * KiB
    c["chunk_bytes"] = 16 * round(_log_uniform(rng, least, max(least + 16, most)) / 16 + 1)
    if op.startswith("reshard"):
        c["to"] = rng.choice([w for w in (1, 2, 3, 4, 6, 7, 8, 16, 64) if w != c["w"]])
    if op in _MOMENT_OPS:
        least = 256 * KiB if op == "moment_sums" else max(4 * MiB, 8 * n // _MOST_CALLS)
        c["moment_chunk_bytes"] = 16 * round(_log_uniform(rng, least, 512 * MiB) / 16)
    return c


def _model(case):
    return tuple(case[k] for k in _SHAPE)


def _source(case, seed):
    """The padded flat fp32 training buffer of the case, on the GPU."""
    model = _model(case)
    flat = datagen.make_flat_torch(model, case["w"], seed)
    if case["specials"]:  # 0.1 % of the weights: ties, subnormals, infinities, NaN, zeros
        n = datagen.flat_sizes(model, case["w"])[0]
        rng = np.random.default_rng(seed)
        k = n // 1000
        pos = np.unique(rng.integers(0, n, k))
        val = datagen.special_values(rng, pos.size).view(np.int32)
        flat.view(torch.int32)[torch.from_numpy(pos).cuda()] = torch.from_numpy(val).cuda()
    return flat


def _cut(flat, w):
    """W views of one flat buffer."""
    s = flat.numel() // w
    return [flat[i * s:(i + 1) * s] for i in range(w)]


def _checksums(n):
    return torch.zeros((n, 2), dtype=torch.int64, device="cuda")


def prepare(case, seed):
    op, w = case["op"], case["w"]
    st = {"op": op}
    if op.startswith("reshard"):
        plan = dr.dr_reshard_plan_create(_model(case), w, case["to"], case["chunk_bytes"])
        info = plan.info
        src = _source(case, seed)
        dst = torch.zeros(info["rollout_bytes"] // 4, dtype=torch.float32, device="cuda")
        st.update(plan=plan, src=_cut(src, w), flat=dst, dst=_cut(dst, case["to"]), cks=_checksums(info["num_chunks"]))
        return st
    plan = dr.dr_plan_create(_model(case), w, case["tp"], case["chunk_bytes"], case["moment_chunk_bytes"])
    info = plan.info
    st["plan"] = plan
    if op in _MOMENT_OPS:
        m, v = datagen.make_moments_torch(info["padded_elems"], seed)
        if op == "restore":
            store = torch.cat([m.cpu(), v.cpu()])
            m.zero_()
            v.zero_()
        else:
            store = torch.zeros(info["moment_bytes"] // 4, dtype=torch.float32) if op == "offload" else None
        st.update(m=m, v=v, ms=_cut(m, w), vs=_cut(v, w), store=store, side=torch.cuda.Stream(),
                  cks=_checksums(info["num_moment_chunks"]))
        return st
    dst = torch.zeros(info["rollout_bytes"] // 2, dtype=torch.bfloat16, device="cuda")
    cks = _checksums(info["num_chunks"])
    st.update(src=_cut(_source(case, seed), w), dst=dst, cks=cks)
    if op == "chunks":  # where each chunk goes, and its checksum
        b = case["chunk_bytes"] // 2
        st["slots"] = [(dst[c * b:(c + 1) * b], cks[c]) for c in range(info["num_chunks"])]
    return st


def run(st):
    op, plan = st["op"], st["plan"]
    if op == "stage":
        dr.dr_stage_all(plan, st["src"], st["dst"], st["cks"])
    elif op == "chunks":
        for c, (dst, ck) in enumerate(st["slots"]):
            dr.dr_stage_chunk(plan, c, st["src"], dst, ck)
    elif op == "stage_host":
        dr.dr_stage_through_host(plan, st["src"], st["dst"], st["cks"])
    elif op == "reshard":
        dr.dr_reshard(plan, st["src"], st["dst"], st["cks"])
        return {"state": st["flat"], "checksums": st["cks"]}
    elif op == "reshard_host":
        dr.dr_reshard_through_host(plan, st["src"], st["dst"], st["cks"])
        return {"state": st["flat"], "checksums": st["cks"]}
    elif op == "moment_sums":
        dr.dr_moment_checksums(plan, st["ms"], st["vs"], st["cks"])
        return {"checksums": st["cks"]}
    elif op == "offload":
        dr.dr_offload_moments(plan, st["ms"], st["vs"], st["store"], st["side"])
        return {"store": st["store"]}
    else:
        dr.dr_restore_moments(plan, st["store"], st["ms"], st["vs"], st["side"])
        return {"m": st["m"], "v": st["v"]}
    return {"rollout": st["dst"], "checksums": st["cks"]}


def work(case):
    model, w, op = _model(case), case["w"], case["op"]
    n, npad = datagen.flat_sizes(model, w)
    if op.startswith("reshard"):
        return {"bytes": 4 * n + 4 * datagen.flat_sizes(model, case["to"])[1], "flops": 0}
    if op in _MOMENT_OPS:  # read once; the transfers also write once
        return {"bytes": 8 * npad * (1 if op == "moment_sums" else 2), "flops": 0}
    norms = (2 * case["n_layers"] + 1) * case["hidden"]  # on every rank
    return {"bytes": 4 * n + 2 * (n + (case["tp"] - 1) * norms), "flops": 0}


def tolerance(case):
    """One rounding per element, the moved bits and integer sums: every correct path gives the same bits."""
    return "exact"


def exact(case, seed):
    op = case["op"]
    if op == "moment_sums":
        return None
    if op in _MOMENT_OPS:
        m, v = datagen.make_moments_torch(datagen.flat_sizes(_model(case), case["w"])[1], seed)
        m, v = m.double(), v.double()
        return {"store": torch.cat([m, v]).cpu()} if op == "offload" else {"m": m, "v": v}
    model = _model(case)
    n = datagen.flat_sizes(model, case["w"])[0]
    flat = _source(case, seed)
    if op.startswith("reshard"):
        out = torch.zeros(datagen.flat_sizes(model, case["to"])[1], dtype=torch.float64, device="cuda")
        out[:n] = flat[:n]
        return {"state": out, "checksums": None}
    layers, h, q, kv, d, f, v = model
    t = case["tp"]
    shapes = {"embed": (v, h), "lm_head": (v, h), "q": (q * d, h), "k": (kv * d, h), "v": (kv * d, h),
              "o": (h, q * d), "gate": (f, h), "up": (f, h), "down": (h, f)}
    src, off = {}, 0
    for name, numel, _ in datagen.tensor_list(model):
        src[name] = flat[off:off + numel].view(shapes.get(name.rpartition(".")[2], (1, numel)))
        off += numel

    def rows(name, r):  # rank r's share of the rows; one row (a norm): all of it
        x = src[name]
        k = x.shape[0] // t
        return x[r * k:(r + 1) * k] if x.shape[0] > 1 else x

    def cols(name, r):
        x = src[name]
        k = x.shape[1] // t
        return x[:, r * k:(r + 1) * k]

    norms = (2 * layers + 1) * h
    out = torch.empty(n + (t - 1) * norms, dtype=torch.float64, device="cuda")
    at = 0
    for r in range(t):
        parts = [rows("embed", r)]
        for i in range(layers):
            p = f"layers.{i}."
            parts += [rows(p + "ln1", r), rows(p + "q", r), rows(p + "k", r), rows(p + "v", r), cols(p + "o", r),
                      rows(p + "ln2", r), rows(p + "gate", r), rows(p + "up", r), cols(p + "down", r)]
        parts += [rows("final_norm", r), rows("lm_head", r)]
        for x in parts:
            out[at:at + x.numel()].view(x.shape).copy_(x)
            at += x.numel()
    return {"rollout": out, "checksums": None}
