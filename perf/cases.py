"""What the speed of this framework is measured on.

Each case is a call, or a short run of calls, that an engine built on the library makes for a batch of
requests, through the public Python entry points:

  hop         one layer from the decode side's paged pool to the prefill side's: kvl_pack_layer into the
              dense transfer buffer, kvl_unpack_layer out of it (also for the appended tail that goes back)
  move        the same between two pools of one device without the buffer: kvl_move_layer
  fullblocks  some layers out of a buffer of Full Blocks into the pool and back into another such buffer
  host        one layer from a pinned host buffer into the pool, and from a pool into a pinned host buffer
  stream      kvl_stream_layers: every layer from pinned host memory under the compute of the one before
  step        a whole batch: both plans made, every layer packed and unpacked, the plans dropped

Sizes are given by the case alone; block tables and contents come from the seed.  Buffers are int64 tensors
where their bytes allow it (bytes are opaque to the library), and results are whole buffers: the transfer
buffer and the destination pool, rows that nothing was written to included.
"""
import math

import numpy as np
import torch

import kvl_workloads as W
import paper_2602_21548_amd as K

SENTINEL = 0x5A


def _case(name, path, bs, rows, requests, hit, append=(0, 0), lengths="uniform", table="random", tokens="hit",
          layers=1, pool=0):
    """A case as a dict of plain values; `hit` and `append` are ranges (lognormal: median and cap)."""
    return {"name": name, "path": path, "block_tokens": bs, "rows": "+".join(str(r) for r in rows),
            "requests": requests, "hit_lo": hit[0], "hit_hi": hit[1], "append_lo": append[0],
            "append_hi": append[1], "lengths": lengths, "table": table, "tokens": tokens, "layers": layers,
            "pool_blocks": pool}


def listed():
    return [
        # the smallest call: four short requests, 16-token blocks of a 576-element bf16 row; its layer is a
        # few MB, so launches and the host's part of them are most of the time
        _case("hop_tiny_mla", "hop", 16, (1152,), 4, (1000, 1000), pool=512),
        # grouped-query attention: K and V in planes of their own, 64 requests of 16-64 K cached tokens
        _case("hop_gqa", "hop", 64, (2048, 2048), 64, (16384, 65536), (256, 1024)),
        # latent attention in bf16, 128 requests around 32 K tokens: the plain large layer
        _case("hop_mla", "hop", 64, (1152,), 128, (32768, 131072), lengths="lognormal"),
        # the largest: latent attention in fp8 with its scales, 656-byte rows that are no multiple of a cache
        # line, 256 requests, no two neighbouring blocks adjacent
        _case("hop_fp8_mla", "hop", 64, (656,), 256, (8192, 131072), (256, 1024), table="fragmented"),
        # pools that are paged token by token: a million blocks of one row
        _case("hop_token_granular", "hop", 1, (1152,), 32, (16384, 49152), (128, 512)),
        # rows that are no multiple of 16 bytes: 128 one-byte values and a 4-byte scale
        _case("hop_odd_rows", "hop", 64, (132,), 64, (16384, 49152), (256, 1024)),
        # the tail a prefill engine sends back: only the appended tokens of each request, many ragged ends
        _case("hop_return_tail", "hop", 64, (2048, 2048), 64, (16384, 65536), (256, 1024), tokens="append"),
        # both engines on one device, or a pool being re-paged
        _case("move_mla", "move", 64, (1152,), 16, (16384, 49152), (256, 1024)),
        # the storage layout next to the pools: four layers of 61-layer blocks in and out again
        _case("fullblocks_mla", "fullblocks", 64, (1152,), 4, (8192, 24576), (0, 64), layers=61),
        # the prefill engine's own host buffer, and the way out to the decode engine's
        _case("host_mla", "host", 64, (1152,), 4, (16384, 49152), (256, 1024)),
        # layer-wise prefill from host memory: eight layers, 200 us of compute each, two resident layers
        _case("stream_mla", "stream", 64, (1152,), 4, (8192, 24576), (256, 1024), layers=8),
        # a batch as an engine serves it, 16-token pages: two plans, 61 layers each way
        _case("step_paged16", "step", 16, (1152,), 4, (16384, 49152), (256, 1024), layers=61),
    ]


def _spread(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """Another case of the ranges above: any block size and row size, a few MB to a few GB a layer."""
    path = rng.choice(["hop"] * 6 + ["move", "fullblocks", "host", "step"])
    bs = rng.choice([1, 8, 16, 24, 32, 64, 64, 100, 128, 256])
    kind = rng.choice(["one", "one", "two", "odd", "apart"])
    r16 = 16 * max(4, round(_spread(rng, 64, 4096) / 16))
    if kind == "one":
        rows = (r16,)
    elif kind == "two":
        rows = (min(r16, 2048),) * 2
    elif kind == "odd":
        r = round(_spread(rng, 20, 2000))
        rows = (r if r % 16 else r + 4,)
        bs = max(bs, 16)
    else:
        rows = (1024, 128)
    row = sum(rows)
    most = {"hop": 6e9, "move": 4e9, "fullblocks": 6e7, "host": 1.5e8, "step": 1.5e8}[path]
    payload = _spread(rng, 2e6, min(most, 3e8) if kind == "odd" else most)
    table = rng.choice(["random", "random", "fragmented", "runs", "contiguous"])
    tokens = rng.choice(["hit", "hit", "hit", "append", "all"]) if path == "hop" else "hit"
    total = min(payload / row, 1_000_000 * bs)        # at most a million blocks
    requests = max(1, min(256, round(_spread(rng, 1, 256)), int(total // 64)))
    mean = max(32, int(total / requests))
    around = (max(1, mean // 2), mean + mean // 2)
    few = (0, max(1, mean // 16))
    if table == "fragmented" and mean < 32 * bs:
        table = "random"                              # too few blocks to keep neighbours apart
    if table == "runs" and total > 100_000 * bs:
        table = "random"                              # such tables take long to draw
    hit, append = (few, around) if tokens == "append" else (around, few)
    layers = {"fullblocks": 61 if bs * row * 61 < 8e6 else 16, "step": rng.choice([8, 32])}.get(path, 1)
    c = _case("", path, bs, rows, requests, hit, append, table=table, tokens=tokens, layers=layers)
    del c["name"]
    return c


def _rows(case):
    return tuple(int(r) for r in case["rows"].split("+"))


def _lengths(case):
    """(hit, append) of every request: drawn from the case's ranges, the same for every seed."""
    rng = np.random.Generator(np.random.PCG64([W.BASE_SEED, case["requests"], case["hit_lo"], case["hit_hi"]]))
    n = case["requests"]
    if case["lengths"] == "lognormal":
        hit = np.minimum(rng.lognormal(math.log(case["hit_lo"]), 0.5, size=n), case["hit_hi"])
        app = np.maximum(1, np.rint(hit * 5.0 / 95.0))
    else:
        hit = rng.integers(case["hit_lo"], case["hit_hi"] + 1, size=n)
        app = rng.integers(case["append_lo"], case["append_hi"] + 1, size=n)
    return hit.astype(np.uint32), app.astype(np.uint32)


def _moved(case):
    """Tokens whose rows one layer's pass moves."""
    hit, app = _lengths(case)
    return int({"hit": hit, "append": app, "all": hit + app}[case["tokens"]].astype(np.int64).sum())


FULLBLOCK_LAYERS = 4        # layers that one pass of the fullblocks path takes in and out


def work(case):
    """Every moved row is read once and written once a copy; descriptors and block tables are not counted."""
    payload = _moved(case) * sum(_rows(case))
    copies = {"hop": 2, "move": 1, "host": 2, "fullblocks": 2 * FULLBLOCK_LAYERS, "stream": case["layers"],
              "step": 2 * case["layers"]}[case["path"]]
    return {"bytes": 2 * payload * copies, "flops": 0}


def tolerance(case):
    return "exact"          # bytes are moved, none is computed


def _buffer(nbytes, parts=1):
    """`parts` buffers of nbytes each, end to end."""
    if nbytes % 8 == 0:
        return torch.empty(parts * nbytes // 8, dtype=torch.int64, device="cuda")
    return torch.empty(parts * nbytes, dtype=torch.uint8, device="cuda")


def _random(nbytes, gen):
    t = _buffer(nbytes)
    return t.random_(generator=gen)


def _marked(nbytes, parts=1):
    t = _buffer(nbytes, parts)
    return t.fill_(int.from_bytes(bytes([SENTINEL] * t.element_size()), "little"))


def _pinned(nbytes, gen=None):
    d = _random(nbytes, gen) if gen is not None else _marked(nbytes)
    h = torch.empty(d.shape, dtype=d.dtype, pin_memory=True)
    h.copy_(d)
    return h


class _Batch:
    """A batch's lengths, its two sides' block tables and layouts, and its pools' plane sizes."""

    def __init__(self, case, seed):
        bs, self.rows = case["block_tokens"], _rows(case)
        self.hit, self.app = _lengths(case)
        blocks = (self.hit.astype(np.int64) + self.app + bs - 1) // bs
        pool = case["pool_blocks"] or int(math.ceil(1.1 * int(blocks.sum()))) + 1
        rng = np.random.Generator(np.random.PCG64([seed, 7]))
        self.src = W.make_tables(blocks, pool, case["table"], rng)
        self.dst = W.make_tables(blocks, pool, case["table"], rng)
        self.layout = K.make_layout(case["layers"], bs, self.rows, pool)
        self.plane_bytes = [pool * bs * r for r in self.rows]
        self.flag = {"hit": 0, "append": K.KVL_TOKENS_APPEND, "all": K.KVL_TOKENS_ALL}[case["tokens"]]
        self.payload = _moved(case) * sum(self.rows)

    def plan(self, side, flags):
        tables = self.src if side == "src" else self.dst
        return K.kvl_plan(self.layout, self.hit, self.app, tables, flags | self.flag)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    b = _Batch(case, seed)
    s = {"path": case["path"], "layers": case["layers"], "batch": b}
    path = case["path"]
    if path in ("hop", "move", "step"):
        resident = 2 if path == "step" else 1           # source layers; every destination layer is kept
        s["src"] = [[_random(n, gen) for n in b.plane_bytes] for _ in range(resident)]
        s["out"] = [_marked(n, case["layers"]) for n in b.plane_bytes]
        s["dst"] = list(zip(*(t.chunk(case["layers"]) for t in s["out"])))
    if path in ("hop", "step"):
        s["xfer"] = _marked(b.payload)
    if path in ("hop", "move"):
        s["gather"], s["scatter"] = b.plan("src", K.KVL_GATHER), b.plan("dst", K.KVL_SCATTER)
    if path == "move":
        s["pair"] = K.kvl_plan_pair(s["gather"], s["scatter"])
    if path == "fullblocks":
        s["gather"] = b.plan("dst", K.KVL_GATHER | K.KVL_NO_MERGE)
        s["scatter"] = b.plan("dst", K.KVL_SCATTER | K.KVL_NO_MERGE)
        size, count = s["scatter"].fullblock_geometry()
        s["blocks"], s["out"] = _random(size * count, gen), _marked(size * count)
        s["dst"] = [[_marked(n) for n in b.plane_bytes] for _ in range(2)]
    if path == "host":
        s["gather"], s["scatter"] = b.plan("src", K.KVL_GATHER), b.plan("dst", K.KVL_SCATTER)
        s["src"] = [_random(n, gen) for n in b.plane_bytes]
        s["dst"] = [_marked(n) for n in b.plane_bytes]
        s["host_in"], s["host_out"] = _pinned(b.payload, gen), _pinned(b.payload)
    if path == "stream":
        s["scatter"] = b.plan("dst", K.KVL_SCATTER)
        s["host"] = [_pinned(b.payload, gen) for _ in range(2)]
        s["slots"] = [[_marked(n) for n in b.plane_bytes] for _ in range(2)]
        s["streams"] = [torch.cuda.Stream() for _ in range(3)]
    return s


def run(s):
    path, b = s["path"], s["batch"]
    if path == "hop":
        K.kvl_pack_layer(s["gather"], s["src"][0], s["xfer"])
        K.kvl_unpack_layer(s["scatter"], s["xfer"], s["dst"][0])
        return [s["xfer"], *s["out"]]
    if path == "move":
        K.kvl_move_layer(s["pair"], s["src"][0], s["dst"][0])
        return s["out"]
    if path == "fullblocks":
        for layer in range(FULLBLOCK_LAYERS):
            pool = s["dst"][layer % 2]
            K.kvl_fullblocks_to_pool_layer(s["scatter"], s["blocks"], layer, pool)
            K.kvl_pool_to_fullblocks_layer(s["gather"], pool, layer, s["out"])
        return [s["out"], *s["dst"][0], *s["dst"][1]]
    if path == "host":
        stream = torch.cuda.current_stream()
        K.kvl_h2d_unpack_layer(s["scatter"], s["host_in"], None, 0, s["dst"], stream, stream)
        K.kvl_pack_layer(s["gather"], s["src"], s["host_out"])
        return [s["host_out"], *s["dst"]]
    if path == "stream":
        K.kvl_stream_layers(s["scatter"], s["host"], s["slots"], None, 0, 200, *s["streams"], n_layers=s["layers"])
        return [p for slot in s["slots"] for p in slot]
    gather, scatter = b.plan("src", K.KVL_GATHER), b.plan("dst", K.KVL_SCATTER)
    for layer in range(s["layers"]):
        K.kvl_pack_layer(gather, s["src"][layer % 2], s["xfer"])
        K.kvl_unpack_layer(scatter, s["xfer"], s["dst"][layer])
    gather.destroy()
    scatter.destroy()
    return [s["xfer"], *s["out"]]
