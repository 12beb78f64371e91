"""The dispatch's edges: sizes at which a launch changes its kernel, its tile or its remainder, against the
CPU oracle, bit for bit (the comparison is exact: bytes are moved, none is computed)."""
import ctypes as C

import numpy as np
import pytest
import torch

import kvl_workloads as W
import oracle
import paper_2602_21548_amd as K
from gpu_util import dev_plan, planes_to_dev, same_bytes, to_dev, to_host

pytestmark = pytest.mark.gpu

GUARD = 256


def hop_at(w, x_off=0, pool_off=0, **tuning):
    """pack and unpack with the transfer buffer x_off and the pools pool_off bytes into their allocations;
    nothing outside them may change."""
    bs, rows = w.layout.block_tokens, w.layout.row_bytes
    src = W.fill_pool(w, 0, "src")
    want_x = oracle.pack(bs, rows, w.hit, w.src.tables, src, threads=8)
    want_dst = W.sentinel_pool(w, "dst")
    oracle.unpack(bs, rows, w.hit, w.dst.tables, want_x, want_dst, threads=8)

    def placed(a, off):
        t = torch.full((a.size + off + GUARD,), 0x3C, dtype=torch.uint8, device="cuda")
        t[off:off + a.size] = to_dev(a)
        return t

    g, s = dev_plan(w, "src", K.KVL_GATHER, **tuning), dev_plan(w, "dst", K.KVL_SCATTER, **tuning)
    d_src = [placed(p, pool_off) for p in src]
    d_dst = [placed(p, pool_off) for p in W.sentinel_pool(w, "dst")]
    n = want_x.size
    d_x = torch.full((n + x_off + GUARD,), 0x3C, dtype=torch.uint8, device="cuda")
    K.kvl_pack_layer(g, [t[pool_off:pool_off + p.size] for t, p in zip(d_src, src)], d_x[x_off:x_off + n])
    K.kvl_unpack_layer(s, d_x[x_off:x_off + n], [t[pool_off:pool_off + p.size] for t, p in zip(d_dst, src)])
    torch.cuda.synchronize()
    got = to_host(d_x)
    assert same_bytes(got[x_off:x_off + n], want_x), "pack differs from the oracle"
    assert np.all(got[:x_off] == 0x3C) and np.all(got[x_off + n:] == 0x3C), "pack wrote outside the payload"
    for t, want in zip(d_dst, want_dst):
        got = to_host(t)
        assert same_bytes(got[pool_off:pool_off + want.size], want), "unpack differs from the oracle"
        assert np.all(got[:pool_off] == 0x3C) and np.all(got[pool_off + want.size:] == 0x3C)
    g.destroy()
    s.destroy()


# spans below one vector, of one vector, around it; 288 and 289 vectors (flat / tiled); around two tiles of 256
@pytest.mark.parametrize("bs,row", [(1, 1), (3, 5), (1, 15), (1, 16), (1, 17), (5, 3), (2, 33), (16, 36), (64, 132),
                                    (16, 287), (16, 288), (17, 271), (1, 4578), (1, 4579), (1, 4594), (8, 1009),
                                    (1, 8065), (1, 8066), (4, 2049), (3, 8191)])
@pytest.mark.parametrize("x_off,pool_off", [(0, 0), (1, 0), (0, 7), (13, 19)])
def test_rows_and_addresses_off_the_16_byte_grid(bs, row, x_off, pool_off):
    w = W.tiny(900 + bs + row, 6, bs, (row,), 90, 10 * bs, kind="runs" if row % 2 else "fragmented")
    hop_at(w, x_off, pool_off)


@pytest.mark.parametrize("tuning", [dict(max_groups=3), dict(block_threads=64), dict(max_groups=2, block_threads=1024)])
@pytest.mark.parametrize("bs,row", [(1, 57), (16, 132), (64, 132)])
def test_odd_rows_split_over_launches_and_walked(bs, row, tuning):
    hop_at(W.tiny(940 + row, 5, bs, (row, row, 16), 120, 20 * bs), 3, 1, **tuning)


# layers that the on-die cache keeps from the gather to the scatter (plain loads), tiled, one and several tiles, and walked; flat
# ones pass it by already, whole lines up to 256 windows among them (200 by 16 and 124 by 32; 70 by 64, 281, is tiled)
@pytest.mark.parametrize("bs,row,tuning", [(64, 132, {}), (64, 1026, {}), (64, 132, dict(max_groups=1000)), (16, 132, {}), (1, 8065, {}), (5, 1009, {}),
                                           (16, 200, {}), (32, 124, {}), (64, 70, {})])
@pytest.mark.parametrize("x_off,pool_off", [(0, 0), (13, 19)])
def test_odd_rows_of_layers_that_are_kept_or_dealt_out_flat(bs, row, tuning, x_off, pool_off):
    w = _uniform(3, (70 << 20) // row // 3, bs, row)
    assert 64 << 20 < oracle.payload_bytes(w.hit, w.layout.row_bytes) < 76 << 20
    hop_at(w, x_off, pool_off, **tuning)


# layers that pass it by: walked, by 128 lanes, by lanes that the caller chose
@pytest.mark.parametrize("bs,row,tuning", [(64, 132, dict(max_groups=1000)), (5, 1009, {}), (64, 333, dict(block_threads=512))])
def test_odd_rows_of_layers_that_pass_the_cache_by(bs, row, tuning):
    w = _uniform(3, (646 << 20) // row // 3, bs, row)
    assert oracle.payload_bytes(w.hit, w.layout.row_bytes) > 640 << 20
    hop_at(w, 13, 19, **tuning)


# two planes of blocks of whole lines: the scatter on the destination's lines after a gather on the source's, the limit of both,
# and the tiles of large descriptors that start late
@pytest.mark.parametrize("row,mb", [(132, 404), (132, 576), (516, 576)])
def test_odd_rows_in_two_planes_of_whole_lines(row, mb):
    w = _uniform(3, (mb << 20) // row // 6, 64, row, row)
    assert oracle.payload_bytes(w.hit, w.layout.row_bytes) > (mb - 2) << 20
    hop_at(w, 0, 19)


# layers that the on-die cache holds in part: both tiles begin on the source's lines, the gather's have 64 lanes, the scatter's
# 256 or 128; beyond that they pass the cache by.  161 windows are the first that are tiled; spans of one line and two tiles
@pytest.mark.parametrize("bs,row,mb,tuning", [(64, 333, 78, {}), (16, 333, 78, {}), (64, 132, 78, dict(max_groups=999)), (1, 2547, 78, {}),
                                              (8, 1009, 78, dict(block_threads=512)), (64, 132, 262, {}), (64, 1026, 642, {})])
@pytest.mark.parametrize("x_off,pool_off", [(0, 0), (13, 19)])
def test_odd_rows_of_layers_that_are_read_once(bs, row, mb, tuning, x_off, pool_off):
    w = _uniform(3, (mb << 20) // row // 3, bs, row)
    assert oracle.payload_bytes(w.hit, w.layout.row_bytes) > (mb - 2) << 20
    hop_at(w, x_off, pool_off, **tuning)


# lanes of a descriptor around the numbers from which a wavefront's lie in at most five, three and two of them
@pytest.mark.parametrize("row", [225, 226, 481, 482, 977, 978, 994])
@pytest.mark.parametrize("kind", ["fragmented", "runs"])
def test_odd_rows_dealt_out_flat(row, kind):
    hop_at(W.tiny(1700 + row, 7, 1, (row,), 333, 40, kind=kind), 13, 19)


@pytest.mark.parametrize("lanes", [1, 15, 16, 31, 32, 62, 63, 64, 129])
@pytest.mark.parametrize("store", [1, 3])
def test_vectors_dealt_out_flat(lanes, store):
    w = W.tiny(1800 + lanes, 7, 1, (16 * lanes, 16 * lanes), 333, 40, kind="fragmented")
    hop_at(w, 16, 32, variant=1 + (128 | 4 | store << 3))
    hop_at(w, 16, 32, variant=1 + (128 | 4 | store << 3), max_groups=3, block_threads=64)


# rows of 1, 15, 16, 31, 32, 63, 64, 65 and 72 vectors (how many rows a wavefront's 64 vectors can touch changes at
# 16, 32 and 64), one to a few to a block, with and without chance neighbours merged into longer descriptors
@pytest.mark.parametrize("row", [16, 240, 256, 496, 512, 1008, 1024, 1040, 1152])
@pytest.mark.parametrize("bs,kind", [(1, "runs"), (1, "random"), (3, "fragmented"), (7, "runs")])
@pytest.mark.parametrize("x_off", [0, 48])
def test_small_descriptors_by_the_row_map(row, bs, kind, x_off):
    hop_at(W.tiny(960 + row + bs, 7, bs, (row, 64, row), 400, 50 * bs, kind=kind), x_off)
    hop_at(W.tiny(970 + row + bs, 5, bs, (row,), 300, 50 * bs, kind=kind), x_off, block_threads=64)


# planes of unlike rows in one launch, by tiles (rows of whole lines, and not; the plain loads of odd lines) or by the row map
# (rows below and from 64 vectors), with a plane repeated; tiles of one wavefront in moves; a range of transfer rows
@pytest.mark.parametrize("bs,rows", [(64, (1024, 128)), (64, (512, 16, 128)), (16, (2048, 656)), (64, (656, 1040)), (1, (1152, 128)),
                                     (3, (16, 1040, 64, 1024)), (128, (128, 2048, 128)), (2, (1008, 1024)), (40, (656, 336))])
@pytest.mark.parametrize("x_off", [0, 48])
def test_planes_of_unlike_rows_at_once(bs, rows, x_off):
    for kind in ("runs", "random"):
        w = W.tiny(1160 + bs + sum(rows), 6, bs, rows, 150, 20 * bs, kind=kind)
        hop_at(w, x_off)
        src = W.fill_pool(w, 0, "src")
        want = W.sentinel_pool(w, "dst")
        oracle.unpack(bs, rows, w.hit, w.dst.tables, oracle.pack(bs, rows, w.hit, w.src.tables, src), want)
        pair = K.kvl_plan_pair(dev_plan(w, "src", K.KVL_GATHER), dev_plan(w, "dst", K.KVL_SCATTER))
        d_src, d_dst = planes_to_dev(src), planes_to_dev(W.sentinel_pool(w, "dst"))
        K.kvl_move_layer(pair, d_src, d_dst)
        torch.cuda.synchronize()
        for a, b in zip(d_dst, want):
            assert same_bytes(to_host(a), b)


# scatters by the row map of layers beyond the on-die cache, or off the lines: rows of 5, 8, 16, 19, 32 and 41 vectors
@pytest.mark.parametrize("bs,rows,mb", [(8, (512, 128), 238), (100, (256, 128), 238), (4, (304, 80), 116), (1, (656, 256), 116)])
def test_planes_of_unlike_rows_of_large_layers(bs, rows, mb):
    w = _uniform(3, (mb << 20) // sum(rows) // 3, bs, *rows)
    assert oracle.payload_bytes(w.hit, w.layout.row_bytes) > (mb - 2) << 20
    hop_at(w, 48)


@pytest.mark.parametrize("bs,row,mb", [(64, 656, 118), (64, 1152, 280), (100, 656, 118), (64, 256, 280)])
def test_layers_about_the_size_of_the_on_die_cache(bs, row, mb):
    """Whole blocks whose scatter takes the row map for the size of the layer (256-byte rows: the tiles)."""
    tokens = (mb << 20) // row // 3
    hop_at(_uniform(3, tokens, bs, row))


def _uniform(requests, tokens, bs, *rows):
    w = W.tiny(981, requests, bs, rows, requests * (tokens // bs + 4), tokens, allow_zero_hit=False)
    w.hit[:] = [tokens - 5 * r for r in range(requests)]
    w.app[:] = 3
    nb = [(int(h) + 3 + bs - 1) // bs for h in w.hit]
    for side, seed in ((w.src, 1), (w.dst, 2)):
        side.tables = W.make_tables(nb, side.pool_blocks, "random", np.random.Generator(np.random.PCG64(seed)))
    return w


@pytest.mark.parametrize("chunk,slots", [(4096, 1), (65536, 3)])
def test_row_map_through_the_staging_slots(chunk, slots):
    """Chunks launch parts of the descriptors, with the transfer rows shifted into a staging slot."""
    w = W.tiny(990, 9, 1, (1152, 272), 3000, 300)
    bs, rows = w.layout.block_tokens, w.layout.row_bytes
    x = W.random_payload(w, 0, oracle.payload_bytes(w.hit, rows))
    want = W.sentinel_pool(w, "dst")
    oracle.unpack(bs, rows, w.hit, w.dst.tables, x, want)
    plan = dev_plan(w, "dst", K.KVL_SCATTER | K.KVL_GATHER)
    host = torch.from_numpy(x).pin_memory()
    back = torch.empty_like(host).pin_memory()
    staging = torch.zeros(chunk * slots, dtype=torch.uint8, device="cuda")
    pool = planes_to_dev(W.sentinel_pool(w, "dst"))
    torch.cuda.synchronize()
    cs, ks = torch.cuda.Stream(), torch.cuda.Stream()
    K.kvl_h2d_unpack_layer(plan, host, staging, chunk, pool, cs, ks)
    K.kvl_d2h_pack_layer(plan, pool, staging, chunk, back, ks, cs)
    torch.cuda.synchronize()
    for a, b in zip(pool, want):
        assert same_bytes(to_host(a), b)
    assert same_bytes(back.numpy(), x)


# one and several planes of unlike rows (their tiles are numbered one plane after the other), on and off the 16-byte
# grid, spans around one and two tiles
@pytest.mark.parametrize("bs,rows", [(64, (64,)), (64, (1024, 128)), (16, (16, 656, 64)), (8, (512, 16, 520, 1024)), (64, (132,)),
                                     (3, (5, 7)), (16, (255, 256, 257, 31)), (1, (4095, 1)), (1, (4096, 8208))])
@pytest.mark.parametrize("off", [0, 5])
@pytest.mark.parametrize("where", ["device", "pinned"])
def test_full_blocks_planes_and_tiles(bs, rows, off, where):
    L, layer = 2, 1
    w = W.tiny(1020 + bs + len(rows), 5, bs, rows, 120, 9 * bs, kind="runs", n_layers=L)
    g, s = dev_plan(w, "src", K.KVL_GATHER | K.KVL_NO_MERGE), dev_plan(w, "dst", K.KVL_SCATTER | K.KVL_NO_MERGE)
    fb, count = g.fullblock_geometry()
    n = fb * count
    first = np.zeros_like(w.hit)
    src = W.fill_pool(w, layer, "src")
    want = np.full(n, 0x5A, dtype=np.uint8)
    oracle.pool_to_fullblocks(bs, L, rows, first, w.hit, w.src.tables, layer, src, want)
    want_pool = W.sentinel_pool(w, "dst")
    oracle.fullblocks_to_pool(bs, L, rows, first, w.hit, w.dst.tables, layer, want, want_pool)
    buf = torch.full((n + off + GUARD,), 0x5A, dtype=torch.uint8)
    buf = buf.cuda() if where == "device" else buf.pin_memory()
    d_src, d_dst = planes_to_dev(src), planes_to_dev(W.sentinel_pool(w, "dst"))
    torch.cuda.synchronize()
    K.kvl_pool_to_fullblocks_layer(g, d_src, layer, buf[off:off + n])
    K.kvl_fullblocks_to_pool_layer(s, buf[off:off + n], layer, d_dst)
    torch.cuda.synchronize()
    got = buf.cpu().numpy()
    assert same_bytes(got[off:off + n], want), "persist differs from the oracle"
    assert np.all(got[:off] == 0x5A) and np.all(got[off + n:] == 0x5A)
    for a, b in zip(d_dst, want_pool):
        assert same_bytes(to_host(a), b), "load differs from the oracle"


# planes alike whose tiles go in runs: below, at and above whole rounds of eight runs (of 256 KiB), ragged last blocks
@pytest.mark.parametrize("bs,rows,blocks", [(64, (1152,), 28), (64, (1152,), 29), (64, (2048, 2048), 16), (64, (2048, 2048), 33), (100, (336, 336), 90),
                                            (16, (336,), 400), (1, (496,), 5000), (256, (80, 80, 80, 80), 103)])
def test_full_blocks_of_planes_alike(bs, rows, blocks):
    L, layer = 3, 2
    w = W.tiny(1060 + blocks, 2, bs, rows, 2 * blocks + 5, blocks // 2 * bs, kind="random", n_layers=L, allow_zero_hit=False)
    w.hit[:] = [blocks // 2 * bs, (blocks - blocks // 2) * bs - bs // 3]
    w.app[:] = 0
    nb = [-(-int(h) // bs) for h in w.hit]
    for side, seed in ((w.src, 1), (w.dst, 2)):
        side.tables = W.make_tables(nb, side.pool_blocks, "random", np.random.Generator(np.random.PCG64(seed)))
    g, s = dev_plan(w, "src", K.KVL_GATHER | K.KVL_NO_MERGE), dev_plan(w, "dst", K.KVL_SCATTER | K.KVL_NO_MERGE)
    fb, count = g.fullblock_geometry()
    assert count == blocks
    first = np.zeros_like(w.hit)
    src = W.fill_pool(w, layer, "src")
    want = np.full(fb * count, 0x5A, dtype=np.uint8)
    oracle.pool_to_fullblocks(bs, L, rows, first, w.hit, w.src.tables, layer, src, want)
    want_pool = W.sentinel_pool(w, "dst")
    oracle.fullblocks_to_pool(bs, L, rows, first, w.hit, w.dst.tables, layer, want, want_pool)
    buf = torch.full((fb * count + GUARD,), 0x5A, dtype=torch.uint8, device="cuda")
    d_src, d_dst = planes_to_dev(src), planes_to_dev(W.sentinel_pool(w, "dst"))
    K.kvl_pool_to_fullblocks_layer(g, d_src, layer, buf[:fb * count])
    K.kvl_fullblocks_to_pool_layer(s, buf[:fb * count], layer, d_dst)
    torch.cuda.synchronize()
    got = to_host(buf)
    assert same_bytes(got[:fb * count], want) and np.all(got[fb * count:] == 0x5A), "persist differs from the oracle"
    for a, b in zip(d_dst, want_pool):
        assert same_bytes(to_host(a), b), "load differs from the oracle"


# tiles of 256, 128 and 64 lanes that begin on lines of the source: spans of whole vectors that begin on a line and off it (the
# last tile holds what the first leaves free: 249, 250 and 256 vectors), and at byte addresses, one wavefront and a byte beyond
@pytest.mark.parametrize("bs,rows", [(16, (336,)), (1, (496,)), (100, (48,)), (3, (1328,)), (1, (3984,)), (1, (4000,)), (1, (4096, 128)), (100, (336,)),
                                     (1, (897,)), (1, (898,)), (1, (1921,)), (100, (46,)), (16, (35,)), (24, (763, 5))])
@pytest.mark.parametrize("first", ["hit", "append"])
def test_full_blocks_on_lines_of_the_source(bs, rows, first):
    L, layer = 3, 1
    w = W.tiny(1200 + bs + sum(rows), 7, bs, rows, 160, 9 * bs, kind="random", n_layers=L)
    flag, lo, n = (0, np.zeros_like(w.hit), w.hit) if first == "hit" else (K.KVL_TOKENS_APPEND, w.hit, w.app)
    g, s = dev_plan(w, "src", K.KVL_GATHER | K.KVL_NO_MERGE | flag), dev_plan(w, "dst", K.KVL_SCATTER | K.KVL_NO_MERGE | flag)
    fb, count = g.fullblock_geometry()
    src = W.fill_pool(w, layer, "src")
    want = np.full(fb * count, 0x5A, dtype=np.uint8)
    oracle.pool_to_fullblocks(bs, L, rows, lo, n, w.src.tables, layer, src, want)
    want_pool = W.sentinel_pool(w, "dst")
    oracle.fullblocks_to_pool(bs, L, rows, lo, n, w.dst.tables, layer, want, want_pool)
    buf = torch.full((fb * count + GUARD,), 0x5A, dtype=torch.uint8, device="cuda")
    d_src, d_dst = planes_to_dev(src), planes_to_dev(W.sentinel_pool(w, "dst"))
    K.kvl_pool_to_fullblocks_layer(g, d_src, layer, buf[:fb * count])
    K.kvl_fullblocks_to_pool_layer(s, buf[:fb * count], layer, d_dst)
    torch.cuda.synchronize()
    got = to_host(buf)
    assert same_bytes(got[:fb * count], want), "persist differs from the oracle"
    assert np.all(got[fb * count:] == 0x5A)
    for a, b in zip(d_dst, want_pool):
        assert same_bytes(to_host(a), b), "load differs from the oracle"


# layers around a gibibyte, in runs and in workgroups of one wavefront, with an odd number of tiles to a descriptor, tiles on lines
# and off them, and a second plane
@pytest.mark.parametrize("bs,rows", [(64, (656,)), (40, (2048, 2048))])
@pytest.mark.parametrize("mb", [1023, 1026])
def test_tiles_of_layers_around_a_gibibyte(bs, rows, mb):
    w = _uniform(2, (mb << 20) // sum(rows) // 2, bs, *rows)
    assert (oracle.payload_bytes(w.hit, w.layout.row_bytes) > 1 << 30) == (mb > 1024)
    hop_at(w, 0)


# tiles in runs: a block's tiles below, at and above whole rounds of eight runs (of 512 KiB), one plane and two, with the lanes of
# layers up to 28 MiB (128) and beyond (256, or 64 where that leaves fewer without work)
@pytest.mark.parametrize("bs,rows,lanes", [(64, (1152,), 256), (64, (656,), 256), (32, (256, 256), 256), (256, (80,), 64)])
@pytest.mark.parametrize("rounds", [1, 8])
@pytest.mark.parametrize("more", [-1, 0, 1])
def test_tiles_around_whole_rounds(bs, rows, lanes, rounds, more):
    vectors = bs * rows[0] // 16 + (7 if rows[0] % 128 else 0)
    threads = 128 if rounds == 1 else lanes
    tiles = -(-vectors // threads)
    per_round = (8 << 19) // (16 * threads)
    if rounds > 1:
        rounds //= len(rows)
    blocks = rounds * per_round // tiles + more
    w = _uniform(1, blocks * bs, bs, *rows)
    assert (oracle.payload_bytes(w.hit, w.layout.row_bytes) <= 28 << 20) == (threads == 128)
    assert abs(blocks * tiles - rounds * per_round) <= 2 * tiles
    hop_at(w, 48 if rows[0] % 128 else 128)


# layers that the gather leaves in the L2 caches and the next larger ones, by tiles, by the row map and of odd rows
@pytest.mark.parametrize("bs,rows,mib", [(64, (1152,), 10), (64, (656,), 12), (64, (512, 512), 10), (1, (1152,), 10), (4, (656,), 12), (64, (333,), 12),
                                         (16, (333,), 12)])
@pytest.mark.parametrize("more", [-20000, 20000])
def test_layers_that_stay_in_the_l2(bs, rows, mib, more):
    w = _uniform(3, ((mib << 20) + more) // 3 // sum(rows) + 5, bs, *rows)
    assert (oracle.payload_bytes(w.hit, w.layout.row_bytes) < mib << 20) == (more < 0)
    hop_at(w, 0 if rows[0] % 16 else 48)


# the limits of run lengths, lanes and order by the layer's size
@pytest.mark.parametrize("bs,rows,mb", [(64, (1152,), 27), (64, (1152,), 29), (64, (1152,), 287), (64, (1152,), 289), (16, (1152,), 223),
                                        (16, (1152,), 225), (64, (656,), 511), (64, (656,), 513), (64, (2048, 2048), 513), (40, (768,), 520)])
def test_hops_at_the_limits_of_runs_and_lanes(bs, rows, mb):
    hop_at(_uniform(5, (mb << 20) // 5 // sum(rows), bs, *rows))


# runs of 1 MiB: short blocks off the lines, above half a GiB (64 rounds of 8 MiB and a rest)
@pytest.mark.parametrize("bs,row", [(64, 176), (24, 400)])
def test_short_blocks_of_large_layers_in_long_runs(bs, row):
    hop_at(_uniform(5, (517 << 20) // 5 // row + 77, bs, row), 48)


# a move's own workgroups: 64 lanes, 128, and 1024 flat; descriptors around one wavefront and one workgroup
@pytest.mark.parametrize("bs,rows", [(1, (16,)), (1, (1152,)), (1, (656, 128)), (2, (1024,)), (1, (2048,)), (1, (2064,)), (16, (1152, 656)),
                                     (64, (656,)), (3, (37,)), (64, (132, 132))])
def test_move_launch_shapes(bs, rows):
    move_of(W.tiny(1080 + bs + sum(rows), 6, bs, rows, 200, 20 * bs, kind="runs" if bs % 2 else "random"))


# the sizes between which scatters and moves store otherwise
@pytest.mark.parametrize("bs,rows", [(64, (1152,)), (8, (256,)), (64, (656,)), (64, (1024, 128))])
@pytest.mark.parametrize("mib", [12, 22])
@pytest.mark.parametrize("more", [-20000, 20000])
def test_hops_at_the_limits_of_the_scatters_stores(bs, rows, mib, more):
    hop_at(_uniform(3, ((mib << 20) + more) // 3 // sum(rows) + 5, bs, *rows))


@pytest.mark.parametrize("bs,rows", [(64, (1152,)), (64, (656,)), (64, (1024, 128))])
@pytest.mark.parametrize("mib", [23, 76])
@pytest.mark.parametrize("more", [-20000, 20000])
def test_moves_at_the_limits_of_their_stores(bs, rows, mib, more):
    move_of(_uniform(3, ((mib << 20) + more) // 3 // sum(rows) + 5, bs, *rows))


def move_of(w):
    bs, rows = w.layout.block_tokens, w.layout.row_bytes
    src = W.fill_pool(w, 0, "src")
    x = oracle.pack(bs, rows, w.hit, w.src.tables, src)
    want = W.sentinel_pool(w, "dst")
    oracle.unpack(bs, rows, w.hit, w.dst.tables, x, want)
    g, s = dev_plan(w, "src", K.KVL_GATHER), dev_plan(w, "dst", K.KVL_SCATTER)
    pair = K.kvl_plan_pair(g, s)
    d_src, d_dst = planes_to_dev(src), planes_to_dev(W.sentinel_pool(w, "dst"))
    K.kvl_move_layer(pair, d_src, d_dst)
    torch.cuda.synchronize()
    for a, b in zip(d_dst, want):
        assert same_bytes(to_host(a), b)


def test_a_plan_used_on_the_default_stream_keeps_its_descriptors_until_they_are_read():
    """Launches on the default stream carry no event: a plan destroyed while its kernel is still queued there must
    not hand its descriptors (or its row map) to the plans made next; they come back once the stream has passed."""
    w = W.tiny(1120, 9, 1, (1152,), 6000, 500)
    other = W.tiny(1120, 9, 1, (1152,), 6000, 500)
    other.src.tables = [t[::-1].copy() for t in other.src.tables]
    bs, rows = w.layout.block_tokens, w.layout.row_bytes
    src = W.fill_pool(w, 0, "src")
    want = [oracle.pack(bs, rows, v.hit, v.src.tables, src) for v in (w, other)]
    d_src = planes_to_dev(src)
    x = [torch.zeros(want[0].size, dtype=torch.uint8, device="cuda") for _ in range(2)]
    side = torch.cuda.Stream()
    K.kvl_release_cached_memory()
    for _ in range(3):
        torch.cuda.synchronize()
        g = dev_plan(w, "src", K.KVL_GATHER)
        torch.cuda._sleep(40_000_000)                       # tens of milliseconds on the default stream
        K.kvl_pack_layer(g, d_src, x[0])
        g.destroy()
        plans = [dev_plan(other, "src", K.KVL_GATHER) for _ in range(4)]
        for p in plans:
            K.kvl_pack_layer(p, d_src, x[1], stream=side)
        torch.cuda.synchronize()
        assert same_bytes(to_host(x[0]), want[0]), "a descriptor array was reused before its kernel had run"
        assert same_bytes(to_host(x[1]), want[1])
        for p in plans:
            p.destroy()
        for t in x:
            t.zero_()
    torch.cuda.synchronize()
    K.kvl_release_cached_memory()
    free0, _ = torch.cuda.mem_get_info()
    for _ in range(100):
        p = dev_plan(w, "src", K.KVL_GATHER)
        K.kvl_pack_layer(p, d_src, x[0])
        p.destroy()
    torch.cuda.synchronize()
    K.kvl_release_cached_memory()
    free1, _ = torch.cuda.mem_get_info()
    assert free0 - free1 < (8 << 20), f"{(free0 - free1) >> 20} MiB of device memory gone"


@pytest.mark.parametrize("row", [1152, 656])
def test_a_move_of_single_rows_with_one_long_run(row):
    """Descriptors that are unlike: every one has the largest one's tiles, most of them empty."""
    n, run = 3000, 113
    w = W.tiny(1100, 1, 1, (row,), n + 2 * run, n + run, allow_zero_hit=False)
    rng = np.random.Generator(np.random.PCG64(4))
    w.hit[:], w.app[:] = n + run, 0
    for side, first in ((w.src, 0), (w.dst, run)):
        single = np.setdiff1d(np.arange(side.pool_blocks), np.arange(first, first + run))
        side.tables = [np.concatenate([rng.permutation(single)[:n], np.arange(first, first + run)]).astype(np.int32)]
    bs, rows = w.layout.block_tokens, w.layout.row_bytes
    src = W.fill_pool(w, 0, "src")
    want = W.sentinel_pool(w, "dst")
    oracle.unpack(bs, rows, w.hit, w.dst.tables, oracle.pack(bs, rows, w.hit, w.src.tables, src), want)
    pair = K.kvl_plan_pair(dev_plan(w, "src", K.KVL_GATHER), dev_plan(w, "dst", K.KVL_SCATTER))
    assert pair.units()[:, 2].max() > 1
    d_src, d_dst = planes_to_dev(src), planes_to_dev(W.sentinel_pool(w, "dst"))
    K.kvl_move_layer(pair, d_src, d_dst)
    torch.cuda.synchronize()
    assert same_bytes(to_host(d_dst[0]), want[0])


@pytest.mark.parametrize("wait", [True, False], ids=["map-made", "at-once"])
def test_a_plan_with_a_row_map_captured_without_an_eager_launch(wait):
    """Its first launches are captured: the map is used if it has been made by then, and every replay is right."""
    w = W.tiny(1130, 9, 1, (1152,), 3000, 300)
    bs, rows = w.layout.block_tokens, w.layout.row_bytes
    g, s = dev_plan(w, "src", K.KVL_GATHER), dev_plan(w, "dst", K.KVL_SCATTER)
    d_src, d_dst = planes_to_dev(W.fill_pool(w, 0, "src")), planes_to_dev(W.sentinel_pool(w, "dst"))
    x = torch.zeros(g.payload_bytes, dtype=torch.uint8, device="cuda")
    st = torch.cuda.Stream()
    if wait:
        torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph, stream=st):
        K.kvl_pack_layer(g, d_src, x, stream=st)
        K.kvl_unpack_layer(s, x, d_dst, stream=st)
    if wait:        # laid out over the transfer rows: as many lanes as there are vectors, and the line-up
        vectors = int(w.hit.sum()) * rows[0] // 16
        assert [grid for grid in _grids(graph)] == [(vectors + 7 + 255) // 256] * 2
    graph.instantiate()
    for rep in range(3):
        fill = W.fill_pool(w, rep + 1, "src")
        d_src[0].copy_(to_dev(fill[0]))
        d_dst[0].fill_(0xA5)
        x.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(st):
            graph.replay()
        st.synchronize()
        want_x = oracle.pack(bs, rows, w.hit, w.src.tables, fill)
        want = W.sentinel_pool(w, "dst")
        oracle.unpack(bs, rows, w.hit, w.dst.tables, want_x, want)
        assert same_bytes(to_host(x), want_x) and same_bytes(to_host(d_dst[0]), want[0]), f"replay {rep}"


def _grids(graph):
    """Workgroups along x of every kernel in a captured graph, in order."""
    class Params(C.Structure):      # hipKernelNodeParams
        _fields_ = [("block", C.c_uint32 * 3), ("extra", C.c_void_p), ("func", C.c_void_p), ("grid", C.c_uint32 * 3),
                    ("params", C.c_void_p), ("shared", C.c_uint32)]
    hip, n = K.binding._lib, C.c_size_t()       # (the library brings the HIP runtime with it)
    raw = C.c_void_p(graph.raw_cuda_graph())
    assert hip.hipGraphGetNodes(raw, None, C.byref(n)) == 0
    nodes = (C.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(raw, nodes, C.byref(n)) == 0
    out = []
    for node in nodes:
        p = Params()
        assert hip.hipGraphKernelNodeGetParams(C.c_void_p(node), C.byref(p)) == 0
        out.append(p.grid[0])
    return out


def test_a_row_map_awaited_by_two_streams():
    """A plan's first launches on two streams at once: both wait for its map, whichever asks first."""
    w = W.tiny(1140, 9, 1, (1152,), 6000, 500)
    bs, rows = w.layout.block_tokens, w.layout.row_bytes
    src = W.fill_pool(w, 0, "src")
    want = oracle.pack(bs, rows, w.hit, w.src.tables, src)
    d_src = planes_to_dev(src)
    streams = [torch.cuda.Stream(), torch.cuda.Stream(), None]
    for _ in range(5):
        x = [torch.zeros(want.size, dtype=torch.uint8, device="cuda") for _ in streams]
        torch.cuda.synchronize()
        g = dev_plan(w, "src", K.KVL_GATHER)
        for s, t in zip(streams, x):
            K.kvl_pack_layer(g, d_src, t, stream=s)
        torch.cuda.synchronize()
        for t in x:
            assert same_bytes(to_host(t), want)
        g.destroy()
