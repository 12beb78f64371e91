"""The dispatch's edges: sizes at which a launch changes its kernel, its tile or its remainder, against the
CPU oracle, bit for bit (the comparison is exact: bytes are moved, none is computed)."""
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
