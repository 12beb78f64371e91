"""The binding's module for the per-layer calls: it takes what is plainly in order and leaves the rest to the general path,
whose results and errors stay what they are."""
import gc
import os
import shutil
import sysconfig

import numpy as np
import pytest
import torch

import kvl_workloads as W
import oracle
import paper_2602_21548_amd as K
from paper_2602_21548_amd import binding as B
from paper_2602_21548_amd import build as kvl_build

NOT_TAKEN = 1


def _plan(w, flags=K.KVL_GATHER | K.KVL_HOST_ONLY, tables=None, hit=None, app=None):
    lay = K.make_layout(w.layout.n_layers, w.layout.block_tokens, w.layout.row_bytes, w.src.pool_blocks)
    return K.kvl_plan(lay, w.hit if hit is None else hit, w.app if app is None else app,
                      w.src.tables if tables is None else tables, flags)


# lists, other integer types, strided and two-dimensional tables, an empty one, a tuple of tables
@pytest.mark.parametrize("form", ["as-is", "int64", "lists", "strided", "two-dimensional", "tuple", "mixed", "iterator"])
def test_requests_in_every_form_give_the_same_plan(form):
    w = W.tiny(7, 6, 16, (64,), 90, 200, kind="runs")
    w.hit[2] = w.app[2] = 0
    tables = list(w.src.tables)
    tables[2] = np.empty(0, dtype=np.int32)
    want = _plan(w, tables=tables).units()
    hit, app = w.hit, w.app
    if form == "int64":
        tables, hit = [t.astype(np.int64) for t in tables], hit.astype(np.int64)
    elif form == "lists":
        tables, hit, app = [t.tolist() for t in tables], hit.tolist(), app.tolist()
    elif form == "strided":
        tables = [np.repeat(t, 2)[::2] for t in tables]
        hit = np.repeat(hit, 3)[::3]
    elif form == "two-dimensional":
        tables = [np.concatenate([t, t]).reshape(2, -1) for t in tables]
    elif form == "tuple":
        tables = tuple(tables)
    elif form == "mixed":
        tables[1] = tables[1].tolist()
    elif form == "iterator":
        class Once:
            def __init__(self, items):
                self.n, self.left = len(items), iter(items)

            def __len__(self):
                return self.n

            def __iter__(self):
                return self.left

        tables = Once([t.astype(np.int64) for t in tables])
    got = _plan(w, tables=tables, hit=hit, app=app).units()
    assert np.array_equal(got, want)


def test_requests_are_refused_as_ever():
    w = W.tiny(7, 4, 16, (64,), 90, 200)
    with pytest.raises(ValueError):
        _plan(w, tables=w.src.tables[:-1])
    with pytest.raises(ValueError):
        _plan(w, app=w.app[:-1])
    with pytest.raises(K.KvlError) as e:
        _plan(w, tables=[t[:-1] for t in w.src.tables])
    assert e.value.code == K.KVL_ERANGE


@pytest.mark.skipif(B._native is None, reason="the module is not built here")
def test_what_is_not_in_order_is_left_to_the_general_path():
    w = W.tiny(7, 4, 16, (64,), 90, 200)
    plan = _plan(w)
    n = w.src.pool_blocks * 16 * 64
    pool, x = [torch.zeros(n, dtype=torch.uint8)], torch.zeros(n, dtype=torch.uint8)
    for args in [(plan, pool, x, None), (plan, pool, None, None), (None, pool, x, None), (plan, None, x, None), (plan, [], x, None),
                 (plan, pool), (plan, [None], x, "s")]:
        assert B._fast_pack(*args) == NOT_TAKEN
    assert B._fast_to_pool(plan, x, -1, pool, None) == B._fast_move(plan, pool, pool, None) == NOT_TAKEN
    with pytest.raises(TypeError):
        K.kvl_pack_layer(plan, pool, x)
    with pytest.raises(ValueError):
        K.kvl_pack_layer(plan, pool + pool, x)
    plan.destroy()
    plan.destroy()
    with pytest.raises(ValueError):
        plan.handle
    del plan
    gc.collect()


@pytest.fixture
def elsewhere(tmp_path, monkeypatch):
    """Built files in a directory of the test's own; the library by a stand-in for hipcc that makes an empty file."""
    hipcc = tmp_path / "hipcc"
    hipcc.write_text('#!/bin/sh\nwhile [ "$1" != -o ]; do shift; done\n: > "$2"\n')
    hipcc.chmod(0o755)
    monkeypatch.setattr(kvl_build, "hipcc", lambda: str(hipcc))
    monkeypatch.setattr(kvl_build, "LIB", str(tmp_path / "libkvl.so"))
    monkeypatch.setattr(kvl_build, "NATIVE", str(tmp_path / os.path.basename(kvl_build.NATIVE)))
    return tmp_path


@pytest.mark.parametrize("compiler", ["/nonexistent/g++", "/bin/false"])
def test_the_library_is_built_without_a_host_compiler(elsewhere, monkeypatch, compiler):
    monkeypatch.setenv("CXX", compiler)
    with pytest.warns(RuntimeWarning, match="module"):
        assert kvl_build.build() == kvl_build.LIB
    assert os.path.exists(kvl_build.LIB) and not os.path.exists(kvl_build.NATIVE)
    with pytest.warns(RuntimeWarning, match="ctypes"):
        assert B._load_native() is None


def test_the_module_is_built_for_this_interpreter_and_from_the_present_sources(elsewhere, monkeypatch):
    assert kvl_build.NATIVE.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    if not shutil.which(os.environ.get("CXX", "g++")):
        pytest.skip("no host compiler")
    kvl_build.build_native()
    assert kvl_build.native_is_current()
    header = elsewhere / "kvl.h"
    with open(kvl_build.NATIVE_SOURCES[0], "rb") as f:
        header.write_bytes(f.read() + b"\n")
    monkeypatch.setattr(kvl_build, "NATIVE_SOURCES", [str(header)] + kvl_build.NATIVE_SOURCES[1:])
    assert not kvl_build.native_is_current()        # built from another header: as good as not there
    monkeypatch.setenv("CXX", "/nonexistent/g++")
    with pytest.warns(RuntimeWarning, match="ctypes"):
        assert B._load_native() is None


@pytest.mark.gpu
def test_each_argument_out_of_order_is_left_to_the_general_path():
    """One at a time, the others in order."""
    assert B._native is not None, "the module is not built"
    w = W.tiny(11, 4, 16, (64,), 90, 200, n_layers=2)
    lay = K.make_layout(2, 16, (64,), w.src.pool_blocks)
    flags = K.KVL_GATHER | K.KVL_SCATTER | K.KVL_NO_MERGE
    plan = K.kvl_plan(lay, w.hit, w.app, w.src.tables, flags)
    size, count = plan.fullblock_geometry()
    n = w.src.pool_blocks * 16 * 64
    pool = [torch.zeros(n, dtype=torch.uint8, device="cuda")]
    x, fb = (torch.zeros(k, dtype=torch.uint8, device="cuda") for k in (plan.payload_bytes, size * count))
    host = torch.zeros(plan.payload_bytes, dtype=torch.uint8)
    two = torch.zeros((2, plan.payload_bytes), dtype=torch.uint8, device="cuda").t()
    gone = K.kvl_plan(lay, w.hit, w.app, w.src.tables, flags)
    gone.destroy()

    class Special(torch.Tensor):
        pass

    short = [pool[0][:-1]]
    calls = [(B._fast_pack, [plan, pool, x, None], {0: [None, gone, "p"], 1: [None, [], pool * 2, short, [None], [host], iter(pool)],
                                                     2: [None, host, two, x.as_subclass(Special), 7], 3: ["s", 1.5]}),
             (B._fast_unpack, [plan, x, pool, None], {0: [gone], 1: [None, host, two], 2: [None, short, pool[0]], 3: ["s"]}),
             (B._fast_to_pool, [plan, fb, 1, pool, None], {0: [gone], 1: [None, host, two], 2: [-1, 1 << 32, True, 1.0, None], 3: [short], 4: ["s"]}),
             (B._fast_to_blocks, [plan, pool, 1, fb, None], {0: [gone], 1: [short], 2: [-1, 1 << 32, True], 3: [None, host, two], 4: ["s"]})]
    for call, args, bad in calls:
        assert call(*args) == K.KVL_OK, call
        for at, values in bad.items():
            for v in values:
                assert call(*args[:at], v, *args[at + 1:]) == NOT_TAKEN, (call, at, v)
        assert call(*args[:-1]) == NOT_TAKEN
    assert B._fast_move(plan, pool, pool, None) == NOT_TAKEN            # (not a paired plan)
    torch.cuda.synchronize()


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [(64,), (1024, 128), (132,)])
@pytest.mark.parametrize("where", ["device", "pinned"])
def test_full_blocks_both_ways(rows, where, monkeypatch):
    assert B._native is not None, "the module is not built"
    L, layer = 3, 2
    w = W.tiny(13, 6, 16, rows, 120, 300, n_layers=L)
    bs = w.layout.block_tokens
    lay = K.make_layout(L, bs, rows, w.src.pool_blocks)
    src = W.fill_pool(w, layer, "src")
    taken = []
    for f in ("_fast_to_pool", "_fast_to_blocks"):
        def spied(*a, call=getattr(B, f)):
            rc = call(*a)
            taken.append(rc)
            return rc
        monkeypatch.setattr(B, f, spied)
    for general in (False, True):
        if general:
            for f in ("_fast_to_pool", "_fast_to_blocks"):
                monkeypatch.setattr(B, f, lambda *a: NOT_TAKEN)
        g = K.kvl_plan(lay, w.hit, w.app, w.src.tables, K.KVL_GATHER | K.KVL_NO_MERGE)
        s = K.kvl_plan(lay, w.hit, w.app, w.dst.tables, K.KVL_SCATTER | K.KVL_NO_MERGE)
        size, count = g.fullblock_geometry()
        want = np.full(size * count, 0x5A, dtype=np.uint8)
        zero = np.zeros_like(w.hit)
        oracle.pool_to_fullblocks(bs, L, rows, zero, w.hit, w.src.tables, layer, src, want)
        want_pool = W.sentinel_pool(w, "dst")
        oracle.fullblocks_to_pool(bs, L, rows, zero, w.hit, w.dst.tables, layer, want, want_pool)
        blocks = torch.full((size * count,), 0x5A, dtype=torch.uint8)
        blocks = blocks.cuda() if where == "device" else blocks.pin_memory()
        d_src, d_dst = ([torch.from_numpy(p).cuda() for p in side] for side in (src, W.sentinel_pool(w, "dst")))
        torch.cuda.synchronize()
        K.kvl_pool_to_fullblocks_layer(g, d_src, layer, blocks)
        K.kvl_fullblocks_to_pool_layer(s, blocks, layer, d_dst)
        torch.cuda.synchronize()
        assert blocks.cpu().numpy().tobytes() == want.tobytes()
        assert all(np.array_equal(p.cpu().numpy(), q) for p, q in zip(d_dst, want_pool))
        for bad in (L, 1 << 20):
            with pytest.raises(K.KvlError) as e:
                K.kvl_fullblocks_to_pool_layer(s, blocks, bad, d_dst)
            assert e.value.code == K.KVL_EINVAL
        with pytest.raises(K.KvlError) as e:
            K.kvl_pool_to_fullblocks_layer(g, d_src, layer, blocks[:-1].clone() if where == "device" else blocks[:-1].clone().pin_memory())
        assert e.value.code == K.KVL_ESPACE
    assert taken.count(0) == 2


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [(64,), (1024, 128), (132,)])
def test_both_ways_move_the_same_bytes_and_refuse_the_same(rows, monkeypatch):
    assert B._native is not None, "the module is not built"
    w = W.tiny(9, 6, 16, rows, 120, 300)
    bs = w.layout.block_tokens
    lay = K.make_layout(1, bs, rows, w.src.pool_blocks)
    src = W.fill_pool(w, 0, "src")
    want_x = oracle.pack(bs, rows, w.hit, w.src.tables, src)
    want = W.sentinel_pool(w, "dst")
    oracle.unpack(bs, rows, w.hit, w.dst.tables, want_x, want)
    d_src = [torch.from_numpy(p).cuda() for p in src]
    side = torch.cuda.Stream()
    taken = []
    for f in ("_fast_pack", "_fast_unpack", "_fast_move"):
        def spied(*a, call=getattr(B, f)):
            rc = call(*a)
            taken.append(rc)
            return rc
        monkeypatch.setattr(B, f, spied)
    for general in (False, True):
        if general:
            for f in ("_fast_pack", "_fast_unpack", "_fast_move"):
                monkeypatch.setattr(B, f, lambda *a: NOT_TAKEN)
        for stream in (None, side, side.cuda_stream):
            g, s = K.kvl_plan(lay, w.hit, w.app, w.src.tables, K.KVL_GATHER), K.kvl_plan(lay, w.hit, w.app, w.dst.tables, K.KVL_SCATTER)
            pair = K.kvl_plan_pair(g, s)
            x = torch.zeros(want_x.size, dtype=torch.uint8, device="cuda")
            host = torch.zeros(want_x.size, dtype=torch.uint8).pin_memory()
            pools = [[torch.from_numpy(p).cuda() for p in W.sentinel_pool(w, "dst")] for _ in range(2)]
            torch.cuda.synchronize()
            K.kvl_pack_layer(g, tuple(d_src), x, stream=stream)
            K.kvl_unpack_layer(s, x, pools[0], stream)
            K.kvl_pack_layer(plan=g, pool_planes=d_src, xfer=host, stream=stream)
            K.kvl_move_layer(pair, d_src, pools[1], stream)
            torch.cuda.synchronize()
            assert x.cpu().numpy().tobytes() == host.numpy().tobytes() == want_x.tobytes()
            for pool in pools:
                assert all(np.array_equal(p.cpu().numpy(), q) for p, q in zip(pool, want))
            if want_x.size > 1:
                with pytest.raises(K.KvlError) as e:
                    K.kvl_pack_layer(g, d_src, x[:-1].clone(), stream)
                assert e.value.code == K.KVL_ESPACE
            with pytest.raises(ValueError):
                K.kvl_unpack_layer(s, x, [p[:-1].clone() for p in pools[0]], stream)
            with pytest.raises(TypeError):
                K.kvl_unpack_layer(s, x, [p.reshape(2, -1).t() for p in pools[0]], stream)
            with pytest.raises(TypeError):
                K.kvl_pack_layer(g, d_src, host.clone(), stream)
            g.destroy()
            with pytest.raises(ValueError):
                K.kvl_pack_layer(g, d_src, x, stream)
        if not general:
            assert taken.count(0) == 3 * 4
