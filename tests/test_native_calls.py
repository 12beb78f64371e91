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
