"""Default launch shapes of a context, over grids from one cell to the
benchmarks' sizes (host only, no device).

Whatever the rule picks is an ordinary shape: valid for the storage, within
the work list that the footprint reserves (jc_set_tiles would refuse it
otherwise), its tiles covering every block once, and independent of
anything but the grid and the options.  A shape that was asked for is kept.
"""
import ctypes

import pytest
from hypothesis import HealthCheck, given, settings
from hypothesis import strategies as hs

from paper_2102_12416_amd import _lib as L

EDGES = hs.one_of(hs.integers(1, 70), hs.sampled_from([95, 96, 97, 127, 128, 129, 255, 256, 257, 400, 512, 1024, 1536]))


def check(st):
    assert st == 0, L.last_error()


def create(grid, block, **kw):
    opt = L.Options()
    opt.ir_dtype = kw.pop("ir_dtype", L.JC_NONE)
    opt.ir_enable = int(opt.ir_dtype != L.JC_NONE)
    for k, v in kw.items():
        setattr(opt, k, v)
    ctx = ctypes.c_void_p()
    g, b = L.i64(grid), L.i64(block)
    check(L.lib.jc_create(g, b, ctypes.byref(opt), ctypes.byref(ctx)))
    return ctx


def tile_of(ctx):
    out = (ctypes.c_int64 * 4)()
    check(L.lib.jc_tile_info(ctx, out))
    return tuple(out)


def blocks_of(ctx):
    out = []
    for i in range(L.lib.jc_num_blocks(ctx)):
        v = (ctypes.c_int64 * 17)()
        check(L.lib.jc_block_info(ctx, i, v))
        out.append(list(v)[:3])
    return out


@settings(max_examples=120, deadline=None, suppress_health_check=[HealthCheck.too_slow])
@given(n=hs.tuples(EDGES, EDGES, EDGES), cut=hs.tuples(*[hs.integers(1, 3)] * 3), mode=hs.sampled_from([0, 1]),
       lo=hs.sampled_from([None, "JC_F64", "JC_F32", "JC_BF16"]))
def test_default_tile_is_valid_and_covers_every_block(n, cut, mode, lo):
    block = [max(1, -(-v // c)) for v, c in zip(n, cut)]
    kw = dict(mode=mode, with_source=1)
    if lo:
        kw["ir_dtype"] = getattr(L, lo)
    ctx = create(n, block, **kw)
    try:
        tx, ty, zc, items = tile_of(ctx)
        blocks = blocks_of(ctx)
        assert items == sum(-(-b[0] // tx) * -(-b[1] // ty) * -(-b[2] // zc) for b in blocks)
        check(L.lib.jc_set_tiles(ctx, tx, ty, zc))
        assert tile_of(ctx) == (tx, ty, zc, items)
    finally:
        L.lib.jc_destroy(ctx)


@settings(max_examples=60, deadline=None)
@given(n=hs.tuples(EDGES, EDGES, EDGES), depth=hs.sampled_from([2, 3]),
       lo=hs.sampled_from([None, "JC_F64", "JC_F32", "JC_BF16"]))
def test_default_multi_sweep_shape(n, depth, lo):
    kw = dict(mode=1, with_source=1, temporal=1, sweeps_per_launch=depth)
    if lo:
        kw["ir_dtype"] = getattr(L, lo)
    ctx = create(n, n, **kw)
    try:
        out = (ctypes.c_int64 * 3)()
        check(L.lib.jc_temporal_info(ctx, out))
        sweeps, rows, planes = out
        assert sweeps == depth
        assert rows in (8, 16) and (rows == 16 or lo == "JC_BF16")
        assert 1 <= planes <= n[2]
        check(L.lib.jc_set_temporal_tiles(ctx, rows, planes))
    finally:
        L.lib.jc_destroy(ctx)


@pytest.mark.parametrize("asked", [dict(tile_x=32), dict(tile_y=4), dict(z_chunk=7), dict(tile_x=64, tile_y=16, z_chunk=5)])
@pytest.mark.parametrize("n", [(17, 9, 30), (64, 64, 64), (300, 200, 250)])
def test_a_shape_that_was_asked_for_is_kept(n, asked):
    ctx = create(n, n, mode=1, **asked)
    try:
        got = dict(zip(("tile_x", "tile_y", "z_chunk"), tile_of(ctx)))
        for k, v in asked.items():
            assert got[k] == v
    finally:
        L.lib.jc_destroy(ctx)
