"""The multi-sweep shape that jc_temporal_info reports can be set again, quads of
cells (32 rows, three sweeps of a binary32 or bfloat16 correction) too (host
only, no device)."""
import ctypes

import pytest

from paper_2102_12416_amd import _lib as L


def create(n, ir=None, depth=3):
    opt = L.Options()
    opt.mode = 1
    opt.ir_dtype = L.JC_NONE if ir is None else ir
    opt.ir_enable = int(ir is not None)
    opt.with_source = 1
    opt.temporal = 1
    opt.sweeps_per_launch = depth
    ctx = ctypes.c_void_p()
    assert L.lib.jc_create(L.i64(n), L.i64(n), ctypes.byref(opt), ctypes.byref(ctx)) == 0, L.last_error()
    return ctx


def info(ctx):
    out = (ctypes.c_int64 * 3)()
    assert L.lib.jc_temporal_info(ctx, out) == 0
    return tuple(out)


@pytest.mark.parametrize("ir", [L.JC_F32, L.JC_BF16])
@pytest.mark.parametrize("n", [(64, 64, 64), (161, 162, 163)])
def test_quads_can_be_set_and_read_back(n, ir):
    ctx = create(n, ir)
    assert L.lib.jc_set_temporal_tiles(ctx, 32, 41) == 0, L.last_error()
    assert info(ctx) == (3, 32, 41)
    assert L.lib.jc_set_temporal_tiles(ctx, 8, 5) == 0
    assert info(ctx) == (3, 8, 5)
    L.lib.jc_destroy(ctx)


@pytest.mark.parametrize("ir,depth", [(None, 3), (L.JC_F64, 3), (L.JC_F32, 2), (L.JC_BF16, 2), (None, 2)])
def test_quads_are_refused_elsewhere(ir, depth):
    ctx = create((161, 162, 163), ir, depth)
    before = info(ctx)
    assert L.lib.jc_set_temporal_tiles(ctx, 32, 41) == L.JC_ERR_INVALID
    assert info(ctx) == before
    L.lib.jc_destroy(ctx)


@pytest.mark.parametrize("ir", [None, L.JC_F32, L.JC_BF16])
def test_a_default_set_again_reports_the_same(ir):
    ctx = create((200, 180, 160), ir)
    before = info(ctx)
    assert L.lib.jc_set_temporal_tiles(ctx, *[int(v) for v in before[1:]]) == 0
    assert info(ctx) == before
    L.lib.jc_destroy(ctx)
