"""Default launch shapes on grids where a rule once picked a slower one than the
rule before it (host only, no device)."""
import ctypes

import pytest

from paper_2102_12416_amd import _lib as L


def check(st):
    assert st == 0, L.last_error()


def create(n, block=None, ir=None, **kw):
    opt = L.Options()
    opt.mode = 1
    opt.ir_dtype = L.JC_NONE if ir is None else ir
    opt.ir_enable = int(ir is not None)
    opt.with_source = int(ir is not None)
    for k, v in kw.items():
        setattr(opt, k, v)
    ctx = ctypes.c_void_p()
    check(L.lib.jc_create(L.i64(n), L.i64(block or n), ctypes.byref(opt), ctypes.byref(ctx)))
    return ctx


def multi_shape(n, **kw):
    ctx = create(n, temporal=1, **kw)
    out = (ctypes.c_int64 * 3)()
    check(L.lib.jc_temporal_info(ctx, out))
    L.lib.jc_destroy(ctx)
    return list(out)[1:]


@pytest.mark.parametrize("n", [(555, 160, 87), (150, 467, 55), (369, 24, 317), (348, 54, 334), (131, 358, 173)])
def test_two_sweeps_of_a_narrow_correction_fill_the_chip_twice(n):
    """More work-groups than compute units: two share one."""
    rows, planes = multi_shape(n, ir=L.JC_BF16)
    assert rows == 16
    groups = -(-n[0] // 64) * -(-n[1] // rows) * -(-n[2] // planes)
    assert 256 < groups <= 512, (planes, groups)


@pytest.mark.parametrize("n,source,depth,most", [((30, 122, 507), 0, 2, 12), ((31, 191, 333), 0, 2, 12),
                                                 ((597, 424, 24), 1, 3, 12), ((631, 428, 28), 0, 2, 14)])
def test_columns_where_one_round_of_long_ones_is_slower(n, source, depth, most):
    """Half-idle tiles without a source, and thin grids of a round and a bit."""
    rows, planes = multi_shape(n, with_source=source, sweeps_per_launch=depth)
    assert rows == 16 and planes <= most, planes


def tile(n, **kw):
    ctx = create(n, **kw)
    out = (ctypes.c_int64 * 4)()
    check(L.lib.jc_tile_info(ctx, out))
    L.lib.jc_destroy(ctx)
    return list(out)[:3]


@pytest.mark.parametrize("n,ir", [((342, 50, 122), None), ((149, 44, 338), None), ((45, 211, 203), None),
                                  ((597, 18, 376), L.JC_F32), ((74, 36, 634), L.JC_F64), ((131, 46, 287), L.JC_F32),
                                  ((193, 347, 343), L.JC_F32)])
def test_no_round_of_tall_tiles_where_their_lanes_idle(n, ir):
    assert tile(n, ir=ir)[1] == 8


@pytest.mark.parametrize("n,ir,rows", [((256, 256, 256), None, 16), ((512, 512, 512), None, 16),
                                       ((384, 320, 448), L.JC_F32, 16), ((285, 592, 67), None, 4)])
def test_one_round_of_long_columns_is_kept(n, ir, rows):
    t = tile(n, ir=ir)
    assert t[1] == rows and t[2] >= 64, t


@pytest.mark.parametrize("n,block,planes", [((106, 624, 274), (106, 123, 84), 11), ((342, 402, 175), (226, 184, 175), 11),
                                            ((579, 576, 78), None, 10)])
def test_short_chunks_are_left_as_they_are(n, block, planes):
    assert tile(n, block=block) == [64, 8, planes]


def test_long_chunks_of_many_blocks_become_short():
    assert tile((371, 402, 310), block=(53, 159, 99)) == [64, 8, 11]
