"""jc_footprint sizes an arena without building the work list (host only): 17
million work items took over a second and half a gigabyte."""
import ctypes
import time

from paper_2102_12416_amd import _lib as L


def test_footprint_builds_no_work_list():
    opt = L.Options()
    opt.ir_dtype = L.JC_NONE
    opt.tile_x, opt.tile_y, opt.z_chunk = 16, 8, 1
    n = L.i64((2048, 2048, 512))
    best, fp = 1e9, ctypes.c_size_t()
    for _ in range(3):
        t0 = time.perf_counter()
        assert L.lib.jc_footprint(n, n, ctypes.byref(opt), ctypes.byref(fp)) == 0, L.last_error()
        best = min(best, time.perf_counter() - t0)
    assert fp.value > 2 * 8 * 2048 * 2048 * 512
    assert best < 0.1, best
