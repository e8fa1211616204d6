"""The helpers that the sweeps share, on the device: bfloat16 rounding over all
2^32 binary32 patterns, the divisions by 6; and edge values through the sweep
paths whose divisions have a branch of their own (resident sweeps, three sweeps
per launch, quads of cells)."""
import ctypes
import os

import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

from paper_2102_12416_amd import JcError, Solver, _lib as L  # noqa: E402
from tests.test_gpu_parity import edge_field, same_bits_or_nan  # noqa: E402

LIB = os.path.join(os.path.dirname(os.path.abspath(__file__)), "libdevice_check.so")


@pytest.fixture(scope="module")
def lib():
    assert os.path.exists(LIB), "not built: run __graft_entry__.build()"
    so = ctypes.CDLL(LIB)
    so.check_bf16_pair.argtypes = so.check_div6_f32.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    so.check_div6_quad.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p]
    return so


def mismatches(call):
    bad = torch.zeros(1, dtype=torch.int64, device="cuda:0")
    stream = torch.cuda.current_stream().cuda_stream
    assert call(ctypes.c_void_p(bad.data_ptr()), ctypes.c_void_p(stream)) == 0
    return int(bad.item())


def test_bf16_rounding_of_every_pattern(lib):
    print("[case] bf16_pair, 2^32 patterns", flush=True)
    assert mismatches(lib.check_bf16_pair) == 0


def test_div6_of_every_binary32_pattern(lib):
    print("[case] div6, 2^32 patterns", flush=True)
    assert mismatches(lib.check_div6_f32) == 0


@pytest.mark.parametrize("place", [0, 1, 2, 3])
def test_div6_quad_edges_in_each_place(lib, place):
    print("[case] div6_quad", place, flush=True)
    rng = np.random.default_rng(place)
    edge = np.array([0.0, -0.0, 5e-324, -5e-324, 3.5e-320, 2.0 ** -1022, -1.5 * 2.0 ** -1000, 1e300, 1.7e308, -1.7e308,
                     np.inf, -np.inf, np.nan])
    v = rng.integers(0, 2 ** 64, 1 << 20, dtype=np.uint64).view(np.float64)
    v[::3] = rng.uniform(-2, 2, v[::3].size)
    v[::5] = rng.choice(edge, v[::5].size)
    t = torch.from_numpy(v.copy()).to("cuda:0")
    assert mismatches(lambda bad, st: lib.check_div6_quad(ctypes.c_void_p(t.data_ptr()), v.size, place, bad, st)) == 0


@pytest.mark.parametrize("n", [(9, 8, 7), (9, 8, 4), (8, 7, 2), (9, 8, 1)])
@pytest.mark.parametrize("kw", [dict(resident=True, mode="fused"), dict(temporal=3)])
def test_division_edge_values(n, kw):
    """As test_division_edge_values_bitwise, on the paths of many sweeps."""
    print("[case] division edge values", n, kw, flush=True)
    u0 = edge_field(n, 31)
    ref = u0
    with np.errstate(all="ignore"):
        for _ in range(3):
            ref = oracle.sweep(ref)
    with Solver(n, **kw) as s:
        s.load(u0)
        s.iterate(3)
        got = s.store().cpu().numpy()
    assert np.isinf(ref).any() and np.isnan(ref).any()
    assert same_bits_or_nan(got, ref)


@pytest.mark.parametrize("shape", [(8, 5), (16, 4), (32, 3)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_refinement_overflow_by_cells(dtype, shape):
    """As test_refinement_overflow_bitwise with three sweeps per launch, by pairs
    and by quads of cells: the values that overflow, vanish or carry a sign of
    zero sit in single cells, in every place of a quad."""
    n, m = (45, 20, 18), 7
    print("[case] refinement overflow by cells", dtype, shape, flush=True)
    rng = np.random.default_rng(5)
    u0 = np.zeros((n[2] + 2, n[1] + 2, n[0] + 2))
    b = np.zeros_like(u0)
    inside = rng.random((n[2], n[1], n[0]))
    inside[rng.random(inside.shape) < 0.2] = -0.0
    inside[rng.random(inside.shape) < 0.1] = 1e-42
    inside[10:, 10:, 20:] = -0.0                          # sums of zeros, signed
    inside[0, 0, :8] = 1e39                               # beyond binary32: r_lo = +inf
    inside[0:3, 15:18, 20:30] = 3.3e38                    # neighbour sums overflow binary32
    b[1:-1, 1:-1, 1:-1] = inside
    with np.errstate(all="ignore"):
        ref = oracle.ir_step(u0, b, dtype, m)
    assert np.isinf(ref).sum() > 100 and np.isfinite(ref[1:-1, 1:-1, 1:-1]).sum() > 5000
    with Solver(n, with_source=True, ir_dtype=dtype, temporal=3) as s:
        s.load(u0, b)
        s.set_temporal_tiles(*shape)
        with pytest.raises(JcError) as e:
            s.solve_ir(inner=m, rtol=0.0, max_inner=m)
        assert e.value.code == L.JC_ERR_NONFINITE
        got = s.store().cpu().numpy()
    assert same_bits_or_nan(got, ref)
