"""Passes over whole rows and faces, at the widths where their lane layouts
change: loading and reading back (8, 16, 32 or 64 lanes of two cells per
row), the refinement's first inner sweep (16 bytes per lane) and outer
update, and the staged halo exchange.  All bitwise."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

from paper_2102_12416_amd import Group, Solver  # noqa: E402

# around 1, 16, 32, 64 and 128 cells: one lane, the lane counts, a second trip
WIDTHS = [1, 2, 15, 16, 17, 18, 31, 33, 34, 63, 64, 65, 66, 127, 129, 131]


def random_field(n, seed):
    rng = np.random.default_rng(seed)
    return rng.uniform(-1.0, 1.0, (n[2] + 2, n[1] + 2, n[0] + 2))


@pytest.mark.parametrize("nx", WIDTHS)
@pytest.mark.parametrize("split", [1, 2, 3])
def test_load_and_store_every_element(nx, split):
    n = (nx, 7, 5)
    if split > nx:
        pytest.skip("more blocks than cells")
    print("[case] load / store", n, split, flush=True)
    u0, b = random_field(n, nx), random_field(n, nx + 1000)
    with Solver(n, block_dims=(-(-nx // split), 3, 2), with_source=True) as s:
        for _ in range(2):                        # a context loaded again
            s.load(u0, b)
            assert np.array_equal(s.store().cpu().numpy(), u0)
            assert np.array_equal(s.store(1).cpu().numpy(), b)
            s.iterate(3)                          # the copies and their ghosts in use
            ref, _ = oracle.c_jacobi(u0, 3, b)
            assert np.array_equal(s.store().cpu().numpy(), ref)
            u0 = u0[::-1, ::-1, ::-1].copy()


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("nx", [1, 2, 3, 4, 5, 7, 8, 9, 15, 17, 63, 64, 65, 130])
def test_first_inner_sweep_and_update_widths(dtype, nx):
    n = (nx, 5, 4)
    print("[case] refinement rows", dtype, n, flush=True)
    u0, b = synth.boundary_field(n, seed=nx), synth.source_field(n, seed=nx)
    ref, _, done, _ = oracle.c_ir_solve(u0, b, storage=dtype, inner=7, rtol=1e-30, max_inner=21)
    for kw in ({}, dict(block_dims=((nx + 1) // 2, 2, 4), mode="fused"), dict(temporal=3)):
        with Solver(n, with_source=True, ir_dtype=dtype, **kw) as s:
            s.load(u0, b)
            info = s.solve_ir(inner=7, rtol=1e-30, max_inner=21)
            assert info["iters"] == done
            assert np.array_equal(s.store().cpu().numpy(), ref), kw


def test_group_update_of_members_at_different_points():
    """Refining members whose pending corrections sit in different copies."""
    print("[case] group update", flush=True)
    sizes = [(20, 9, 8), (33, 8, 7), (17, 6, 9), (12, 12, 12)]
    windows = [7, 8, 8, 7]

    def make(i):
        s = Solver(sizes[i], with_source=True, ir_dtype="f32")
        return s.load(synth.boundary_field(sizes[i], seed=i), synth.source_field(sizes[i], seed=i))

    def start(s, w):
        with Group([s]) as g:
            g.residuals()
            g.iterate(w)

    alone = []
    for i, w in enumerate(windows):
        s = make(i)
        start(s, w)
        with Group([s]) as g:
            g.residuals()
        alone.append(s.store().cpu().numpy())
        s.close()
    mix = [make(i) for i in range(len(sizes))]
    for s, w in zip(mix, windows):
        start(s, w)
    with Group(mix) as g:
        g.residuals()
    for s, a in zip(mix, alone):
        assert np.array_equal(s.store().cpu().numpy(), a)
        s.close()


@pytest.mark.parametrize("bd", [(1, 1, 1), (16, 17, 15), (40, 9, 33)])
def test_faces_of_small_and_large_planes(bd):
    n = (40, 34, 33) if bd != (1, 1, 1) else (4, 3, 5)
    print("[case] faces", n, bd, flush=True)
    u0 = random_field(n, 5)
    ref, _ = oracle.c_jacobi(u0, 4, None)
    with Solver(n, block_dims=bd, mode="staged") as s:
        s.load(u0)
        for _ in range(4):
            s.pack_faces()
            s.exchange()
            s.unpack_faces()
            s.sweep()
        assert np.array_equal(s.store().cpu().numpy(), ref)
