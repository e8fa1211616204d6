"""Windows long enough to be captured (8 launches or more), replayed several times
from both ping-pong copies, with eager work, synchronisations, windows of other
lengths and changes of the launch shape between the replays.  Every field is
compared bitwise with the CPU oracle's sweep or with eager launches."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

from paper_2102_12416_amd import Group, Solver  # noqa: E402


def between(rep):
    """Unrelated eager work and a synchronisation."""
    junk = torch.ones(1000, device="cuda") * rep
    torch.cuda.synchronize()
    assert float(junk.sum()) == 1000.0 * rep


@pytest.mark.parametrize("kw", [dict(mode="staged"), dict(mode="fused"),
                                dict(mode="staged", block_dims=(24, 20, 18)), dict(mode="fused", block_dims=(24, 20, 18))])
@pytest.mark.parametrize("source", [False, True])
def test_one_sweep_windows(kw, source):
    n = (48, 40, 36)
    print("[case] graph windows, one sweep per launch", kw, source, flush=True)
    u, b = synth.boundary_field(n, seed=6), synth.source_field(n, seed=6) if source else None
    shapes = [None, (32, 8, 9), (64, 16, 5), (32, 8, 9)]
    with Solver(n, with_source=source, use_graphs=True, **kw) as s:
        s.load(u, b)
        for rep, shape in enumerate(shapes):
            if shape:
                s.set_tiles(*shape)
            for k in (9, 9, 9, 10, 3, 9):         # odd windows: replays from either copy
                s.iterate(k)
                u, _ = oracle.c_jacobi(u, k, b)
                between(rep + 1)
                assert np.array_equal(s.store().cpu().numpy(), u), (rep, k)


@pytest.mark.parametrize("temporal,window,shapes", [(True, 16, [None, (24, 7), (8, 50), (24, 7)]),
                                                    (3, 24, [None, (8, 7), (16, 50), (8, 7)])])
@pytest.mark.parametrize("source", [False, True])
def test_multi_sweep_windows(temporal, window, shapes, source):
    n = (90, 41, 50)
    print("[case] graph windows, temporal", temporal, source, flush=True)
    u, b = synth.boundary_field(n, seed=13), synth.source_field(n, seed=13) if source else None
    with Solver(n, mode="fused", temporal=temporal, with_source=source, use_graphs=True) as s:
        s.load(u, b)
        for rep, shape in enumerate(shapes):
            if shape:
                s.set_temporal_tiles(*shape)
            # 16 or 24 sweeps: 8 launches; one more: 9, from the other copy next
            for k in (window, window, window + 1, window, window + 1, 4, window):
                s.iterate(k)
                u, _ = oracle.c_jacobi(u, k, b)
                between(rep + 1)
                assert np.array_equal(s.store().cpu().numpy(), u), (rep, k)


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("temporal,inner", [(False, 12), (True, 19), (3, 28)])
def test_refinement_windows(dtype, temporal, inner):
    n = (61, 37, 29)
    print("[case] graph windows, refinement", dtype, temporal, flush=True)
    u, b = synth.boundary_field(n, seed=21), synth.source_field(n, seed=21)
    kw = dict(mode="fused", with_source=True, ir_dtype=dtype)
    with Solver(n, use_graphs=False, **kw) as e, Solver(n, use_graphs=True, temporal=temporal, **kw) as g:
        e.load(u, b)
        g.load(u, b)
        for rep in range(3):
            if temporal and rep == 1:
                g.set_temporal_tiles(8, 6)
            if temporal == 3 and rep == 2 and dtype != "f64":
                g.set_temporal_tiles(32, 11)
            for s in (e, g):
                s.solve_ir(inner=inner, rtol=0.0, max_inner=3 * inner)
            between(rep + 1)
            assert np.array_equal(g.store().cpu().numpy(), e.store().cpu().numpy()), rep
            for s in (e, g):
                s.iterate(1)                      # the next refinement starts from the other copy


@pytest.mark.parametrize("temporal,window", [(False, 8), (True, 16), (3, 24)])
@pytest.mark.parametrize("dtype", [None, "f32", "bf16"])
def test_group_windows(temporal, window, dtype):
    sizes = [(40, 33, 20), (17, 64, 9), (65, 15, 31)]
    print("[case] graph windows, group", temporal, dtype, flush=True)
    fields = []
    for graphs in (False, True):
        solvers = []
        for i, n in enumerate(sizes):
            kw = dict(ir_dtype=dtype) if dtype and i % 2 == 0 else {}
            s = Solver(n, with_source=True, **kw)
            s.load(synth.boundary_field(n, seed=50 + i), synth.source_field(n, seed=50 + i))
            solvers.append(s)
        got = []
        with Group(solvers, use_graphs=graphs, temporal=temporal) as g:
            for rep, k in enumerate((window, window, window + 1, window, window + 1, window)):
                got.append(g.residuals())
                g.iterate(k)
                between(rep + 1)
            got.append(g.residuals())
        fields.append((got, [s.store().cpu().numpy() for s in solvers]))
        for s in solvers:
            s.close()
    assert fields[0][0] == fields[1][0]
    for a, b in zip(*(f[1] for f in fields)):
        assert np.array_equal(a, b)
