"""Default multi-sweep shapes against one sweep per launch, on both sides of
the sizes where the rule changes: columns of a plane or two, one round of
long columns, several rounds, and the binary32 and bfloat16 correction from
2^22 cells on (three sweeps by quads of cells; rows that end in each place of
a quad).  Same sums in the same order, so the
iterates are equal, not close."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

from paper_2102_12416_amd import Solver  # noqa: E402


def field(n, kw, temporal, sweeps):
    with Solver(n, mode="fused", temporal=temporal, **kw) as s:
        s.load(synth.boundary_field(n, seed=77), synth.source_field(n, seed=77) if kw.get("with_source") else None)
        if kw.get("ir_dtype"):
            s.solve_ir(inner=sweeps, rtol=0.0, max_inner=sweeps)
        else:
            s.iterate(sweeps)
        return s.store().cpu().numpy()


@pytest.mark.parametrize("n", [(66, 1, 5), (64, 64, 64), (130, 50, 97), (257, 129, 140)])
@pytest.mark.parametrize("src", [False, True])
def test_binary64_default_shapes(n, src):
    print("[case] default multi-sweep shape", n, src, flush=True)
    kw = dict(with_source=src)
    ref = field(n, kw, False, 8)
    for depth in (True, 3):
        assert np.array_equal(field(n, kw, depth, 8), ref), depth


@pytest.mark.parametrize("n", [(128, 128, 255), (128, 128, 256), (259, 253, 130), (1, 257, 16400),
                               (2, 2100, 1000), (62, 262, 261), (63, 250, 270), (64, 33, 2000), (65, 1, 65000)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_correction_default_shapes(n, dtype):
    print("[case] default multi-sweep shape", n, dtype, flush=True)
    kw = dict(with_source=True, ir_dtype=dtype)
    ref = field(n, kw, False, 9)
    for depth in (True, 3):
        assert np.array_equal(field(n, kw, depth, 9), ref), depth
