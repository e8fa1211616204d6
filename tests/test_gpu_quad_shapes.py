"""Three sweeps of a binary32 or bfloat16 correction by quads of cells in shapes
that are set (32 rows): rows that end in each place of a quad, one and several
tiles and z chunks.  The same sums in the same order as one sweep per launch:
equal, not close."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

from paper_2102_12416_amd import Solver  # noqa: E402


def refined(n, dtype, temporal, shape=None, inner=10):
    with Solver(n, mode="fused", with_source=True, ir_dtype=dtype, temporal=temporal) as s:
        s.load(synth.boundary_field(n, seed=8), synth.source_field(n, seed=8))
        if shape:
            s.set_temporal_tiles(*shape)
            i = s.temporal_info()
            assert (i["rows"], i["z_chunk"]) == shape
        s.solve_ir(inner=inner, rtol=0.0, max_inner=3 * inner)
        return s.store().cpu().numpy()


@pytest.mark.parametrize("n,planes", [((1, 1, 1), 1), ((61, 33, 9), 4), ((62, 32, 8), 8), ((63, 31, 7), 3),
                                      ((64, 64, 20), 7), ((65, 65, 5), 9), ((130, 40, 33), 11)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_quads_match_one_sweep_per_launch(n, planes, dtype):
    print("[case] quads set", n, planes, dtype, flush=True)
    assert np.array_equal(refined(n, dtype, 3, (32, planes)), refined(n, dtype, False))
