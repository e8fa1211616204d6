"""Groups that sweep two or three times per launch, in the shape chosen from
their members' sizes: edges around the tile's 32 and 64 cells and 16 and 32
rows, from a group whose columns are a few planes each to one of several
rounds of columns.  The sweeps take the same sums in the same order as one
sweep per launch, so the fields and norms are equal, not close."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

from paper_2102_12416_amd import Group, Solver  # noqa: E402

# one member: short columns; edges on and next to the tile's; several rounds
SIZES = {
    "one": [(5, 3, 2)],
    "edges": [(31, 33, 9), (32, 32, 32), (33, 31, 65), (63, 17, 16), (64, 16, 17), (65, 15, 1), (1, 1, 7)],
    "rounds64": [(64, 63, 48)] * 40,
    "rounds": [(97, 66, 70), (65, 33, 64)] * 13,
}


@pytest.mark.parametrize("dtype", [None, "f64", "f32", "bf16"])
@pytest.mark.parametrize("sizes", sorted(SIZES))
def test_group_shapes_match_one_sweep_per_launch(sizes, dtype):
    print("[case] group shapes", sizes, dtype, flush=True)
    kw = dict(with_source=True, **({"ir_dtype": dtype} if dtype else {}))
    runs = []
    for temporal in (False, True, 3):
        solvers = []
        for i, n in enumerate(SIZES[sizes]):
            s = Solver(n, **kw)
            s.load(synth.boundary_field(n, seed=90 + i), synth.source_field(n, seed=90 + i))
            solvers.append(s)
        norms = []
        with Group(solvers, temporal=temporal) as g:
            for window in (12, 11, 10, 7):
                norms.append(g.residuals())
                g.iterate(window)
            norms.append(g.residuals())
        runs.append((norms, [s.store().cpu().numpy() for s in solvers]))
        for s in solvers:
            s.close()
    for norms, fields in runs[1:]:
        assert norms == runs[0][0]
        for i, (a, b) in enumerate(zip(runs[0][1], fields)):
            assert np.array_equal(a, b), (sizes, dtype, i)
