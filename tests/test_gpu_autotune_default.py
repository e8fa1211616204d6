"""jc_autotune keeps the shape a context has where no candidate beats it: small
one-block grids, whose default columns of a few planes (about 1.4 to 1.8 times
as fast as the best of the search's own list) are not in that list."""
import pytest

import synth

pytestmark = pytest.mark.gpu

from paper_2102_12416_amd import Solver  # noqa: E402


@pytest.mark.parametrize("n,kw", [((64, 64, 64), dict()), ((64, 64, 64), dict(mode="fused", with_source=True)),
                                  ((100, 90, 80), dict(mode="fused")), ((32, 32, 32), dict()),
                                  ((64, 64, 64), dict(with_source=True, ir_dtype="bf16"))])
def test_autotune_keeps_a_default_that_nothing_beats(n, kw):
    print("[case] autotune default", n, kw, flush=True)
    with Solver(n, **kw) as s:
        s.load(synth.boundary_field(n, seed=4), synth.source_field(n, seed=4) if kw.get("with_source") else None)
        before = s.tile_info()
        tuned = s.autotune(reps=3)
        assert before["z_chunk"] < 16
        assert tuned[:3] == (before["tile_x"], before["tile_y"], before["z_chunk"])
        assert s.tile_info() == before
