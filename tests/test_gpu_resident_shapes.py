"""Resident sweeps over the kernel's variants: buffer sizes (up to 16^3, up to
32^3, long thin blocks), work-groups of one to eight waves, even and odd rows,
and groups whose members differ in all of these in one launch.  Bitwise."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

from paper_2102_12416_amd import Group, Solver  # noqa: E402

SHAPES = [(16, 16, 16), (15, 16, 17), (17, 16, 16), (32, 16, 32), (32, 17, 8), (33, 16, 31), (32, 32, 32),
          (31, 32, 30), (1024, 1, 1), (800, 1, 2), (2, 300, 9), (1, 310, 9), (1, 512, 3), (2, 1, 32), (3, 2, 31)]


def fields(n, seed, src):
    return synth.boundary_field(n, seed=seed), synth.source_field(n, seed=seed) if src else None


@pytest.mark.parametrize("src", [False, True])
@pytest.mark.parametrize("n", SHAPES)
def test_variants_alone(n, src):
    print("[case] resident", n, src, flush=True)
    u0, b = fields(n, 3, src)
    with Solver(n, mode="fused", with_source=src, resident=True) as s:
        s.load(u0, b)
        done = 0
        for k in (1, 2, 5):                       # windows that end going up and going down
            s.iterate(k)
            done += k
            ref, _ = oracle.c_jacobi(u0, done, b)
            assert np.array_equal(s.store().cpu().numpy(), ref), done


@pytest.mark.parametrize("src", [False, True])
def test_group_of_all_variants(src):
    print("[case] resident group", src, flush=True)
    data = [fields(n, 10 + i, src) for i, n in enumerate(SHAPES)]
    solvers = [Solver(n, mode="fused", with_source=src).load(*d) for n, d in zip(SHAPES, data)]
    solvers[2].iterate(3)                         # a member in the other copy
    with Group(solvers, resident=True) as g:
        g.iterate(4)
        g.residuals()
        g.iterate(3)
    for i, (s, (u0, b)) in enumerate(zip(solvers, data)):
        ref, _ = oracle.c_jacobi(u0, 7 + (3 if i == 2 else 0), b)
        assert np.array_equal(s.store().cpu().numpy(), ref), SHAPES[i]
        s.close()
