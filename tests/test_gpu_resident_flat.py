"""Resident sweeps of blocks of up to four planes (a build of their own: one or
two steps per sweep) in each of its buffer sizes, alone, in groups of their own
and beside taller blocks, in windows that end going up and going down.
Bitwise against the oracle."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

from paper_2102_12416_amd import Group, Solver  # noqa: E402

SHAPES = [(1, 1, 1), (7, 5, 1), (8, 5, 2), (9, 4, 3), (8, 6, 4), (31, 20, 1), (32, 20, 2), (33, 16, 3), (32, 32, 4),
          (1023, 1, 1), (256, 2, 2), (2, 400, 2), (1, 512, 3), (500, 2, 4)]


def fields(n, seed, src):
    return synth.boundary_field(n, seed=seed), synth.source_field(n, seed=seed) if src else None


@pytest.mark.parametrize("src", [False, True])
@pytest.mark.parametrize("n", SHAPES)
def test_flat_blocks_alone(n, src):
    print("[case] flat resident", n, src, flush=True)
    u0, b = fields(n, 5, src)
    with Solver(n, mode="fused", with_source=src, resident=True) as s:
        s.load(u0, b)
        done = 0
        for k in (1, 2, 5, 8):
            s.iterate(k)
            done += k
            ref, _ = oracle.c_jacobi(u0, done, b)
            assert np.array_equal(s.store().cpu().numpy(), ref), done


@pytest.mark.parametrize("src", [False, True])
@pytest.mark.parametrize("tall", [[], [(6, 5, 5)], [(16, 10, 32), (32, 32, 32)]])
def test_flat_blocks_in_groups(tall, src):
    print("[case] flat resident group", tall, src, flush=True)
    shapes = SHAPES + tall
    data = [fields(n, 20 + i, src) for i, n in enumerate(shapes)]
    solvers = [Solver(n, mode="fused", with_source=src).load(*d) for n, d in zip(shapes, data)]
    solvers[3].iterate(1)                         # a member in the other copy
    with Group(solvers, resident=True) as g:
        g.iterate(4)
        g.iterate(3)
    for i, (s, (u0, b)) in enumerate(zip(solvers, data)):
        ref, _ = oracle.c_jacobi(u0, 7 + (i == 3), b)
        assert np.array_equal(s.store().cpu().numpy(), ref), shapes[i]
        s.close()
