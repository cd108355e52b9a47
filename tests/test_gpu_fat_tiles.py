"""Fat links and path force where the tiles of the passes change their order with the size, and
with remainders of every part of the tile walk (blocks of z, the last slab of t, planes that
are not whole tiles): a field repeated along t has the repeated links and forces.

Every link goes through the same operations on the same values whatever its tile (both
lattices are above the size where links are shared between waves), so they agree bitwise. The
short lattice's sizes are among those compared with the oracle elsewhere or larger.
"""
import numpy as np
import pytest
import torch

import gaugegen

from gpu_util import cdtype, device

pytestmark = pytest.mark.gpu

C = (0.61, -0.071, 0.013, -0.0029, -0.055, -0.043)

CASES = [
    ((16, 32, 6, 4), 11),  # walk, z in four and two, slabs of six t and one of two; gather over two planes
    ((32, 16, 8, 4), 9),   # walk, slabs of five and one of one; gather over four planes
    ((24, 24, 6, 4), 10),  # planes of no whole tiles
    ((16, 16, 8, 6), 6),   # below the size where the order changes; gather with a short slab
]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("L,reps", CASES, ids=str)
def test_repeated_field(L, reps, prec):
    import paper_1808_02281_amd as sym

    big = (L[0], L[1], L[2], L[3] * reps)
    rng = np.random.default_rng(9)
    U = gaugegen.near_thermal_links(L, 0.3, 9)
    fields = [U] + [rng.standard_normal(U.shape) + 1j * rng.standard_normal(U.shape) for _ in range(2)]
    aos = [torch.from_numpy(f).to(cdtype(prec)).to(device()) for f in fields]

    def results(a, shape):
        Us, GV, GW = (sym.pack(f, shape) for f in a)
        nan = lambda: torch.full_like(Us, float("nan"))  # a link left out shows
        V, W = sym.fat_links(Us, shape, C, out=(nan(), nan()))
        F = sym.fat_force(Us, shape, C, GV, GW, mode="force", out=nan())
        return [sym.unpack(r, shape) for r in (V, W, F)]

    short = results(aos, L)
    long = results([f.repeat(reps, 1, 1, 1, 1, 1, 1) for f in aos], big)
    for name, a, b in zip("VWF", short, long):
        assert torch.equal(b, a.repeat(reps, 1, 1, 1, 1, 1, 1)), f"case {L} x {reps} {prec} {name}"
