"""Wilson-clover force where four waves share 64 links: a field repeated along t until the whole-link
kernel takes it has the repeated forces, bitwise (the same operations in the same order)."""
import numpy as np
import pytest
import torch

import gaugegen

from gpu_util import cdtype, device

pytestmark = pytest.mark.gpu

CASES = [
    ((4, 6, 4, 10), 10),  # half a wave past the lattice -> 600 workgroups of 64 links
    ((8, 8, 8, 16), 2),   # the largest with shared links -> 1024
]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("L,reps", CASES, ids=str)
def test_shared_equals_whole(L, reps, prec):
    import paper_1808_02281_amd as sym

    big = (L[0], L[1], L[2], L[3] * reps)
    rng = np.random.default_rng(12)
    U = gaugegen.near_thermal_links(L, 0.35, 12)
    X, Y = (rng.standard_normal(U.shape[:4] + (4, 3)) + 1j * rng.standard_normal(U.shape[:4] + (4, 3)) for _ in range(2))
    u, x, y = (torch.from_numpy(f).to(cdtype(prec)).to(device()) for f in (U, X, Y))

    def force(shape, n):
        rep = lambda f: f.repeat((n,) + (1,) * (f.dim() - 1))
        Us = sym.pack(rep(u), shape)
        out = torch.full_like(Us, float("nan"))
        return sym.unpack(sym.wilson_force(Us, sym.pack_spinor(rep(x), shape), sym.pack_spinor(rep(y), shape), shape,
                                           0.1242, 1.37, out=out), shape)

    short, long = force(L, 1), force(big, reps)
    assert torch.equal(long, short.repeat(reps, 1, 1, 1, 1, 1, 1))
