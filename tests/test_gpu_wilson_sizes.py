"""Wilson-clover force on both sides of the size where four waves stop sharing links, with and
without the clover term, against the FP64 oracle on every link; gates as in the Wilson
parity tests."""
import numpy as np
import pytest
import torch

import gaugegen
import oracle

from gpu_util import cdtype, device, force_errors, from_soa, rounded, to_soa

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-5}

SHAPES = [
    (4, 6, 4, 10),  # shared links, half a wave past the lattice
    (8, 8, 8, 16),  # the largest with shared links
    (8, 8, 8, 18),  # the first without
]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("csw", [1.37, 0.0])
@pytest.mark.parametrize("L", SHAPES, ids=str)
def test_sizes(L, csw, prec):
    import paper_1808_02281_amd as sym

    rng = np.random.default_rng(6)
    U = rounded(gaugegen.near_thermal_links(L, 0.35, 6), prec)
    shape = (L[3], L[2], L[1], L[0], 4, 3)
    X, Y = (rounded(rng.standard_normal(shape) + 1j * rng.standard_normal(shape), prec) for _ in range(2))
    spinor = lambda f: sym.pack_spinor(torch.from_numpy(np.ascontiguousarray(f)).to(cdtype(prec)).to(device()), L)
    G = from_soa(sym, sym.wilson_force(to_soa(sym, U, L, prec, device()), spinor(X), spinor(Y), L, 0.1242, csw), L)
    assert force_errors(G, oracle.wilson_force(U, X, Y, L, 0.1242, csw))[0] <= TOL[prec]
