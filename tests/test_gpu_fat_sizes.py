"""Fat links and path force on both sides of the size where the passes stop sharing links
between waves, and where the tile walk over z and t applies (planes of 256 sites per
parity) or not, against the FP64 oracle on every link; gates as in the fat parity tests."""
import numpy as np
import pytest

import gaugegen
import oracle

from gpu_util import device, force_errors, from_soa, rounded, to_soa

pytestmark = pytest.mark.gpu

C = (0.61, -0.071, 0.013, -0.0029, -0.055, -0.043)
TOL = {"f64": 1e-12, "f32": 1e-5}

SHAPES = [
    (4, 6, 4, 10),   # shared links, half a wave past the lattice
    (8, 8, 8, 16),   # the largest with shared links
    (8, 8, 8, 18),   # the first without
    (16, 32, 6, 4),  # tile walk, blocks of four and two z; gather in workgroups of two planes
    (16, 8, 8, 10),  # gather in workgroups of four planes (FP32) or none, slabs of two t
    (32, 16, 4, 6),  # of four planes, slabs of one t on six XCDs
]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("L", SHAPES, ids=str)
def test_sizes(L, prec):
    import paper_1808_02281_amd as sym

    rng = np.random.default_rng(5)
    U = rounded(gaugegen.near_thermal_links(L, 0.35, 5), prec)
    GV, GW = (rounded(rng.standard_normal(U.shape) + 1j * rng.standard_normal(U.shape), prec) for _ in range(2))
    Us, GVs, GWs = (to_soa(sym, f, L, prec, device()) for f in (U, GV, GW))
    rel = lambda a, b: np.abs(from_soa(sym, a, L) - b).max() / np.abs(b).max()
    V, W = sym.fat_links(Us, L, C)
    Vo, Wo = oracle.fat_links(U, L, C)
    assert rel(V, Vo) <= TOL[prec] and rel(W, Wo) <= TOL[prec]
    go = oracle.fat_grad(U, L, C, GV, GW)
    assert rel(sym.fat_force(Us, L, C, GVs, GWs, mode="grad"), go) <= TOL[prec]
    G = from_soa(sym, sym.fat_force(Us, L, C, GVs, GWs, mode="force"), L)
    assert force_errors(G, oracle.fat_force_from_grad(U, go))[0] <= TOL[prec]
    # no Naik term
    go = oracle.fat_grad(U, L, C, GV, None)
    assert rel(sym.fat_force(Us, L, C, GVs, None, mode="grad"), go) <= TOL[prec]
