"""The factored force on lattices whose last slab of t is shorter than the others, in each of the
tile walks (planes that are whole workgroups; in FP64 planes of whole halves), against the FP64
oracle on every link. Gates as in the parity tests: 1e-12 and 1e-5 of the largest force, the
FP32 oracle on the rounded links."""
import pytest

import gaugegen
import oracle

from gpu_util import device, force_errors, from_soa, rounded, to_soa

pytestmark = pytest.mark.gpu

U0, BETA = gaugegen.U0, gaugegen.BETA
TOL = {"f64": 1e-12, "f32": 1e-5}

SHAPES = [
    (16, 16, 6, 20),  # planes of one (FP32) and two workgroups, z in four and two; slabs of three t, the last of two
    (16, 32, 4, 34),  # of two and four; slabs of five, the last of four
    (8, 8, 10, 22),   # FP64: half a workgroup a plane; slabs of three, the last of one
    (8, 24, 6, 20),   # FP64: three halves; slabs of three, the last of two
]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("L", SHAPES, ids=str)
def test_short_last_slab(L, prec):
    import paper_1808_02281_amd as sym

    U = gaugegen.haar_links(L, 43)
    c = oracle.coeffs(U0)[0]
    Uin = rounded(U, prec)
    F, S = sym.force(to_soa(sym, U, L, prec, device()), L, U0, BETA, with_action=True)
    gmax, _, _ = force_errors(from_soa(sym, F, L), oracle.force(Uin, L, c, BETA))
    S_ref = oracle.action(Uin, L, c, BETA)[0]
    assert gmax <= TOL[prec]
    assert abs(S[0].item() - S_ref) <= TOL[prec] * abs(S_ref)
