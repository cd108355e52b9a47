"""The factored force on lattices whose (x, y) planes are whole workgroups (the blocked walk
over z and t), with remainders of every part of the walk, against the FP64 oracle on every
link; FP32 planes of one and two workgroups, FP64 of two and four and of one and three halves. Gates as in the parity
tests: 1e-12 and 1e-5 of the largest force, the FP32 oracle on the rounded links."""
import pytest

import gaugegen
import oracle

from gpu_util import device, force_errors, from_soa, rounded, to_soa

pytestmark = pytest.mark.gpu

U0, BETA = gaugegen.U0, gaugegen.BETA
TOL = {"f64": 1e-12, "f32": 1e-5}

SHAPES = [
    (16, 16, 4, 4),    # one block of z, slabs of one t-slice on four of the eight XCDs
    (32, 8, 6, 10),    # a block of two z, slabs of two t-slices, the last XCDs' share uneven
    (16, 32, 10, 18),  # two chunks (FP32) a plane, blocks 4 4 2 of z, slabs of three
    (8, 8, 10, 14),    # FP64: one half workgroup a plane, slabs of two
    (8, 24, 6, 18),    # FP64: three half workgroups a plane, slabs of three
]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("L", SHAPES, ids=str)
def test_blocked_walk(L, prec):
    import paper_1808_02281_amd as sym

    U = gaugegen.haar_links(L, 41)
    c = oracle.coeffs(U0)[0]
    Uin = rounded(U, prec)
    F, S = sym.force(to_soa(sym, U, L, prec, device()), L, U0, BETA, with_action=True)
    gmax, _, _ = force_errors(from_soa(sym, F, L), oracle.force(Uin, L, c, BETA))
    S_ref = oracle.action(Uin, L, c, BETA)[0]
    assert gmax <= TOL[prec]
    assert abs(S[0].item() - S_ref) <= TOL[prec] * abs(S_ref)
