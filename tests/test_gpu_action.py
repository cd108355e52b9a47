"""The action kernel against the FP64 oracle at the edges of its tiles (64 sites of one
parity per workgroup), in both tile orders, and for matrices off SU(3), which the action
takes as they are.

Tolerance. Every loop is six (four) matrices of norm about one: with unit roundoff u its
trace carries at most 6 x 6 x 3 u, relative to the 3 of a loop near the identity; the sums
over loops are in double. 36 u relative to the loop sum n_X V x 3 bounds the FP64 figure far
below 1e-12, and in FP32 gives 36 x 2^-24 = 2.2e-6, below the 1e-5 of the parity gates.
"""
import numpy as np
import pytest

import gaugegen
import oracle

from gpu_util import device, rounded, to_soa

pytestmark = pytest.mark.gpu

U0, BETA = gaugegen.U0, gaugegen.BETA
TOL = {"f64": 1e-12, "f32": 36 * 2.0 ** -24}

SHAPES = [
    (4, 4, 4, 4),    # two whole tiles per parity, wraps on every side
    (6, 4, 4, 4),    # three tiles per parity: tile count rounded up to a multiple of 8
    (4, 6, 10, 6),   # 11.25 tiles per parity: a ragged last tile
    (16, 16, 4, 8),  # t-slab order, one t-slice per XCD, two 256-site chunks per slice
    (8, 16, 4, 16),  # t-slab order, two slices per XCD
]


def check(U, L, prec):
    import paper_1808_02281_amd as sym

    c = oracle.coeffs(U0)[0]
    S_ref, W_ref = oracle.action(rounded(U, prec), L, c, BETA)
    got = sym.action(to_soa(sym, U, L, prec, device()), L, U0, BETA).cpu().numpy()
    V = np.prod(L)
    loops = 3.0 * V * np.array([6, 12, 16])
    np.testing.assert_array_less(np.abs(got[1:] - W_ref), TOL[prec] * loops)
    assert abs(got[0] - S_ref) <= TOL[prec] * BETA / 3 * np.abs(np.array(c)) @ loops


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("L", SHAPES, ids=str)
def test_action_tiles(L, prec):
    check(gaugegen.haar_links(L, 31), L, prec)


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_action_of_matrices_off_su3(prec):
    L = (4, 6, 4, 6)
    rng = np.random.default_rng(8)
    U = gaugegen.near_thermal_links(L, 0.3, 8)
    # Frobenius norms below one: the bound above holds with room
    U = 0.5 * (U + 0.2 * (rng.standard_normal(U.shape) + 1j * rng.standard_normal(U.shape)))
    check(U, L, prec)
