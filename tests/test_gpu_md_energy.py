"""The energies of a trajectory at the sizes where the force pass changes its split: the kinetic
energy is summed in the first and the last kick and has to be that of the momenta before the
first and after the last, next to the action of the fields at either end."""
import pytest

import gaugegen

from gpu_util import device, rounded, to_soa

pytestmark = pytest.mark.gpu

U0, BETA = gaugegen.U0, gaugegen.BETA

SHAPES = [
    (4, 4, 4, 4),     # two workgroups per direction and parity
    (4, 6, 4, 10),    # half a wave past the lattice
    (8, 8, 8, 8),     # the largest split force pass
    (8, 8, 8, 10),    # the first whole one
    (6, 10, 14, 12),  # ragged workgroups
]


# The energies are sums of at most 1e5 terms in 64 bits: rounding 2^-53 times the terms'
# count at worst, 1e-11; FP32 links give the action FP32 traces, 2^-24 with a few roundings.
@pytest.mark.parametrize("prec,tol", [("f32", 1e-5), ("f64", 1e-11)])
@pytest.mark.parametrize("L", SHAPES, ids=str)
def test_energies_at_both_ends(L, prec, tol):
    import paper_1808_02281_amd as sym

    U = to_soa(sym, rounded(gaugegen.near_thermal_links(L, 0.3, 3), prec), L, prec, device())
    P = to_soa(sym, rounded(gaugegen.momenta(L, 4), prec), L, prec, device())

    def energy():  # no steps: the kernels that only measure
        return sym.md_leapfrog(U, P, L, U0, BETA, 0.02, 0)[0].item()

    before = energy()
    H = sym.md_leapfrog(U, P, L, U0, BETA, 0.02, 2)
    after = energy()
    print(f"case {L} {prec}: H0 {H[0].item():.12e} {before:.12e} H1 {H[1].item():.12e} {after:.12e}", flush=True)
    assert abs(H[0].item() - before) <= tol * abs(before)
    assert abs(H[1].item() - after) <= tol * abs(after)
