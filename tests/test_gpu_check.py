"""sym_check_links where its workgroups take one tile each and where they loop over several:
planted defects in the last tiles are found, and counted once."""
import pytest
import torch

import gaugegen

from gpu_util import device, to_soa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("L", [(6, 4, 4, 6), (16, 16, 16, 32), (16, 16, 16, 36)], ids=str)  # 16, 2048, 2304 tiles
def test_planted_defects(L, prec):
    import paper_1808_02281_amd as sym

    U = to_soa(sym, gaugegen.unit_links(L), L, prec, device())
    assert sym.check_links(U, L).tolist() == [0.0, 0.0, 0.0]
    # links (direction 3, odd parity): one scaled by 1.5, U^+U - 1 = 1.25 and det = 3.375
    U[3, 1, :, -1] *= 1.5
    U[0, 0, 4, 0, 0] = float("nan")
    U[3, 1, 0, -2, 1] = float("inf")
    assert sym.check_links(U, L).tolist() == [pytest.approx(1.25 * 3 ** 0.5, rel=1e-15), 2.375, 2.0]
