"""Small lattices: the force and staple passes that split a link's and a site's work over
waves give bitwise the forces of the batched call, which runs the whole-link code at every
size, on both sides of the sizes where the split ends."""
import pytest
import torch

import gaugegen

from gpu_util import device, to_soa

pytestmark = pytest.mark.gpu

U0, BETA = gaugegen.U0, gaugegen.BETA

SHAPES = [
    (4, 4, 4, 4),      # two chunks per parity
    (4, 6, 4, 10),     # 7.5 chunks per parity: half a wave past the lattice
    (8, 8, 8, 8),      # the largest split force
    (8, 8, 8, 10),     # the first whole one
    (8, 8, 8, 20),     # the largest split FP64 staples
    (8, 8, 10, 18),    # whole FP64 staples
    (12, 12, 12, 12),  # the largest split FP32 staples
    (12, 12, 12, 14),  # whole FP32 staples
]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("L", SHAPES, ids=str)
def test_split_equals_whole(L, prec):
    import paper_1808_02281_amd as sym

    U = to_soa(sym, gaugegen.haar_links(L, 17), L, prec, device())
    F = sym.force(U, L, U0, BETA)
    Fb = sym.force_batch([U], [L], U0, BETA)
    assert torch.equal(F, Fb[0])
