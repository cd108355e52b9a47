"""Batched force over the sizes where its default schedule changes (workgroups of 256 or 128
links in FP32) and over lattices whose planes are whole tiles, which it walks in blocks of z
and t, mixed with others: bitwise the single-lattice forces, the actions to rounding.

The actions are sums of at most 7e5 terms in 64 bits, grouped differently by the two calls: no
more than the terms' count times 2^-53, 8e-11 of the sum of their absolute values; the terms
are deficits of one sign up to the mixed class, whose two weights differ in sign by a factor
of ten, so the bound below holds with room (FP32 traces are the same in both calls).
"""
import math

import pytest
import torch

import gaugegen

from gpu_util import device, to_soa

pytestmark = pytest.mark.gpu

U0, BETA = gaugegen.U0, gaugegen.BETA
S = 2048  # waves of 64 links resident at a time in FP32

# name: lattices, the range of their number of waves
BATCHES = {
    # FP32 256 links, nothing walked
    "half a round": ([(8, 8, 8, 8)] * 4, (0, S // 2)),
    # 128 links: z in fours and two, t in a slab of eight and one of two; neighbours in the
    # table that are not walked and end in half a wave
    "most of a round": ([(4, 6, 4, 10), (16, 16, 6, 10), (6, 6, 6, 8)], (S // 2 + 1, S - 1)),
    # FP32 256 links: one chunk a plane, slabs of eight and four; half a chunk, not walked
    "two rounds": ([(32, 16, 6, 12), (4, 4, 4, 4), (16, 16, 6, 10)], (S, 3 * S)),
    # 128 links: two chunks a plane, slabs of eight, eight and four
    "four rounds, walked": ([(32, 16, 4, 20)] * 3 + [(8, 8, 8, 8)], (3 * S + 1, 6 * S)),
    # FP32 256 links
    "four rounds": ([(8, 8, 8, 14)] * 20, (3 * S + 1, 6 * S)),
    # 128 links
    "seven rounds": ([(12, 12, 12, 12)] * 11, (6 * S + 1, 8 * S)),
}


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("name", BATCHES)
def test_batch_equals_single(name, prec):
    import paper_1808_02281_amd as sym

    shapes, (least, most) = BATCHES[name]
    assert least <= sum(8 * -(-math.prod(L) // 128) for L in shapes) <= most
    fields = {L: to_soa(sym, gaugegen.haar_links(L, 60 + i), L, prec, device()) for i, L in enumerate(set(shapes))}
    single = {L: sym.force(U, L, U0, BETA, with_action=True) for L, U in fields.items()}
    out = [torch.full_like(fields[L], float("nan")) for L in shapes]  # a link left out shows
    Fs, act = sym.force_batch([fields[L] for L in shapes], shapes, U0, BETA, with_action=True, out=out)
    for i, L in enumerate(shapes):
        F, A = single[L]
        assert torch.equal(Fs[i], F), f"lattice {i} {L}"
        scale = 3.0 * math.prod(L) * BETA / 3 * 34
        assert abs(act[i, 0].item() - A[0].item()) <= 1e-10 * scale, f"lattice {i} {L}"
