"""The split kernels of small lattices in captured HIP graphs (their launches reserve up to 153 KiB
of LDS): force with action, gradient, action and trajectory, replayed with eager work in
between, are bitwise the eager results."""
import pytest
import torch

import gaugegen

from gpu_util import device, to_soa

pytestmark = pytest.mark.gpu

U0, BETA = gaugegen.U0, gaugegen.BETA


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("L", [(4, 4, 4, 4), (8, 8, 8, 8)], ids=str)
def test_replays(L, prec):
    import paper_1808_02281_amd as sym

    U = to_soa(sym, gaugegen.near_thermal_links(L, 0.3, 21), L, prec, device())
    P = to_soa(sym, gaugegen.momenta(L, 22), L, prec, device())
    Um, Pm = U.clone(), P.clone()

    def work():
        F, S = sym.force(U, L, U0, BETA, with_action=True)
        g, Sg = sym.action_grad(U, L, U0, BETA, with_action=True)
        W = sym.action(U, L, U0, BETA)
        H = sym.md_leapfrog(Um, Pm, L, U0, BETA, 0.02, 3)
        return F, S, g, Sg, W, H, Um, Pm

    eager = [t.clone() for t in work()]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = work()
    for rep in range(4):
        for t in out[:6]:
            t.zero_()
        Um.copy_(U)
        Pm.copy_(P)
        sym.force(P, L, U0, BETA)  # eager work that overwrites the workspace
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for k, (a, b) in enumerate(zip(out, eager)):
            assert torch.equal(a, b), f"replay {rep} output {k}"
