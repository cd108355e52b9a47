"""Layout kernels at the edges of their runs of 64 (FP64) and 128 (FP32) sites, links and
spinors, against a numpy statement of the layouts. They are copies: bitwise."""
import numpy as np
import pytest
import torch

from gpu_util import cdtype, device, soa_reference

pytestmark = pytest.mark.gpu

SHAPES = [
    (4, 4, 4, 4),   # whole runs
    (6, 4, 4, 4),   # six FP64 runs, three FP32 runs
    (6, 6, 6, 6),   # a last run of 16 sites in both precisions
    (4, 6, 4, 10),  # 15 FP64 runs, a half FP32 run
    (10, 6, 4, 6),  # a last run of 32 sites
]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("L", SHAPES, ids=str)
def test_layouts(L, prec):
    import paper_1808_02281_amd as sym

    rng = np.random.default_rng(3)
    real = np.float32 if prec == "f32" else np.float64
    grid = (L[3], L[2], L[1], L[0])
    field = lambda *c: (rng.standard_normal(grid + c).astype(real) + 1j * rng.standard_normal(grid + c).astype(real))
    U, X = field(4, 3, 3), field(4, 3)
    a = torch.from_numpy(U).to(cdtype(prec)).to(device())
    S = sym.pack(a, L)
    np.testing.assert_array_equal(S.cpu().numpy().astype(np.float64), soa_reference(U.astype(np.complex128), L))
    assert torch.equal(sym.unpack(S, L), a)

    x = torch.from_numpy(X).to(cdtype(prec)).to(device())
    R = sym.pack_spinor(x, L)
    t, z, y, xx = np.meshgrid(*[np.arange(n) for n in grid], indexing="ij")
    par = ((t + z + y + xx) & 1).reshape(-1)
    flat = X.reshape(-1, 12)
    want = np.stack([flat[par == p].T for p in (0, 1)])  # (2, 12, V/2): sites of a parity in order
    got = R.cpu().numpy()
    np.testing.assert_array_equal(got[..., 0], want.real)
    np.testing.assert_array_equal(got[..., 1], want.imag)
    assert torch.equal(sym.unpack_spinor(R, L), x)
