"""The stored Gram operator's tiles: grids narrower than a tile, with a partial
last tile, just wide enough for the window (K = 2 J), and every width, whose
plane quads wrap differently at the grid's edges.  Q through the planes against
the oracle's Q; tolerances of the operators, 1e-5 (FP32) and 1e-12 (FP64)."""
import numpy as np
import pytest

import workloads as W
from oracle import nufft
from tests.gpu_helpers import TOL, announce, device, host, rel, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n,J", [(8, 6), (12, 6), (16, 16), (24, 14), (36, 8), (72, 10), (72, 12)])
def test_gram_tiles(n, J, prec):
    device()
    announce(f"Gram tiles n={n} J={J} {prec}")
    from paper_1307_4370_amd import Plan
    uv = W.rng(610, n, J).uniform(-np.pi, np.pi, size=(3 * n * n, 2))
    x = W.random_complex((n, n), W.rng(611, n + J))
    if prec == "f32":
        uv = uv.astype(np.float32).astype(np.float64)
        uv = np.clip(uv, -np.pi, np.pi)
        x = x.astype(np.complex64).astype(np.complex128)
    plan = Plan(n, to_dev(uv, prec), J=J, levels=1, prec=prec, tile=8 if n == 36 else 0)  # 2n = 72 = 9 x 8
    plan.gram_build()
    op = nufft.Operator(n, uv, J)
    assert rel(host(plan.apply_q(to_dev(x, prec))), op.phi_adj(op.phi(x)) + 2 * x) <= TOL[prec]
