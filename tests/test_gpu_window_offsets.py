"""Windows at every offset inside the 8-aligned column block in which gridding
stages its column weights: the two halves of a wavefront clear the block's rows
and then write their weights over rows that the other half may have cleared.
Slices that hold one offset, all offsets in turn, and offsets that change at every
entry; Phi^dagger and the fused Phi^dagger Phi against the oracle, tolerances of
the operators, 1e-5 (FP32) and 1e-12 (FP64)."""
import numpy as np
import pytest

import workloads as W
from oracle import nufft
from tests.gpu_helpers import TOL, announce, device, host, rel, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("J", [6, 8])
@pytest.mark.parametrize("offsets", [[0], [3], [5], [7], list(range(8)), [7, 0, 4]])
def test_window_offsets(J, offsets, prec):
    device()
    announce(f"window offsets J={J} {offsets} {prec}")
    from paper_1307_4370_amd import Plan
    n, M = 32, 37 * 8
    g = W.rng(341, J, 10 * len(offsets) + offsets[0])
    # The window's first column is floor(g - J/2) + 1: column 8 k + offset.
    col = 8 * g.integers(-3, 3, size=M) + np.resize(offsets, M) - 1 + J // 2 + g.uniform(0.05, 0.95, size=M)
    row = g.integers(-n, n - 1, size=M) + g.uniform(0.05, 0.95, size=M)
    uv = np.stack([row, col], axis=1) * (np.pi / n)
    w, x = W.random_complex(M, g), W.random_complex((n, n), g)
    if prec == "f32":
        uv = uv.astype(np.float32).astype(np.float64)
        w, x = (a.astype(np.complex64).astype(np.complex128) for a in (w, x))
    op = nufft.Operator(n, uv, J)
    plan = Plan(n, to_dev(uv, prec), J=J, levels=1, prec=prec)
    first = plan.layout()[1].cpu().numpy().astype(np.int64) >> 16
    assert set((first % 8).tolist()) == set(offsets)
    assert rel(host(plan.phi_adj(to_dev(w, prec))), op.phi_adj(w)) <= TOL[prec]
    assert rel(host(plan.apply_q(to_dev(x, prec))), op.phi_adj(op.phi(x)) + 2 * x) <= TOL[prec]
