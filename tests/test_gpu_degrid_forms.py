"""Degridding's two forms, a block per work unit and blocks for parts of a unit,
on both sides of the rule that chooses: units of at most 256 visibilities, of
257 and of the full 1024 and one more; few units; regions so wide that staging
them again per part costs more than it gives (64-wide tiles, the region wider
than a wavefront); a window wider than its tile's remainder at the grid's edge.
Phi in both orders against the oracle; tolerances of the operators, 1e-5 (FP32)
and 1e-12 (FP64)."""
import numpy as np
import pytest

import workloads as W
from oracle import nufft
from tests.gpu_helpers import TOL, announce, device, host, rel, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n,M,J,tile,one", [
    (16, 256, 8, 8, 1), (16, 257, 8, 8, 1), (32, 1024, 6, 16, 1), (32, 1025, 6, 16, 1), (64, 9000, 8, 8, 0),
    (32, 600, 8, 64, 0), (64, 5000, 8, 64, 0), (64, 5000, 16, 16, 0), (64, 9000, 12, 32, 0), (128, 40000, 6, 32, 0),
    # More parts than are in flight at once, their restaging too costly: whole units.
    (128, 70000, 12, 64, 0), (256, 140000, 8, 64, 0), (256, 270000, 6, 64, 0),
])
def test_degrid_forms(n, M, J, tile, one, prec):
    device()
    announce(f"degridding n={n} M={M} J={J} tile={tile} one={one} {prec}")
    from paper_1307_4370_amd import Plan
    g = W.rng(340, n, M + tile)
    uv = g.uniform(-np.pi, np.pi, size=(M, 2))
    if one:  # all windows start in the last tile and wrap
        uv = np.pi * (1.0 - 1e-3 - g.random((M, 2)) / n)
    x = W.random_complex((n, n), g)
    if prec == "f32":
        uv = uv.astype(np.float32).astype(np.float64)
        x = x.astype(np.complex64).astype(np.complex128)
    op = nufft.Operator(n, uv, J)
    plan = Plan(n, to_dev(uv, prec), J=J, levels=1, prec=prec, tile=tile)
    want = op.phi(x)
    assert rel(host(plan.phi(to_dev(x, prec))), want) <= TOL[prec]
    perm = host(plan.layout()[0]).real.astype(np.int64)
    assert rel(host(plan.phi(to_dev(x, prec), sorted=True)), want[perm]) <= TOL[prec]
