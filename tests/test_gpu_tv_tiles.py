"""The TV prox's tiles: images smaller than a tile, ending inside one and at its
edge, iteration counts around the launches' limits (one iteration, uneven
splits, both limits), weights with zeros.  Two SDMM iterations against the oracle;
tolerances 1e-10 (FP64) and 1e-4 (FP32), the TV solver's."""
import numpy as np
import pytest

import workloads as W
from oracle import nufft, tv
from tests.gpu_helpers import announce, device, host, rel, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [("f64", 1e-10), ("f32", 1e-4)])
@pytest.mark.parametrize("n,inner,weighted", [(8, 1, 0), (16, 2, 1), (24, 7, 0), (32, 8, 1), (48, 15, 0), (96, 20, 1),
                                              (64, 13, 1), (384, 7, 0), (512, 6, 1)])
def test_tv_tiles(n, inner, weighted, prec, tol):
    device()
    announce(f"TV tiles n={n} inner={inner} weighted={weighted} {prec}")
    from paper_1307_4370_amd import Plan
    g = W.rng(350, 1, n + inner)
    M = 400
    uv, y = W.coverage(M, g), W.random_complex(M, g)
    w = np.maximum(g.uniform(-0.3, 1.5, size=(n, n)), 0.0) if weighted else None
    if prec == "f32":
        uv = uv.astype(np.float32).astype(np.float64)
        y = y.astype(np.complex64).astype(np.complex128)
        w = None if w is None else w.astype(np.float32).astype(np.float64)
    op = nufft.Operator(n, uv, 6)
    eps = 0.4 * float(np.linalg.norm(y))
    xo, _, hist, _ = tv.sdmm_tv(y, eps, op, T=3, n_cg=3, n_inner=inner, weights=w)
    plan = Plan(n, to_dev(uv, prec), J=6, levels=1, prec=prec)
    xg, _, ghist, _, _ = plan.sdmm_tv(to_dev(y, prec), eps, T=3, n_cg=3, n_inner=inner,
                                      weights=None if w is None else to_dev(w, prec))
    assert rel(host(xg), xo) <= tol
    assert ghist[-1][0] == pytest.approx(hist[-1]["f1"], rel=tol)
