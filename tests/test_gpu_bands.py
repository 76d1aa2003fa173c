"""Gridding bands: TB rows of a sort tile per workgroup, TB chosen from the
coverage's counts.  Coverages that lead to every band height the rule can
choose (sparse: the whole tile; dense in few cells: the narrowest), windows that
straddle band, tile and grid edges, and widths with J - 1 above and below the
narrowest band.  Phi^dagger against the oracle, Phi^dagger Phi through a
grid whose halos the adjoint row pass adds (a power of two), that have their own
kernel (72 = 2^3 9), and with the l2-ball prox fused in (one SDMM iteration).
Tolerances: relative L2 of 1e-5 (FP32) and 1e-12 (FP64), as for the operators;
10 times that for the SDMM iterate (CG, condition number below 10).
Which height and which form of G^T G a coverage takes follows the library's cost
rule; test_gpu_band_choice.py asserts both, with coverages that reach every height
and the two launches.
"""
import math

import numpy as np
import pytest

import workloads as W
from oracle import nufft, sdmm as osdmm, wavelets
from tests.gpu_helpers import TOL, announce, device, host, rel, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _uv(n, M, kind, g):
    """sparse: uniform; edges: cells around multiples of 8 rows of the grid, its
    wrap included; dense: most of M within a few cells."""
    uv = g.uniform(-math.pi, math.pi, size=(M, 2))
    if kind == "edges":
        row = 8 * g.integers(-n // 8, n // 8 + 1, size=M) + g.uniform(-4.0, 4.0, size=M)
        uv[:, 0] = np.clip(row * math.pi / n, -math.pi, 3.1415)
    elif kind == "dense":
        uv[M // 4:] = 0.05 * uv[M // 4:] / math.pi + 0.3
    return uv


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n,M,J,kind", [
    (64, 700, 8, "sparse"), (64, 9000, 6, "edges"), (128, 30000, 8, "dense"), (128, 30000, 8, "edges"),
    (72, 9000, 8, "dense"), (128, 30000, 10, "dense"), (128, 20000, 16, "dense"), (192, 40000, 8, "dense"),
])
def test_bands(prec, n, M, J, kind):
    device()
    announce(f"bands n={n} M={M} J={J} {kind} {prec}")
    from paper_1307_4370_amd import Plan
    g = W.rng(320, 1, n * 31 + J)
    uv, w = _uv(n, M, kind, g), W.random_complex(M, g)
    if prec == "f32":
        uv = uv.astype(np.float32).astype(np.float64)
        w = w.astype(np.complex64).astype(np.complex128)
    op = nufft.Operator(n, uv, J)
    plan = Plan(n, to_dev(uv, prec), J=J, levels=1, prec=prec)
    want = op.phi_adj(w)
    assert rel(host(plan.phi_adj(to_dev(w, prec))), want) <= TOL[prec]
    perm = host(plan.layout()[0]).real.astype(np.int64)
    assert rel(host(plan.phi_adj(to_dev(w[perm], prec), sorted=True)), want) <= TOL[prec]
    sara = wavelets.Sara(n, 1)
    eps = 0.5 * float(np.linalg.norm(w))
    got, _, _, _ = plan.sdmm(to_dev(w, prec), eps, 2, n_cg=3)
    x, _, _, _ = osdmm.sdmm(w, eps, op, sara, 2, n_cg=3)
    assert rel(host(got), x) <= 10 * TOL[prec]


@pytest.mark.parametrize("n,M,J,tile", [(32, 1, 8, 8), (64, 33, 6, 16), (64, 5000, 8, 16), (64, 5000, 8, 64),
                                        (96, 20000, 6, 64), (128, 60000, 8, 32), (48, 255, 8, 32)])
def test_fused_gram(n, M, J, tile):
    """Single-precision Q through the fused kernel at every tile side (64: the two
    launches it replaces), one visibility, slices with 1 and 31 live entries, a
    dense corner that wraps the grid's edges."""
    device()
    announce(f"fused G^T G n={n} M={M} J={J} tile={tile}")
    from paper_1307_4370_amd import Plan
    g = W.rng(321, 1, n * 31 + tile)
    uv = g.uniform(-math.pi, math.pi, size=(M, 2))
    uv[M // 2:] = math.pi - 0.02 - 0.1 * g.random((M - M // 2, 2))
    uv = uv.astype(np.float32).astype(np.float64)
    x = W.random_complex((n, n), g).astype(np.complex64).astype(np.complex128)
    op = nufft.Operator(n, uv, J)
    plan = Plan(n, to_dev(uv, "f32"), J=J, levels=1, prec="f32", tile=tile)
    got = host(plan.apply_q(to_dev(x, "f32"))) - 2 * x
    assert rel(got, op.phi_adj(op.phi(x))) <= TOL["f32"]
