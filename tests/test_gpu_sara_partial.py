"""SARA on sides whose sub-bands the filter tiles do not divide: bands of an odd
side, one or two samples past a tile, shorter than a tile and than the filters,
down to a last level of 3 samples, where regions wrap more than once.
Psi^dagger and Psi against the oracle, and the l1 step with its f1 (two SDMM
iterations); tolerances of the operators, 1e-5 (FP32) and 1e-12 (FP64), 10 times
that for the SDMM iterate and f1."""
import numpy as np
import pytest

import workloads as W
from oracle import nufft, sdmm as osdmm, wavelets
from tests.gpu_helpers import TOL, announce, device, host, rel, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n,levels", [(12, 2), (24, 3), (36, 1), (36, 2), (72, 2), (108, 2), (144, 4), (324, 2)])
def test_partial_tiles(n, levels, prec):
    device()
    announce(f"SARA partial tiles n={n} levels={levels} {prec}")
    from paper_1307_4370_amd import Plan
    g = W.rng(342, n, levels)
    M = 200
    uv, x, alpha, y = W.coverage(M, g), W.random_complex((n, n), g), W.random_complex((9, n, n), g), W.random_complex(M, g)
    if prec == "f32":
        uv = uv.astype(np.float32).astype(np.float64)
        x, alpha, y = (a.astype(np.complex64).astype(np.complex128) for a in (x, alpha, y))
    plan = Plan(n, to_dev(uv, prec), J=6, levels=levels, prec=prec, tile=8)
    sara = wavelets.Sara(n, levels)
    assert rel(host(plan.psi_adj(to_dev(x, prec))), sara.psi_adj(x)) <= TOL[prec]
    assert rel(host(plan.psi(to_dev(alpha, prec))), sara.psi(alpha)) <= TOL[prec]
    if n <= 144:
        eps = 0.4 * float(np.linalg.norm(y))
        xo, _, hist, _ = osdmm.sdmm(y, eps, nufft.Operator(n, uv, 6), sara, 2, n_cg=3)
        xg, _, ghist, _ = plan.sdmm(to_dev(y, prec), eps, 2, n_cg=3)
        assert rel(host(xg), xo) <= 10 * TOL[prec]
        assert ghist[-1][0] == pytest.approx(hist[-1]["f1"], rel=10 * TOL[prec])


# Tiles of 1 to 16, whole and partial, of each kernel: one, three and eight bases,
# with and without the Dirac plane.
@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n,levels,mask", [
    (16, 4, 511), (64, 3, 511), (96, 3, 140), (192, 2, 257), (192, 2, 510), (108, 1, 256), (108, 2, 257), (216, 2, 256),
    (288, 2, 140),
])
def test_tile_sides(n, levels, mask, prec):
    device()
    announce(f"SARA tile sides n={n} levels={levels} mask={mask} {prec}")
    from paper_1307_4370_amd import Plan
    g = W.rng(345, n, mask)
    q = bin(mask).count("1")
    uv, x, alpha = W.coverage(8, g), W.random_complex((n, n), g), W.random_complex((q, n, n), g)
    if prec == "f32":
        x, alpha = (a.astype(np.complex64).astype(np.complex128) for a in (x, alpha))
    plan = Plan(n, to_dev(uv, prec), J=6, levels=levels, dict_mask=mask, prec=prec, tile=8)
    sara = wavelets.Sara(n, levels, mask)
    assert rel(host(plan.psi_adj(to_dev(x, prec))), sara.psi_adj(x)) <= TOL[prec]
    assert rel(host(plan.psi(to_dev(alpha, prec))), sara.psi(alpha)) <= TOL[prec]
