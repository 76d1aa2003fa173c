"""The compile-time FFT passes over their line lengths K = 2n: the smallest and
largest of each family (2^a and 3 2^a), lengths that end in each last radix,
lines shorter than a wavefront, and a length left to the generic kernel.

Phi and Phi^dagger against the oracle, and CG, whose direction update and p.q
sums ride on the column passes (halos are added by the row pass where it can).
Tolerances: the operators' relative L2 of 1e-5 (FP32) and 1e-12 (FP64); CG
solves a system of condition number at most (||Phi||^2 + 2) / 2 < 10 here, so
its iterate is held to 10 times that.
Of the families' largest lengths K = 2048 and K = 3072 are in test_gpu_fft_large.py,
K = 6144 in test_gpu_limits.py.
"""
import numpy as np
import pytest

import workloads as W
from oracle import nufft, sdmm as osdmm
from tests.gpu_helpers import TOL, announce, device, host, rel, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n", [8, 12, 16, 24, 48, 72, 96, 192, 384, 512, 768])
def test_lengths(prec, n):
    device()
    announce(f"fft length K={2 * n} {prec}")
    from paper_1307_4370_amd import Plan
    g = W.rng(310, 1, n)
    M, J = min(1501, n * n // 2 + 1), 6
    uv, x, w = W.coverage(M, g), W.random_complex((n, n), g), W.random_complex(M, g)
    if prec == "f32":
        uv = uv.astype(np.float32).astype(np.float64)
        x, w = (a.astype(np.complex64).astype(np.complex128) for a in (x, w))
    op = nufft.Operator(n, uv, J)
    plan = Plan(n, to_dev(uv, prec), J=J, levels=1, prec=prec)
    assert rel(host(plan.phi(to_dev(x, prec))), op.phi(x)) <= TOL[prec]
    assert rel(host(plan.phi_adj(to_dev(w, prec))), op.phi_adj(w)) <= TOL[prec]
    got, _ = plan.cg(to_dev(x, prec), n_iter=4)
    want = osdmm.conjugate_gradient(lambda v: op.phi_adj(op.phi(v)) + 2.0 * v, x, np.zeros_like(x), 4)
    assert rel(host(got), want) <= 10 * TOL[prec]
