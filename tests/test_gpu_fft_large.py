"""The compile-time FFT passes at K = 2048 and K = 3072.  At K = 3072 a column block
holds one or two columns and there are more blocks (768, 1536) than partial-sum
slots: Q's 2 x rides on the adjoint column pass without sums, and CG's direction
update and p.q sums run as kernels of their own.  Phi, Phi^dagger, Q and two CG
iterations against the oracle on inputs of single precision; tolerances of the
operators, 1e-5 (FP32) and 1e-12 (FP64), 10 times that for CG (condition number
below 10)."""
import functools

import numpy as np
import pytest

import workloads as W
from oracle import nufft, sdmm as osdmm
from tests.gpu_helpers import TOL, announce, device, host, rel, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@functools.lru_cache(maxsize=1)
def _case(n):
    g = W.rng(311, 1, n)
    M, J = 3001, 6
    uv = W.coverage(M, g).astype(np.float32).astype(np.float64)
    x, w = (a.astype(np.complex64).astype(np.complex128) for a in (W.random_complex((n, n), g), W.random_complex(M, g)))
    op = nufft.Operator(n, uv, J)
    y = op.phi(x)
    cg = osdmm.conjugate_gradient(lambda v: op.phi_adj(op.phi(v)) + 2.0 * v, x, np.zeros_like(x), 2)
    return uv, J, x, w, y, op.phi_adj(w), op.phi_adj(y) + 2.0 * x, cg


@pytest.mark.parametrize("n,prec", [(1024, "f32"), (1024, "f64"), (1536, "f32"), (1536, "f64")])
def test_large_lengths(n, prec):
    device()
    announce(f"fft length K={2 * n} {prec}")
    from paper_1307_4370_amd import Plan
    uv, J, x, w, y, xa, q, cg = _case(n)
    plan = Plan(n, to_dev(uv, prec), J=J, levels=1, dict_mask=1, prec=prec)
    assert rel(host(plan.phi(to_dev(x, prec))), y) <= TOL[prec]
    assert rel(host(plan.phi_adj(to_dev(w, prec))), xa) <= TOL[prec]
    assert rel(host(plan.apply_q(to_dev(x, prec))), q) <= TOL[prec]
    got, _ = plan.cg(to_dev(x, prec), n_iter=2)
    assert rel(host(got), cg) <= 10 * TOL[prec]
    plan.close()
