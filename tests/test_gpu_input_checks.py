"""Non-finite inputs are reported by the pass that first loads them: the forward
column pass (compile-time and generic lengths), the gridding (both orders, matrix
and vector paths, first and last visibility, one visibility in all), the
gather of the solvers' data and CG's first kernel.  Clean inputs report nothing and
leave Q = Phi^dagger Phi + 2 I as the oracle has it (the 2 x is added in the adjoint
column pass where the length allows).  Tolerance: the operators' 1e-12."""
import numpy as np
import pytest

import workloads as W
from oracle import nufft
from tests.gpu_helpers import TOL, announce, device, host, rel, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,M,J", [(16, 1, 6), (16, 333, 8), (72, 700, 8), (48, 130, 10)])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_input_checks(n, M, J, prec):
    device()
    announce(f"input checks n={n} M={M} J={J} {prec}")
    from paper_1307_4370_amd import Plan, RiopError
    uv, x = W.coverage(M, W.rng(340, n)), W.random_complex((n, n), W.rng(341, n))
    plan = Plan(n, to_dev(uv, prec), J=J, levels=1, prec=prec, tile=8 if n == 72 else 0)  # 2n = 144 = 9 x 16
    good_x, good_y = to_dev(x, prec), plan.phi(to_dev(x, prec))
    if prec == "f64":
        op = nufft.Operator(n, uv, J)
        assert rel(host(plan.apply_q(good_x)), op.phi_adj(op.phi(x)) + 2 * x) <= TOL[prec]
    plan.phi_adj(good_y), plan.phi_adj(good_y, sorted=True), plan.apply_q(good_x), plan.cg(good_x, n_iter=1)
    plan.sync()
    for bad in (complex("nan"), complex(0.0, float("inf"))):
        for at in ((0, 0), (n - 1, n - 1), (n // 2, 1)):
            bx = good_x.clone()
            bx[at] = bad
            for call in (lambda: plan.phi(bx), lambda: plan.phi(bx, sorted=True), lambda: plan.apply_q(bx),
                         lambda: plan.cg(bx, n_iter=1), lambda: plan.cg(good_x, x0=bx, n_iter=1)):
                with pytest.raises(RiopError):
                    call()
                    plan.sync()
        for at in {0, M // 2, M - 1}:
            by = good_y.clone()
            by[at] = bad
            for call in (lambda: plan.phi_adj(by), lambda: plan.phi_adj(by, sorted=True), lambda: plan.gamma(by),
                         lambda: plan.sdmm(by, 1.0, 1, n_cg=1)):
                with pytest.raises(RiopError):
                    call()
                    plan.sync()
        plan.sync()
