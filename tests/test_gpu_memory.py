"""What the library holds on the device, by riop_device_bytes: the sizes that the
interface states, and the smallest RIOP_DEVICE_MEMORY_LIMIT under which a call
fits.  Counts are exact; nothing depends on a tolerance."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_helpers import announce, device, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _plan(n, M, J=8, prec="f32", levels=1, **more):
    from paper_1307_4370_amd import Plan
    return Plan(n, to_dev(W.coverage(M, W.rng(360, n, J)), prec), J=J, levels=levels, prec=prec, **more)


@pytest.mark.parametrize("prec,rb", [("f32", 4), ("f64", 8)])
@pytest.mark.parametrize("n,J", [(8, 6), (12, 8), (24, 8), (36, 8), (48, 16), (64, 8), (72, 6)])
def test_stored_gram_takes_its_planes(n, J, prec, rb):
    """J + (J - 1)(2J - 1) planes of K^2 values, at every K: no padding of a row."""
    device()
    announce(f"Gram bytes n={n} J={J} {prec}")
    from paper_1307_4370_amd import device_bytes
    plan = _plan(n, 200, J, prec, tile=8 if n == 36 else 0)
    held = device_bytes()
    plan.gram_build()
    assert device_bytes() - held == (J + (J - 1) * (2 * J - 1)) * (2 * n) ** 2 * rb
    plan.gram_release()
    assert device_bytes() == held


@pytest.mark.parametrize("prec,cb", [("f32", 8), ("f64", 16)])
@pytest.mark.parametrize("n,inner", [(16, 1), (64, 8), (48, 33)])
def test_tv_takes_six_images(n, inner, prec, cb):
    """Beyond the solver's workspace the TV prior holds six complex images, whatever
    the number of inner iterations."""
    device()
    announce(f"TV bytes n={n} inner={inner} {prec}")
    from paper_1307_4370_amd import device_bytes
    M = 300
    plan = _plan(n, M, 6, prec)
    y = to_dev(W.random_complex(M, W.rng(361, n)), prec)
    eps = 0.5 * float(torch.linalg.vector_norm(y))
    plan.sdmm(y, eps, 2, n_cg=2)
    held = device_bytes()
    plan.sdmm_tv(y, eps, 2, n_cg=2, n_inner=inner)
    assert device_bytes() - held == 6 * n * n * cb
