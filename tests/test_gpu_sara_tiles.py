"""SARA's tiles: every sub-band tile side (16 down to 1), levels whose region
wraps the periodic line more than once, each basis alone (its own filter code),
dictionaries without the Dirac plane, and image sizes whose last synthesis level
runs one, two and four groups per block.  Psi^dagger and Psi against the oracle,
and a NaN in any part of the input reported.  Tolerances: relative L2 of 1e-5
(FP32) and 1e-12 (FP64), as for the operators."""
import numpy as np
import pytest

import workloads as W
from oracle import wavelets
from tests.gpu_helpers import TOL, announce, device, host, rel, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FULL = wavelets.FULL_MASK


def _plan(n, levels, mask, prec):
    from paper_1307_4370_amd import Plan
    uv = W.coverage(4, W.rng(330, n))
    return Plan(n, to_dev(uv, prec), J=6, levels=levels, dict_mask=mask, prec=prec)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n,levels,mask", [
    (8, 3, FULL), (16, 4, FULL), (24, 3, FULL), (48, 4, FULL), (64, 1, FULL), (96, 5, FULL),
    (32, 5, FULL & ~1), (512, 1, FULL), (768, 2, FULL), (64, 2, 1), *[(32, 2, 1 << b) for b in range(1, 9)],
    (1024, 1, 0b100000110),
])
def test_sara_tiles(n, levels, mask, prec):
    device()
    announce(f"SARA tiles n={n} levels={levels} mask={mask:#x} {prec}")
    q = bin(mask).count("1")
    x, alpha = W.random_complex((n, n), W.rng(331, n)), W.random_complex((q, n, n), W.rng(332, n))
    if prec == "f32":
        x, alpha = (v.astype(np.complex64).astype(np.complex128) for v in (x, alpha))
    sara = wavelets.Sara(n, levels, mask)
    plan = _plan(n, levels, mask, prec)
    assert rel(host(plan.psi_adj(to_dev(x, prec))), sara.psi_adj(x)) <= TOL[prec]
    assert rel(host(plan.psi(to_dev(alpha, prec))), sara.psi(alpha)) <= TOL[prec]
    plan.sync()


@pytest.mark.parametrize("mask", [FULL, FULL & ~1, 1])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
def test_nonfinite_inputs_reported(mask, bad):
    """Each pass checks what it loads: pixels in every quarter, coefficients in every band."""
    device()
    from paper_1307_4370_amd import RiopError
    n, levels, q = 64, 2, bin(mask).count("1")
    plan = _plan(n, levels, mask, "f32")
    for at in ((0, 0), (63, 63), (31, 40), (17, 2)):
        x = torch.zeros(n, n, dtype=torch.complex64, device="cuda")
        x[at] = complex(0.0, bad)
        plan.psi_adj(x)
        with pytest.raises(RiopError):
            plan.sync()
    for plane in {0, q - 1}:
        for at in ((0, 0), (3, 20), (20, 3), (20, 20), (5, 50), (50, 5), (63, 63)):
            a = torch.zeros(q, n, n, dtype=torch.complex64, device="cuda")
            a[(plane, *at)] = complex(bad, 0.0)
            plan.psi(a)
            with pytest.raises(RiopError):
                plan.sync()
    plan.psi(torch.zeros(q, n, n, dtype=torch.complex64, device="cuda"))
    plan.sync()
