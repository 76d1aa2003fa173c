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


@pytest.mark.parametrize("prec,cb", [("f32", 8), ("f64", 16)])
@pytest.mark.parametrize("n,J", [(128, 8), (64, 6), (128, 10)])
def test_capped_plans_keep_the_smallest_halo(n, J, prec, cb, monkeypatch):
    """A coverage that narrow gridding bands serve best: under a cap the plan keeps
    one band per tile, (J - 1)(K tps + ntiles (T + J - 1)) halo cells, and gives the
    same results."""
    device()
    announce(f"capped plan n={n} J={J} {prec}")
    g = W.rng(362, n, J)
    M = 30000
    uv = np.clip(g.standard_normal((M, 2)) * 0.3, -np.pi, np.pi).astype(np.float32).astype(np.float64)
    y = to_dev(W.random_complex(M, g), prec)
    from paper_1307_4370_amd import Plan, device_bytes
    held = device_bytes()
    free = Plan(n, to_dev(uv, prec), J=J, levels=1, prec=prec)
    free_bytes = device_bytes() - held
    monkeypatch.setenv("RIOP_DEVICE_MEMORY_LIMIT", str(1 << 36))
    held = device_bytes()
    capped = Plan(n, to_dev(uv, prec), J=J, levels=1, prec=prec)
    extra = free_bytes - (device_bytes() - held)
    info = capped.info()
    T = info["tile"]
    # Per extra band: its bottom strip, and its place in the list of bands.
    per_band = cb * (J - 1) * (T + J - 1) + 16
    assert extra % (per_band * info["ntiles"]) == 0
    assert extra // (per_band * info["ntiles"]) + 1 in (2, 4, 8)
    a, b = free.phi_adj(y), capped.phi_adj(y)
    assert float(torch.linalg.vector_norm(a - b) / torch.linalg.vector_norm(a)) <= (1e-6 if prec == "f32" else 1e-14)


@pytest.mark.parametrize("n,levels,tiles", [(36, 1, [5]), (72, 2, [5, 5]), (108, 1, [7]), (24, 2, [3, 3]), (64, 2, [2, 1])])
def test_solver_workspace(n, levels, tiles):
    """The solver's workspace at its first use: 8 images, two sets of nine
    coefficient planes, three sets of visibilities, the partial sums of the
    reductions, of which the l1 norm has one per analysis tile and basis and at
    most one per 256 pixels for the Dirac basis, and the scalars."""
    device()
    announce(f"solver workspace n={n} levels={levels}")
    from paper_1307_4370_amd import device_bytes
    M, N = 300, n * n
    plan = _plan(n, M, 6, "f32", levels, tile=8 if n % 16 else 0)
    held = device_bytes()
    b = to_dev(W.random_complex((n, n), W.rng(363, n)), "f32")
    plan.cg(b, n_iter=1)
    f1 = 8 * sum(t * t for t in tiles) + min(tiles[0] ** 2, -(-N // 256))
    got = device_bytes() - held - 8 * (8 * N + 2 * 9 * N + 3 * M) - 8 * f1
    assert got == 8 * (7 * 512 + 10)
