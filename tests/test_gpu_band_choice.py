"""The gridding's band heights and G^T G's two forms, each reached by a coverage
that asks for it: whole tiles, 16 and 8 rows of a 32-row tile, on the matrix and
the vector path; one launch for even coverages, two where a clustered coverage's
heaviest band would degrid alone or whole 64-row tiles leave no LDS (a plan made
under a memory cap).  The height is read off the halo a plan holds beyond one made
under a cap (which keeps whole tiles), the form off the kernel timings.
Phi^dagger, with and without the cap, and Q against the oracle; tolerances of the
operators, 1e-5 (FP32) and 1e-12 (FP64)."""
import numpy as np
import pytest

import workloads as W
from oracle import nufft
from tests.gpu_helpers import TOL, announce, device, host, rel, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _uv(n, M, kind):
    g = W.rng(343, n, M)
    uv = g.uniform(-np.pi, np.pi, size=(M, 2))
    if kind == "gauss":
        uv = np.clip(g.standard_normal((M, 2)) * np.pi / 4, -np.pi, 3.1415)
    elif kind == "cluster":
        uv[M // 3:] = 0.02 * uv[M // 3:] + 0.3
    return uv.astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("prec,n,M,J,tile,kind,rows,launches", [
    ("f32", 256, 20000, 8, 32, "uniform", 32, 1), ("f32", 256, 20000, 6, 32, "uniform", 32, 1),
    ("f32", 256, 20000, 12, 32, "uniform", 32, 2), ("f32", 256, 20000, 8, 32, "gauss", 16, 1),
    ("f32", 128, 20000, 8, 32, "uniform", 16, 1), ("f32", 128, 20000, 6, 32, "uniform", 8, 1),
    ("f32", 128, 3000, 8, 32, "gauss", 8, 1), ("f32", 128, 20000, 8, 32, "gauss", 8, 1),
    ("f32", 128, 20000, 8, 32, "cluster", 8, 2), ("f32", 128, 20000, 6, 32, "cluster", 8, 2),
    ("f32", 64, 600, 8, 64, "uniform", 8, 1), ("f32", 256, 30000, 8, 8, "uniform", 8, 2),
    ("f32", 128, 9000, 12, 32, "uniform", 16, 2), ("f32", 128, 9000, 12, 32, "gauss", 16, 2),
    ("f64", 256, 20000, 8, 32, "uniform", 32, 2), ("f64", 128, 20000, 6, 32, "uniform", 8, 2),
    ("f64", 128, 20000, 8, 32, "gauss", 8, 2), ("f64", 128, 9000, 12, 32, "gauss", 16, 2),
])
def test_band_choice(prec, n, M, J, tile, kind, rows, launches, monkeypatch):
    device()
    announce(f"band choice n={n} M={M} J={J} tile={tile} {kind} {prec}")
    from paper_1307_4370_amd import Plan, device_bytes
    g = W.rng(344, n, M)
    uv, w, x = _uv(n, M, kind), W.random_complex(M, g), W.random_complex((n, n), g)
    if prec == "f32":
        w, x = (a.astype(np.complex64).astype(np.complex128) for a in (w, x))
    op = nufft.Operator(n, uv, J)
    want, wantq = op.phi_adj(w), op.phi_adj(op.phi(x)) + 2 * x
    held = []
    for cap in (None, 1 << 36):
        if cap:
            monkeypatch.setenv("RIOP_DEVICE_MEMORY_LIMIT", str(cap))
        before = device_bytes()
        plan = Plan(n, to_dev(uv, prec), J=J, levels=1, prec=prec, tile=tile)
        held.append(device_bytes() - before)
        assert rel(host(plan.phi_adj(to_dev(w, prec))), want) <= TOL[prec]
        plan.timing(True)
        got = plan.apply_q(to_dev(x, prec))
        kinds = {k for k, (_, count) in plan.timing_read().items() if count}
        plan.timing(False)
        assert rel(host(got), wantq) <= TOL[prec]
        one = launches == 1 and not (cap and tile == 64)
        assert ("gram_fused" in kinds) == one and ("degrid" in kinds) != one
        plan.close()
    per_band = (8 if prec == "f32" else 16) * (J - 1) * (tile + J - 1) + 16
    assert held[0] - held[1] == (tile // rows - 1) * (2 * n // tile) ** 2 * per_band
