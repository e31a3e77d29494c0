"""The direction scan of lbm_diagnostics against a scan of every node in FP64 torch, and the
initialisation from rest (no u0, F = I) against the general one."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _solver(nx, ny, storage, law, bc, seed, fields):
    from paper_2605_26677_amd.solver import Solver
    rng = np.random.default_rng(seed)
    mu, lam = 0.1, 0.2
    if fields:
        mu = (0.1 * np.exp(0.3 * rng.standard_normal((ny, nx)))).astype(np.float32)
        lam = (0.2 * np.exp(0.3 * rng.standard_normal((ny, nx)))).astype(np.float32)
    return Solver(nx, ny, c=4.0, omega=1.99, material=law, storage=storage, bc=(bc,) * 4, mu=mu, lam=lam,
                  force_unstable=True), rng


def _scan(sv):
    """max over nodes and 180 directions of sqrt(lam_max(Q)) / c in FP64 (log-NH)."""
    U = sv.moments()
    mu = sv.mu_t.double() if sv.mu_t is not None else torch.full_like(U[0], sv.s.mu0)
    lam = sv.lam_t.double() if sv.lam_t is not None else torch.full_like(U[0], sv.s.lam0)
    F = [1 + U[2], U[3], U[4], 1 + U[5]]
    J = F[0] * F[3] - F[1] * F[2]
    H = [F[3] / J, -F[2] / J, -F[1] / J, F[0] / J]
    a = mu - lam * torch.log(J)
    best = torch.zeros_like(J)
    for t in range(180):
        n = (math.cos(math.pi * t / 180), math.sin(math.pi * t / 180))
        h = [H[2 * i] * n[0] + H[2 * i + 1] * n[1] for i in range(2)]
        q = [[(a + lam) * h[i] * h[k] + (mu if i == k else 0) for k in range(2)] for i in range(2)]
        top = 0.5 * (q[0][0] + q[1][1]) + torch.sqrt((0.5 * (q[0][0] - q[1][1])) ** 2 + q[0][1] ** 2)
        best = torch.maximum(best, top)
    return float(torch.sqrt(best.max()) / sv.p.c)


# FP32: the recovered F (rounding 1e-7) and the scan's own arithmetic, whose rotated direction
# drifts by up to 180 roundings of 6e-8; FP64 the same in double
@pytest.mark.parametrize("storage,tol", [("f32", 2e-5), ("f64", 1e-12), ("f16", 2e-5)])
@pytest.mark.parametrize("nx,ny", [(3, 5), (64, 64), (300, 211), (1031, 517)])
@pytest.mark.parametrize("amp", [0.0, 1e-3, 0.2])
@pytest.mark.parametrize("fields", [False, True])
def test_wave_speed_audit(nx, ny, storage, tol, amp, fields):
    sv, rng = _solver(nx, ny, storage, "lognh", "periodic", 3, fields)
    sv.init(amp * rng.standard_normal((2, ny, nx)), 0.5 * amp * rng.standard_normal((2, ny, nx)))
    got = float(sv.diagnostics()[9])
    want = _scan(sv)
    assert abs(got - want) <= tol * want


@pytest.mark.parametrize("storage", ["f32", "f64", "f16"])
@pytest.mark.parametrize("bc", ["periodic", "velocity", "traction"])
@pytest.mark.parametrize("law", ["lognh", "nh", "svk", "mr", "yeoh", "gent"])
@pytest.mark.parametrize("nx,ny", [(4, 5), (130, 33)])
def test_init_from_rest_equals_general_init(nx, ny, storage, bc, law):
    """A zero u0 takes the general kernels: the same populations, displacement and faults."""
    a, rng = _solver(nx, ny, storage, law, bc, 7, True)
    b, _ = _solver(nx, ny, storage, law, bc, 7, True)
    v0 = 1e-2 * rng.standard_normal((2, ny, nx))
    a.init(v0)
    b.init(v0, np.zeros((2, ny, nx)))
    assert torch.equal(a.populations(), b.populations())
    assert torch.equal(a.displacement(), b.displacement())
    assert a.faults() == b.faults()
