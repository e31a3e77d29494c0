"""The wave-speed audit of lbm_diagnostics (out[9]), which scans only the nodes whose bounds let
them hold the largest value, against the oracle's tangent scanned at every node over the same 180
directions: prescribed states of every law, up to strong compression and stretch."""
import numpy as np
import pytest
import torch

from oracle import material as om

pytestmark = pytest.mark.gpu


def _scan(law, F, mu, lam):
    """(largest eigenvalue of Q over the 180 directions, |C|) of the states F (2, 2, n)."""
    C = om.tangent(law, F, mu, lam)
    top = np.full(F.shape[2], -np.inf)
    for t in range(180):
        n = np.array([np.cos(np.pi * t / 180), np.sin(np.pi * t / 180)])
        Q = np.einsum("A,iAkBn,B->ikn", n, C, n)
        top = np.maximum(top, 0.5 * (Q[0, 0] + Q[1, 1])
                         + np.sqrt((0.5 * (Q[0, 0] - Q[1, 1])) ** 2 + (0.5 * (Q[0, 1] + Q[1, 0])) ** 2))
    return top, np.sqrt((C ** 2).sum(axis=(0, 1, 2, 3)))


def _audit(law, F, storage, mu, lam, c):
    """(the library's value, the scan of every node, |C| over the largest eigenvalue there)."""
    from paper_2605_26677_amd.solver import Solver
    ny, nx = F.shape[2:]
    sv = Solver(nx, ny, c=c, omega=1.9, material=law, storage=storage, mu=mu, lam=lam, force_unstable=True)
    U0 = np.zeros((6, ny, nx))
    U0[2:] = (F - np.eye(2)[:, :, None, None]).reshape(4, ny, nx)
    zero = np.zeros_like(U0)
    sv.init_state(U0, zero, zero)
    got = float(sv.diagnostics()[9])
    U = sv.moments().cpu().numpy()
    F = U[2:].reshape(2, 2, -1) + np.eye(2)[:, :, None]
    top, norm = _scan(law, F, mu, lam)
    k = int(np.argmax(top))
    return got, np.sqrt(top[k]) / c, norm[k] / top[k]


# Rounding of the library's scan, relative to |C|: FP32 rotated directions drift by 5e-6 in |n|^2
# and 6e-7 in angle, FP64 by 1e-14; the tangent and Q add some 20 roundings.  The speed is a square
# root (half the relative error).
TOL = {"f32": 1e-5, "f16": 1e-5, "f64": 2e-14}


def _rotation(t):
    return np.array([[np.cos(t), -np.sin(t)], [np.sin(t), np.cos(t)]])


def _dilation(law, target, mu, lam, low, high):
    """s in [low, high] whose state s I scans to `target` (decreasing with low > high)."""
    for _ in range(60):
        s = 0.5 * (low + high)
        if _scan(law, s * np.eye(2)[:, :, None], mu, lam)[0][0] < target:
            low = s
        else:
            high = s
    return s


def test_a_peak_between_directions_does_not_hide_a_larger_scan():
    """A compressed St. Venant-Kirchhoff state whose largest eigenvalue at multiples of 11.25
    degrees exceeds that of the whole degrees by 1e-3, next to a pure dilation whose scan, the
    larger of the two, lies between them."""
    mu, lam = 1.0, 2.0
    F = np.empty((2, 2, 4, 6))
    F[:] = np.array([[0.013754, 0.410202], [-0.664567, -0.174563]])[:, :, None, None]
    target = _scan("svk", F[:, :, 0, :1], mu, lam)[0][0] * (1 + 6e-4)
    F[:, :, 1, 2] = _dilation("svk", target, mu, lam, 0.6, 0.9) * np.eye(2)
    got, want, cond = _audit("svk", F, "f64", mu, lam, 8.0)
    assert abs(want * want * 64.0 / target - 1) < 1e-12
    assert abs(got - want) <= TOL["f64"] * cond * want


@pytest.mark.parametrize("scale", [1e-24, 1e-12, 1.0, 1e12, 1e24])
def test_moduli_of_any_size(scale):
    """The bounds are formed in FP32: their powers of the moduli must not leave its range."""
    mu, lam = scale, 2.0 * scale
    F = np.empty((2, 2, 3, 5))
    B = np.array([[0.2093, -1.2362], [0.73, 0.5282]])
    target = _scan("lognh", B[:, :, None], mu, lam)[0][0]
    F[:] = _dilation("lognh", target * (1 - 1e-3), mu, lam, 1.4, 0.4) * np.eye(2)[:, :, None, None]
    F[:, :, 2, 1] = B
    got, want, cond = _audit("lognh", F, "f64", mu, lam, 8.0 * scale ** 0.5)
    assert abs(want * want * 64.0 * scale / target - 1) < 1e-12
    assert abs(got - want) <= TOL["f64"] * cond * want


@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("amp", [0.02, 0.3, 1.0])
@pytest.mark.parametrize("law", om.ALL_LAWS)
def test_audit_of_prescribed_states(law, amp, storage):
    rng = np.random.default_rng(17)
    ny, nx = 40, 131
    F = np.empty((2, 2, ny, nx))
    for b in range(ny):
        for a in range(nx):
            s = np.exp(rng.uniform(-amp, min(amp, 0.6), 2))
            F[:, :, b, a] = _rotation(rng.uniform(0, 6.3)) @ np.diag(s) @ _rotation(rng.uniform(0, 6.3))
    got, want, cond = _audit(law, F, storage, 1.0, 4.0, 8.0)
    assert abs(got - want) <= TOL[storage] * cond * want
