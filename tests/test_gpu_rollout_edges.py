"""Rollouts whose edges function refills what it returns: the displacement and the gradients are
bit for bit those with data of their own for every step, over spans of one and of several calls
of the library, forward, replay and adjoint."""
import numpy as np
import pytest
import torch

import lbm_inputs as li

pytestmark = pytest.mark.gpu

NX, NY = 40, 24
BC = ("velocity", "traction", "traction", "traction")


def _load(n, device):
    k = torch.arange(NX, dtype=torch.float64, device=device)
    return torch.stack([1e-5 * torch.sin(0.3 * k + 0.2 * n), -2e-5 * torch.cos(0.1 * k - 0.3 * n)])


def _run(edges, steps, every, levels=(), revolve=0):
    from paper_2605_26677_amd.rollout import RolloutConfig, rollout
    dev = torch.device("cuda")
    rng = np.random.default_rng(2)
    mu = torch.tensor(li.lognormal_field(NX, NY, 11, 0.1, 0.2, 4.0), device=dev)
    lam = torch.tensor(li.lognormal_field(NX, NY, 12, 0.3, 0.2, 4.0), device=dev)
    v0 = torch.tensor(1e-3 * rng.standard_normal((2, NY, NX)), device=dev)
    leaves = [t.double().requires_grad_(True) for t in (mu, lam, torch.zeros_like(v0), v0)]
    cfg = RolloutConfig(nx=NX, ny=NY, c=10.0, omega=1.95, nsteps=steps, probes=torch.arange(0, NX * NY, 37), bc=BC,
                        edges=edges, checkpoint_every=every, levels=list(levels), revolve=revolve, force_unstable=True)
    u = rollout(*leaves, cfg)
    (u * u).sum().backward()
    return [u.detach()] + [t.grad for t in leaves]


@pytest.mark.parametrize("steps,every,levels,revolve", [(30, 12, (), 0), (230, 230, (), 0), (60, 20, (20, 5), 0),
                                                        (60, 10, (), 3)])
@pytest.mark.parametrize("how", ["tensor", "list"])
def test_refilled_wall_data(how, steps, every, levels, revolve):
    dev = torch.device("cuda")
    buf, data = torch.zeros((2, NX), dtype=torch.float64, device=dev), [(0.0, 0.0)] * 4

    def own(n):
        return [(0.0, 0.0), (1e-5 * n, 0.0), (0.0, 0.0), _load(n, dev) if how == "tensor" else (0.0, -1e-5 * n)]

    def refilled(n):
        data[1] = (1e-5 * n, 0.0)
        data[3] = buf.copy_(_load(n, dev)) if how == "tensor" else (0.0, -1e-5 * n)
        return data
    for a, b in zip(_run(own, steps, every, levels, revolve), _run(refilled, steps, every, levels, revolve)):
        assert torch.equal(a, b)
