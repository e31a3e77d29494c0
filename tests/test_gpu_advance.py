"""lbm_advance (Solver.steps) against as many single lbm_step calls: populations, displacement,
records and fault word bit for bit, over storages, laws, wall layouts, grid shapes from the
smallest to several patches with remainders, and step counts that are no multiple of the
levels of a launch."""
import numpy as np
import pytest
import torch

import lbm_inputs as li

pytestmark = pytest.mark.gpu

LAYOUTS = {
    "periodic": ("periodic",) * 4,
    "all_traction": ("traction",) * 4,
    "mixed": ("velocity", "traction", "traction", "velocity"),
    "x_periodic": ("periodic", "periodic", "traction", "velocity"),
    "y_periodic": ("traction", "velocity", "periodic", "periodic"),
}
DATA = [(1e-4, -2e-4), (3e-4, 1e-4), (-2e-4, 2e-4), (0.0, 1e-4)]


def make(nx, ny, storage, law, walls, fields, seed=5):
    from paper_2605_26677_amd.solver import Solver
    rng = np.random.default_rng(seed)
    mu, lam, body = 0.1, 0.25, (1e-5, -3e-5)
    if fields:
        mu = (0.1 * np.exp(0.2 * rng.standard_normal((ny, nx)))).astype(np.float32)
        lam = (0.25 * np.exp(0.2 * rng.standard_normal((ny, nx)))).astype(np.float32)
        body = (1e-5 * rng.standard_normal((2, ny, nx))).astype(np.float32)
    sv = Solver(nx, ny, c=3.0, omega=1.95, material=law, storage=storage, bc=LAYOUTS[walls], mu=mu, lam=lam,
                body=body, force_unstable=True)
    v0 = 2e-3 * rng.standard_normal((2, ny, nx))
    sv.init(v0, 0.02 * rng.standard_normal((2, ny, nx)), r0=0.5)
    return sv


def edge_fn(walls, nx, ny, device):
    if walls == "periodic":
        return lambda n: None
    L = (ny, ny, nx, nx)

    def at(n):
        out = [(a * (1 + 0.1 * n), b) for a, b in DATA]
        for e in (1, 2):                                 # per-node data on two edges
            k = torch.arange(L[e], dtype=torch.float64, device=device)
            out[e] = torch.stack([out[e][0] + 1e-5 * torch.sin(k + n), out[e][1] + 0 * k])
        return out
    return at


def ramp(n):
    return 0.5 + 0.03 * n


def compare(nx, ny, storage, law, walls, fields, count, n0=3, records=0):
    a, b = (make(nx, ny, storage, law, walls, fields) for _ in range(2))
    at = edge_fn(walls, nx, ny, a.device)
    want = [torch.zeros_like(a.new_record()) for _ in range(count)] if records else [None] * count
    got = [torch.zeros_like(t) if records else None for t in want]
    edges = [at(n0 + i) for i in range(count)]
    for i in range(count):
        a.step(n0 + i, ramp(n0 + i), ramp(n0 + i + 1), edges=edges[i], record=want[i], ustar=not records)
    b.steps(n0, [ramp(n0 + i) for i in range(count + 1)], edges=edges, records=got if records else None,
            ustar=not records, record_planes=records or 6)
    torch.cuda.synchronize()
    assert torch.equal(a.populations(), b.populations())
    if records:
        tiles = lambda t: t.view(ny, a.tiles_per_row, 6, 64).permute(2, 0, 1, 3).reshape(6, ny, -1)[:, :, :nx]
        for w, g in zip(want, got):
            assert torch.equal(tiles(w)[6 - records:], tiles(g)[6 - records:])
    else:
        assert torch.equal(a.displacement(ramp(n0 + count)), b.displacement(ramp(n0 + count)))
    assert a.faults() == b.faults()


@pytest.mark.parametrize("walls", list(LAYOUTS))
@pytest.mark.parametrize("storage", ["f32", "f64", "f16"])
@pytest.mark.parametrize("nx,ny", [(4, 4), (5, 7), (16, 16), (33, 17), (130, 61)])
def test_steps_equal_single_steps(nx, ny, storage, walls):
    compare(nx, ny, storage, "lognh", walls, False, 21)
    compare(nx, ny, storage, "nh", walls, True, 6, n0=30)


@pytest.mark.parametrize("walls", ["periodic", "mixed"])
@pytest.mark.parametrize("law", ["svk", "mr", "yeoh", "gent"])
def test_steps_of_every_law(law, walls):
    for storage in ("f32", "f64"):
        compare(37, 45, storage, law, walls, True, 11)


@pytest.mark.parametrize("walls", ["periodic", "all_traction"])
@pytest.mark.parametrize("storage", ["f32", "f64", "f16"])
@pytest.mark.parametrize("planes", [4, 6])
def test_steps_with_records(storage, walls, planes):
    compare(75, 41, storage, "lognh", walls, True, 10, records=planes)


@pytest.mark.parametrize("count", list(range(1, 18)))
def test_every_step_count(count):
    compare(50, 34, "f32", "lognh", "mixed", False, count, n0=count)
    compare(50, 34, "f64", "lognh", "periodic", True, count, n0=0)


def test_three_node_periodic_grid():
    compare(3, 3, "f32", "lognh", "periodic", True, 9)


def test_steps_from_a_lent_buffer_leave_it_unchanged():
    a = make(70, 40, "f32", "lognh", "mixed", True)
    b = make(70, 40, "f32", "lognh", "mixed", True)
    at = edge_fn("mixed", 70, 40, a.device)
    snap = a.pop[a.s.cur].clone()
    keep = snap.clone()
    b.lend(snap)
    edges = [at(i) for i in range(13)]
    r = [ramp(i) for i in range(14)]
    a.steps(0, r, edges=edges)
    b.steps(0, r, edges=edges)
    torch.cuda.synchronize()
    assert torch.equal(snap, keep)
    assert torch.equal(a.populations(), b.populations())


@pytest.mark.parametrize("walls", ["all_traction", "mixed", "x_periodic", "y_periodic"])
@pytest.mark.parametrize("nx,ny", [(1151, 1103), (256, 4900), (4899, 260)])
def test_large_walled_grids(nx, ny, walls):
    """The inner rectangle in multi-level launches and the patches around it: widths that leave
    4 and more columns beyond the last whole tile, every remainder of the levels."""
    compare(nx, ny, "f32", "lognh", walls, True, 9, n0=11)
    compare(nx, ny, "f16", "svk", walls, False, 6)


@pytest.mark.parametrize("nx", [1152, 1154, 1155, 1156, 1157])
def test_large_walled_grid_widths(nx):
    compare(nx, 1103, "f32", "nh", "mixed", False, 5, n0=13)


@pytest.mark.parametrize("planes", [4, 6])
def test_large_walled_grid_records(planes):
    compare(1151, 1103, "f32", "lognh", "mixed", True, 10, records=planes)
    compare(1151, 1103, "f16", "gent", "x_periodic", True, 5, records=planes)


# walls that are all velocity walls take a kernel of their own
VELOCITY = {
    "x_channel": ("periodic", "periodic", "velocity", "velocity"),
    "y_channel": ("velocity", "velocity", "periodic", "periodic"),
    "all_velocity": ("velocity",) * 4,
}
LAYOUTS.update(VELOCITY)


@pytest.mark.parametrize("walls", list(VELOCITY))
@pytest.mark.parametrize("storage", ["f32", "f64", "f16"])
@pytest.mark.parametrize("nx,ny", [(4, 4), (5, 7), (64, 64), (130, 61), (385, 384)])
def test_steps_between_velocity_walls(nx, ny, storage, walls):
    """The smallest grids, whole patches, remainders, and grids of more patches than compute
    units: levels that end on odd and even steps, corners of two velocity walls, records."""
    compare(nx, ny, storage, "lognh", walls, False, 21)
    compare(nx, ny, storage, "gent", walls, True, 5, n0=30)
    compare(nx, ny, storage, "nh", walls, True, 8, records=4)


@pytest.mark.parametrize("walls", list(VELOCITY))
def test_large_grids_between_velocity_walls(walls):
    compare(1151, 1103, "f32", "lognh", walls, True, 9, n0=11)
