"""The route of lbm_advance on large grids, read from the levels of its first launch (no GPU): four
where march_kernel takes the grid, two where the pairs are faster, one patch plan on small ones."""
import ctypes

import pytest

from paper_2605_26677_amd import _lib as L

WALLS = {
    "periodic": ("periodic",) * 4,
    "traction": ("traction",) * 4,
    "channel": ("periodic", "periodic", "velocity", "velocity"),
}
LAW_K = {"mr": (0.3, 0.2, 0.0), "yeoh": (0.5, 0.05, 0.01), "gent": (20.0, 0.0, 0.0)}


def levels(nx, ny, storage, law, walls, left=32, records=False):
    p, s = L.lbm_params(), L.lbm_state()
    p.nx, p.ny, p.material, p.storage = nx, ny, L.MATERIAL[law], L.STORAGE[storage]
    for e in range(4):
        p.bc[e] = L.BC[WALLS[walls][e]]
    for i, k in enumerate(LAW_K.get(law, (0.0, 0.0, 0.0))):
        p.law_k[i] = k
    p.dx, p.c, p.omega = 1.0, 10.0, 1.9
    s.ustar = None if records else 1
    rec = ctypes.cast((ctypes.c_void_p * left)(*([1] * left)), ctypes.c_void_p) if records else None
    return L.lib().lbm_advance_levels(ctypes.byref(p), ctypes.byref(s), left, rec)


@pytest.mark.parametrize("storage,law,walls,nx,ny,want", [
    ("f64", "lognh", "periodic", 2048, 2048, 4), ("f64", "lognh", "periodic", 64, 12000, 2),
    ("f64", "lognh", "periodic", 192, 5000, 4), ("f64", "mr", "periodic", 256, 8000, 2),
    ("f64", "mr", "periodic", 1536, 1500, 4), ("f64", "gent", "traction", 1400, 1400, 2),
    ("f64", "lognh", "traction", 1500, 1500, 4), ("f64", "lognh", "traction", 320, 6000, 2),
    ("f16", "gent", "traction", 640, 2500, 2), ("f16", "lognh", "traction", 4096, 4096, 4),
    ("f32", "lognh", "traction", 257, 5000, 4), ("f32", "lognh", "channel", 4500, 300, 4),
    ("f32", "gent", "channel", 2048, 2048, 4), ("f32", "lognh", "traction", 200, 8000, 2),
])
def test_march_or_pairs(storage, law, walls, nx, ny, want):
    assert levels(nx, ny, storage, law, walls) == want
    assert levels(nx, ny, storage, law, walls, left=1) == 1
    # a pair or a march is never followed by a single step where two launches can share the rest
    assert levels(nx, ny, storage, law, walls, left=5) == (3 if want == 4 else 2)


@pytest.mark.parametrize("storage,law,nx,ny,want", [("f32", "lognh", 2048, 2048, 4), ("f16", "gent", 640, 2500, 2),
                                                    ("f64", "lognh", 2048, 2048, 2)])
def test_replay_route(storage, law, nx, ny, want):
    assert levels(nx, ny, storage, law, "traction", records=True) == want


@pytest.mark.parametrize("storage,law,nx,ny,want", [
    ("f16", "lognh", 545, 545, 2), ("f16", "lognh", 800, 800, 3), ("f32", "lognh", 400, 400, 4),
    ("f32", "yeoh", 370, 370, 2), ("f32", "lognh", 900, 900, 3), ("f64", "gent", 500, 500, 3)])
def test_plans_of_periodic_grids(storage, law, nx, ny, want):
    assert levels(nx, ny, storage, law, "periodic") == want
