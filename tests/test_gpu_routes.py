"""The launches that lbm_advance and lbm_adjoint_advance pick on larger grids, against single
steps bit for bit: double precision between walls (march_kernel's rectangle with 3-tile spans, the
patches around it), the patch plans of large periodic grids, the march with its remainders, and
the adjoint above its patches."""
import pytest

import test_gpu_adjoint_advance as adjoint
from test_gpu_advance import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("walls", ["all_traction", "mixed", "x_periodic", "y_periodic", "x_channel", "all_velocity"])
@pytest.mark.parametrize("nx,ny", [(861, 853), (300, 2603), (2600, 300)])
def test_double_precision_between_walls(nx, ny, walls):
    compare(nx, ny, "f64", "lognh", walls, True, 9, n0=11)
    compare(nx, ny, "f64", "svk", walls, False, 6)


@pytest.mark.parametrize("nx", [896, 897, 898, 899, 900, 901, 960, 1025])
def test_double_precision_widths(nx):
    """0 to 5 columns beyond the last whole tile, and rectangles of every number of tiles mod 3."""
    compare(nx, 859, "f64", "nh", "mixed", False, 7, n0=13)


@pytest.mark.parametrize("law", ["gent", "mr"])
def test_double_precision_invariant_laws(law):
    compare(1261, 1255, "f64", law, "mixed", True, 7)


@pytest.mark.parametrize("count", [2, 3, 4, 5, 6, 7])
def test_double_precision_periodic_march(count):
    compare(801, 790, "f64", "lognh", "periodic", True, count, n0=12)


@pytest.mark.parametrize("nx,ny", [(1001, 777), (720, 731), (2000, 390), (411, 1900), (1023, 1024)])
def test_large_periodic_patches(nx, ny):
    compare(nx, ny, "f32", "lognh", "periodic", True, 8, n0=13)
    compare(nx, ny, "f16", "gent", "periodic", False, 7)


@pytest.mark.parametrize("nx,ny", [(470, 471), (638, 339), (440, 432), (527, 531)])
def test_half_precision_pairs_and_patches(nx, ny):
    compare(nx, ny, "f16", "lognh", "periodic", True, 9, n0=11)


@pytest.mark.parametrize("count", [2, 3, 4, 5, 9])
def test_periodic_march(count):
    compare(1031, 1027, "f32", "svk", "periodic", True, count, n0=12)
    compare(1157, 1151, "f16", "lognh", "periodic", False, count, n0=12)


@pytest.mark.parametrize("planes", [4, 6])
def test_replay_march(planes):
    compare(2049, 2053, "f32", "lognh", "periodic", True, 9, records=planes)


@pytest.mark.parametrize("walls", ["mixed", "x_channel", "y_periodic"])
def test_adjoint_above_its_patches(walls):
    adjoint.compare(1461, 1457, "f32", "lognh", walls, True, 19, 19, 8)
    adjoint.compare(1053, 1051, "f64", "lognh", walls, True, 19, 18, 5)


def test_adjoint_march():
    adjoint.compare(2051, 2049, "f32", "lognh", "periodic", True, 18, 18, 10)
    adjoint.compare(2051, 2049, "f32", "gent", "periodic", True, 18, 17, 8)


@pytest.mark.parametrize("storage,nx,ny", [("f32", 360, 361), ("f32", 396, 410), ("f16", 399, 370), ("f64", 375, 380),
                                           ("f64", 291, 300), ("f64", 128, 900)])
def test_ranged_plans(storage, nx, ny):
    """Periodic grids whose plan, or pairs instead, was read off sweeps."""
    compare(nx, ny, storage, "lognh", "periodic", True, 9, n0=11)
    compare(nx, ny, storage, "yeoh", "periodic", True, 8, records=4)


def test_half_precision_between_velocity_walls():
    compare(381, 390, "f16", "lognh", "all_velocity", True, 7, n0=13)


@pytest.mark.parametrize("storage,law,walls,nx,ny",
                         [("f32", "svk", "periodic", 340, 352), ("f32", "yeoh", "periodic", 361, 350),
                          ("f64", "svk", "periodic", 321, 300), ("f64", "gent", "periodic", 340, 333),
                          ("f64", "yeoh", "periodic", 230, 240), ("f64", "mr", "periodic", 190, 200),
                          ("f32", "mr", "x_channel", 851, 830), ("f64", "yeoh", "all_velocity", 661, 650)])
def test_ranged_adjoint_plans(storage, law, walls, nx, ny):
    adjoint.compare(nx, ny, storage, law, walls, True, 19, 19, 10)
