"""The FP64 traction Newton solve against the oracle's, which tries every step length at every
iteration, while the library's tries the full step alone once |r| is at the rounding floor of the
plain F (16 eps (|T| + 2 mu)): one step of a block with loaded traction walls on all sides, over
ratios lam / mu and loads, the wall lines element by element.

Bound.  F^b of either solve is within 4e-15 of the 64-bit solution (evaluated in extended precision
over these ranges, the same for both rules), a wall node's F sums four populations of that and 24
roundings of values below 1 on either side: 5e-14 on F.  v carries the rounding of P / c, of the
size eps sqrt(lam + 2 mu) with c proportional to that root: 5e-14 (1 + sqrt(lam + 2 mu))."""
import numpy as np
import pytest

import lbm_inputs as li
from gpu_cases import Case, run_library, run_oracle, wall_lines

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("load", [1e-6, 1e-3, 3e-2])
@pytest.mark.parametrize("ratio", [0.1, 1.0, 10.0, 100.0, 1000.0])
@pytest.mark.parametrize("law", ["lognh", "nh", "svk", "mr"])
def test_wall_state_after_one_step(law, ratio, load):
    nx, ny, mu = 36, 28, 0.1
    lam = ratio * mu
    cp = np.sqrt(lam + 2 * mu)
    T = load * mu
    u0 = np.stack([li.gaussian_random_field(nx, ny, 21, 0.3 * load), li.gaussian_random_field(nx, ny, 22, 0.3 * load)])
    v0 = np.stack([li.gaussian_random_field(nx, ny, 23, 1e-2 * load), li.gaussian_random_field(nx, ny, 24, 1e-2 * load)])
    case = Case(f"{law}_{ratio}_{load}", nx, ny, 8.0 * cp, 1.9, 1, law=law, mu=mu, lam=lam, kinds=("traction",) * 4,
                data=[(T, -0.5 * T), (0.3 * T, T), (-0.7 * T, 0.2 * T), (0.1 * T, 0.6 * T)], v0=v0, u0=u0,
                force_unstable=True)
    Uo, _, _ = run_oracle(case)
    sv, Ug, _ = run_library(case, "f64")
    if sv.faults():
        # the library's default of 8 updates does not reach the solution of stiff svk at the largest
        # load and says so; with the oracle's 50 it does
        assert sv.faults() == 4
        sv.p.newton_max_iter = 50
        sv.init(case.v0, case.u0)
        sv.step(0, edges=list(case.data))
        Ug = sv.moments().cpu().numpy()
    assert sv.faults() == 0
    Uo[2] -= 1.0
    Uo[5] -= 1.0
    err = np.abs(wall_lines(Ug, case.kinds) - wall_lines(Uo, case.kinds))
    assert err[2:6].max() <= 5e-14
    assert err[0:2].max() <= 5e-14 * (1 + cp)
