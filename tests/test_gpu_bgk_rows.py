"""The population step at the widths where a lane's vector of nodes can go
wrong (rows below, at and beside a vector, a wavefront and two of them; walls and
periodic wraps) against the FP64 oracle.

Tolerances as for the other population tests: FP64 1e-12, FP32 1e-5 relative L2."""
import pytest

import oracle
from conftest import rel_l2, to_problem
from paper_1901_02716_amd import BGK, workloads

pytestmark = pytest.mark.gpu

WIDTHS = [3, 31, 63, 64, 65, 127, 128, 129, 130, 131, 254, 256, 257, 300, 515]


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32", 1e-5)])
@pytest.mark.parametrize("q", [9, 19])
@pytest.mark.parametrize("nx", WIDTHS)
def test_rows_of_any_width(nx, q, precision, tol):
    for walls in ("", "xy", "y", "x"):
        n = (nx, 7, 1) if q == 9 else (nx, 5, 6)
        case = workloads.random_field(q, n, seed=nx, amp=0.03)
        for ax in walls:
            case.fixed[ax + "lo"] = (1.0, (0.0, 0.01, 0.0))
            case.fixed[ax + "hi"] = (1.002, (0.02, 0.0, 0.0))
        case.G = (0.1, -0.2, 0.05)
        sim = BGK(q, n, case.dx, case.nu, precision=precision, body_force=case.G)
        for f, (rb, ub) in case.fixed.items():
            sim.set_bc(f, rb, ub)
        sim.set_fields(case.rho, case.u)
        sim.step(4)
        rho, u = sim.fields()
        orho, ou = oracle.run(to_problem(case), case.rho, case.u, 4)
        assert rel_l2(u, ou) < tol and rel_l2(rho, orho) < tol, walls
