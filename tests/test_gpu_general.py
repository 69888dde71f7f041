"""The D3Q19 step at the edges of the tiles of its FP64 kernel (segments of 64
and 128 nodes, workgroups of 6 and 14 rows) against the FP64 oracle.

Tolerance: the FP64 bar of the other parity tests, 1e-12 relative L2 (a step
rounds about 40 operations on values of the size of u, 1e-15 per step)."""
import pytest

import oracle
from conftest import rel_l2, to_problem
from paper_1901_02716_amd import Simulation, workloads

pytestmark = pytest.mark.gpu

# widths beside one, two and four segments; rows beside a workgroup's; one to many planes
SIZES = [(3, 3, 3), (63, 7, 9), (64, 14, 5), (65, 15, 4), (66, 8, 5), (127, 6, 3), (128, 9, 17), (129, 20, 7),
         (130, 17, 6), (192, 5, 30), (250, 13, 8), (256, 7, 5), (258, 16, 6), (300, 29, 4)]


@pytest.mark.parametrize("walls", ["", "xyz", "yz", "x"])
@pytest.mark.parametrize("n", SIZES)
def test_fp64_step_at_tile_edges(n, walls):
    case = workloads.random_field(19, n, seed=3, amp=0.03)
    for ax in walls:
        case.fixed[ax + "lo"] = (1.0, (0.0, 0.01, 0.0))
        case.fixed[ax + "hi"] = (1.002, (0.02, 0.0, 0.0))
    case.G = (0.1, 0.2, -0.1)
    sim = Simulation(19, n, case.dx, case.nu, precision="fp64", body_force=case.G)
    sim.set_fields(case.rho, case.u)
    for f, (rb, ub) in case.fixed.items():
        sim.set_bc(f, rb, ub)
    s0 = sim.save_state()
    sim.step(5)
    rho, u = sim.fields()
    orho, ou = oracle.run(to_problem(case), case.rho, case.u, 5)
    assert rel_l2(u, ou) < 1e-12 and rel_l2(rho, orho) < 1e-12
    # faces changed after the first step: the tiling follows them
    if walls == "":
        sim.load_state(s0)
        case.fixed = {"ylo": (1.0, (0.0, 0.0, 0.0)), "yhi": (1.0, (0.03, 0.0, 0.0))}
        for f, (rb, ub) in case.fixed.items():
            sim.set_bc(f, rb, ub)
        sim.step(3)
        rho, u = sim.fields()
        orho, ou = oracle.run(to_problem(case), case.rho, case.u, 3)
        assert rel_l2(u, ou) < 1e-12 and rel_l2(rho, orho) < 1e-12
