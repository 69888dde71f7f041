"""Forms of the step kernels that only larger lattices reach, against the FP64
oracle or against a form that is itself checked against it."""
import numpy as np
import pytest

import oracle
from conftest import rel_l2, to_problem
from paper_1901_02716_amd import BGK, workloads

pytestmark = pytest.mark.gpu


def _boxed(q, n, walls, seed=3):
    case = workloads.random_field(q, n, seed=seed, amp=0.03)
    for ax in walls:
        case.fixed[ax + "lo"] = (1.0, (0.0, 0.01, 0.0))
        case.fixed[ax + "hi"] = (1.002, (0.02, 0.0, 0.0))
    case.G = (0.1, 0.2 if q == 19 else -0.2, -0.1)
    return case


# Populations past 256 MB, whose stores stream, in rows that end in part of a vector
# (four nodes FP32, two FP64). Tolerances as for the other population tests.
@pytest.mark.parametrize("precision,n,tol", [("fp32", (157, 155, 150), 1e-5), ("fp32", (1030, 60, 60), 1e-5),
                                             ("fp64", (125, 130, 110), 1e-12)])
@pytest.mark.parametrize("walls", ["", "xyz"])
def test_population_rows_past_the_memory_side_cache(precision, n, tol, walls):
    print(f"[bgk] {n} {walls} {precision}", flush=True)
    case = _boxed(19, n, walls)
    sim = BGK(19, n, case.dx, case.nu, precision=precision, body_force=case.G)
    assert 19 * np.prod(n) * (4 if precision == "fp32" else 8) > 256 << 20
    for f, (rb, ub) in case.fixed.items():
        sim.set_bc(f, rb, ub)
    sim.set_fields(case.rho, case.u)
    sim.step(2)
    rho, u = sim.fields()
    orho, ou = oracle.run(to_problem(case), case.rho, case.u, 2)
    assert rel_l2(u, ou) < tol and rel_l2(rho, orho) < tol
