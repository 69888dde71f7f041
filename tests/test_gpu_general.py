"""The general D3Q19 step against the FP64 oracle at the edges of its tiles:
the FP64 kernel (segments of 64 and 128 nodes, workgroups of 6 and 14 rows, from
40960 nodes; fewer take one thread per node) and that of the other storages
(segments of 62 nodes, chunks of planes).

Tolerances: the bars of the other parity tests, relative L2: FP64 1e-12 (a step
rounds about 40 operations on values of the size of u, 1e-15 per step), FP32 1e-5,
split storage 2e-3 (a few units of its resolution)."""
import numpy as np
import pytest
import torch

import oracle
from conftest import rel_l2, to_problem
from paper_1901_02716_amd import Simulation, _lib, workloads

pytestmark = pytest.mark.gpu

# widths beside one, two and four segments; rows beside a workgroup's; one to many planes
SIZES = [(3, 3, 3), (63, 7, 9), (64, 14, 5), (65, 15, 4), (66, 8, 5), (127, 6, 3), (128, 9, 17), (129, 20, 7),
         (130, 17, 6), (192, 5, 30), (250, 13, 8), (256, 7, 5), (258, 16, 6), (300, 29, 4)]

LARGE = [(3, 120, 115), (63, 30, 23), (64, 29, 23), (65, 31, 22), (66, 28, 23), (127, 20, 17), (128, 27, 13),
         (129, 20, 17), (130, 17, 19), (192, 15, 15), (250, 13, 13), (256, 13, 13), (258, 16, 11), (300, 29, 5)]
ROWS = [(1, 1, 1), (2, 3, 2), (3, 3, 3), (4, 1, 9), (24, 11, 7), (61, 7, 4), (62, 5, 5), (63, 9, 4), (64, 8, 6),
        (65, 5, 9), (124, 5, 3), (125, 6, 4), (126, 7, 3), (127, 4, 4), (187, 60, 40)]


@pytest.mark.parametrize("precision,tol", [("fp32", 1e-5), ("hilo", 2e-3), ("s16", 2e-3)])
@pytest.mark.parametrize("walls", ["", "xyz", "yz", "x"])
@pytest.mark.parametrize("n", ROWS)
def test_rows_at_segment_edges(n, walls, precision, tol):
    if any(n["xyz".index(ax)] < 3 for ax in walls):
        pytest.skip("a bounded axis needs three nodes")
    case = workloads.random_field(19, n, seed=3, amp=0.03)
    for ax in walls:
        case.fixed[ax + "lo"] = (1.0, (0.0, 0.01, 0.0))
        case.fixed[ax + "hi"] = (1.002, (0.02, 0.0, 0.0))
    case.G = (0.1, 0.2, -0.1)
    sim = Simulation(19, n, case.dx, case.nu, precision=precision, body_force=case.G, seed=2)
    sim.set_fields(case.rho, case.u)
    for f, (rb, ub) in case.fixed.items():
        sim.set_bc(f, rb, ub)
    sim.set_tiling(kernel="general")
    sim.step(5)
    rho, u = sim.fields()
    orho, ou = oracle.run(to_problem(case), case.rho, case.u, 5)
    assert rel_l2(u, ou) < tol and rel_l2(rho, orho) < tol


@pytest.mark.parametrize("walls", ["", "xyz", "yz", "x"])
@pytest.mark.parametrize("n", SIZES + LARGE)
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


@pytest.mark.parametrize("precision", ["fp64", "fp32", "hilo", "s16"])
@pytest.mark.parametrize(
    "n", [(3, 5), (2, 3), (64, 64), (1023, 4), (1024, 3), (1025, 7), (1030, 9), (7, 300), (5, 4, 3), (61, 17, 9),
          (100, 9, 8), (250, 6, 5), (210, 205, 200), (209, 205, 201)])
def test_fields_on_the_device_are_those_on_the_host(n, precision):
    """Reading the fields in one launch (pairs of nodes or single ones, arrays past
    the caches or not) gives the bits of reading them a field at a time."""
    lattice = 9 if len(n) == 2 else 19
    sim = Simulation(lattice, n, 0.1, 0.05, precision=precision)
    case = workloads.random_field(lattice, tuple(n) + (1,) * (3 - len(n)), seed=3, amp=0.03)
    sim.set_fields(case.rho, case.u)
    rho, u = sim.fields()
    r, v = sim.fields(on_device=True)
    assert np.array_equal(r.cpu().numpy(), rho) and np.array_equal(v.cpu().numpy(), u)
    if sim.N > 1 << 20:
        return
    # arrays that are not aligned for pairs
    N = rho.size
    flat = torch.empty((sim.d + 1) * N + 3, dtype=torch.float64, device=sim.device)
    r, v = flat[1 : 1 + N], flat[2 + N : 2 + N + sim.d * N]
    _lib.check(sim.lib.maclab_get_fields(sim.h, r.data_ptr(), v.data_ptr(), 1), sim.h)
    assert np.array_equal(r.cpu().numpy(), rho.ravel()) and np.array_equal(v.cpu().numpy(), u.ravel())
