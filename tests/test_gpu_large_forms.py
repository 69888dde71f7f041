"""Forms of the step kernels that only larger lattices reach, against the FP64
oracle or against a form that is itself checked against it."""
import numpy as np
import pytest
import torch

import oracle
from conftest import rel_l2, to_problem
from paper_1901_02716_amd import BGK, Simulation, workloads

pytestmark = pytest.mark.gpu


def _boxed(q, n, walls, seed=3):
    case = workloads.random_field(q, n, seed=seed, amp=0.03)
    for ax in walls:
        case.fixed[ax + "lo"] = (1.0, (0.0, 0.01, 0.0))
        case.fixed[ax + "hi"] = (1.002, (0.02, 0.0, 0.0))
    case.G = (0.1, 0.2 if q == 19 else -0.2, -0.1)
    return case


# The population step's forms: (lattice, nodes, storage, nodes per lane, streaming stores).
# Rows that end in part of a vector and rows that do not, a wavefront's pass and more;
# test_host_sequence.py checks that these lattices take these forms.
POPULATIONS = [
    (9, (129, 17, 1), "fp32", 4, False), (9, (130, 17, 1), "fp32", 4, False),
    (9, (131, 33, 1), "fp32", 4, False), (9, (256, 16, 1), "fp32", 4, False),
    (9, (449, 18, 1), "fp32", 4, False), (9, (515, 20, 1), "fp32", 4, False),
    (9, (512, 17, 1), "fp64", 2, False), (9, (641, 16, 1), "fp64", 2, False), (9, (513, 7, 1), "fp64", 1, True),
    (9, (400, 16, 1), "fp64", 1, False), (9, (263, 54, 1), "fp32", 1, False),
    (19, (129, 66, 67), "fp32", 4, False), (19, (130, 66, 67), "fp32", 4, False),
    (19, (450, 33, 40), "fp32", 4, False), (19, (193, 48, 48), "fp64", 2, False),
    (19, (254, 42, 42), "fp64", 2, False), (19, (20, 260, 380), "fp32", 1, True),
    (19, (157, 155, 150), "fp32", 4, True), (19, (1030, 60, 60), "fp32", 4, True),
    (19, (125, 130, 110), "fp64", 2, True), (19, (128, 110, 80), "fp64", 2, True),
]


# Tolerances as for the other population tests.
@pytest.mark.parametrize("q,n,precision,lanes,streams", POPULATIONS)
@pytest.mark.parametrize("walls", ["", "xyz", "x"])
def test_population_forms(q, n, precision, lanes, streams, walls):
    print(f"[bgk] {n} {walls} {precision}", flush=True)
    case = _boxed(q, n, walls[: 2 if q == 9 else 3])
    sim = BGK(q, n, case.dx, case.nu, precision=precision, body_force=case.G)
    for f, (rb, ub) in case.fixed.items():
        sim.set_bc(f, rb, ub)
    sim.set_fields(case.rho, case.u)
    sim.step(2)
    rho, u = sim.fields()
    orho, ou = oracle.run(to_problem(case), case.rho, case.u, 2)
    tol = 1e-5 if precision == "fp32" else 1e-12
    assert rel_l2(u, ou) < tol and rel_l2(rho, orho) < tol


# (lattice, nodes, copies along each axis, storage): the first lattice takes one node per
# lane, the one made of its copies another form.
COPIES = [
    (19, (64, 16, 16), (4, 4, 4), "fp32"), (19, (43, 16, 16), (3, 5, 5), "fp32"),
    (19, (64, 16, 16), (4, 8, 6), "fp32"), (19, (53, 16, 16), (3, 10, 10), "fp32"),
    (9, (64, 32, 1), (4, 2, 1), "fp32"), (9, (77, 16, 1), (7, 1, 1), "fp32"),
    (19, (50, 16, 16), (4, 4, 4), "fp64"), (19, (65, 16, 16), (3, 4, 4), "fp64"),
    (19, (64, 16, 16), (2, 8, 6), "fp64"), (19, (39, 16, 16), (5, 10, 10), "fp64"),
    (9, (90, 40, 1), (7, 1, 1), "fp64"),
]


@pytest.mark.parametrize("q,n,copies,precision", COPIES)
def test_population_forms_have_the_same_bits(q, n, copies, precision):
    case = workloads.random_field(q, n, seed=11, amp=0.05)
    d = 2 if q == 9 else 3
    rho, u = np.asarray(case.rho).reshape(n[::-1]), np.asarray(case.u).reshape((d,) + n[::-1])
    pops = []
    for c in ((1, 1, 1), copies):
        m = tuple(a * b for a, b in zip(n, c))
        sim = BGK(q, m, 0.1, 0.05, precision=precision, body_force=(0.1, -0.2, 0.05))
        sim.set_fields(np.tile(rho, c[::-1]), np.tile(u, (1,) + c[::-1]))
        sim.step(3)
        state = sim.save_state().view(torch.float32 if precision == "fp32" else torch.float64)
        pops.append(state.reshape(q, -1)[:, : int(np.prod(m))].reshape((q,) + m[::-1]))
    assert torch.equal(pops[0].repeat((1,) + copies[::-1]), pops[1])

# The FP64 D3Q19 march: (nodes, walls, (nodes per lane, output rows of a workgroup, nodes
# beside a segment evaluated, streaming stores)). Odd and even widths, with and without
# padding of the row, a segment that the row ends in or fills; workgroups whose rows do
# not divide the lattice's. test_host_sequence.py checks that they take these forms.
SEGMENTS = [
    ((64, 60, 50), "", (1, 6, 0, 0)), ((42, 40, 198), "xyz", (1, 6, 0, 0)), ((129, 40, 40), "", (1, 6, 1, 0)),
    ((199, 155, 14), "xyz", (1, 6, 1, 0)), ((295, 104, 286), "xyz", (1, 6, 1, 1)),
    ((44, 195, 141), "xyz", (1, 14, 0, 0)),
    ((28, 122, 220), "", (1, 14, 1, 0)), ((130, 129, 131), "xyz", (1, 14, 1, 0)), ((255, 169, 141), "", (1, 14, 1, 0)),
    ((259, 185, 181), "yz", (1, 14, 1, 1)), ((60, 380, 375), "xyz", (1, 14, 0, 1)), ((98, 143, 60), "xy", (2, 6, 0, 0)),
    ((119, 145, 50), "xy", (2, 6, 0, 0)), ((128, 128, 128), "xyz", (2, 6, 0, 0)), ((128, 128, 128), "", (2, 6, 0, 0)),
    ((70, 297, 17), "", (2, 6, 1, 0)), ((96, 96, 96), "", (2, 6, 1, 0)), ((249, 130, 130), "xyz", (2, 6, 1, 0)),
    ((250, 64, 64), "yz", (2, 6, 1, 0)), ((200, 60, 60), "xyz", (2, 6, 1, 0)), ((119, 239, 308), "x", (2, 6, 0, 1)),
    ((106, 266, 315), "xyz", (2, 6, 0, 1)), ((251, 187, 183), "xyz", (2, 6, 1, 1)), ((150, 189, 303), "", (2, 6, 1, 1)),
]


# Tolerance of the other FP64 parity tests (a step rounds about 40 operations on values of
# the size of u). Two steps: the second reads what the first stored, walls included.
@pytest.mark.parametrize("n,walls,form", SEGMENTS)
def test_fp64_march_forms(n, walls, form):
    print(f"[march] {n} {walls} {form}", flush=True)
    case = _boxed(19, n, walls)
    sim = Simulation(19, n, case.dx, case.nu, precision="fp64", body_force=case.G)
    sim.set_fields(case.rho, case.u)
    for f, (rb, ub) in case.fixed.items():
        sim.set_bc(f, rb, ub)
    sim.step(2)
    rho, u = sim.fields()
    orho, ou = oracle.run(to_problem(case), case.rho, case.u, 2)
    assert rel_l2(u, ou) < 1e-12 and rel_l2(rho, orho) < 1e-12
    assert np.abs(u - ou).max() < 4e-12 * np.abs(ou).max()  # no single node stands out either


def _random_state(sim, seed):
    """Fields of the amplitudes of workloads.random_field, made on the device."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    shape = (sim.n[2], sim.n[1], sim.n[0])
    e = sim.params()["e"]
    rho = 1 + 0.01 * torch.randn(shape, generator=g, device="cuda", dtype=torch.float64)
    u = 0.01 * e * torch.randn((sim.d,) + shape, generator=g, device="cuda", dtype=torch.float64)
    sim.set_fields(rho, u)


# Several D2Q9 steps per launch under the default and the tuned plan against one step per
# launch, past 256 MB (streaming stores) and at the benchmark's sizes: the same bits.
@pytest.mark.parametrize("n,walls,precision", [((4096, 4096), "xy", "fp64"), ((4700, 4901), "x", "fp32"),
                                               ((4901, 4700), "", "hilo"), ((6700, 6901), "y", "s16"),
                                               ((1024, 1024), "xy", "fp64"), ((1024, 1024), "xy", "fp32"),
                                               ((512, 512), "", "fp32")])
def test_several_steps_of_large_d2q9_lattices(n, walls, precision):
    print(f"[multi] {n} {walls} {precision}", flush=True)
    a, b = (Simulation(9, n, 1 / (n[1] - 1), 1e-4, precision=precision, seed=6) for _ in range(2))
    _random_state(a, 9)
    for ax in walls:
        for side, v in (("lo", 0.0), ("hi", 0.05)):
            a.set_bc(ax + side, 1.0, (v, 0.0, 0.0))
            b.set_bc(ax + side, 1.0, (v, 0.0, 0.0))
    b.load_state(a.save_state())
    for tuned in (False, True):
        if tuned:
            a.autotune(reps=3)
        a.step(18)
        for _ in range(18):
            b.step(1)
        assert torch.equal(a.save_state(), b.save_state()), tuned
        assert a.residual() == b.residual()


def test_general_d3q19_lattice_whose_grid_needs_two_dimensions():
    """A thin lattice with more workgroups than one grid dimension takes, periodic with a
    period of seven rows: every period has the bits of the lattice of one."""
    n, period = (65, 7 * 1198373, 1), (65, 7, 1)
    small, big = (Simulation(19, m, 0.1, 0.05, precision="fp32", body_force=(0.1, 0.2, -0.1)) for m in (period, n))
    assert 2 * n[1] > 4 << 22  # wavefronts: two segments a row, four to a workgroup, 2^22 workgroups
    _random_state(small, 3)
    cells = 65 * 7

    def planes(sim, state):
        return state.view(torch.float32).view(4, -1)[:, : sim.N]

    s = planes(small, small.save_state())
    start = torch.zeros(big.state_bytes(), dtype=torch.uint8, device="cuda")
    planes(big, start).view(4, -1, cells).copy_(s.view(4, 1, cells).expand(4, n[1] // 7, cells))
    big.load_state(start)
    small.step(3)
    big.step(3)
    s = planes(small, small.save_state())
    got = planes(big, big.save_state(out=start))
    for f in range(4):
        assert bool((got[f].view(-1, cells) == s[f]).all()), f


@pytest.mark.parametrize("n", [(200, 2, 130), (61, 390, 2), (62, 1, 662), (63, 720, 1), (187, 3, 2), (330, 2, 131)])
@pytest.mark.parametrize("walls", ["", "x"])
def test_fp64_rows(n, walls):
    """FP64 lattices with an axis too short for the march in segments: by rows from 40960
    nodes, below with one thread per node. Tolerance as above."""
    case = _boxed(19, n, walls)
    sim = Simulation(19, n, case.dx, case.nu, precision="fp64", body_force=case.G)
    sim.set_fields(case.rho, case.u)
    for f, (rb, ub) in case.fixed.items():
        sim.set_bc(f, rb, ub)
    sim.step(4)
    rho, u = sim.fields()
    orho, ou = oracle.run(to_problem(case), case.rho, case.u, 4)
    assert rel_l2(u, ou) < 1e-12 and rel_l2(rho, orho) < 1e-12


# Split storage keeps a value to 2^-17 of it (7.6e-6); six roundings (the start and five
# steps) and FP32 arithmetic stay under 1e-4.
@pytest.mark.parametrize("n", [(3, 3, 3), (24, 11, 7), (61, 7, 4), (63, 9, 4), (125, 6, 4), (187, 60, 40)])
@pytest.mark.parametrize("walls", ["", "xyz"])
def test_split_storage_rows(n, walls):
    case = _boxed(19, n, walls)
    sim = Simulation(19, n, case.dx, case.nu, precision="hilo", body_force=case.G)
    sim.set_fields(case.rho, case.u)
    for f, (rb, ub) in case.fixed.items():
        sim.set_bc(f, rb, ub)
    sim.set_tiling(kernel="general")
    sim.step(5)
    rho, u = sim.fields()
    orho, ou = oracle.run(to_problem(case), case.rho, case.u, 5)
    assert rel_l2(u, ou) < 1e-4 and rel_l2(rho - 1, orho - 1) < 1e-4
