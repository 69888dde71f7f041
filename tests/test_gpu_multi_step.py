"""Several D2Q9 steps per launch against one step per launch (the tiling asked
for by set_tiling, itself checked against the oracle elsewhere): the same bits,
state and change over the last step, for lattices at and beside the edges of
the tiles, every storage, and step counts beside those of a launch."""
import pytest
import torch

from paper_1901_02716_amd import Batch, Simulation, workloads

pytestmark = pytest.mark.gpu

# (nx, ny, walled axes): one tile, beside it, beside several, wrapped onto itself, large
SIZES = [(3, 3, "xy"), (5, 4, ""), (20, 51, "y"), (63, 40, "xy"), (64, 64, ""), (64, 16, "x"), (65, 17, "xy"),
         (66, 64, ""), (104, 65, "xy"), (105, 33, "y"), (131, 77, "xy"), (300, 210, ""), (513, 300, "x"),
         (1400, 1100, "xy"), (2050, 2000, "")]


def _sim(nx, ny, walls, precision):
    case = workloads.random_field(9, (nx, ny, 1), seed=nx + ny, amp=0.03)
    for ax in walls:
        case.fixed[ax + "lo"] = (1.0, (0.0, 0.0, 0.0))
        case.fixed[ax + "hi"] = (1.003, (0.06, 0.0, 0.0))
    sim = Simulation(9, case.n, case.dx, case.nu, precision=precision, body_force=(0.1, -0.05, 0.0), seed=4)
    sim.set_fields(case.rho, case.u)
    for f, (rb, ub) in case.fixed.items():
        sim.set_bc(f, rb, ub)
    return sim


@pytest.mark.parametrize("precision", ["fp64", "fp32", "hilo", "s16"])
@pytest.mark.parametrize("nx,ny,walls", SIZES)
def test_steps_per_launch_do_not_change_bits(nx, ny, walls, precision):
    print(f"[multi] {nx}x{ny} {walls} {precision}", flush=True)
    a, b = _sim(nx, ny, walls, precision), _sim(nx, ny, walls, precision)
    b.set_tiling(W=1, nzb=1 if ny < 100 else 16, kernel="fast2d")
    for n in (1, 2, 3, 4, 14, 37):
        a.step(n)
        b.step(n)
        assert torch.equal(a.save_state(), b.save_state()), n
        assert a.residual() == b.residual(), n
    a.autotune(reps=1)
    a.step(19)
    b.step(19)
    assert torch.equal(a.save_state(), b.save_state())
    assert a.params()["steps"] == b.params()["steps"] == 80


@pytest.mark.parametrize("precision", ["fp64", "fp32", "s16"])
def test_batch_steps_per_launch_do_not_change_bits(precision):
    sizes = [(20, 30), (64, 64), (65, 17), (131, 77), (300, 10), (3, 3), (200, 200)]

    def make():
        b = Batch([(n, 0.1, 0.05, (0.1, -0.05)) for n in sizes], precision=precision, seed=2)
        for i, (nx, ny) in enumerate(sizes):
            case = workloads.random_field(9, (nx, ny, 1), seed=i, amp=0.03)
            b[i].set_fields(case.rho, case.u)
            if i % 2 or min(nx, ny) < 4:
                for f in ("xlo", "xhi", "ylo", "yhi"):
                    b[i].set_bc(f, 1.0, (0.02 if f == "yhi" else 0.0, 0.0, 0.0))
        return b

    a, b = make(), make()
    b.set_tiling(1, 8)
    b.set_graph(0)
    for n in (1, 2, 5, 33, 34, 70, 3):
        a.step(n)
        b.step(n)
        for i in range(len(sizes)):
            assert torch.equal(a[i].save_state(), b[i].save_state()), (n, i)
            assert a[i].residual() == b[i].residual(), (n, i)
    a.set_graph(6)
    a.step(21)
    b.step(21)
    a.autotune(reps=1)
    a.step(40)
    b.step(40)
    for i in range(len(sizes)):
        assert torch.equal(a[i].save_state(), b[i].save_state()), i


def test_lattices_of_a_batch_stepped_alike_go_on_together():
    """Lattices that were each stepped on their own by the same number of steps
    are in step: the batch takes them further."""
    sizes = [(20, 30), (200, 200), (64, 64)]

    def make():
        b = Batch([(n, 0.1, 0.05, (0.1, -0.05)) for n in sizes], precision="fp32")
        for i, (nx, ny) in enumerate(sizes):
            case = workloads.random_field(9, (nx, ny, 1), seed=i, amp=0.03)
            b[i].set_fields(case.rho, case.u)
        return b

    a, b = make(), make()
    for i in range(len(sizes)):
        a[i].step(16)
    b.step(16)
    a.step(5)
    b.step(5)
    for i in range(len(sizes)):
        assert torch.equal(a[i].save_state(), b[i].save_state())
