"""Several reverse steps per launch against one per launch (the reverse tiling
asked for by set_adjoint_tiling, itself checked against the oracle elsewhere), at
and beside the edges of the tiles.

The velocity gradient has the same bits. The force gradient sums the same FP64
terms in another order. Lanes and slots are summed in pairs, and a slot's chain is a
few thousand additions at most (rows of a tile times steps): its rounding is under
1e4 x 2^-53, so 1e-12 of the sum of the terms' sizes covers every size here."""
import numpy as np
import pytest
import torch

from paper_1901_02716_amd import Simulation, rollout, workloads

pytestmark = pytest.mark.gpu

SIZES = [(3, 3, "xy"), (5, 4, ""), (20, 51, "y"), (64, 64, ""), (64, 16, "x"), (65, 17, "xy"), (105, 33, "y"),
         (131, 77, "xy"), (300, 210, ""), (900, 700, "xy")]


def _grad(nx, ny, walls, precision, steps, single, K=None):
    case = workloads.random_field(9, (nx, ny, 1), seed=nx + ny, amp=0.03)
    for ax in walls:
        case.fixed[ax + "lo"] = (1.0, (0.0, 0.0, 0.0))
        case.fixed[ax + "hi"] = (1.003, (0.06, 0.0, 0.0))
    sim = Simulation(9, case.n, case.dx, case.nu, precision=precision, seed=4)
    for f, (rb, ub) in case.fixed.items():
        sim.set_bc(f, rb, ub)
    if single:
        sim.set_tiling(W=1, nzb=1, kernel="fast2d")
        sim.set_adjoint_tiling("fast2d", 1, 1)
    u0 = torch.tensor(case.u, dtype=torch.float64, device=sim.device, requires_grad=True)
    G = torch.tensor([0.1, -0.05, 0.0], dtype=torch.float64, requires_grad=True)
    tgt = torch.tensor(workloads.random_field(9, (nx, ny, 1), seed=5).u, device=sim.device) + 0.02
    uT = rollout(sim, case.rho, u0, G, steps, checkpoint_every=K)
    ((uT - tgt) ** 2).sum().backward()
    return uT.detach(), u0.grad, G.grad.numpy()


@pytest.mark.parametrize("precision", ["fp64", "fp32", "hilo", "s16"])
@pytest.mark.parametrize("nx,ny,walls", SIZES)
def test_reverse_steps_per_launch(nx, ny, walls, precision):
    print(f"[reverse] {nx}x{ny} {walls} {precision}", flush=True)
    for steps in (1, 2, 17):
        a, b = (_grad(nx, ny, walls, precision, steps, single) for single in (False, True))
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]), steps
        scale = np.abs(b[2]).max() + 1e-3 * np.abs(a[1].cpu().numpy()).sum()
        assert np.all(np.abs(a[2] - b[2]) <= 1e-12 * scale), steps


def test_force_gradient_does_not_depend_on_the_checkpoints():
    ref = _grad(131, 77, "xy", "fp32", 40, False)
    for K in (1, 2, 7, 40):
        got = _grad(131, 77, "xy", "fp32", 40, False, K)
        assert torch.equal(got[1], ref[1]) and np.array_equal(got[2], ref[2]), K
