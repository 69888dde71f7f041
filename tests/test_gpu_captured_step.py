"""A call of an even number of steps captured in a caller's HIP graph and
replayed, with eager work and synchronisation between the replays, against the
same calls made one by one: the same bits (FP64, FP32 and split storage; S16 keys
its rounding per step)."""
import pytest
import torch

from paper_1901_02716_amd import Simulation, workloads

pytestmark = pytest.mark.gpu


def _sim(n, walls, precision):
    case = workloads.random_field(9, n + (1,), seed=7, amp=0.03)
    sim = Simulation(9, case.n, case.dx, case.nu, precision=precision, body_force=(0.1, -0.05, 0.0))
    sim.set_fields(case.rho, case.u)
    for ax in walls:
        sim.set_bc(ax + "lo", 1.0, (0.0, 0.0, 0.0))
        sim.set_bc(ax + "hi", 1.0, (0.06, 0.0, 0.0))
    return sim


@pytest.mark.parametrize("precision", ["fp64", "fp32", "hilo"])
@pytest.mark.parametrize("n,walls", [((64, 64), ""), ((131, 77), "xy")])
def test_a_captured_call_of_an_even_number_of_steps_is_replayed(n, walls, precision):
    stream = torch.cuda.Stream()
    for steps in (2, 10, 14, 20):
        print(f"[capture] {n} {walls} {precision} {steps}", flush=True)
        with torch.cuda.stream(stream):
            a, b = _sim(n, walls, precision), _sim(n, walls, precision)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            a.step(steps)
        for _ in range(3):
            with torch.cuda.stream(stream):
                graph.replay()
                b.step(steps)
                same = torch.equal(a.save_state(), b.save_state())
            torch.cuda.synchronize()
            assert same, steps
