"""What the library enqueues, checked without a GPU: launches, their order and
their buffers, over a stand-in HIP runtime (standin.py)."""
import standin


def test_an_even_number_of_steps_ends_in_the_buffer_it_began_in(tmp_path):
    """The two buffers alternate with the steps, however many a launch takes, so
    that a caller's captured call of an even number of steps can be replayed."""
    standin.run(tmp_path, """
r = standin.load()
for precision in range(4):
    for n, walls in (((20, 51), "y"), ((64, 64), ""), ((300, 200), "xy"), ((1024, 1024), "xy"), ((2048, 2048), "")):
        h = r.handle(9, n, precision, walls)
        at = r.buffer(h)
        several = 0
        for steps in list(range(1, 60)) + [100, 199, 200, 1000]:
            rc, log = r.launches(r.lib.maclab_step, h, steps)
            assert rc == 0 and "multi" not in log[-1][0], "the last step goes alone"
            several += len(log) < steps
            assert all(a[3] == b[3][::-1] for a, b in zip(log, log[1:])), "each launch reads what the last one wrote"
            now = r.buffer(h)
            assert (now == at) == (steps % 2 == 0), (n, precision, steps)
            at = now
        assert several > 50
    b = r.batch([(64, 64), (200, 131)], precision)
    assert r.lib.maclab_batch_set_graph(b, 0) == 0
    h = r.m.ctypes.c_void_p(r.lib.maclab_batch_lattice(b, 0))
    at = r.buffer(h)
    for steps in range(1, 60):
        assert r.lib.maclab_batch_step(b, steps) == 0
        now = r.buffer(h)
        assert (now == at) == (steps % 2 == 0), (precision, steps)
        at = now
""")
