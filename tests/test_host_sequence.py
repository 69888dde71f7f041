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


def test_a_batch_goes_on_as_before_after_its_autotuner_failed(tmp_path):
    """An error at any of the autotuner's timings leaves the tiling, the shape of
    several steps and the tables that belong to them as they were."""
    standin.run(tmp_path, """
r = standin.load()
sizes = [(64, 64), (131, 77), (300, 200), (512, 512)]
def launched(b):
    out = []
    for steps in (1, 40, 45):
        rc, log = r.launches(r.lib.maclab_batch_step, b, steps)
        assert rc == 0
        out += [e[:3] for e in log]
    return out
for before in (None, 0, "tiling"):  # the first call that needs tables; after steps; after a tiling was set
    def make():
        b = r.batch(sizes, r.m.FP32)
        assert r.lib.maclab_batch_set_graph(b, 0) == 0
        if before == 0:
            assert r.lib.maclab_batch_step(b, 3) == 0
        if before == "tiling":
            assert r.lib.maclab_batch_set_tiling(b, 1, 16) == 0
        return b
    want = launched(make())
    failed = 0
    for at in range(40):
        b = make()
        r.fail_event.value = at
        rc = r.lib.maclab_batch_autotune(b, 1, None)
        r.fail_event.value = -1
        if rc == 0:
            break
        failed += 1
        assert launched(b) == want, (before, at)
    assert failed == 8  # two shapes of several steps, six heights of a band
""")


def test_a_lattice_of_a_batch_is_tuned_for_the_steps_it_takes(tmp_path):
    """Stepped on its own it goes step by step, so its autotuner times and reports
    single steps; so does a lattice with derived faces."""
    standin.run(tmp_path, """
import ctypes
r = standin.load()
u = (ctypes.c_double * 3)()
view = ctypes.c_void_p(r.lib.maclab_batch_lattice(r.batch([(300, 200), (64, 64)], r.m.FP32), 0))
derived = r.handle(9, (300, 200), r.m.FP32, "xy")
assert r.lib.maclab_set_bc(derived, r.m.YHI, r.m.RHO_NEUMANN, 1.0, u) == 0
for h, single in ((view, True), (derived, True), (r.handle(9, (300, 200), r.m.FP32, "xy"), False)):
    best = ctypes.c_double()
    rc, log = r.launches(r.lib.maclab_autotune, h, 2, ctypes.byref(best))
    assert rc == 0 and single == (not any("multi" in e[0] for e in log))
    assert single == (best.value == 1.0), best.value  # every timed launch takes 1 ms
    rc, log = r.launches(r.lib.maclab_step, h, 20)
    assert rc == 0 and single == (not any("multi" in e[0] for e in log))
""")


def test_the_default_d3q19_tiling_loads_two_planes_ahead_only_where_that_was_faster(tmp_path):
    standin.run(tmp_path, """
import ctypes
r = standin.load()
out = (ctypes.c_int * 5)()
planes = {(n, p): 2 for n in (64, 128, 256) for p in (r.m.FP32, r.m.HILO, r.m.S16)}
planes[128, r.m.S16] = planes[256, r.m.FP32] = 1  # measured slower with two
planes.update({(251, p): 1 for p in (r.m.FP32, r.m.HILO, r.m.S16)})  # padded rows: not built
for (nx, p), want in planes.items():
    for n in ((nx, 128, 128), (nx, 30, 20)):
        h = r.handle(19, n, p, "xyz")
        assert r.lib.maclab_get_tiling(h, out) == 0 and out[0] == 1 and out[4] == want, (n, p, list(out))
""")


def test_a_step_costs_the_host_about_the_same_on_every_lattice(tmp_path):
    """The shapes are ranked once for a lattice and its faces, not on every call: host
    time of single-step calls and of one call of many steps, the smallest of ten
    repeats, against a small cube's (0.5 us a step; ranking the chunks of the thinnest
    lattice takes 18 us)."""
    standin.run(tmp_path, """
import time
r = standin.load()
def cost(h, calls, steps):
    best = 1e9
    for _ in range(10):
        r._count.value = 0
        t = time.perf_counter()
        for _ in range(calls):
            r.lib.maclab_step(h, steps)
        best = min(best, (time.perf_counter() - t) / (calls * steps))
    return best
small = r.handle(19, (16, 17, 18), r.m.FP64)
many, single = cost(small, 1, 300), cost(small, 300, 1)
for n, p in (((3, 3, 3000), r.m.FP32), ((8, 8, 4096), r.m.S16), ((3, 3, 100000), r.m.HILO), ((48, 40, 36), r.m.FP64)):
    h = r.handle(19, n, p)
    assert cost(h, 1, 300) < 5 * many and cost(h, 300, 1) < 5 * single, n
""")
    # (a handle whose faces change gets the shapes of the new faces)
    standin.run(tmp_path, """
r = standin.load()
for q, n, p, walls in ((19, (300, 67, 93), r.m.FP32, "yz"), (19, (130, 129, 131), r.m.FP64, "xyz"),
                       (9, (300, 200), r.m.FP64, "xy"), (9, (65, 130), r.m.FP32, "y"), (19, (64, 30, 20), r.m.S16, "xz")):
    a, b = r.handle(q, n, p), r.handle(q, n, p, walls)
    assert r.lib.maclab_step(a, 5) == 0
    r.walls(a, walls)
    la, lb = r.launches(r.lib.maclab_step, a, 9), r.launches(r.lib.maclab_step, b, 9)
    assert [e[:3] for e in la[1]] == [e[:3] for e in lb[1]], (n, walls)
""")


def test_population_forms(tmp_path):
    """Nodes per lane and store policy: the lattices of the GPU test of these forms, and
    the sizes where the policy was measured to change sides."""
    from test_gpu_large_forms import POPULATIONS

    more = [(19, (128, 128, 128), "fp32", 4, True), (19, (104, 104, 104), "fp64", 2, True), (19, (64, 64, 64), "fp32", 1, False),
            (19, (129, 16, 16), "fp32", 1, False), (19, (129, 59, 3), "fp64", 1, False), (19, (400, 64, 70), "fp32", 4, False),
            (19, (160, 90, 90), "fp64", 1, True), (19, (256, 256, 256), "fp32", 4, True), (9, (2048, 2048, 1), "fp32", 4, False),
            (9, (1024, 1024, 1), "fp64", 2, False), (9, (140, 4, 1), "fp64", 1, True)]
    standin.run(tmp_path, f"""
import ctypes
r = standin.load()
lib, m = r.lib, r.m
for q, n, p, lanes, streams in {POPULATIONS + more}:
    c = r.config(q, n, m.FP64 if p == "fp64" else m.FP32)
    c.workspace, c.workspace_bytes = standin.WORKSPACE, lib.maclab_bgk_workspace_bytes(ctypes.byref(c))
    h = ctypes.c_void_p()
    assert lib.maclab_bgk_init(ctypes.byref(c), ctypes.byref(h)) == 0
    rc, log = r.launches(lib.maclab_bgk_step, h, 1)
    assert rc == 0 and len(log) == 1
    tail = lanes > 1 and n[0] % lanes != 0
    want = f"bgk_step_kernelILi{{q}}E{{'d' if p == 'fp64' else 'f'}}Li{{lanes}}ELb{{int(tail)}}ELb{{int(streams)}}E"
    assert want in log[0][0], (q, n, p, want, log[0][0])
""")


def test_fp64_d3q19_marches_where_that_was_faster(tmp_path):
    standin.run(tmp_path, """
r = standin.load()
nodes, march = "step_generic_kernel", "step_d3q19_seg"
for n, walls, want in (((40, 32, 32), "", nodes), ((63, 32, 32), "xyz", nodes), ((40, 33, 32), "", march), ((130, 8, 40), "xyz", nodes),
                       ((130, 8, 50), "", march), ((80, 3, 800), "xyz", nodes), ((80, 3, 800), "", march), ((300, 3, 800), "xyz", nodes),
                       ((48, 40, 36), "xyz", march), ((12, 100, 30), "", nodes), ((251, 251, 251), "xyz", march),
                       ((200, 2, 130), "", "step_d3q19_rows"), ((100, 2, 130), "", nodes)):
    h = r.handle(19, n, r.m.FP64, walls)
    rc, log = r.launches(r.lib.maclab_step, h, 1)
    assert rc == 0 and want in log[0][0], (n, walls, log)
""")


def test_fp64_march_forms(tmp_path):
    """The lattices of the GPU test of these forms."""
    from test_gpu_large_forms import SEGMENTS

    standin.run(tmp_path, f"""
import re
r = standin.load()
for n, walls, (kx, w, halo, streams) in {SEGMENTS}:
    rc, log = r.launches(r.lib.maclab_step, r.handle(19, n, r.m.FP64, walls), 1)
    got = re.search("step_d3q19_segI.*?Li(\\d+)ELi(\\d+)ELb(\\d)ELi(\\d+)E", log[0][0])
    policy = 2 if streams else 16
    assert rc == 0 and got and tuple(map(int, got.groups())) == (kx, w, halo, policy), (n, walls, log[0][0])
""")


def test_a_batch_of_millions_of_lattices_stays_within_a_grid(tmp_path):
    """One tile of a thousand threads for each of 4.2 million lattices would be more than
    2^32 work-items; single steps take 64 for each."""
    standin.run(tmp_path, """
import ctypes
r = standin.load()
count = 4200000
c = r.config(9, (3, 3), r.m.FP32)
cfgs = (r.m.Config * count).from_buffer_copy(bytes(c) * count)
b = ctypes.c_void_p()
need = r.lib.maclab_batch_workspace_bytes(cfgs, count)
assert r.lib.maclab_batch_init(cfgs, count, standin.WORKSPACE, need, ctypes.byref(b)) == 0
assert r.lib.maclab_batch_step(b, 5) == 0, r.lib.maclab_batch_last_error(b)
""")


def test_a_batch_reports_that_host_memory_ran_out(tmp_path):
    """Tables that do not fit the process's memory are an error code, not an exception
    across the ABI, and the batch goes on once they fit."""
    standin.run(tmp_path, """
import resource
r = standin.load()
lib = r.lib
sizes = [((1 << 19) + i, 1000) for i in range(6)]  # tables of 40 MB
def limit(mb):
    used = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
    resource.setrlimit(resource.RLIMIT_AS, (resource.RLIM_INFINITY if mb is None else used + (mb << 20), resource.RLIM_INFINITY))
want = None
calls = (lambda b: lib.maclab_batch_step(b, 40), lambda b: lib.maclab_batch_get_tiling(b, (r.m.ctypes.c_int * 3)()),
         lambda b: lib.maclab_batch_set_tiling(b, 1, 4), lambda b: lib.maclab_batch_autotune(b, 1, None))
for call in calls:
    for stepped in (False, True):
        b, fresh = r.batch(sizes, r.m.FP32), r.batch(sizes, r.m.FP32)
        for h in (b, fresh):
            assert lib.maclab_batch_set_graph(h, 0) == 0
            if stepped:
                assert lib.maclab_batch_step(h, 1) == 0
        limit(3)
        rc = call(b)
        limit(None)
        assert rc == r.m.EINVAL or (stepped and rc == 0), rc
        assert rc == 0 or b"out of host memory" in lib.maclab_batch_last_error(b)
        if rc:
            assert r.launches(lib.maclab_batch_step, b, 5)[1][0][:3] == r.launches(lib.maclab_batch_step, fresh, 5)[1][0][:3]
        lib.maclab_batch_destroy(b)
        lib.maclab_batch_destroy(fresh)
""")


def test_a_batch_call_takes_few_launches_beside_its_graphs(tmp_path):
    """The steps a batch makes outside its graphs, and the buffer the call ends in."""
    standin.run(tmp_path, """
r = standin.load()
b = r.batch([(300 + i, 400) for i in range(200)], r.m.FP32)
h = r.m.ctypes.c_void_p(r.lib.maclab_batch_lattice(b, 0))
assert r.lib.maclab_batch_step(b, 40) == 0  # (the graph is captured)
at = r.buffer(h)
for steps in list(range(1, 130)) + [200, 1001]:
    rc, log = r.launches(r.lib.maclab_batch_step, b, steps)
    now = r.buffer(h)
    assert rc == 0 and (now == at) == (steps % 2 == 0) and "multi" not in log[-1][0], steps
    assert len(log) <= 16, (steps, len(log))  # two graphs of steps at most
    at = now
""")
