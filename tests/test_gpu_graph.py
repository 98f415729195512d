"""Graph mode (``bd_set_graph_mode``): each step replayed from captured HIP
graphs must give exactly the results of launching the same kernels one by one
-- positions, angles, the triangulation and every counter -- including steps
whose round budget runs out and are finished by the host, neighbour-list
rebuilds, batches, and an adjoint pass whose replays run launch by launch."""
import numpy as np
import pytest

from paper_1703_02484_amd import binding, synth
from tests._checks import tri_set
from tests.conftest import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _same(a, b):
    xa, ta, sa, sta = a.state()
    xb, tb, sb, stb = b.state()
    assert np.array_equal(xa, xb) and np.array_equal(ta, tb) and sa == sb
    # every counter but host_continued: graph mode holds the round budgets for a
    # whole queued batch, so its steps may hand over to the host where launch
    # by launch (budgets adapted after every step) they did not
    sta.pop("host_continued")
    stb.pop("host_continued")
    assert sta == stb
    assert tri_set(a.triangles()) == tri_set(b.triangles())


def _pair(make):
    a, b = make(), make()
    b.set_graph_mode(True)
    return a, b


@pytest.mark.parametrize("chunk", [1, 5])
def test_graph_equals_eager_c2_reduced(chunk):
    w = synth.make("C2", n=3000)
    a, b = _pair(lambda: binding.Sim.from_workload(w))
    for _ in range(20 // chunk):
        a.step(chunk)
        b.step(chunk)
    _same(a, b)


def test_graph_equals_eager_with_halts_and_continuations():
    # dense box and strong noise: budgets run out, the host finishes steps,
    # budgets adapt (several captured settings)
    n = 600
    L = synth.box_side(n, 0.5)
    xy = synth.rsa(n, L, 1.0, seed=8)
    mk = lambda: binding.Sim(xy, np.ones(n), np.zeros(n, np.int32), None, np.array([[0.0]]), L=L, D=1.0,
                             dt=2e-2, seed=2)
    a, b = _pair(mk)
    for _ in range(12):
        a.step(1)
        b.step(1)
        _same(a, b)
    assert b.state()[3]["overlap_rounds_max"] >= 3


def test_graph_equals_eager_verlet():
    w = synth.make("C3", n=6000)
    a, b = _pair(lambda: binding.Sim.from_workload(w))
    a.step(40)
    b.step(40)
    _same(a, b)
    assert b.state()[3]["verlet_rebuilds"] >= 2


def test_graph_rebuilds_lists_inside_queued_steps_and_grows_them():
    # self-propelled disks pile up against a wall: the lists are rebuilt inside
    # queued steps, and after ~40 steps a disk has more neighbours within
    # cutoff + skin than the initial capacity (32), so one queued step stops
    # before its force, the host grows the lists and runs it again
    from scipy.spatial import cKDTree

    n = 400
    L = synth.box_side(n, 0.4)
    xy = synth.rsa(n, L, 1.0, seed=3)
    mk = lambda: binding.Sim(xy, np.ones(n), np.zeros(n, np.int32), np.full(n, np.pi), np.array([[0.0]]), L=L,
                             D=0.1, dt=1e-2, seed=1, kind="power", q=2.0, cutoff=6.0, skin=0.5, v0=20.0, Dr=0.0)
    a, b = _pair(mk)
    for _ in range(6):
        a.step(10)
        b.step(10)
        _same(a, b)
    t = cKDTree(b.state()[0])
    assert max(len(v) - 1 for v in t.query_ball_point(b.state()[0], 6.5)) > 32
    assert b.state()[3]["verlet_rebuilds"] >= 30


def test_graph_equals_eager_batch():
    ws = synth.make_batch(4, seed=3, lo=200, hi=1500)
    a, b = _pair(lambda: binding.Sim.from_workloads(ws))
    a.step(15)
    b.step(15)
    _same(a, b)


def test_graph_forward_gives_same_gradients():
    w = synth.make("C5", n=700)
    lamT = np.random.default_rng(2).normal(size=(w.n, 2))
    out = []
    for graph in (False, True):
        g = binding.Sim.from_workload(w)
        g.set_graph_mode(graph)
        g.adjoint_begin(9, 4)
        out.append((g.state()[0], *g.adjoint_backward(lamT)))
    for u, v in zip(out[0], out[1]):
        assert np.array_equal(u, v)


def test_switching_modes_midway():
    # launch-by-launch steps, then graph batches, then launch-by-launch again, in a
    # dense box where steps halt and the host finishes them: identical to all-eager
    n = 600
    L = synth.box_side(n, 0.5)
    xy = synth.rsa(n, L, 1.0, seed=9)
    mk = lambda: binding.Sim(xy, np.ones(n), np.zeros(n, np.int32), None, np.array([[0.0]]), L=L, D=1.0,
                             dt=2e-2, seed=4)
    a, b = mk(), mk()
    a.step(5)
    b.step(5)
    b.set_graph_mode(True)
    a.step(10)
    b.step(10)
    _same(a, b)
    b.set_graph_mode(False)
    a.step(3)
    b.step(3)
    _same(a, b)


@pytest.mark.parametrize("graph", [False, True])
def test_tail_mode_with_more_rounds_than_one_workgroup_takes(graph):
    # contact factor 1/2: ~20 overlap rounds per step, so the round budget
    # outgrows what one workgroup runs and the step falls back to launches per
    # phase while the repair after the move still runs in one workgroup
    w = synth.make("C5", n=2048)
    a, b, c = binding.Sim.from_workload(w), binding.Sim.from_workload(w), binding.Sim.from_workload(w)
    a.set_tail_mode(0)
    b.set_tail_mode(1)
    c.set_tail_mode(2)
    for h in (a, b, c):
        h.set_graph_mode(graph)
    for _ in range(4):
        for h in (a, b, c):
            h.step(2)
        _same(a, b)
        _same(a, c)
    assert b.state()[3]["overlap_rounds_max"] > 8


@pytest.mark.parametrize("graph", [False, True])
def test_tail_in_one_workgroup_equals_launch_per_phase(graph):
    # overlap rounds after the first detection run by one workgroup or launched
    # phase by phase: same results, including steps that halt and are finished
    # by the host
    n = 600
    L = synth.box_side(n, 0.5)
    xy = synth.rsa(n, L, 1.0, seed=12)
    mk = lambda: binding.Sim(xy, np.ones(n), np.zeros(n, np.int32), None, np.array([[0.0]]), L=L, D=1.0,
                             dt=2e-2, seed=6)
    a, b, c = mk(), mk(), mk()
    a.set_tail_mode(0)
    b.set_tail_mode(1)
    c.set_tail_mode(2)
    for h in (a, b, c):
        h.set_graph_mode(graph)
    for _ in range(10):
        for h in (a, b, c):
            h.step(1)
        _same(a, b)
        _same(a, c)
    assert b.state()[3]["overlap_rounds_max"] >= 3
    w = synth.make("C2", n=3000)
    a, b, c = binding.Sim.from_workload(w), binding.Sim.from_workload(w), binding.Sim.from_workload(w)
    a.set_tail_mode(0)
    b.set_tail_mode(1)
    c.set_tail_mode(2)
    for h in (a, b, c):
        h.set_graph_mode(graph)
        h.step(25)
    _same(a, b)
    _same(a, c)


@pytest.mark.parametrize("name,over", [("C1", {}), ("C2", {}), ("C3", {}), ("C3", {"overlap": "verlet"})])
def test_graph_forms_bitwise_equal_eager(name, over):
    """The captured forms of a step -- one step, several steps in one graph (captured once the budgets have held),
    and a step cut around its timed force -- against launch by launch, batch sizes that use each of them."""
    w = synth.make(name, n=1500)
    a = binding.Sim.from_workload(w, **over)
    b = binding.Sim.from_workload(w, **over)
    b.set_graph_mode(True)
    for k, n in enumerate([1, 40, 3, 33, 8, 70, 5]):
        if k in (4, 6):
            b.enable_kernel_timing(k == 4)
        a.step(n)
        b.step(n)
        if k == 4:
            assert b.kernel_time()[1] == n
        if "overlap" in over:   # the list method keeps no triangulation
            xa, ta, sa, _ = a.state()
            xb, tb, sb, _ = b.state()
            assert np.array_equal(xa, xb) and np.array_equal(ta, tb) and sa == sb
        else:
            _same(a, b)


@pytest.mark.parametrize("name,over", [("C2", {}), ("C3", {}), ("C3", {"overlap": "verlet"})])
def test_untimed_steps_after_a_handles_first_steps_were_timed(name, over):
    """A fresh handle whose first steps all run cut around their timed force, with moves so small that the round
    budgets settle and hold (they shrink by one after 64 steps that needed less), and then untimed batches that need
    single steps (3), both graphs (11) and several in one graph (8)."""
    w = synth.make(name, n=600)
    a = binding.Sim.from_workload(w, dt=1e-9, **over)
    b = binding.Sim.from_workload(w, dt=1e-9, **over)
    b.set_graph_mode(True)
    b.enable_kernel_timing(True)
    a.step(600)
    b.step(600)
    assert b.kernel_time()[1] == 600
    b.enable_kernel_timing(False)
    for n in (3, 11, 8):
        a.step(n)
        b.step(n)
        xa, ta, sa, _ = a.state()
        xb, tb, sb, _ = b.state()
        assert np.array_equal(xa, xb) and np.array_equal(ta, tb) and sa == sb


def test_rounds_launched_per_phase_after_a_step_of_many():
    """Launch form 2 launches the overlap rounds that recently moved many disks.  After one step of more than a
    hundred rounds of thousands of disks the next one launches all 48 that a step holds, those after it 24; the
    results are those of the other forms."""
    torch = pytest.importorskip("torch")
    from torch.profiler import ProfilerActivity, profile

    m, c = 12, 12   # c x c patches of m x m disks on a hexagonal lattice

    def patches(d):
        p = d * np.array([[i + 0.5 * (j & 1) - m / 2, 0.8660254 * (j - m / 2)] for i in range(m) for j in range(m)])
        return np.concatenate([p + [20.0 + 32.0 * a, 20.0 + 32.0 * b] for a in range(c) for b in range(c)])

    xy0 = patches(2.1)
    n = len(xy0)
    xy = patches(1.99) + np.random.default_rng(3).uniform(0, 0.001, (n, 2))
    launched = {}
    sims = []
    for mode in (1, 2):
        g = binding.Sim(xy0, np.ones(n), np.zeros(n, np.int32), None, np.array([[0.0]]), L=32.0 * c + 8, D=0.0,
                        dt=1e-6, seed=1, overlap_factor=0.5, contact_tol=1e-4)
        g.set_tail_mode(mode)
        g.set_positions(xy)
        g.step(1)
        assert g.state()[3]["overlap_rounds_max"] > 100
        for _ in range(3):
            with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
                g.step(1)
                torch.cuda.synchronize()
            names = [e.name for e in prof.events()]
            assert any("k_em" in k for k in names)   # the trace holds this library's kernels
            launched.setdefault(mode, []).append(sum("k_ovl_gather" in k for k in names))
        sims.append(g)
    assert launched == {1: [0, 0, 0], 2: [48, 24, 24]}
    _same(*sims)


def test_first_queued_steps_of_many_overlaps_cost_no_more_than_launched_ones():
    """A fresh handle of 66,000 disks that overlap much in every step: the first twenty steps queued together take no
    longer than launched one by one (which adapt after each step), with half as much again for the captures."""
    import time

    n = 66000
    L = synth.box_side(n, 0.5)
    xy = synth.rsa(n, L, 1.0, seed=8)
    best = {}
    for graph in (True, False) * 3:
        g = binding.Sim(xy, np.ones(n), np.zeros(n, np.int32), None, np.array([[0.0]]), L=L, D=1.0, dt=2e-2, seed=2,
                        kind="screened", A=1.0, lam=0.5, cutoff=2.5, skin=0.5)
        g.set_graph_mode(graph)
        g.state()
        t = time.perf_counter()
        g.step(20)
        g.state()
        best[graph] = min(best.get(graph, 1e9), time.perf_counter() - t)
        g.close()
    assert best[True] <= 1.5 * best[False], best


@pytest.mark.parametrize("graph", [False, True])
def test_launch_forms_agree_where_overlap_rounds_fold_the_triangulation(graph):
    """A compressed patch whose first overlap rounds throw disks across edges: repairs that end with inverted triangles
    and edges whose flip is blocked, at different rounds in the three launch forms, and a move that the host replays."""
    m = 64

    def patch(d):
        p = np.array([[i + 0.5 * (j & 1) - m / 2, 0.8660254 * (j - m / 2)] for i in range(m) for j in range(m)])
        return 106.0 + d * p

    n = m * m
    xy = patch(1.95) + np.random.default_rng(4).uniform(0.0, 0.01, (n, 2))
    sims = []
    for mode in (0, 1, 2):
        g = binding.Sim(patch(2.1), np.ones(n), np.zeros(n, np.int32), None, np.array([[0.0]]), L=212.0, D=0.0,
                        dt=1e-6, seed=1)
        g.set_tail_mode(mode)
        g.set_graph_mode(graph)
        g.set_positions(xy)
        g.step(2)
        sims.append(g)
    assert sims[0].state()[3]["kinetic_repairs"] >= 2 and sims[0].state()[3]["inversion_flips"] > 0
    _same(sims[0], sims[1])
    _same(sims[0], sims[2])


@pytest.mark.parametrize("c", [6, 12])   # 5,184 disks (all rounds in one workgroup by default) and 20,736
def test_a_step_of_many_large_rounds_is_not_left_to_one_workgroup(c):
    """A step of more than a hundred rounds that each move most of the disks: the default launch form takes no longer
    than launching its rounds (form 0, which hands them to the host after a few), with half as much again for the rounds
    it takes before it sees that, and gives the same state and counters."""
    import time

    m = 12

    def patches(d):
        p = np.array([[i + 0.5 * (j & 1) - m / 2, 0.8660254 * (j - m / 2)] for i in range(m) for j in range(m)])
        return np.concatenate([d * p + [20.0 + 32.0 * a, 20.0 + 32.0 * b] for a in range(c) for b in range(c)])

    xy0 = patches(2.1)
    n = len(xy0)
    xy = patches(1.99) + np.random.default_rng(3).uniform(0, 0.001, (n, 2))
    best, sims = {}, []
    for mode in (0, -1):
        for rep in range(3):
            g = binding.Sim(xy0, np.ones(n), np.zeros(n, np.int32), None, np.array([[0.0]]), L=32.0 * c + 8, D=0.0,
                            dt=1e-6, seed=1, kind="screened", A=1.0, lam=0.5, cutoff=2.5, skin=0.5, overlap_factor=0.5,
                            contact_tol=1e-4)
            g.set_tail_mode(mode)
            g.step(2)
            g.set_positions(xy)
            t = time.perf_counter()
            g.step(1)
            best[mode] = min(best.get(mode, 1e9), time.perf_counter() - t)
            g.step(3)
        sims.append(g)
    assert sims[0].state()[3]["overlap_rounds_max"] > 100
    _same(*sims)
    assert best[-1] <= 1.5 * best[0], best
