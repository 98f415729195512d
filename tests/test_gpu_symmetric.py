"""The symmetric form of the all-pairs force (``force_chunk = -1``): every
pair of chunks of a system evaluated once by one workgroup, which writes the
partial sums of both chunks (the pair's geometric factor is the same for both
orders; K weights each side in the reduction).  Checked against the oracle
like the ordinary form: forces, trajectories, a batch, the adjoint, and
run-to-run determinism.  Chunks are cut to at most 1024 disks, so the sizes
below give ragged last chunks and several chunk pairs per system."""
import numpy as np
import pytest

import oracle
from paper_1703_02484_amd import binding, synth
from tests._checks import rel_err, tri_set
from tests.conftest import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _scale(f):
    return np.abs(f).max()


@pytest.mark.parametrize("pin", [-1, -2, -3])
@pytest.mark.parametrize("n", [3, 65, 1000, 1025, 4099])
def test_symmetric_forces_fp32(n, pin):
    w = synth.make("C2", n=n)
    g = binding.Sim.from_workload(w, force_chunk=pin)
    cfg = g.force_config()
    assert cfg["persistent"] == 2 and cfg["per_lane"] == {-1: 4, -2: 2, -3: 8}[pin]
    fo = oracle.forces(w.xy, w.species, w.K)
    assert np.abs(g.forces() - fo).max() <= 1e-4 * _scale(fo)


@pytest.mark.parametrize("pin", [-1, -2, -3])
@pytest.mark.parametrize("n", [700, 2500])
def test_symmetric_forces_fp64(n, pin):
    w = synth.make("C1", n=n)
    g = binding.Sim.from_workload(w, force_chunk=pin)
    fo = oracle.forces(w.xy, w.species, w.K)
    assert np.abs(g.forces() - fo).max() <= 1e-12 * _scale(fo)


@pytest.mark.parametrize("pin", [-1, -3])
def test_symmetric_full_size_c2_sampled(pin):
    w = synth.make("C2")
    g = binding.Sim.from_workload(w, force_chunk=pin)
    fg = g.forces()
    idx = np.sort(np.random.default_rng(0).choice(w.n, 512, replace=False))
    fo = oracle.forces(w.xy, w.species, w.K, idx=idx)
    assert np.abs(fg[idx] - fo).max() <= 1e-4 * _scale(fo)


def test_symmetric_trajectory_c2_fp32():
    w = synth.make("C2", n=3000)
    g = binding.Sim.from_workload(w, force_chunk=-1)
    o = oracle.OracleSim.from_workload(w)
    for _ in range(5):
        g.step(10)
        o.step(10)
        assert rel_err(g.state()[0], o.state()[0]) <= 1e-4
        assert tri_set(g.triangles()) == tri_set(o.triangles())


def test_symmetric_batch_fp64_matches_oracle():
    ws = synth.make_batch(5, seed=4, lo=300, hi=2600)
    b = binding.Sim.from_workloads(ws, force_chunk=-1)
    _, doff, _ = b.layout()
    f = b.forces()
    for r, w in enumerate(ws):
        fo = oracle.forces(w.xy, w.species, w.K)
        assert np.abs(f[doff[r]:doff[r + 1]] - fo).max() <= 1e-12 * _scale(fo)


def test_symmetric_bitwise_run_to_run():
    w = synth.make("C2", n=5000)
    a = binding.Sim.from_workload(w, force_chunk=-1)
    b = binding.Sim.from_workload(w, force_chunk=-1)
    a.step(8)
    b.step(8)
    assert np.array_equal(a.state()[0], b.state()[0])


@pytest.mark.parametrize("pin", [-1, -2, -3])
def test_symmetric_adjoint_matches_oracle_jvp(pin):
    w = synth.make("C5", n=1500)
    steps = 8
    g = binding.Sim.from_workload(w, force_chunk=pin)
    g.adjoint_begin(steps, 3)
    o = oracle.OracleSim.from_workload(w)
    rng = np.random.default_rng(2)
    v = rng.normal(size=(w.n, 2))
    tK = rng.normal(size=w.K.shape)
    o.set_tangent(v, tK)
    o.step(steps)
    assert np.abs(g.state()[0] - o.state()[0]).max() <= 1e-9 * w.L
    lam = rng.normal(size=(w.n, 2))
    g0, gK = g.adjoint_backward(lam)
    lhs = np.sum(g0 * v) + np.sum(gK * tK)
    rhs = np.sum(lam * o.tangent())
    assert abs(lhs - rhs) <= 1e-10 * abs(rhs)


def test_symmetric_form_needs_the_inverse_square_law():
    w = synth.make("C1", n=300)
    with pytest.raises(binding.BDError):
        binding.Sim.from_workload(w, force_chunk=-1, kind="power", q=6.0)


@pytest.mark.parametrize("n", [700, 769, 2561, 4097, 5003, 12289])
@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("periodic", [False, True])
def test_fixed_rule_forms_match_oracle(n, fp32, periodic):
    """The forms the library takes without timing, at the sizes where they change: small ordinary tiles, then one
    wavefront per pair of chunks of 128 (and 256 in a periodic box), with ragged last chunks of three species whose
    padding must not act (in a periodic box padding has a nearest image)."""
    w = synth.make("C1", n=n, periodic=periodic)
    species = (np.arange(n) % 5 % 3).astype(np.int32)
    K = np.array([[1e-2, -5e-3, 4e-3], [2e-3, 1e-2, 0.0], [-1e-3, 3e-3, 7e-3]])
    g = binding.Sim(w.xy, w.radii, species, None, K, L=w.L, fp32=fp32, periodic=periodic)
    cfg = g.force_config()
    if cfg["tuned"] == 0:
        assert cfg["persistent"] == (2 if n > 4096 else 0)
    idx = np.unique(np.concatenate([[0, n - 1], np.random.default_rng(1).integers(0, n, 500)])).astype(np.int32)
    fo = oracle.forces(w.xy, species, K, idx=idx, period=w.L if periodic else 0.0)
    tol = 1e-4 if fp32 else 1e-12
    assert np.abs(g.forces()[idx] - fo).max() <= tol * _scale(fo)


@pytest.mark.parametrize("pin, sizes", [(-1, (129, 1023, 2050)), (-2, (129, 1023, 2050)), (-3, (129, 1023, 2050)),
                                        (0, (4100,)), (0, (12301,))])
def test_symmetric_adjoint_matches_ordinary_tiles(pin, sizes):
    """Ragged chunks (one disk over, one short) of two species in every symmetric form (0: the library's, of 128 and
    256), against the ordered pair sum."""
    ws = [synth.make("C5", n=n, seed=n) for n in sizes]
    rng = np.random.default_rng(5)
    lam = rng.normal(size=(sum(w.n for w in ws), 2))
    out = []
    for chunk in (pin, 256):
        b = binding.Sim.from_workloads(ws, force_chunk=chunk)
        b.adjoint_begin(5, 2)
        out.append(b.adjoint_backward(lam))
    for got, ref in zip(*out):   # the two trajectories differ by the rounding of their force sums
        assert np.abs(got - ref).max() <= 1e-9 * np.abs(ref).max()


@pytest.mark.parametrize("n", [1500, 14000])
def test_adjoint_of_large_overlap_rounds_matches_oracle_jvp(n):
    """A first round of some hundred, and of more than 4,096 moved disks (with later ones of fewer than 1,024)."""
    L = synth.box_side(n, 0.5)
    xy = synth.rsa(n, L, 1.0, seed=8)
    sp = (np.arange(n) % 2).astype(np.int32)
    w = synth.Workload("dense", xy, np.ones(n), sp, np.zeros(n), 2, np.array([[0.05, -0.02], [0.03, 0.04]]), L=L,
                       D=1.0, dt=2e-2, seed=2)
    g = binding.Sim.from_workload(w)
    g.adjoint_begin(1, 1)
    o = oracle.OracleSim.from_workload(w)
    rng = np.random.default_rng(2)
    v, tK = rng.normal(size=(n, 2)), rng.normal(size=(2, 2))
    o.set_tangent(v, tK)
    o.step(1)
    assert np.abs(g.state()[0] - o.state()[0]).max() <= 1e-9 * w.L
    lam = rng.normal(size=(n, 2))
    g0, gK = g.adjoint_backward(lam)
    lhs = np.sum(g0 * v) + np.sum(gK * tK)
    rhs = np.sum(lam * o.tangent())
    assert abs(lhs - rhs) <= 1e-10 * max(abs(rhs), np.abs(lam * o.tangent()).sum() * 1e-2)
