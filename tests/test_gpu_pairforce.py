"""The stateless pair-force call bd_pair_forces_dev (device arrays in, device
forces out, no handle) against the oracle's brute-force forces, element by
element: every law, FP64 and FP32, non-reciprocal two-species K, ragged sizes
that span several workgroups and j splits with a short last one, the
single-particle and two-particle edge cases, and the full 65,536-disk
two-species workload on sampled rows."""
import numpy as np
import pytest

import oracle
from paper_1703_02484_amd import binding, synth
from tests.conftest import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

LAWS = {
    "q2": dict(kind="power", q=2.0),
    "q6": dict(kind="power", q=6.0),
    "screened_cut": dict(kind="screened", A=1.0, lam=0.5, cutoff=2.5),
    "q2_cut": dict(kind="power", q=2.0, cutoff=6.0),
}


def _dev(w):
    import torch

    xy = torch.from_numpy(np.ascontiguousarray(w.xy)).cuda()
    sp = torch.from_numpy(np.ascontiguousarray(w.species, dtype=np.int32)).cuda()
    return xy, sp


@pytest.mark.parametrize("law", sorted(LAWS))
@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("n", [1, 2, 513, 3001])
def test_pair_forces_dev_matches_oracle(law, fp32, n):
    import torch

    w = synth.make("C2", n=max(n, 3))
    if n < 3:   # the workload generator's smallest system; keep its first n disks
        w.xy, w.species = w.xy[:n].copy(), w.species[:n].copy()
    kw = LAWS[law]
    xy, sp = _dev(w)
    f = binding.pair_forces_dev(xy, sp, w.K, fp32=fp32, **kw)
    torch.cuda.synchronize()
    fo = oracle.forces(w.xy, w.species, w.K, **kw)
    got = f.cpu().numpy()
    scale = max(np.abs(fo).max(), 1e-300)
    tol = 1e-4 if fp32 else 1e-12
    assert np.abs(got - fo).max() <= tol * scale
    if n == 1:
        assert np.all(got == 0.0)


def test_pair_forces_dev_full_size_sampled():
    import torch

    w = synth.make("C2")
    xy, sp = _dev(w)
    f = binding.pair_forces_dev(xy, sp, w.K, fp32=True).cpu().numpy()
    torch.cuda.synchronize()
    rng = np.random.default_rng(5)
    idx = np.concatenate([[0, w.n - 1], rng.choice(w.n, 510, replace=False)]).astype(np.int32)
    fo = oracle.forces(w.xy, w.species, w.K, idx=idx)
    assert np.abs(f[idx] - fo).max() <= 1e-4 * np.abs(fo).max()


def test_pair_forces_dev_rejects_bad_arguments():
    import torch

    w = synth.make("C1", n=100)
    xy, sp = _dev(w)
    with pytest.raises(ValueError):
        binding.pair_forces_dev(xy.float(), sp, w.K)
    with pytest.raises(binding.BDError):
        binding.pair_forces_dev(xy, sp, np.zeros((9, 9)))   # S above BD_MAX_SPECIES
    with pytest.raises(binding.BDError):
        binding.pair_forces_dev(xy, sp, w.K, kind="screened", lam=-1.0)


@pytest.mark.parametrize("law", ["q2", "q6", "screened_cut"])
@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("n", [63, 64, 4096, 4097, 6144, 6145])
def test_pair_forces_dev_layout_edges(law, fp32, n):
    """Sizes around the layouts' limits (one wavefront per particle; staged tiles), ragged blocks, three species of
    uneven number, one of them absent from whole staged blocks."""
    import torch

    w = synth.make("C1", n=n)
    species = np.where(np.arange(n) < n // 2, 0, np.where(np.arange(n) % 7 == 0, 2, 1)).astype(np.int32)
    K = np.array([[1e-2, -5e-3, 4e-3], [2e-3, 1e-2, 0.0], [-1e-3, 3e-3, 7e-3]])
    xy = torch.from_numpy(np.ascontiguousarray(w.xy)).cuda()
    sp = torch.from_numpy(species).cuda()
    f = binding.pair_forces_dev(xy, sp, K, fp32=fp32, **LAWS[law]).cpu().numpy()
    idx = np.unique(np.concatenate([[0, n // 2, n - 1], np.random.default_rng(3).integers(0, n, 400)])).astype(np.int32)
    fo = oracle.forces(w.xy, species, K, idx=idx, **LAWS[law])
    tol = 1e-4 if fp32 else 1e-12
    assert np.abs(f[idx] - fo).max() <= tol * np.abs(fo).max()


@pytest.mark.parametrize("n", [200, 7000])
@pytest.mark.parametrize("law", ["q2", "screened_cut"])
@pytest.mark.parametrize("fp32", [False, True])
def test_pair_forces_dev_singular_positions(n, law, fp32):
    """Two particles at one place: both forces non-finite, the others as without the pair's mutual term.  A particle
    at infinity: its pairs give 0 * inf along x in every force, with and without a cutoff, and nothing along y."""
    import torch

    w = synth.make("C1", n=n)
    sp = torch.zeros(n, dtype=torch.int32, device="cuda")
    K = np.array([[1.0]])
    xy = w.xy.copy()
    xy[n - 1] = xy[3]
    f = binding.pair_forces_dev(torch.from_numpy(xy).cuda(), sp, K, fp32=fp32, **LAWS[law]).cpu().numpy()
    bad = np.zeros(n, bool)
    bad[[3, n - 1]] = True
    assert not np.isfinite(f[bad]).any() and np.isfinite(f[~bad]).all()
    xy = w.xy.copy()
    xy[5, 0] = np.inf
    f = binding.pair_forces_dev(torch.from_numpy(xy).cuda(), sp, K, fp32=fp32, **LAWS[law]).cpu().numpy()
    rest = np.arange(n) != 5
    assert np.isnan(f[:, 0]).all() and np.isfinite(f[rest, 1]).all()


@pytest.mark.parametrize("law", ["q2", "q6", "screened"])
@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("n", [4097, 32768, 32769])
def test_pair_forces_dev_cells_match_oracle(law, fp32, n):
    """With a cutoff: cells around the origin (both signs of the coordinates), more of them than the grid has (the
    torus closes), and beside an empty half; three species; the edges of the layout's sizes."""
    rng = np.random.default_rng(n)
    m = int(np.ceil(np.sqrt(n)))
    k = rng.permutation(m * m)[:n]
    xy = np.stack([k % m, k // m], 1) * 2.5 + rng.uniform(-0.4, 0.4, (n, 2)) - [0.5 * 2.5 * m, 300.0]
    xy[xy[:, 0] > 0.0] += [5000.0, 0.0]
    species = rng.integers(0, 3, n).astype(np.int32)
    K = np.array([[1e-2, -5e-3, 4e-3], [2e-3, 1e-2, 0.0], [-1e-3, 3e-3, 7e-3]])
    kw = dict(cutoff=7.0, **{"q2": dict(kind="power", q=2.0), "q6": dict(kind="power", q=6.0),
                             "screened": dict(kind="screened", A=1.0, lam=2.0)}[law])
    import torch

    f = binding.pair_forces_dev(torch.from_numpy(xy).cuda(), torch.from_numpy(species).cuda(), K, fp32=fp32, **kw)
    g = binding.pair_forces_dev(torch.from_numpy(xy).cuda(), torch.from_numpy(species).cuda(), K, fp32=fp32,
                                noalloc=True, **kw)
    f = f.cpu().numpy()
    assert np.array_equal(f, g.cpu().numpy())   # the order in which particles reach their cells does not show
    idx = np.unique(np.concatenate([[0, n - 1], rng.integers(0, n, 400)])).astype(np.int32)
    # FP32 rounds the positions (to 2.4e-4 at 5,000) and a pair within that of the cutoff may fall on either side
    fo = oracle.forces(xy.astype(np.float32).astype(np.float64) if fp32 else xy, species, K, idx=idx, **kw)
    edge = np.zeros(len(idx), bool)
    if fp32:
        xr = xy.astype(np.float32).astype(np.float64)
        for a, i in enumerate(idx):
            d = np.hypot(*(xr - xr[i]).T)
            edge[a] = (np.abs(d - 7.0) < 1e-3).any()
        assert edge.mean() < 0.5
    tol = 1e-4 if fp32 else 1e-12
    assert np.abs(f[idx] - fo)[~edge].max() <= tol * np.abs(fo).max()


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("how", ["one_cell", "far_away", "cluster"])
def test_pair_forces_dev_cells_fall_back(how, fp32):
    """Positions the cells leave to the all-pairs tiles: within the cutoff of one another, too far from the origin to
    bin, and most of them in a few cells."""
    import torch

    n = 5000
    rng = np.random.default_rng(3)
    w = synth.make("C1", n=n)
    xy, cutoff = w.xy.copy(), 6.0
    if how == "one_cell":
        cutoff = 4.0 * w.L
    elif how == "far_away":
        xy = np.round((xy + 2.0**23 - 1000.0) * 2.0) / 2.0   # halves: exact in FP32 too
    else:
        xy[: n // 2] *= 0.05
    species = rng.integers(0, 2, n).astype(np.int32)
    K = np.array([[1e-2, -5e-3], [2e-3, 1e-2]])
    kw = dict(kind="screened", A=1.0, lam=2.0, cutoff=cutoff)
    f = binding.pair_forces_dev(torch.from_numpy(xy).cuda(), torch.from_numpy(species).cuda(), K, fp32=fp32, **kw)
    f = f.cpu().numpy()
    idx = rng.integers(0, n, 300).astype(np.int32)
    fo = oracle.forces(xy, species, K, idx=idx, **kw)
    ok = np.isfinite(fo).all(1)
    assert ok.sum() > 100 and np.array_equal(np.isfinite(f[idx]).all(1), ok)
    assert np.abs(f[idx] - fo)[ok].max() <= (2e-4 if fp32 else 1e-12) * np.abs(fo[ok]).max()


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("n, S", [(16385, 1), (20001, 8), (20480, 2), (31001, 3), (46001, 2), (64001, 2)])
def test_pair_forces_dev_every_pair_once_matches_oracle(n, S, fp32):
    """The inverse-square law without a cutoff above the rows: every chunk length, ragged last chunks, species of
    uneven number with one absent, and sizes whose sums do not fit and stay with the tiles (64,001 in FP64)."""
    import torch

    w = synth.make("C1", n=n)
    rng = np.random.default_rng(n)
    species = np.minimum(rng.integers(0, 4 * S, n), S - 1).astype(np.int32)   # the last one holds most
    if S == 8:
        species[species == 2] = 3
    K = rng.normal(size=(S, S)) * 1e-2
    xy, sp = torch.from_numpy(np.ascontiguousarray(w.xy)).cuda(), torch.from_numpy(species).cuda()
    f = binding.pair_forces_dev(xy, sp, K, fp32=fp32)
    g = binding.pair_forces_dev(xy, sp, K, fp32=fp32, noalloc=True)
    f = f.cpu().numpy()
    assert np.array_equal(f, g.cpu().numpy())
    idx = np.unique(np.concatenate([[0, n // 2, n - 1], rng.integers(0, n, 300)])).astype(np.int32)
    fo = oracle.forces(w.xy, species, K, idx=idx)
    assert np.abs(f[idx] - fo).max() <= (1e-4 if fp32 else 1e-12) * np.abs(fo).max()


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("n", [20100, 20480])
def test_pair_forces_dev_every_pair_once_singular(n, fp32):
    """Two particles at one place give non-finite forces to both, within one chunk and across two, and to nobody else;
    a particle at infinity gives 0 * inf along x."""
    import torch

    w = synth.make("C1", n=n)
    sp = torch.zeros(n, dtype=torch.int32, device="cuda")
    for a, b in ((3, 4), (0, n - 1), (100, 100 + 64)):
        xy = w.xy.copy()
        xy[b] = xy[a]
        f = binding.pair_forces_dev(torch.from_numpy(xy).cuda(), sp, np.array([[1.0]]), fp32=fp32).cpu().numpy()
        bad = np.zeros(n, bool)
        bad[[a, b]] = True
        assert not np.isfinite(f[bad]).any() and np.isfinite(f[~bad]).all()
    xy = w.xy.copy()
    xy[n - 1, 0] = np.inf
    f = binding.pair_forces_dev(torch.from_numpy(xy).cuda(), sp, np.array([[1.0]]), fp32=fp32).cpu().numpy()
    rest = np.arange(n) != n - 1
    assert np.isnan(f[:, 0]).all() and np.isfinite(f[rest, 1]).all()


@pytest.mark.parametrize("n, cutoff", [(5000, 0.0), (9000, 6.0), (9000, 0.0), (17000, 0.0)])
def test_noalloc_layouts_in_a_graph(n, cutoff):
    """Each layout captured once and replayed with other positions in the same buffers, among them ones the cells leave
    to the tiles, with eager work between the replays: bitwise the eager forces."""
    import torch

    w = synth.make("C1", n=n)
    sp = torch.from_numpy((np.arange(n) % 2).astype(np.int32)).cuda()
    K = np.array([[1e-2, -5e-3], [2e-3, 1e-2]])
    xy = torch.from_numpy(np.ascontiguousarray(w.xy)).cuda()
    out = torch.empty_like(xy)
    kw = dict(kind="power", q=2.0, cutoff=cutoff, noalloc=True)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        binding.pair_forces_dev(xy, sp, K, out=out, **kw)
    torch.cuda.current_stream().wait_stream(s)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        binding.pair_forces_dev(xy, sp, K, out=out, **kw)
    base = xy.clone()
    for scale in (1.0, 0.02, 1.3, 1.0):   # 0.02: most pairs within the cutoff
        xy.copy_(base * scale)
        g.replay()
        torch.cuda.synchronize()
        got = out.clone()
        ref = binding.pair_forces_dev(xy, sp, K, **{**kw, "noalloc": False})
        torch.cuda.synchronize()
        assert torch.equal(got, ref), scale


@pytest.mark.parametrize("fp32, n, S", [(True, 40001, 1), (True, 60001, 2), (True, 64101, 2), (True, 71600, 2),
                                        (True, 66001, 8), (False, 28001, 2), (False, 44001, 2)])
def test_pair_forces_dev_every_pair_once_in_long_chunks(fp32, n, S):
    """Chunks of 512, 1,024 and (FP32) 1,280 particles, whose wavefronts add into one copy of the sums: against the
    oracle, with two particles at one place (neighbours, in different wavefronts of a chunk, in different chunks), with
    one at infinity, and captured and replayed with other positions, bitwise the eager forces."""
    import torch

    w = synth.make("C1", n=n)
    rng = np.random.default_rng(n)
    species = np.minimum(rng.integers(0, 4 * S, n), S - 1).astype(np.int32)
    K = rng.normal(size=(S, S)) * 1e-2
    base, sp = torch.from_numpy(np.ascontiguousarray(w.xy)).cuda(), torch.from_numpy(species).cuda()
    f = binding.pair_forces_dev(base, sp, K, fp32=fp32).cpu().numpy()
    idx = np.unique(np.concatenate([[0, n // 2, n - 1], rng.integers(0, n, 300)])).astype(np.int32)
    fo = oracle.forces(w.xy, species, K, idx=idx)
    assert np.abs(f[idx] - fo).max() <= (1e-4 if fp32 else 1e-12) * np.abs(fo).max()

    for a, b in ((3, 4), (0, n - 1), (100, 100 + 450)):
        xy = base.clone()
        xy[b] = xy[a]
        f = binding.pair_forces_dev(xy, sp, K, fp32=fp32).cpu().numpy()
        bad = np.zeros(n, bool)
        bad[[a, b]] = True
        assert not np.isfinite(f[bad]).any() and np.isfinite(f[~bad]).all()
    xy = base.clone()
    xy[n - 1, 0] = np.inf
    f = binding.pair_forces_dev(xy, sp, K, fp32=fp32).cpu().numpy()
    rest = np.arange(n) != n - 1
    assert np.isnan(f[:, 0]).all() and np.isfinite(f[rest, 1]).all()

    xy = base.clone()
    out = torch.empty_like(xy)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        binding.pair_forces_dev(xy, sp, K, fp32=fp32, out=out, noalloc=True)
    torch.cuda.current_stream().wait_stream(s)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        binding.pair_forces_dev(xy, sp, K, fp32=fp32, out=out, noalloc=True)
    for scale in (1.0, 1.3, 0.9, 1.0):
        xy.copy_(base * scale)
        g.replay()
        torch.cuda.synchronize()
        got = out.clone()
        ref = binding.pair_forces_dev(xy, sp, K, fp32=fp32)
        assert torch.equal(got, ref), scale


@pytest.mark.parametrize("law", ["q2", "q6", "screened"])
@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("frac", [0.35, 0.5, 2.0])
def test_pair_forces_dev_wide_cutoffs_match_oracle(law, fp32, frac):
    """Cutoffs that the cells leave to the tiles, with a quarter to all of the pairs inside: blocks whose pairs are
    noted and blocks evaluated pair by pair, particles in no order in space and in rows."""
    import torch

    n = 9001
    w = synth.make("C1", n=n)
    rng = np.random.default_rng(2)
    cutoff = frac * w.L
    kw = dict(cutoff=cutoff, **{"q2": dict(kind="power", q=2.0), "q6": dict(kind="power", q=6.0),
                                "screened": dict(kind="screened", A=1.0, lam=20.0)}[law])
    K = np.array([[1e-2, -5e-3, 4e-3], [2e-3, 1e-2, 0.0], [-1e-3, 3e-3, 7e-3]])
    species = rng.integers(0, 3, n).astype(np.int32)
    for xy in (w.xy, w.xy[np.argsort(w.xy[:, 1])]):
        x = np.ascontiguousarray(xy.astype(np.float32).astype(np.float64) if fp32 else xy)
        f = binding.pair_forces_dev(torch.from_numpy(x).cuda(), torch.from_numpy(species).cuda(), K, fp32=fp32, **kw)
        f = f.cpu().numpy()
        idx = np.unique(np.concatenate([[0, n - 1], rng.integers(0, n, 300)])).astype(np.int32)
        fo = oracle.forces(x, species, K, idx=idx, **kw)
        edge = np.array([(np.abs(np.hypot(*(x - x[i]).T) - cutoff) < (1e-3 if fp32 else 1e-9)).any() for i in idx])
        assert edge.mean() < 0.9
        assert np.abs(f[idx] - fo)[~edge].max() <= (1e-4 if fp32 else 1e-12) * np.abs(fo).max()


@pytest.mark.parametrize("fp32", [False, True])
def test_pair_forces_dev_cutoff_beyond_the_system_costs_no_more(fp32):
    """With every pair inside the cutoff the call does the work of the one without, and the tests of the distances: of
    some 30 instructions a pair 2 more, 7 %; the limit is twice that."""
    import time

    import torch

    n = 40001
    w = synth.make("C1", n=n)
    xy, sp = torch.from_numpy(np.ascontiguousarray(w.xy)).cuda(), torch.zeros(n, dtype=torch.int32, device="cuda")
    out = torch.empty_like(xy)

    def best(cutoff):
        ts = []
        for _ in range(12):
            torch.cuda.synchronize()
            t = time.perf_counter()
            binding.pair_forces_dev(xy, sp, np.array([[1.0]]), kind="screened", A=1.0, lam=0.5, fp32=fp32,
                                    cutoff=cutoff, out=out)
            ts.append(time.perf_counter() - t)
        return min(ts[2:])

    t0, t1 = best(0.0), best(2.0 * w.L)
    assert t1 <= 1.14 * t0, (t0, t1)
