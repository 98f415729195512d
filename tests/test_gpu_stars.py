"""Overlap rounds at disks of high degree: a large disk inside a ring of touching small ones, at the degrees where
the star of a disk changes its form on the device (8 half-edges in one pass of a group of lanes, 16 in two, more by
one lane), in every launch form of the rounds, against the oracle."""
import math

import numpy as np
import pytest

import oracle
from paper_1703_02484_amd import binding, synth
from tests._checks import rel_err, tri_set
from tests.conftest import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def ring_system(m):
    """A disk with m radius-1 neighbours around it and a jittered lattice of radius-1 disks outside."""
    R = 1.01 / math.sin(math.pi / m) - 1.0
    ring = R + 1.0
    L = 2.0 * (ring + 12.0)
    c = 0.5 * L
    a = 2.0 * math.pi * np.arange(m) / m
    pts = [[c, c]] + [[c + (ring + 0.004) * math.cos(t), c + (ring + 0.004) * math.sin(t)] for t in a]
    rng = np.random.default_rng(m)
    k = int((L - 2.0) / 2.2)
    for i in range(k):
        for j in range(k):
            x, y = 1.05 + 2.2 * i + rng.uniform(0.0, 0.15), 1.05 + 2.2 * j + rng.uniform(0.0, 0.15)
            if math.hypot(x - c, y - c) > ring + 2.1 and x <= L - 1.0 and y <= L - 1.0:
                pts.append([x, y])
    xy = np.array(pts)
    rad = np.ones(len(xy))
    rad[0] = R
    return xy, rad, L


@pytest.mark.parametrize("m", [7, 8, 9, 15, 16, 17, 25])
@pytest.mark.parametrize("tail_mode", [0, 1, 2])
def test_high_degree_stars_match_oracle(m, tail_mode):
    xy, rad, L = ring_system(m)
    n = len(xy)
    kw = dict(L=L, D=1.0, dt=2e-4, seed=m, overlap_factor=0.5)
    sp, K = np.zeros(n, np.int32), np.array([[1e-2]])
    g = binding.Sim(xy, rad, sp, None, K, **kw)
    g.set_tail_mode(tail_mode)
    g.set_graph_mode(tail_mode != 0)
    o = oracle.OracleSim(xy, rad, sp, None, K, **kw)
    deg = np.bincount(np.concatenate([np.asarray(t)[np.asarray(t) != 0] for t in g.triangles() if 0 in t]))
    assert np.count_nonzero(deg) == m
    g.step(12)
    o.step(12)
    assert rel_err(g.state()[0], o.state()[0]) <= 1e-9
    assert tri_set(g.triangles()) == tri_set(o.triangles())
    sg, so = g.state()[3], o.state()[3]
    assert sg["overlap_rounds_total"] == so["overlap_rounds_total"] > 0


@pytest.mark.parametrize("pairs", [1, 63, 64, 65, 150])
@pytest.mark.parametrize("periodic", [False, True])
def test_tail_rounds_around_one_star_per_group_match_oracle(pairs, periodic):
    """Rounds of 2 * pairs disks in the one-workgroup tail: below, at and above the 128 stars it keeps in registers."""
    k = 40
    L = 2.3 * k
    rng = np.random.default_rng(pairs)
    xy = np.array([[1.15 + 2.3 * i, 1.15 + 2.3 * j] for i in range(k) for j in range(k)])
    xy += rng.uniform(-0.1, 0.1, xy.shape)
    odd = rng.choice(np.arange(k // 2) * 2 * k + 1, k // 2, replace=False)   # rows 0, 2, ...: pairs along y
    first = np.concatenate([odd + 4 * c for c in range(k // 4 - 1)])[:pairs]
    assert len(first) == pairs
    xy[first + 1] = xy[first] + [0.0, 2.0 + 1e-6]   # each pair pulled 0.02 into an overlap by every step; no other forces
    n = len(xy)
    kw = dict(L=L, D=1.0, dt=1e-7, seed=pairs, overlap_factor=0.5, periodic=periodic, cutoff=2.05)
    sp, K = np.zeros(n, np.int32), np.array([[-4e5]])
    g = binding.Sim(xy, np.ones(n), sp, None, K, **kw)
    g.set_tail_mode(2)
    o = oracle.OracleSim(xy, np.ones(n), sp, None, K, **kw)
    g.step(3)
    o.step(3)
    assert rel_err(g.state()[0], o.state()[0]) <= 1e-9
    assert tri_set(g.triangles()) == tri_set(o.triangles())
    sg, so = g.state()[3], o.state()[3]
    assert sg["overlap_rounds_total"] == so["overlap_rounds_total"] > 0


@pytest.mark.parametrize("tail_mode", [0, 1, 2])
@pytest.mark.parametrize("graph", [False, True])
def test_many_overlap_rounds_match_oracle(tail_mode, graph):
    """Steps of 35 to 60 rounds: within and beyond what one launch of the tail holds (48)."""
    n = 300
    L = synth.box_side(n, 0.5)
    xy = synth.rsa(n, L, 1.0, seed=3)
    kw = dict(L=L, dt=2e-3, seed=1, overlap_factor=0.4)
    sp, K = np.zeros(n, np.int32), np.array([[1e-2]])
    g = binding.Sim(xy, np.ones(n), sp, None, K, **kw)
    g.set_tail_mode(tail_mode)
    g.set_graph_mode(graph)
    o = oracle.OracleSim(xy, np.ones(n), sp, None, K, **kw)
    g.step(8)
    o.step(8)
    assert rel_err(g.state()[0], o.state()[0]) <= 1e-9
    sg, so = g.state()[3], o.state()[3]
    assert so["overlap_rounds_max"] > 48
    for k in ("overlap_rounds_total", "overlap_rounds_max", "overlap_edges_total"):
        assert sg[k] == so[k]
