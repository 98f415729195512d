"""Performance cases: the work a program has this library do, through its public entry points.

A case is a dict of plain values.  Three kinds cover the library:

* ``forces``  the stateless pair force of device arrays (``binding.pair_forces_dev``);
* ``steps``   a running simulation: ``steps`` time steps of a ``Sim`` handle (one system or a batch), then its
              positions and angles into device memory;
* ``adjoint`` a rollout with checkpoints followed by its reverse sweep (gradients of the positions and of K).

The sizes are those of the workloads of ``synth`` (1,024, 16,384, 65,536 and 1,048,576 disks, the batch of log-uniform
sizes in [2048, 32768]) and generic ones around them, odd ones among them.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1703_02484_amd import binding, synth


def listed():
    return [
        # a few hundred particles whose forces another program asks for one call at a time: launches and allocation
        dict(name="forces_777_fp64", kind="forces", n=777, phi=0.3, S=1, law="power", q=2.0, cutoff=0.0, fp32=False,
             noalloc=False),
        # medium system, three species, the screened law with its cutoff, inside a serving loop that may not allocate
        dict(name="forces_20011_screened", kind="forces", n=20011, phi=0.45, S=3, law="screened", q=2.0, cutoff=12.0,
             fp32=False, noalloc=True),
        # the size of the 65,536-disk workload, two species, FP32 pair sums for a program that keeps 32-bit data
        dict(name="forces_65536_fp32", kind="forces", n=65536, phi=0.4, S=2, law="power", q=2.0, cutoff=0.0, fp32=True,
             noalloc=False),
        # the plain method at its smallest: 1,024 disks, FP64, graph replay; the chain of launches is the time
        dict(name="steps_1024_fp64", kind="steps", n=1024, phi=0.30, S=1, force="pairs", overlap="delaunay",
             fp32=False, periodic=False, factor=1.0, graph=True, steps=16, active=False),
        # an odd size stepped launch by launch, the library's default mode
        dict(name="steps_5003_eager", kind="steps", n=5003, phi=0.40, S=2, force="pairs", overlap="delaunay",
             fp32=False, periodic=False, factor=1.0, graph=False, steps=4, active=True),
        # the headline workload: 65,536 self-propelled disks of two species, FP32 all-pairs forces
        dict(name="steps_65536_fp32", kind="steps", n=65536, phi=0.40, S=2, force="pairs", overlap="delaunay",
             fp32=True, periodic=False, factor=1.0, graph=True, steps=4, active=True),
        # the paper's own domain: a periodic box, all pairs in FP64 at the nearest image
        dict(name="steps_16001_periodic", kind="steps", n=16001, phi=0.35, S=1, force="pairs", overlap="delaunay",
             fp32=False, periodic=True, factor=1.0, graph=True, steps=4, active=False),
        # short-range forces of a medium system in FP64, a periodic box, overlaps over Delaunay edges
        dict(name="steps_40009_lists_fp64", kind="steps", n=40009, phi=0.45, S=2, force="lists", overlap="delaunay",
             fp32=False, periodic=True, factor=1.0, graph=True, steps=8, active=True),
        # the largest system, short-range forces, overlaps over Delaunay edges (the default method)
        dict(name="steps_1m_lists", kind="steps", n=1048576, phi=0.50, S=1, force="lists", overlap="delaunay",
             fp32=True, periodic=False, factor=1.0, graph=True, steps=8, active=False),
        # the same with the paper's short-range algorithm: overlaps over the neighbour lists
        dict(name="steps_1m_lists_verlet", kind="steps", n=1048576, phi=0.50, S=1, force="lists", overlap="verlet",
             fp32=True, periodic=False, factor=1.0, graph=True, steps=8, active=False),
        # many independent FP64 systems of uneven size in one handle
        dict(name="steps_batch64_fp64", kind="steps", n=0, R=64, lo=2048, hi=32768, phi=0.35, S=1, force="pairs",
             overlap="delaunay", fp32=False, periodic=False, factor=1.0, graph=True, steps=1, active=False),
        # gradients through 10 steps of the differentiation workload (contact factor 1/2, 16,384 disks)
        dict(name="adjoint_16384", kind="adjoint", n=16384, phi=0.35, S=2, steps=10, every=5, factor=0.5),
    ]


def _log(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    kind = rng.choice(["forces", "forces", "steps", "steps", "steps", "adjoint"])
    phi = round(rng.uniform(0.2, 0.5), 3)
    if kind == "forces":
        law = rng.choice(["power", "power", "screened"])
        return dict(kind="forces", n=_log(rng, 200, 65536), phi=phi, S=rng.randint(1, 3), law=law,
                    q=rng.choice([2.0, 2.0, 6.0]) if law == "power" else 2.0,
                    cutoff=rng.choice([0.0, 12.0]) if law == "screened" else 0.0, fp32=rng.random() < 0.5,
                    noalloc=rng.random() < 0.5)
    if kind == "adjoint":
        return dict(kind="adjoint", n=_log(rng, 500, 16384), phi=min(phi, 0.4), S=rng.randint(1, 2), steps=6, every=3,
                    factor=rng.choice([0.5, 1.0]))
    force = rng.choice(["pairs", "lists"])
    c = dict(kind="steps", phi=phi, S=rng.randint(1, 3), force=force, overlap="delaunay", fp32=rng.random() < 0.5,
             periodic=rng.random() < 0.3, factor=rng.choice([1.0, 1.0, 0.5]), graph=rng.random() < 0.7, steps=4,
             active=rng.random() < 0.5)
    if force == "lists":
        c["n"] = _log(rng, 2000, 400000)
        c["overlap"] = rng.choice(["delaunay", "verlet"])
    elif rng.random() < 0.25:
        c.update(n=0, R=rng.randint(3, 24), lo=rng.randint(300, 2048), hi=rng.randint(4096, 16384), periodic=False,
                 steps=2)
    else:
        c["n"] = _log(rng, 500, 40000)
    return c


# ---------------------------------------------------------------- inputs
def _lattice(case, seed):
    """Disks of radius 1 at area fraction phi on a jittered square lattice, in random order: positions and species."""
    n = case["n"]
    g = torch.Generator().manual_seed(seed)
    m = math.isqrt(n - 1) + 1
    a = math.sqrt(math.pi / case["phi"])
    k = torch.randperm(m * m, generator=g)[:n]
    xy = torch.stack([k % m, k // m], 1).to(torch.float64) * a + 0.5 * a
    xy += (torch.rand(n, 2, generator=g, dtype=torch.float64) - 0.5) * 0.9 * (a - 2.0)
    return xy, torch.randint(0, case["S"], (n,), generator=g, dtype=torch.int32)


def _strengths(S, scale):
    """A strength matrix that is not symmetric."""
    a, b = np.meshgrid(np.arange(S), np.arange(S), indexing="ij")
    return scale * np.where(a == b, 1.0, np.where(a < b, -0.5, 0.2))


def _disks(n, phi, seed, periodic):
    """Random sequential insertion; the largest systems repeat one periodically placed tile 4 x 4 times."""
    if n < 500000:
        L = synth.box_side(n, phi)
        return synth.rsa(n, L, 1.0, seed, periodic=periodic), L
    side = synth.box_side(n // 16, phi)
    tile = synth.rsa(n // 16, side, 1.0, seed, periodic=True)
    shifts = np.array([[i * side, j * side] for j in range(4) for i in range(4)])
    xy = (shifts[:, None, :] + tile[None, :, :]).reshape(-1, 2)
    return xy + 1.0, 4.0 * side + 2.0


def _sizes(case):
    rng = np.random.Generator(np.random.PCG64(case["R"]))
    return [int(v) for v in np.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"]), size=case["R"]))]


def _handle(case, seed):
    S = case["S"]
    opts = dict(D=1.0, dt=1e-4, overlap_factor=case["factor"], fp32=case.get("fp32", False))
    if case.get("active"):
        opts.update(v0=1.0, Dr=1.0)
    if case.get("force") == "lists":
        opts.update(kind="screened", A=1.0, lam=0.5, cutoff=2.5, skin=0.5, overlap=case["overlap"])
        K = _strengths(S, 1.0)
    else:
        K = _strengths(S, 1e-2)
    if case["n"]:
        xy, L = _disks(case["n"], case["phi"], seed, case.get("periodic", False))
        n = len(xy)
        th = np.random.Generator(np.random.PCG64(seed + 7)).uniform(0.0, 2.0 * math.pi, n)
        return binding.Sim(xy, np.ones(n), (np.arange(n) % S).astype(np.int32), th, K, L=L, seed=seed,
                           periodic=case.get("periodic", False), **opts)
    sizes = _sizes(case)
    made = [_disks(n, case["phi"], 1000003 * seed + r, False) for r, n in enumerate(sizes)]
    return binding.Sim.batch([xy for xy, _ in made], [np.ones(n) for n in sizes],
                             [(np.arange(n) % S).astype(np.int32) for n in sizes], [np.zeros(n) for n in sizes],
                             [L for _, L in made], [seed + r for r in range(len(sizes))], K, **opts)


def prepare(case, seed):
    """Device arrays for a force call; otherwise a handle as a program holds it in the middle of a run (a few steps
    behind it), with the device buffers its results go to."""
    st = dict(case)
    if case["kind"] == "forces":
        xy, sp = _lattice(case, seed)
        st.update(xy=xy.cuda(), sp=sp.cuda(), K=_strengths(case["S"], 1.0),
                  out=torch.empty(case["n"], 2, dtype=torch.float64, device="cuda"))
        return st
    sim = _handle(case, seed)
    st.update(sim=sim, xy=torch.empty(sim.n, 2, dtype=torch.float64, device="cuda"),
              th=torch.empty(sim.n, dtype=torch.float64, device="cuda"))
    if case["kind"] == "steps":
        sim.set_graph_mode(case["graph"])
        sim.step(8)
    else:
        g = torch.Generator().manual_seed(seed + 1)
        st.update(grad=torch.randn(sim.n, 2, generator=g, dtype=torch.float64).cuda(),
                  g0=torch.empty(sim.n, 2, dtype=torch.float64, device="cuda"),
                  gK=torch.empty(case["S"], case["S"], dtype=torch.float64, device="cuda"))
        torch.cuda.synchronize()   # the handle runs on its own stream
    return st


def run(st):
    if st["kind"] == "forces":
        f = binding.pair_forces_dev(st["xy"], st["sp"], st["K"], kind=st["law"], q=st["q"], A=1.0, lam=2.0,
                                    cutoff=st["cutoff"], fp32=st["fp32"], out=st["out"], noalloc=st["noalloc"])
        return f.float() if st["fp32"] else f   # FP32 pair sums go on as 32-bit data
    sim = st["sim"]
    if st["kind"] == "steps":
        sim.step(st["steps"])
        sim.state_dev(st["xy"].data_ptr(), st["th"].data_ptr())
        return st["xy"], st["th"]
    sim.adjoint_begin(st["steps"], st["every"])
    sim.state_dev(st["xy"].data_ptr())
    sim.adjoint_backward_dev(st["grad"].data_ptr(), st["g0"].data_ptr(), st["gK"].data_ptr())
    return st["xy"], st["g0"], st["gK"]


def work(case):
    """Inputs read once and outputs written once; 12 operations per ordered pair where all pairs act through a
    strength matrix that is not symmetric, 16 per unordered pair inside a step (both sides from one evaluation)."""
    n = case["n"]
    if case["kind"] == "forces":
        return {"bytes": 36.0 * n, "flops": 12.0 * n * (n - 1)}
    if case["kind"] == "adjoint":   # forward, recomputed forward, reverse pair sum
        return {"bytes": case["steps"] * 300.0 * n, "flops": case["steps"] * (8.0 + 8.0 + 28.0) * n * (n - 1)}
    sizes = [n] if n else _sizes(case)
    total = float(sum(sizes))
    # per disk and step: positions in and out 32, radius and species 12, angle 16; two triangles of the
    # triangulation 48; the neighbour list (about 4 ids and the count) 20
    per = 44.0 + (16.0 if case["active"] else 0.0) + (48.0 if case["overlap"] == "delaunay" else 0.0)
    if case["force"] == "lists":
        return {"bytes": case["steps"] * (per + 20.0) * total, "flops": case["steps"] * 100.0 * total}
    return {"bytes": case["steps"] * per * total, "flops": case["steps"] * 8.0 * sum(float(m) * (m - 1) for m in sizes)}


def exact(case, seed):
    """Forces by plain torch in 64 bits.  A step has no such value: its end state goes through thresholds (overlap
    rounds on a Delaunay triangulation) that plain array code does not give."""
    if case["kind"] != "forces":
        return None
    xy, sp = (t.cuda() if torch.cuda.is_available() else t for t in _lattice(case, seed))
    K = torch.from_numpy(_strengths(case["S"], 1.0)).to(xy.device)
    out = torch.empty_like(xy)
    rows = max(1, 16_000_000 // case["n"])
    for i in range(0, case["n"], rows):
        d = xy[i:i + rows, None, :] - xy[None, :, :]
        r = d.square().sum(-1).sqrt()
        ok = r > 0
        r = torch.where(ok, r, torch.ones_like(r))
        g = torch.exp(-r / 2.0) / r if case["law"] == "screened" else r ** -case["q"]
        if case["cutoff"] > 0:
            ok &= r <= case["cutoff"]
        w = torch.where(ok, K[sp[i:i + rows].long()][:, sp.long()] * g / r, torch.zeros_like(r))
        out[i:i + rows] = (w[..., None] * d).sum(1)
    return out
