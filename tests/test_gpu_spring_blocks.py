"""The spring kernels with positions staged in LDS (k_spring_block), against the oracle where their
tables can go wrong: one vertex past a workgroup, vertices with no edge, edges from a vertex to
itself and repeated edges, springs of zero, tiny and huge length; and graphs that the tables do not
take (a hub, scrambled vertices).

Tolerances (normwise), as in test_gpu_springs: forces 1e-12, ten steps 1e-10."""
import numpy as np
import pytest
import torch

import oracle
from paper_1506_07577_amd import meshgen as mg

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1506_07577_amd import ebbx
else:  # collected on a CPU host only to be deselected
    ebbx = None


def _ring(nv, reach=6):
    """Vertex i with the `reach` after it, cyclically, in both directions: vertices near each other in
    number share neighbours."""
    X = np.random.default_rng(1).uniform(0.0, 1.0, (nv, 3))
    i = np.arange(nv)
    pairs = [(i, (i + k) % nv) for k in range(1, reach + 1)]
    tail = np.concatenate([a for a, b in pairs] + [b for a, b in pairs])
    head = np.concatenate([b for a, b in pairs] + [a for a, b in pairs])
    return X, tail.astype(np.int32), head.astype(np.int32)


def _cube(n, **kw):
    m = mg.jitter(mg.kuhn_cube(n), 0.02, seed=0)
    return (m.X, *mg.directed_edges(m.tets, m.nv))


def _odd():
    """A ring with loops, repeated edges and a stretch of vertices that no edge leaves."""
    X, tail, head = _ring(700)
    keep = (tail < 100) | (tail >= 230)
    tail, head = tail[keep], head[keep]
    loops = np.arange(300, 340, dtype=np.int32)
    return X, np.concatenate([tail, loops, tail[:50]]), np.concatenate([head, loops, head[:50]])


def _hub():
    X, tail, head = _ring(600)
    spokes = np.arange(1, 600, dtype=np.int32)
    return X, np.concatenate([tail, 0 * spokes]), np.concatenate([head, spokes])


def _scrambled():
    m, _, _ = mg.scramble(mg.kuhn_cube(9), seed=1)
    return (m.X, *mg.directed_edges(m.tets, m.nv))


GRAPHS = {"ring_64": lambda: _ring(64), "ring_65": lambda: _ring(65), "ring_321": lambda: _ring(321),
          "cube": lambda: _cube(9), "large": lambda: _cube(41), "odd": _odd, "hub": _hub, "scrambled": _scrambled}


@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_forces_and_steps(name):
    X, tail, head = GRAPHS[name]()
    nv = len(X)
    rng = np.random.default_rng(4)
    mass = (1.0 + 0.5 * rng.uniform(-1, 1, nv)) / nv
    q = X + 0.01 * rng.uniform(-1, 1, X.shape)
    q[nv // 2] = q[nv // 2 - 1]   # a spring of zero length, where the two are neighbours
    qd = 0.05 * rng.uniform(-1, 1, X.shape)
    sm = ebbx.SpringMesh(X, tail, head, 0.5)
    ref = oracle.Springs(X, tail, head, mass, 0.5)
    f0 = rng.uniform(-1, 1, X.shape)
    f = sm.to_dev(f0)
    sm.springs.forces(sm.to_dev(q), f, accumulate=True)
    want = ref.forces(q)
    assert np.abs(sm.from_dev(f) - f0 - want).max() <= 1e-12 * max(np.abs(want).max(), 1.0)
    qs, qds = q.copy(), qd.copy()
    for _ in range(10):
        qs, qds = ref.step(qs, qds, 1e-4)
    a, b = sm.to_dev(q), sm.to_dev(qd)
    sm.springs.run(sm.scalar_to_dev(mass), 1e-4, 10, a, b, torch.zeros_like(a))
    assert np.abs(sm.from_dev(a) - qs).max() <= 1e-10 * np.abs(qs).max()
    assert np.abs(sm.from_dev(b) - qds).max() <= 1e-10 * np.abs(qds).max()


@pytest.mark.parametrize("scale", [1e-145, 1e-100, 1e100, 1e145])
def test_extreme_lengths(scale):
    """Lengths whose squares leave the range of the fast path: the library's root and division."""
    X, tail, head = _ring(321)
    X = X * scale
    q = X * (1.0 + 0.01 * np.random.default_rng(2).uniform(-1, 1, X.shape))
    sm = ebbx.SpringMesh(X, tail, head, 0.5)
    ref = oracle.Springs(X, tail, head, np.ones(len(X)), 0.5)
    want = ref.forces(q)
    got = sm.from_dev(sm.springs.forces(sm.to_dev(q)))
    assert np.abs(got - want).max() <= 1e-12 * np.abs(want).max()
